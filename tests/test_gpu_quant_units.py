"""The 8-bit copy at numbers of units where the maxima change their place, few rows and many, twice with the second call's values
below the first's (a maximum that is not cleared would show), against torch's conversion."""
import pytest
import torch

import paper_2502_08246_amd as saap

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("units,rows", [(1, 1), (1, 70001), (2, 3000), (9, 63), (512, 5), (513, 5), (4096, 2), (4097, 2)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_quantize_units(units, rows, dtype):
    g = torch.Generator(device=DEV).manual_seed(units + rows)
    for size in (1e4, 1.0, 1e-3):
        K, V = ((size * torch.randn(1, units, rows, 128, generator=g, device=DEV)).to(dtype) for _ in range(2))
        K[0, -1] = 0                                       # the last unit's keys: scale 1
        got = saap.quantize_kv(K, V)
        for x, codes, scale in ((K, got[0], got[2]), (V, got[1], got[3])):
            mx = x.float().abs().amax((2, 3))
            want = torch.where(mx > 0, torch.exp2(torch.ceil(torch.log2(mx.double() / 448))).float(), torch.ones_like(mx))
            assert torch.equal(scale.view_as(want), want)
            assert torch.equal(codes, (x.float() / want[:, :, None, None]).to(torch.float8_e4m3fn).view(torch.uint8))


@pytest.mark.parametrize("units,rows", [(600, 15), (600, 16), (600, 17), (1000, 64), (1000, 65), (2048, 130), (8192, 3), (64, 1040), (3, 33)])
def test_quantize_short_units(units, rows):
    """Fewer workgroups than usual for a unit: rows on both sides of what they take."""
    test_quantize_units(units, rows, torch.bfloat16)
