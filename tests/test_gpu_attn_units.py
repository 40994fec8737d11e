"""Sparse attention at numbers of (sequence, KV head) units where three workgroups, or one, share a unit: the first and last such numbers
and their neighbours on a device of 256 compute units, list lengths on both sides of the line, buckets of very unequal sizes with
empty ones among them, against plain softmax attention in float64."""
import math

import pytest
import torch

import paper_2502_08246_amd as saap

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALE = 1.0 / math.sqrt(128)


@pytest.mark.parametrize("S,Hkv", [(128, 1), (43, 3), (18, 8), (85, 2), (57, 3)])
@pytest.mark.parametrize("G,dtype", [(1, "fp8"), (4, "fp8"), (8, "fp8"), (1, "f32"), (4, "f32"), (8, "f32"), (4, "bf16"), (8, "bf16")])
@pytest.mark.parametrize("nprobe", [23, 24, 39, 40])       # 1536 keys are expected of 24 of these buckets, 2560 of 40
def test_units_sharing(S, Hkv, G, dtype, nprobe):
    B, N = 128, 8192
    g = torch.Generator(device=DEV).manual_seed(S * Hkv + G)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    weights = torch.rand(S * Hkv, B, generator=g, device=DEV) ** 4
    weights[:, 3] = 0
    ids = torch.multinomial(weights, N, replacement=True, generator=g).to(torch.int32).view(S, Hkv, N)
    K, V = (torch.randn(S, Hkv, N, 128, generator=g, device=DEV).to(kind) for _ in range(2))
    q = (2.0 * torch.randn(S, Hkv * G, 128, generator=g, device=DEV)).to(kind)
    off, ln, idx, Ks, Vs = saap.build_bucket_index(ids, K, V, B, 0)
    logits = torch.randn(S, Hkv * G, B, generator=g, device=DEV)
    selected = saap.select_buckets_from_logits(logits, Hkv, nprobe)
    index, Kd, Vd = (Ks, Vs), Ks.double(), Vs.double()
    if dtype == "fp8":
        K8, V8, ks, vs = saap.quantize_kv(Ks, Vs)
        index = (K8, V8, ks, vs)
        Kd, Vd = (c.view(torch.float8_e4m3fn).double() * s.double().view(S, Hkv, 1, 1) for c, s in ((K8, ks), (V8, vs)))
    attend, both = (saap.sparse_decode_attention_fp8, saap.select_attend_fp8) if dtype == "fp8" else (saap.sparse_decode_attention, saap.select_attend)
    out, lse = attend(q, *index, off, ln, selected, SCALE)
    picked, out2, lse2 = both(logits, q, *index, off, ln, nprobe, SCALE)
    assert torch.equal(picked, selected)
    bucket = torch.gather(ids, 2, idx.long())              # of each slot
    seen = torch.zeros(S, Hkv, B, dtype=torch.bool, device=DEV).scatter_(2, selected.long(), True).gather(2, bucket.long())
    qd = q.double().view(S, Hkv, G, 128)
    scores = torch.stack([(Kd * qd[:, :, i:i + 1]).sum(-1) for i in range(G)], 2) * SCALE
    scores = scores.masked_fill(~seen.unsqueeze(2), -math.inf)
    p = scores.softmax(-1)
    want = torch.stack([(p[:, :, i].unsqueeze(-1) * Vd).sum(2) for i in range(G)], 2).view(S, Hkv * G, 128)
    want_lse = scores.logsumexp(-1).view(S, Hkv * G)
    absolute, relative = (1e-5, 1e-5) if dtype == "f32" else (2e-3, 1e-2)
    for got, ref in ((out, want), (out2, want), (lse, want_lse), (lse2, want_lse)):
        assert ((got.double() - ref).abs() <= absolute + relative * ref.abs()).all()
