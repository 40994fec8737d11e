"""The classifier's row-tiled output layer in tiles of 64 x 128: edges of rows and buckets, hidden units that fill their chunks and
units that do not, against the oracle."""
import pytest

from test_gpu_classify_rows import saap, test_logits as check_logits  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,Hq,Hkv,Hw,hidden,B", [(69, 64, 8, 8, 96, 880), (1100, 1, 1, 1, 128, 1008), (1025, 1, 1, 1, 32, 2064), (65, 64, 8, 8, 160, 784)])
def test_logits_of_many_rows(saap, S, Hq, Hkv, Hw, hidden, B):  # noqa: F811
    check_logits(saap, S, Hq, Hkv, Hw, hidden, B, "bf16")
