"""Prefill-time sparse attention where its key and query tiles end: groups of 1 to 8 heads, blocks that do not fill a tile of
query rows, buckets of less than a key tile and of many, tokens that list the same buckets and tokens that list none."""
import numpy as np
import pytest
import torch

from oracle import ref
from test_gpu_prefill import DEV, SCALE, assert_close, h, setup
from test_gpu_prefill import saap  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,Hq,Hkv,Nt,B,Tq,nprobe,n_sink,n_recent,pos0,same", [
    (1, 2, 2, 700, 16, 33, 3, 1, 40, (600,), False),             # one head per group: 32 tokens a tile, and one more
    (2, 4, 2, 900, 64, 17, 9, 0, 33, (0, 883), False),           # buckets below a key tile; a block that opens its prompt
    (1, 8, 2, 5000, 4, 35, 2, 3, 129, (4965,), False),            # buckets long enough to be shared out over waves
    (1, 8, 1, 5000, 8, 67, 3, 2, 64, (3000,), True),             # every token lists the same buckets; keys beyond the block
    (4, 16, 2, 1300, 40, 8, 40, 1, 1, (1292, 0, 7, 640), False), # as few tokens as come here, every bucket
    (3, 4, 1, 600, 8, 130, 1, 600, 0, (0, 100, 470), False),     # a sink as large as the cache
    (1, 4, 4, 2500, 300, 65, 250, 0, 500, (2000,), False),       # hundreds of lists per token
])
def test_prefill_tiles(saap, S, Hq, Hkv, Nt, B, Tq, nprobe, n_sink, n_recent, pos0, same):  # noqa: F811
    cache, ids, (off, ln, idx, Ks, Vs), q = setup(saap, "bf16", S, Hq, Hkv, Nt, B, Tq, 5 + Tq, slack=2)
    rng = np.random.default_rng(Tq + nprobe)
    sel = np.stack([rng.permutation(B)[:nprobe] for _ in range(S * Hkv * Tq)]).reshape(S, Hkv, Tq, nprobe).astype(np.int32)
    if same:
        sel[:] = sel[:, :, :1]
    p0 = np.array(pos0, dtype=np.int32)
    args = (cache["K"], cache["V"], Ks, Vs, off, ln, idx, torch.from_numpy(sel).to(DEV), torch.from_numpy(p0).to(DEV), n_sink, n_recent)
    out, lse = saap.prefill_sparse_attention(q, *args, SCALE)
    again, _ = saap.prefill_sparse_attention(q, *args, SCALE)
    torch.cuda.synchronize()
    ro, rl = ref.prefill_sparse_attention(h(q), h(cache["K"]), h(cache["V"]), ids.cpu().numpy(), sel, p0, n_sink, n_recent, SCALE, B)
    assert_close(out.cpu().numpy(), ro, "bf16", "out")
    assert_close(lse.cpu().numpy(), rl, "bf16", "lse")
    assert torch.equal(out, again)                               # whatever order the work is taken in


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_scores_that_are_no_numbers(saap, bad):  # noqa: F811
    """A key or a query that is not finite: the block gives what its tokens give four at a time (too few for shared tiles)."""
    S, Hq, Hkv, Nt, B, Tq, nprobe, p0 = 1, 8, 2, 1500, 24, 40, 6, 1400
    cache, ids, _, q = setup(saap, "bf16", S, Hq, Hkv, Nt, B, Tq, 11)
    K = cache["K"].clone()
    K[0, 0, 700], K[0, 1, p0 + 20] = bad, bad                    # a bucket's member; a key the block's second half sees
    off, ln, idx, Ks, Vs = saap.build_bucket_index(ids, K, cache["V"], B, 0)
    q = q.clone()
    q[0, 9, 5] = bad
    rng = np.random.default_rng(3)
    sel = np.stack([rng.permutation(B)[:nprobe] for _ in range(Hkv * Tq)]).reshape(S, Hkv, Tq, nprobe).astype(np.int32)
    sel = torch.from_numpy(sel).to(DEV)

    def attend(t0, t1):
        return saap.prefill_sparse_attention(q[:, t0:t1].contiguous(), K, cache["V"], Ks, Vs, off, ln, idx,
                                             sel[:, :, t0:t1].contiguous(), torch.tensor([p0 + t0], dtype=torch.int32, device=DEV),
                                             1, 64, SCALE)
    out, lse = attend(0, Tq)
    parts = [attend(t, t + 4) for t in range(0, Tq, 4)]
    want, want_lse = torch.cat([p[0] for p in parts], 1), torch.cat([p[1] for p in parts], 1)
    none = torch.isinf(want_lse)
    assert 0 < none.sum() < none.numel()
    assert torch.equal(torch.isinf(lse), none)
    assert torch.isnan(out[none]).all()
    assert_close(out[~none].cpu().numpy(), want[~none].cpu().numpy(), "bf16", "out")
    assert_close(lse[~none].cpu().numpy(), want_lse[~none].cpu().numpy(), "bf16", "lse")


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("Hq,Hkv,B,same", [(8, 2, 24, False), (8, 2, 24, True), (8, 2, 3, True), (2, 2, 6, False), (16, 2, 24, False)])
def test_values_that_are_no_numbers_stay_with_the_tokens_that_attend_them(saap, Hq, Hkv, B, same, bad):  # noqa: F811
    """Values that are not finite at a later token of the block, at the edge of the recent keys, at a sink key beyond some
    tokens' range and at a bucket's member: what does not attend them (by the oracle) has the numbers of a cache without them,
    bit for bit, also where the tokens of a tile differ in what they see.  B = 3: buckets shared out over waves."""
    S, Nt, Tq, nprobe, p0, n_sink, n_recent = 2, 1500, 40, max(1, B // 4), np.array([1400, 0], dtype=np.int32), 12, 64
    cache, ids, (off, ln, idx, Ks, Vs), q = setup(saap, "bf16", S, Hq, Hkv, Nt, B, Tq, 12)
    rng = np.random.default_rng(4)
    sel = np.stack([rng.permutation(B)[:nprobe] for _ in range(S * Hkv * Tq)]).reshape(S, Hkv, Tq, nprobe).astype(np.int32)
    if same:
        sel[:] = sel[:, :, :1]
    V = cache["V"].clone()
    V[0, 0, 1421, 3] = V[0, 1, 1400 - 64 + 20, 77] = V[0, 1, 700] = bad       # later token; edge of the recent keys; a member
    V[1, 0, 5, 0], V[1, 0, 9, 127], V[1, 1, 30, 64] = bad, -bad, bad          # sink keys of the prompt's first tokens; a later one
    sel_d, p0_d = torch.from_numpy(sel).to(DEV), torch.from_numpy(p0).to(DEV)

    def attend(values):
        index = saap.build_bucket_index(ids, cache["K"], values, B, 0)
        return saap.prefill_sparse_attention(q, cache["K"], values, index[3], index[4], *index[:3], sel_d, p0_d, n_sink, n_recent, SCALE)
    out, lse = attend(V)
    clean, clean_lse = attend(cache["V"])
    ro, _ = ref.prefill_sparse_attention(h(q), h(cache["K"]), h(V), ids.cpu().numpy(), sel, p0, n_sink, n_recent, SCALE, B)
    fin = torch.from_numpy(np.isfinite(ro)).to(DEV)
    assert 0 < (~fin).sum() < fin.numel() // 2
    assert torch.equal(torch.isfinite(out), fin)
    assert torch.equal(out[fin], clean[fin]) and torch.equal(lse, clean_lse)
