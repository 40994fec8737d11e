"""The native call layer: arguments by position and by name, what it raises, and that outputs passed in come back as
the objects they are."""
import inspect
import math

import pytest
import torch

import paper_2502_08246_amd as saap
from paper_2502_08246_amd import binding

DEV = "cuda:0"


def test_every_native_call_states_its_signature():
    for name in binding.NATIVE:
        assert len(inspect.signature(getattr(saap, name)).parameters) >= 3, name


def test_arguments_are_checked_like_a_python_call():
    x, c = torch.zeros(1, 1, 8, 128), torch.zeros(1, 4, 128)
    with pytest.raises(TypeError):
        saap.assign_keys(x)                                   # a mandatory argument is missing
    with pytest.raises(TypeError):
        saap.assign_keys(x, c, nothing=1)
    with pytest.raises(TypeError):
        saap.assign_keys(x, c, centroids=c)                   # given twice
    with pytest.raises(TypeError):
        saap.assign_keys(x, [1, 2])                           # not a tensor
    with pytest.raises(ValueError):
        saap.assign_keys(x[0], c)                             # a dimension short
    with pytest.raises(ValueError):
        saap.assign_keys(x, c[:, :, :64])
    with pytest.raises(ValueError):
        saap.assign_keys(x, c)                                # host memory
    with pytest.raises(TypeError):
        saap.sparse_decode_attention_fp8(*[x] * 8, 1.0)       # not an 8-bit cache


@pytest.mark.gpu
def test_names_positions_and_outputs_passed_in():
    g = torch.Generator(device=DEV).manual_seed(1)
    S, Hkv, G, N, B, nprobe = 2, 2, 4, 700, 16, 3
    rand = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    x, q, cent = rand(S, Hkv, N, 128), rand(S, Hkv * G, 128), rand(Hkv, B, 128)
    ids = saap.assign_keys(x, cent)
    off, ln, _, Ks, Vs = saap.build_bucket_index(ids, x, x, B, slack=2)
    logits = torch.randn(S, Hkv * G, B, generator=g, device=DEV)
    sel = saap.select_buckets_from_logits(logits, nprobe=nprobe, Hkv=Hkv)
    scale = 1 / math.sqrt(128)
    want, want_lse = saap.sparse_decode_attention(q, Ks, Vs, off, ln, sel, scale)
    out = torch.empty_like(q)
    got = saap.sparse_decode_attention(scale=scale, selected=sel, ln=ln, off=off, Vs=Vs, Ks=Ks, q=q, out=out)
    assert isinstance(got, tuple) and got[0] is out and got[0].dtype == torch.bfloat16
    assert torch.equal(out, want.to(torch.bfloat16)) and torch.equal(got[1], want_lse)
    half, _ = saap.sparse_decode_attention(q, Ks, Vs, off, ln, sel, scale, out_dtype=torch.bfloat16)
    assert torch.equal(half, out)
    with pytest.raises(ValueError):
        saap.sparse_decode_attention(q.transpose(0, 1), Ks, Vs, off, ln, sel, scale)      # not contiguous
    with pytest.raises(saap.SaapError) as e:
        saap.sparse_decode_attention(q, Ks, Vs, off, ln, sel, scale, ws=torch.zeros(64, dtype=torch.uint8, device=DEV))
    assert e.value.status == -3


@pytest.mark.gpu
def test_a_missing_pointer_is_the_librarys_error():
    """Arguments that are only passed on: None is the library's invalid argument, whatever the call."""
    S, Hkv, G, N, B, nprobe = 1, 2, 4, 64, 16, 3
    bf16 = dict(dtype=torch.bfloat16, device=DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    q, K, cent = torch.zeros(S, Hkv * G, 128, **bf16), torch.zeros(S, Hkv, N, 128, **bf16), torch.zeros(Hkv, B, 128, **bf16)
    K8, one = torch.zeros(S, Hkv, N, 128, dtype=torch.uint8, device=DEV), torch.ones(S, Hkv, device=DEV)
    ids, idx = torch.zeros(S, Hkv, N, **i32), torch.zeros(S, Hkv, N, **i32)
    off, ln = torch.zeros(S, Hkv, B + 1, **i32), torch.zeros(S, Hkv, B, **i32)
    sel, logits, new = torch.zeros(S, Hkv, nprobe, **i32), torch.zeros(S, Hkv * G, B, device=DEV), K[:, :, 0].contiguous()
    pos = torch.zeros(S, **i32)
    plan = saap.build_visit_plan(sel, off, ln, Hkv * G)
    calls = [
        ("build_bucket_index", (ids, K, K, B), (0, 2)),
        ("build_windowed_index", (ids, K, K, B, 2, 1, 8), (0, 2)),
        ("quantize_kv", (K, K), (1,)),
        ("build_visit_plan", (sel, off, ln, Hkv * G), (1,)),
        ("select_buckets_planned", (logits, off, ln, Hkv, nprobe), (1, 2)),
        ("sparse_decode_attention", (q, K, K, off, ln, sel, 0.1), (2, 3)),
        ("windowed_decode_attention", (q, K, K, off, ln, sel, -1, 0.1), (2, 3)),
        ("dense_decode_attention", (q, K, K, 0.1), (2,)),
        ("select_attend", (logits, q, K, K, off, ln, nprobe, 0.1), (0, 3, 4)),
        ("planned_decode_attention", (q, K, K, plan, nprobe, 0.1), (2, 3)),
        ("sparse_decode_attention_fp8", (q, K8, K8, one, one, off, ln, sel, 0.1), (3, 4, 5)),
        ("windowed_decode_attention_fp8", (q, K8, K8, one, one, off, ln, sel, -1, 0.1), (3, 4, 5)),
        ("dense_decode_attention_fp8", (q, K8, K8, one, one, 0.1), (3, 4)),
        ("select_attend_fp8", (logits, q, K8, K8, one, one, off, ln, nprobe, 0.1), (0, 4, 5, 6)),
        ("planned_decode_attention_fp8", (q, K8, K8, one, one, plan, nprobe, 0.1), (3, 4, 5)),
        ("prefill_sparse_attention", (q.view(S, 1, Hkv * G, 128), K, K, K, K, off, ln, idx, sel.view(S, Hkv, 1, nprobe),
                                      pos, 1, 8, 0.1), (2, 4, 5, 7, 9)),
        ("append_keys", (new, new, new, pos, cent, None, off, ln, idx, K, K), (1, 2, 6, 7, 9, 10)),
        ("append_keys_fp8", (new, new, new, pos, cent, None, off, ln, idx, K8, K8, one, one), (6, 7, 9, 10, 11, 12)),
        ("window_push", (new, new, new, pos, cent, None, off, ln, idx, K, K, ids, 1, 8), (1, 2, 6, 7, 9, 10, 11)),
        ("window_push_fp8", (new, new, new, pos, cent, None, off, ln, idx, K8, K8, one, one, ids, 1, 8), (6, 7, 9, 10, 11, 12, 13)),
    ]
    for name, args, pointers in calls:
        for i in pointers:
            with pytest.raises(saap.SaapError) as e:
                getattr(saap, name)(*args[:i], None, *args[i + 1:])
            assert e.value.status == -1, (name, i)
            with pytest.raises(TypeError):
                getattr(saap, name)(*args[:i], [1], *args[i + 1:])


@pytest.mark.gpu
def test_every_stream_has_its_own_workspace_and_graphs_have_theirs():
    """The default workspace: one per stream, a zeroed header each, kept while it is large enough; a capture takes the
    one that the calls before it used, which no later eager call gets, or the one of an earlier capture."""
    here = saap.workspace(1 << 20, DEV)
    assert saap.workspace(0, DEV).data_ptr() == here.data_ptr()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        there = saap.workspace(0, DEV)
        assert there.data_ptr() == saap.workspace(0, DEV).data_ptr() != here.data_ptr()
        assert not there[:saap.binding.WS_HEADER_BYTES].any()
    g = torch.Generator(device=DEV).manual_seed(2)
    logits = torch.randn(2, 8, 64, generator=g, device=DEV)
    want = saap.select_buckets_from_logits(logits, 2, 5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = saap.select_buckets_from_logits(logits, 2, 5)
        inside = saap.workspace(0, DEV).data_ptr()
        with pytest.raises(RuntimeError):
            saap.workspace(1 << 40, DEV)                       # a capture cannot make one
    after = saap.workspace(0, DEV).data_ptr()
    if inside == here.data_ptr():                              # the process's first capture took this stream's
        assert after not in (inside, there.data_ptr())
    else:                                                      # an earlier capture's serves all graphs
        assert after == here.data_ptr() and inside != there.data_ptr()
    again = torch.cuda.CUDAGraph()
    with torch.cuda.graph(again):
        saap.select_buckets_from_logits(logits, 2, 5)
        assert saap.workspace(0, DEV).data_ptr() == inside
    with torch.cuda.stream(side):
        assert saap.workspace(0, DEV).data_ptr() == there.data_ptr()
    for _ in range(3):
        got.zero_()
        graph.replay()
        assert torch.equal(got, want)
        assert torch.equal(saap.select_buckets_from_logits(logits, 2, 5), want)


@pytest.mark.gpu
def test_two_streams_at_once_give_what_one_gives():
    """Several launches and counters per call: two streams that enqueue them by turns, with the default workspace."""
    S, Hq, Hkv, N, B, Tq, nprobe, scale = 1, 8, 8, 6000, 48, 64, 6, 1 / math.sqrt(128)
    g = torch.Generator(device=DEV).manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    K, V = rand(S, Hkv, N, 128), rand(S, Hkv, N, 128)
    ids = torch.randint(0, B, (S, Hkv, N), generator=g, device=DEV, dtype=torch.int32)
    off, ln, idx, Ks, Vs = saap.build_bucket_index(ids, K, V, B)
    pos0 = torch.tensor([N - Tq], dtype=torch.int32, device=DEV)
    jobs = []
    for _ in range(2):
        sel = torch.rand(S, Hkv, Tq, B, generator=g, device=DEV).topk(nprobe, dim=-1).indices.to(torch.int32).contiguous()
        jobs.append((rand(S, Tq, Hq, 128), K, V, Ks, Vs, off, ln, idx, sel, pos0, 1, 200, scale))
    want = [saap.prefill_sparse_attention(*j) for j in jobs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in jobs]
    got = [[], []]
    for _ in range(20):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[i].append(saap.prefill_sparse_attention(*jobs[i]))
    torch.cuda.synchronize()
    for w, results in zip(want, got):
        for r in results:
            assert torch.equal(r[0], w[0]) and torch.equal(r[1], w[1])


@pytest.mark.gpu
def test_two_threads_on_one_stream_give_what_one_gives():
    """Calls of several launches on the default workspace, from two threads on the same stream."""
    import threading
    S, Hkv, R, N, B, scale = 1, 2, 64, 3000, 32, 1 / math.sqrt(128)
    g = torch.Generator(device=DEV).manual_seed(4)
    rand = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)  # noqa: E731
    K, q, xq = rand(S, Hkv, N, 128), rand(2, S, Hkv, R, 128), rand(2, 64, Hkv, 128)
    ids = torch.randint(0, B, (S, Hkv, N), generator=g, device=DEV, dtype=torch.int32)
    off, ln, _, Ks, _ = saap.build_bucket_index(ids, K, K, B)
    W1, W2 = rand(Hkv, 64, 128) / 11, rand(Hkv, B, 64) / 8

    def once(i):
        mass, lse = saap.bucket_attention_mass_batch(q[i], Ks, off, ln, scale)
        return mass, lse, saap.classify_queries(xq[i], W1, None, W2, None, Hkv)
    want = [once(i) for i in range(2)]
    torch.cuda.synchronize()
    got = [[], []]
    threads = [threading.Thread(target=lambda i=i: got[i].extend(once(i) for _ in range(50))) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for w, results in zip(want, got):
        assert len(results) == 50
        for r in results:
            assert all(torch.equal(a, b) for a, b in zip(r, w))
