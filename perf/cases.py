"""What a program built on this library has it do, as cases that can be timed and compared.

Five paths: a decode step ("decode"), the indexing of a prompt ("prefill"), sparse attention for a block of
prompt tokens ("block"), a training step of the query model ("train") and the k-means that makes the centroids
("kmeans").  Inputs have the shapes and the structure of the library's workloads: per KV head the keys are a
Gaussian mixture (centres N(0,4I), within-component sigma 1) plus one shared offset of norm 20, the queries come
from another mixture without the offset, values are N(0,I), classifiers are random-init.
"""
import math

import torch

import paper_2502_08246_amd as saap

D = 128                       # features per head, the only size the library takes
DEV = "cuda:0"
SCALE = 1.0 / math.sqrt(D)
N_SINK, N_RECENT = 1, 2047    # the dense block of the paper's default setting
ROW_BYTES = {"f32": 4 * D, "bf16": 2 * D, "fp8": D}
MAX_KEYS = 8 * 131072         # keys per KV head, over all sequences, of the largest prefill


def _decode(name, **kw):
    case = dict(name=name, path="decode", S=1, Hq=32, Hkv=8, N=131072, B=1024, hidden=512, nprobe=51, skew=False,
                dtype="bf16", route="separate", store="none", layers=1, graph=False)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: one fp32 head over a short context; launches and host time are all there is
        _decode("decode_tiny_f32", Hq=1, Hkv=1, N=4096, B=64, hidden=256, nprobe=8, dtype="f32"),
        # one token of one layer of a Llama-3.1-8B-shaped model at 128k, called from Python as it comes
        _decode("decode_128k"),
        # a serving loop: one token through several layers, each with its own cache, replayed as a HIP graph
        _decode("decode_128k_8_layers_graph", layers=8, graph=True),
        # the longest context, buckets of very unequal sizes, 5 % of the keys
        _decode("decode_500k_skewed", N=500000, B=4096, nprobe=205, skew=True),
        # batched decoding; every step also stores the token's keys in their buckets
        _decode("decode_batch8_append", S=8, store="append"),
        # the paper's default setting: sink and recent keys always attended, the token's key enters the window
        _decode("decode_128k_window", route="attend", store="window"),
        # the largest decode launch: 32 sequences on an 8-bit cache, selection inside the attention launch
        _decode("decode_batch32_fp8", S=32, dtype="fp8", route="attend"),
        # a short prompt of odd length gets its index
        dict(name="prefill_short_ragged", path="prefill", S=1, Hkv=8, N=5003, B=128, slack=8, dtype="bf16", window=False,
             kv8=False),
        # prompts of a batch are indexed with room for the tokens to come
        dict(name="prefill_batch8_128k", path="prefill", S=8, Hkv=8, N=131072, B=1024, slack=64, dtype="bf16",
             window=False, kv8=False),
        # the last block of a long prompt: routing of every token, then sparse attention for the block
        dict(name="block_128_of_128k", path="block", S=1, Hq=32, Hkv=8, N=131072, Tq=128, B=1024, hidden=512, nprobe=51),
        # one iteration of the query model's training: target rows for the batch, loss and gradients, Adam
        dict(name="train_1000_queries", path="train", Hkv=8, R=1000, N=131072, B=1024, hidden=512),
        # spherical k-means over a sample of the keys of every head
        dict(name="kmeans_64k_samples", path="kmeans", Hkv=8, N=65536, B=1024, iters=2),
    ]


# ------------------------------------------------------------------------------------------ drawn cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _buckets(rng, N, most=4096):
    """A bucket holds 32 to 256 keys on average; the classifier wants a multiple of 16."""
    b = N / math.exp(rng.uniform(math.log(32), math.log(256)))
    return max(16, min(most, 16 * int(round(b / 16))))


def _probe(rng, B):
    """1 to 12 % of the buckets."""
    return max(1, int(round(B * math.exp(rng.uniform(math.log(0.01), math.log(0.12))))))


def _heads(rng):
    return rng.choice([(32, 8), (32, 8), (32, 8), (64, 8), (16, 8), (8, 8), (4, 1), (16, 4), (1, 1)])


def _draw_decode(rng):
    Hq, Hkv = _heads(rng)
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp8", "fp8", "f32"])
    N = _log_int(rng, 1000, 32768 if dtype == "f32" else 500000)
    S = min(_log_int(rng, 1, 32), max(1, 32 * 131072 // N))
    graph = rng.random() < 0.3
    layers = min(_log_int(rng, 1, 8), max(1, 8 * 131072 // (S * N))) if graph else 1
    if dtype == "f32":
        S = min(S, 4)
    B = _buckets(rng, N)
    store = rng.choice(["none", "none", "append", "window"])
    if layers > 1 or S * N > MAX_KEYS:
        store = "none"
    route = "separate" if dtype == "fp8" and store == "window" else rng.choice(["separate", "attend"])
    return dict(path="decode", S=S, Hq=Hq, Hkv=Hkv, N=N, B=B, hidden=32 * rng.randint(2, 16), nprobe=_probe(rng, B),
                skew=rng.random() < 0.3, dtype=dtype, route=route, store=store, layers=layers, graph=graph)


def _draw_prefill(rng):
    f32 = rng.random() < 0.15
    N = _log_int(rng, 1000, 8192 if f32 else 500000)
    S = 1 if f32 else min(_log_int(rng, 1, 8), max(1, MAX_KEYS // N))
    B = _buckets(rng, N, 4096 if S * N <= MAX_KEYS // 4 else 1024)
    return dict(path="prefill", S=S, Hkv=rng.choice([1, 4, 8, 8]), N=N, B=B, slack=rng.choice([0, 8, 64]),
                dtype="f32" if f32 else "bf16", window=rng.random() < 0.3, kv8=rng.random() < 0.3)


def _draw_block(rng):
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (64, 8), (8, 8), (16, 4)])
    S = rng.choice([1, 1, 2, 4])
    N = _log_int(rng, 8192, 131072)
    B = _buckets(rng, N, 1024)
    return dict(path="block", S=S, Hq=Hq, Hkv=Hkv, N=N, Tq=_log_int(rng, 16, 4096 // (S * Hkv)), B=B,
                hidden=32 * rng.randint(2, 16), nprobe=min(_probe(rng, B), 64))


def _draw_train(rng):
    N = _log_int(rng, 4096, 131072)
    return dict(path="train", Hkv=rng.choice([1, 4, 8, 8]), R=_log_int(rng, 64, 1024), N=N, B=_buckets(rng, N, 1024),
                hidden=32 * rng.randint(2, 16))


def _draw_kmeans(rng):
    N = _log_int(rng, 4096, 131072)
    return dict(path="kmeans", Hkv=rng.choice([1, 4, 8, 8]), N=N, B=_buckets(rng, N, 1024), iters=rng.choice([1, 2, 3]))


def draw(rng):
    kind = rng.choice([_draw_decode] * 6 + [_draw_prefill] * 2 + [_draw_block, _draw_train, _draw_kmeans])
    return kind(rng)


# ------------------------------------------------------------------------------------------ inputs
class _Mixture:
    """One layer's key distribution: B components per KV head, the heads' shared offsets, component weights."""

    def __init__(self, gen, Hkv, B, skew):
        self.gen, self.Hkv, self.B = gen, Hkv, B
        self.centres = 2.0 * self.randn(Hkv, B, D)
        offset = self.randn(Hkv, 1, D)
        self.offset = 20.0 * offset / offset.norm(dim=-1, keepdim=True)
        if skew:       # one draw of Dirichlet(0.3): Gamma(0.3) variates, Gamma(1.3) * U^(1/0.3)
            u = torch.rand(Hkv, B, generator=gen, device=DEV).clamp_min(1e-6)
            gamma = self._gamma(1.3, (Hkv, B)) * u.pow(1.0 / 0.3)
            self.weights = gamma / gamma.sum(-1, keepdim=True)
        else:
            self.weights = torch.full((Hkv, B), 1.0 / B, device=DEV)

    def randn(self, *shape):
        return torch.randn(*shape, generator=self.gen, device=DEV)

    def _gamma(self, shape, size):
        """Wilson-Hilferty's cubed normal, close enough to a Gamma variate for drawing weights."""
        z = self.randn(*size)
        return (shape * (1 - 1 / (9 * shape) + z / math.sqrt(9 * shape)).clamp_min(0.05).pow(3)).clamp_min(1e-6)

    def components(self, n):
        """Component of each of n keys per head: [Hkv,n] int64."""
        cdf = self.weights.cumsum(-1)
        u = torch.rand(self.Hkv, n, generator=self.gen, device=DEV) * cdf[:, -1:]
        return torch.searchsorted(cdf, u).clamp_max(self.B - 1)

    def keys(self, comp, dtype):
        """Keys [Hkv,n,D] of the given components."""
        out = torch.empty(*comp.shape, D, dtype=dtype, device=DEV)
        for h in range(self.Hkv):
            out[h] = (self.centres[h][comp[h]] + self.randn(comp.shape[1], D) + self.offset[h]).to(dtype)
        return out

    def values(self, n, dtype):
        out = torch.empty(self.Hkv, n, D, dtype=dtype, device=DEV)
        for h in range(self.Hkv):
            out[h] = self.randn(n, D).to(dtype)
        return out

    def centroids(self, dtype):
        """Unit vectors along the components' means: what spherical k-means finds on such keys."""
        c = self.centres + self.offset
        return (c / c.norm(dim=-1, keepdim=True)).to(dtype).contiguous()


def _queries(gen, shape, dtype):
    """Rows of the query mixture: centre N(0,4I) plus N(0,I), no offset."""
    return (math.sqrt(5.0) * torch.randn(*shape, D, generator=gen, device=DEV)).to(dtype)


def _classifier(gen, Hw, hidden, B, dtype):
    W1 = (torch.randn(Hw, hidden, D, generator=gen, device=DEV) / math.sqrt(D)).to(dtype)
    W2 = (torch.randn(Hw, B, hidden, generator=gen, device=DEV) / math.sqrt(hidden)).to(dtype)
    b1 = 0.05 * torch.randn(Hw, hidden, generator=gen, device=DEV)
    b2 = 0.05 * torch.randn(Hw, B, generator=gen, device=DEV)
    return W1, b1, W2, b2


def _layer(case, gen):
    """One layer as decoding finds it: classifier, the bucket-sorted cache with its index, the token's vectors."""
    S, Hq, Hkv, N, B = (case[k] for k in ("S", "Hq", "Hkv", "N", "B"))
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    mix = _Mixture(gen, Hkv, B, case["skew"])
    slack = 0 if case["store"] == "none" else 64
    parts = []
    for _ in range(S):
        comp = mix.components(N)
        ids = comp.to(torch.int32).unsqueeze(0)
        K, V = mix.keys(comp, dtype).unsqueeze(0), mix.values(N, dtype).unsqueeze(0)
        if case["store"] == "window":
            index = saap.build_windowed_index(ids, K, V, B, slack, N_SINK, N_RECENT)
        else:
            index = saap.build_bucket_index(ids, K, V, B, slack)
        if case["dtype"] == "fp8":
            index = index[:3] + saap.quantize_kv(index[3], index[4]) + index[5:]
        parts.append(index)
        del K, V
    index = parts[0] if S == 1 else [torch.cat(t) for t in zip(*parts)]
    del parts
    L = dict(zip(("off", "len", "idx", "Ks", "Vs"), index[:5]))
    L["scales"] = tuple(index[5:7]) if case["dtype"] == "fp8" else ()
    L["resident_ids"] = index[-1].contiguous() if case["store"] == "window" else None
    L["classifier"] = _classifier(gen, Hkv, case["hidden"], B, dtype)
    L["xq"], L["q"] = _queries(gen, (S, Hq), dtype), _queries(gen, (S, Hq), dtype)
    if case["store"] != "none":
        L["centroids"] = mix.centroids(dtype)
        L["x_new"] = torch.stack([mix.keys(mix.components(1), dtype)[:, 0] for _ in range(S)])
        L["k_new"], L["v_new"] = L["x_new"].roll(1, -1).contiguous(), mix.randn(S, Hkv, D).to(dtype)
        L["pos_new"] = torch.full((S,), N, dtype=torch.int32, device=DEV)
        L["len_before"] = L["len"].clone()
        L["flag"] = torch.zeros(4, dtype=torch.int32, device=DEV)
    return L


def _decode_layer(case, L):
    """One token of one layer: route, attend and, where generation stores its keys, store the token's key."""
    Hkv, nprobe, fp8, window = case["Hkv"], case["nprobe"], case["dtype"] == "fp8", case["store"] == "window"
    resident = case["B"] if window else -1
    if case["store"] != "none":
        # the bucket lengths as before the token (what a rejected draft token leaves behind), so that a pass can
        # be repeated without filling the slack
        L["len"].copy_(L["len_before"])
    logits = saap.classify_queries(L["xq"], *L["classifier"], Hkv, output_kind=saap.LOGITS)
    index = (L["Ks"], L["Vs"]) + L["scales"] + (L["off"], L["len"])
    if case["route"] == "attend":
        if fp8:
            selected, out, lse = saap.select_attend_fp8(logits, L["q"], *index, nprobe, SCALE)
        else:
            selected, out, lse = saap.select_attend(logits, L["q"], *index, nprobe, SCALE, resident_run=resident)
    else:
        selected = saap.select_buckets_from_logits(logits, Hkv, nprobe)
        if window:
            attend = saap.windowed_decode_attention_fp8 if fp8 else saap.windowed_decode_attention
            out, lse = attend(L["q"], *index, selected, resident, SCALE)
        else:
            attend = saap.sparse_decode_attention_fp8 if fp8 else saap.sparse_decode_attention
            out, lse = attend(L["q"], *index, selected, SCALE)
    result = {"logits": logits, "selected": selected, "out": out, "lse": lse}
    if case["store"] != "none":
        rows = (L["x_new"], L["k_new"], L["v_new"], L["pos_new"], L["centroids"], None, L["off"], L["len"], L["idx"],
                L["Ks"], L["Vs"]) + L["scales"]
        if window:
            push = saap.window_push_fp8 if fp8 else saap.window_push
            new_ids, flag = push(*rows, L["resident_ids"], N_SINK, N_RECENT, overflow_flag=L["flag"])
            result["resident_ids"] = L["resident_ids"]
        else:
            append = saap.append_keys_fp8 if fp8 else saap.append_keys
            new_ids, flag = append(*rows, overflow_flag=L["flag"])
        result.update(new_ids=new_ids, flag=flag, len=L["len"], idx=L["idx"], Ks=L["Ks"], Vs=L["Vs"])
    return result


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 17)
    path, state = case["path"], {"case": case}
    if path == "decode":
        state["layers"] = [_layer(case, gen) for _ in range(case["layers"])]
        if case["graph"]:
            for L in state["layers"]:
                _decode_layer(case, L)                 # workspaces exist before the capture
            torch.cuda.synchronize()
            state["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(state["graph"]):
                state["results"] = [_decode_layer(case, L) for L in state["layers"]]
    elif path == "prefill":
        S, Hkv, N = case["S"], case["Hkv"], case["N"]
        dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        mix = _Mixture(gen, Hkv, case["B"], False)
        state["x"], state["K"], state["V"] = (torch.empty(S, Hkv, N, D, dtype=dtype, device=DEV) for _ in range(3))
        for s in range(S):
            state["x"][s] = mix.keys(mix.components(N), dtype)
            state["K"][s] = state["x"][s].roll(1, -1)
            state["V"][s] = mix.values(N, dtype)
        state["centroids"] = mix.centroids(dtype)
    elif path == "block":
        S, Hq, Hkv, N, Tq, B = (case[k] for k in ("S", "Hq", "Hkv", "N", "Tq", "B"))
        mix = _Mixture(gen, Hkv, B, False)
        comp = torch.stack([mix.components(N) for _ in range(S)])
        state["K"] = torch.stack([mix.keys(comp[s], torch.bfloat16) for s in range(S)])
        state["V"] = torch.stack([mix.values(N, torch.bfloat16) for _ in range(S)])
        state["index"] = saap.build_bucket_index(comp.to(torch.int32).contiguous(), state["K"], state["V"], B, 0)
        state["classifier"] = _classifier(gen, Hkv, case["hidden"], B, torch.bfloat16)
        state["xq"], state["q"] = _queries(gen, (S, Tq, Hq), torch.bfloat16), _queries(gen, (S, Tq, Hq), torch.bfloat16)
        state["pos0"] = torch.full((S,), N - Tq, dtype=torch.int32, device=DEV)
    elif path == "train":
        Hkv, R, N, B = case["Hkv"], case["R"], case["N"], case["B"]
        mix = _Mixture(gen, Hkv, B, False)
        comp = mix.components(N)
        K = mix.keys(comp, torch.bfloat16).unsqueeze(0)
        state["off"], state["len"], _, state["Ks"], _ = saap.build_bucket_index(comp.to(torch.int32).unsqueeze(0), K, K, B, 0)
        state["q"] = _queries(gen, (1, Hkv, R), torch.bfloat16)
        state["x"] = state["q"][0].roll(1, -1).contiguous()
        W1, b1, W2, b2 = _classifier(gen, Hkv, case["hidden"], B, torch.float32)
        state["params"] = (W1, b1, W2, b2)
        state["m"] = tuple(torch.zeros_like(p) for p in state["params"])
        state["v"] = tuple(torch.zeros_like(p) for p in state["params"])
        state["grads"] = tuple(torch.empty_like(p) for p in state["params"])
        state["step"] = 0
    else:
        mix = _Mixture(gen, case["Hkv"], case["B"], False)
        x = mix.keys(mix.components(case["N"]), torch.bfloat16)
        first = x[:, :case["B"]].float()
        state["x"] = x.unsqueeze(0)
        state["centroids"] = (first / first.norm(dim=-1, keepdim=True)).to(torch.bfloat16).contiguous()
    return state


def run(state):
    case = state["case"]
    path = case["path"]
    if path == "decode":
        if case["graph"]:
            state["graph"].replay()
            results = state["results"]
        else:
            results = [_decode_layer(case, L) for L in state["layers"]]
        return results[0] if len(results) == 1 else results
    if path == "prefill":
        ids = saap.assign_keys(state["x"], state["centroids"])
        if case["window"]:
            off, ln, idx, Ks, Vs, resident = saap.build_windowed_index(ids, state["K"], state["V"], case["B"], case["slack"],
                                                                       N_SINK, N_RECENT)
        else:
            off, ln, idx, Ks, Vs = saap.build_bucket_index(ids, state["K"], state["V"], case["B"], case["slack"])
            resident = None
        result = {"ids": ids, "off": off, "len": ln, "idx": idx, "Ks": Ks, "Vs": Vs, "resident_ids": resident}
        if case["kv8"]:
            result["K8"], result["V8"], result["kscale"], result["vscale"] = saap.quantize_kv(Ks, Vs)
        return result
    if path == "block":
        S, Hq, Hkv, Tq, nprobe = (case[k] for k in ("S", "Hq", "Hkv", "Tq", "nprobe"))
        logits = saap.classify_queries(state["xq"].view(S * Tq, Hq, D), *state["classifier"], Hkv, output_kind=saap.LOGITS)
        lists = saap.select_buckets_from_logits(logits, Hkv, nprobe)
        lists = lists.view(S, Tq, Hkv, nprobe).permute(0, 2, 1, 3).contiguous()
        off, ln, idx, Ks, Vs = state["index"]
        out, lse = saap.prefill_sparse_attention(state["q"], state["K"], state["V"], Ks, Vs, off, ln, idx, lists, state["pos0"],
                                                 N_SINK, N_RECENT, SCALE)
        return {"lists": lists, "out": out, "lse": lse}
    if path == "train":
        state["step"] += 1
        target, lse = saap.bucket_attention_mass_batch(state["q"], state["Ks"], state["off"], state["len"], SCALE)
        loss, grads = saap.query_model_loss_grads(state["x"], target[0], state["params"], grads=state["grads"])
        for p, g, m, v in zip(state["params"], grads, state["m"], state["v"]):
            saap.adam_update(p, g, m, v, state["step"], 1e-5)
        return {"target": target, "lse": lse, "loss": loss, "grads": grads, "params": state["params"], "m": state["m"],
                "v": state["v"]}
    return saap.lloyd_iterations(state["x"], state["centroids"], case["iters"])


# ------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    path = case["path"]
    if path == "decode":
        S, Hq, Hkv, N, B, hidden, nprobe = (case[k] for k in ("S", "Hq", "Hkv", "N", "B", "hidden", "nprobe"))
        row = ROW_BYTES[case["dtype"]]
        elem = 4 if case["dtype"] == "f32" else 2
        dense = min(N, N_SINK + N_RECENT) if case["store"] == "window" else 0
        keys = S * Hkv * (dense + (N - dense) * nprobe / B)
        nbytes = Hkv * (D * hidden + hidden * B) * elem + 2 * row * keys + 2 * S * Hq * D * elem + 4 * S * Hq * (D + 1)
        flops = 2 * S * Hq * (D * hidden + hidden * B) + 4 * D * (Hq // Hkv) * keys
        if case["store"] != "none":
            nbytes += Hkv * B * D * elem + S * Hkv * (3 * D * elem + 2 * row)
            flops += 2 * S * Hkv * B * D
        return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * flops}
    if path == "prefill":
        S, Hkv, N, B = case["S"], case["Hkv"], case["N"], case["B"]
        row = ROW_BYTES[case["dtype"]]
        keys = S * Hkv * N
        free = S * Hkv * B * case["slack"]             # free slots are written too: they come back as zeros
        nbytes = keys * (row + 4) + Hkv * B * row + keys * 4 * row + free * 2 * row + 4 * (keys + free)
        if case["kv8"]:
            nbytes += (keys + free) * 2 * D
        return {"bytes": nbytes, "flops": 2 * keys * B * D}
    if path == "block":
        S, Hq, Hkv, N, Tq, B, hidden, nprobe = (case[k] for k in ("S", "Hq", "Hkv", "N", "Tq", "B", "hidden", "nprobe"))
        dense = min(N, N_SINK + N_RECENT)
        pairs = S * Hkv * Tq * (dense + (N - dense) * nprobe / B)      # (token, key) pairs
        touched = S * Hkv * (dense + Tq + (N - dense) * (1 - (1 - nprobe / B) ** Tq))     # keys some token attends
        nbytes = touched * 4 * D + Hkv * (D * hidden + hidden * B) * 2 + S * Tq * Hq * (4 * D + 4 * D + 4)
        return {"bytes": nbytes, "flops": 2 * S * Tq * Hq * (D * hidden + hidden * B) + 4 * D * (Hq // Hkv) * pairs}
    if path == "train":
        Hkv, R, N, B, hidden = case["Hkv"], case["R"], case["N"], case["B"], case["hidden"]
        params = Hkv * (hidden * D + hidden + B * hidden + B)
        nbytes = Hkv * N * 2 * D + Hkv * R * (4 * D + 4 * B + 4) + 4 * params * 7
        return {"bytes": nbytes, "flops": 2 * Hkv * R * N * D + Hkv * R * (4 * D * hidden + 6 * hidden * B)}
    Hkv, N, B = case["Hkv"], case["N"], case["B"]
    return {"bytes": case["iters"] * Hkv * (N * 2 * D + B * 4 * D), "flops": case["iters"] * Hkv * N * (2 * B * D + D)}


def tolerance(case):
    path = case["path"]
    if path == "prefill":
        return "exact"                                  # ids, positions, copied rows and codes
    if path == "train":
        # fp32 sums over up to 1024 terms; the targets are exponentials of fp32 scores of magnitude 10 to 30
        return {"rel": 1e-4, "max": 1e-2}
    if path == "kmeans":
        return {"rel": 3e-3, "max": 0.1}                # centroids are rounded to bf16
    # lists: an fp32 logit may round differently where two buckets score alike.  Attention: fp32 caches throughout in
    # fp32; bf16 and 8-bit caches weigh values with bf16 parts on the matrix cores
    if case.get("dtype") == "f32":
        return {"rel": 2e-5, "differ": 1e-2}
    return {"rel": 2e-3, "differ": 1e-2}
