"""The work a program has this library do, as measurable cases: expert layers of a decode
step, of a prompt's prefill and of a small all-fp32 model, stacks of layers, and the gating
and batching around an expert FFN that the program runs itself.

Shapes (d, f, E, k): the Mixtral-shaped layer (4096, 14336, 8, 2), the 16-expert layer
(4096, 6400, 16, 2), a generic layer of many small experts (2048, 1408, 64, 6) and the tiny
all-fp32 layer (256, 512, 8, 2).  Expert matrices are N(0, 1/fan_in), activations N(0, 1),
router logits N(0, 1), with `zipf` > 0 skewed by the log of a Zipf pmf over the experts
(expert 0 hottest), as router outputs are in earnest."""
import math

import numpy as np
import torch

import paper_2402_07033_amd as moe

MIXTRAL = dict(d=4096, f=14336, E=8, k=2, w="bf16")
SIXTEEN = dict(d=4096, f=6400, E=16, k=2, w="bf16")
SIXTYFOUR = dict(d=2048, f=1408, E=64, k=6, w="bf16")
TINY = dict(d=256, f=512, E=8, k=2, w="f32")
EPS = 1e-5


def listed():
    return [
        # the smallest calls: the tiny all-fp32 layer through the four boundary calls, where
        # launches and latency are everything
        dict(name="tiny_fp32", kind="calls", T=16, x="f32", zipf=0.0, layers=1, **TINY),
        # single-batch decoding, one token per step: every active expert's matrices read once
        dict(name="decode_t1", kind="decode", T=1, x="f32", zipf=0.0, layers=1, **MIXTRAL),
        # a few concurrent sequences on smaller experts (odd token count, ragged row counts)
        dict(name="decode_e16_t5", kind="decode", T=5, x="f32", zipf=1.2, layers=1, **SIXTEEN),
        # beam search, width 16: the largest decode step
        dict(name="beam_t16", kind="decode", T=16, x="f32", zipf=1.2, layers=1, **MIXTRAL),
        # single-batch decoding through consecutive blocks (norm, router, experts, residual)
        dict(name="stack_t1", kind="stack", T=1, x="f32", zipf=0.0, layers=4, **MIXTRAL),
        # a short prompt of odd length: tens of rows per expert
        dict(name="prompt_t77", kind="layer", T=77, x="f32", zipf=1.2, layers=1, **MIXTRAL),
        # a chunk of a prompt on many small experts
        dict(name="chunk_e64_t300", kind="layer", T=300, x="bf16", zipf=0.0, layers=1, **SIXTYFOUR),
        # a whole transformer block's expert part on a 512-token prompt
        dict(name="block_t512", kind="stack", T=512, x="f32", zipf=0.0, layers=1, **MIXTRAL),
        # a prompt of odd length, compute and weight traffic both in sight
        dict(name="prefill_t1531", kind="layer", T=1531, x="bf16", zipf=1.2, layers=1, **MIXTRAL),
        # the longest prefill step
        dict(name="prefill_t4096", kind="layer", T=4096, x="bf16", zipf=1.2, layers=1, **MIXTRAL),
        # the same on the 16-expert layer
        dict(name="prefill_e16_t4096", kind="layer", T=4096, x="bf16", zipf=1.2, layers=1, **SIXTEEN),
        # gating, batching and combine of a prefill step around a program's own expert FFN
        dict(name="gating_t4096", kind="gating", T=4096, x="bf16", zipf=1.2, layers=1, **MIXTRAL),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["calls", "decode", "decode", "layer", "layer", "layer", "layer", "stack",
                       "gating"])
    zipf = rng.choice([0.0, 0.6, 1.2])
    if kind == "calls":
        return dict(kind=kind, T=_log_int(rng, 1, 128), x="f32", zipf=zipf, layers=1,
                    d=64 * rng.randint(2, 8), f=64 * rng.randint(4, 16), E=rng.randint(2, 8), k=2,
                    w="f32")
    if kind == "decode":
        return dict(kind=kind, T=rng.randint(1, 16), x="f32", zipf=zipf, layers=1,
                    **rng.choice([MIXTRAL, SIXTEEN]))
    if kind == "layer":
        shape = rng.choice([MIXTRAL, MIXTRAL, SIXTEEN, SIXTYFOUR])
        return dict(kind=kind, T=_log_int(rng, 17, 4096), x=rng.choice(["bf16", "f32"]), zipf=zipf,
                    layers=1, **shape)
    if kind == "stack":
        small = rng.random() < 0.5
        return dict(kind=kind, T=rng.randint(1, 4) if small else _log_int(rng, 32, 1024), x="f32",
                    zipf=0.0, layers=rng.randint(2, 4) if small else 1,
                    **rng.choice([MIXTRAL, SIXTEEN]))
    return dict(kind=kind, T=_log_int(rng, 64, 8192), x=rng.choice(["bf16", "f32"]), zipf=zipf,
                layers=1, **rng.choice([MIXTRAL, SIXTYFOUR]))


# ---- inputs ----------------------------------------------------------------------------

def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _normal(gen, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000 + stream)
    return g


def _expert_matrices(case, seed, layer):
    g, dt = _generator(seed, 100 + layer), _dtype(case["w"])
    d, f, E = case["d"], case["f"], case["E"]
    return (_normal(g, (E, d, f), d ** -0.5, dt), _normal(g, (E, d, f), d ** -0.5, dt),
            _normal(g, (E, f, d), f ** -0.5, dt))


def _log_pmf(case):
    p = np.arange(1, case["E"] + 1, dtype=np.float64) ** -case["zipf"]
    return np.log(p / p.sum())


def _tokens(case, seed):
    """Token rows and router logits of a single layer."""
    g = _generator(seed, 1)
    x = _normal(g, (case["T"], case["d"]), 1.0, _dtype(case["x"]))
    logits = _normal(g, (case["T"], case["E"]), 1.0, torch.float32)
    return x, logits + torch.from_numpy(_log_pmf(case).astype(np.float32)).cuda()


def _router_matrix(case, seed, layer):
    return _normal(_generator(seed, 50 + layer), (case["d"], case["E"]), case["d"] ** -0.5,
                   torch.float32)


def _expert_rows(case, seed):
    """What a program's own expert FFN leaves: one row per (token, expert), in expert order."""
    return _normal(_generator(seed, 2), (case["T"] * case["k"], case["d"]), 1.0, torch.float32)


def _index_buffers(case):
    i32 = dict(dtype=torch.int32, device="cuda")
    T, E, k = case["T"], case["E"], case["k"]
    return dict(idx=torch.empty((T, k), **i32),
                w=torch.empty((T, k), dtype=torch.float32, device="cuda"),
                out=(torch.empty(E, **i32), torch.empty(E + 1, **i32), torch.empty(T * k, **i32),
                     torch.empty(T * k, **i32)))


def prepare(case, seed):
    T, d, f, E, k = (case[n] for n in ("T", "d", "f", "E", "k"))
    f32 = dict(dtype=torch.float32, device="cuda")
    st = dict(case=case)
    if case["kind"] == "gating":
        st["x"], st["logits"] = _tokens(case, seed)
        st["yg"] = _expert_rows(case, seed)
        st.update(_index_buffers(case))
        st["xg"] = torch.empty((T * k, d), dtype=st["x"].dtype, device="cuda")
        st["y"] = torch.empty((T, d), **f32)
        return st
    packed = []
    for layer in range(case["layers"]):
        packed.append(moe.moe_weights_pack(*_expert_matrices(case, seed, layer)))
    if case["kind"] == "stack":
        st["layers"] = [(W, _router_matrix(case, seed, n)) for n, W in enumerate(packed)]
        st["x"] = _tokens(case, seed)[0]
        st["bufs"] = moe.StackBuffers(T, E, k, d, f)
        return st
    st["W"] = packed[0]
    st["x"], st["logits"] = _tokens(case, seed)
    if case["kind"] == "calls":
        return st
    st.update(_index_buffers(case))
    act = moe.MOE_BF16 if case["x"] == "bf16" else moe.MOE_F32
    st["ws"] = torch.empty(moe.moe_expert_ffn_workspace(T * k, E, d, f, act), dtype=torch.uint8,
                           device="cuda")
    st["y"] = torch.empty((T, d), **f32)
    if case["kind"] == "layer":
        st["yg"] = torch.empty((T * k, d), **f32)
    return st


# ---- one pass --------------------------------------------------------------------------

def run(state):
    case = state["case"]
    k, kind = case["k"], case["kind"]
    if kind == "calls":
        out = moe.moe_layer(state["W"], state["x"], state["logits"], k)
        return dict(y=out["y"], idx=out["idx"], w=out["w"])
    if kind == "decode":
        out = moe.moe_decode_layer(state["W"], state["x"], state["logits"], k, idx=state["idx"],
                                   weights=state["w"], out=state["out"] + (None,),
                                   workspace=state["ws"], y=state["y"])
        return dict(y=out["y"], idx=out["idx"], w=out["w"])
    if kind == "stack":
        x = state["x"].clone()  # the residual stream, updated in place
        return moe.moe_stack_forward(state["layers"], x, k, EPS, bufs=state["bufs"])
    idx, w = moe.moe_route(state["logits"], k, state["idx"], state["w"])
    if kind == "layer":
        _, offsets, perm, inv_perm, _ = moe.moe_permute(idx, case["E"], None,
                                                        out=state["out"] + (None,))
        yg = moe.moe_expert_ffn_tokens(state["W"], state["x"], k, perm, offsets,
                                       workspace=state["ws"], yg=state["yg"])
        return dict(y=moe.moe_combine(yg, inv_perm, w, state["y"]), idx=idx, w=w)
    counts, offsets, perm, inv_perm, xg = moe.moe_permute(idx, case["E"], state["x"],
                                                          out=state["out"] + (state["xg"],))
    y = moe.moe_combine(state["yg"], inv_perm, w, state["y"])
    return dict(y=y, idx=idx, w=w, counts=counts, offsets=offsets, perm=perm, inv_perm=inv_perm,
                xg=xg)


# ---- what a pass cannot do without, and what its outputs may be off by -----------------

def _active_experts(case):
    """Experts that get at least one token, on average over draws of the router logits."""
    T, E, k = case["T"], case["E"], case["k"]
    if T == 1 or T * k >= 64 * E:
        return float(min(E, T * k))
    rng = np.random.default_rng(7)
    n = []
    for _ in range(32):
        lg = rng.standard_normal((T, E)) + _log_pmf(case)[None, :]
        n.append(len(np.unique(np.argsort(-lg, axis=1)[:, :k])))
    return float(np.mean(n))


def work(case):
    T, d, f, E, k, L = (case[n] for n in ("T", "d", "f", "E", "k", "layers"))
    N = T * k
    xb = 2 if case["x"] == "bf16" else 4
    wb = 2 if case["w"] == "bf16" else 4
    index = T * E * 4 + 2 * N * 4
    if case["kind"] == "gating":
        return {"bytes": index + 2 * N * 4 + T * d * xb + N * d * xb + N * d * 4 + T * d * 4,
                "flops": 2 * N * d}
    experts = _active_experts(case) * 3 * d * f * wb
    flops = 6 * N * d * f + 2 * N * d
    if case["kind"] == "stack":
        return {"bytes": L * (experts + d * E * 4) + 2 * T * d * 4,
                "flops": L * (flops + 2 * T * d * E)}
    return {"bytes": experts + index + T * d * xb + T * d * 4, "flops": flops}


def tolerance(case):
    """Relative 2-norm errors against 64-bit arithmetic, about four times what the path shows
    where that is set by the data types: fp32 throughout (6e-7 measured); up to 72 routed rows
    the activations and the intermediate kept as bf16 pairs (4.3e-6); bf16 activations and
    intermediate beyond (1.7e-3 with bf16 rows, 2.9e-3 with fp32 rows)."""
    if case["w"] == "f32" or case["kind"] == "gating":
        return {"rel": 5e-6}
    if case["T"] * case["k"] <= 72:
        return {"rel": 2e-5}
    return {"rel": 1e-2}


# ---- the same in 64 bits, without the library -------------------------------------------

def _route64(logits, k):
    lg = logits.double()
    idx = torch.sort(lg, dim=1, descending=True, stable=True)[1][:, :k]
    return idx, torch.softmax(torch.gather(lg, 1, idx), dim=1)


def _layer64(x, idx, w, mats):
    w1, w3, w2 = mats
    y = torch.zeros((x.shape[0], w1.shape[1]), dtype=torch.float64, device="cuda")
    for e in range(w1.shape[0]):
        tok, slot = torch.nonzero(idx == e, as_tuple=True)
        if tok.numel() == 0:
            continue
        a = x[tok]
        h = torch.nn.functional.silu(a @ w1[e].double()) * (a @ w3[e].double())
        y.index_add_(0, tok, (h @ w2[e].double()) * w[tok, slot, None])
    return y


def exact(case, seed):
    k = case["k"]
    if case["kind"] == "stack":
        x = _tokens(case, seed)[0].double()
        for n in range(case["layers"]):
            h = x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS)
            idx, w = _route64(h @ _router_matrix(case, seed, n).double(), k)
            x = x + _layer64(h, idx, w, _expert_matrices(case, seed, n))
        return x
    x, logits = _tokens(case, seed)
    idx, w = _route64(logits, k)
    if case["kind"] != "gating":
        y = _layer64(x.double(), idx, w, _expert_matrices(case, seed, 0))
        return dict(y=y, idx=idx.int(), w=w)
    flat = idx.reshape(-1)
    perm = torch.sort(flat, stable=True)[1]
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(perm.numel(), device="cuda")
    counts = torch.bincount(flat, minlength=case["E"])
    offsets = torch.cat([counts.new_zeros(1), torch.cumsum(counts, 0)])
    rows = _expert_rows(case, seed).double()[inv].reshape(case["T"], k, case["d"])
    return dict(y=(rows * w[:, :, None]).sum(dim=1), idx=idx.int(), w=w, counts=counts.int(),
                offsets=offsets.int(), perm=perm.int(), inv_perm=inv.int(),
                xg=x[torch.div(perm, k, rounding_mode="floor")].double())
