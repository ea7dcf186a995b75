"""The calls that a user of this framework makes, at the sizes they make them, for timing and
comparing two builds of it: listed() names twelve, draw() gives more of the same ranges,
prepare() makes what a program holds before the call (inputs, weights, plan), run() is one call
through the public entry points, exact() the same result in float64 by plain torch.

The layer shapes are those of workloads/configs.py (Mixtral-, OLMoE-, fine-grained- and
decode-shaped, and the float32 one), generic ones beside them; the distributions are the
workloads' (hidden states N(0, 1), weights N(0, 0.02), logits by shape)."""
import math

import torch

import paper_2609_01024_amd as pcm
from paper_2609_01024_amd import binding
from paper_2609_01024_amd.stack import random_stack

DEV = "cuda"

# (H, n, F, k, mask density, logits, shared F, most tokens)
FAMILIES = {
    "mixtral": (4096, 8, 14336, 2, 0.5, "normal_bias", 0, 4096),
    "olmoe": (2048, 64, 1024, 8, 0.25, "zipf", 0, 8192),
    "finegrained": (2048, 60, 1408, 4, 0.3, "normal", 5632, 16384),
    "decode": (7168, 256, 2048, 8, 0.2, "normal", 0, 32),
}


def family(name, kind, T, **more):
    H, n, F, k, density, logits, shared_F, _ = FAMILIES[name]
    c = dict(kind=kind, T=T, H=H, n=n, F=F, k=k, dtype="bf16", density=density, logits=logits,
             shared_F=shared_F, down="f16", beta=0)
    c.update(more)
    return c


def listed():
    return [
        # the float32 layer of the tests and the benchmark: 64 tokens, bound by its launches
        dict(name="f32 small layer", kind="layer", T=64, H=256, n=8, F=512, k=2, dtype="f32",
             density=0.5, logits="normal", shared_F=0, down="f32", beta=0),
        # a float32 layer with a few hundred ragged tokens (float32 checks of a model, small models)
        dict(name="f32 ragged layer", kind="layer", T=777, H=768, n=16, F=960, k=4, dtype="f32",
             density=0.3, logits="normal", shared_F=0, down="f32", beta=2),
        # prefill at the three large shapes; the first is the benchmark's headline
        dict(family("mixtral", "layer", 4096), name="mixtral prefill"),
        dict(family("olmoe", "layer", 8192), name="olmoe prefill"),
        dict(family("finegrained", "layer", 16384), name="fine-grained prefill, shared expert"),
        # one step of a decode batch at the widest layer: streams the weights of most experts
        dict(family("decode", "layer", 32), name="decode batch 32"),
        # a handful of sequences decoding on the Mixtral shape, bf16 projection weights
        dict(family("mixtral", "layer", 3, down="bf16"), name="mixtral decode batch 3"),
        # a mid-size batch (chunked prefill, speculative decoding): 50 rows per expert
        dict(family("mixtral", "layer", 203), name="mixtral batch 203"),
        # the scored compositional router, the one used at inference, on a ragged prefill chunk
        dict(family("olmoe", "scored", 3001), name="olmoe scored prefill 3001"),
        # a decode step through a stack of layers with its own router GEMMs and residuals
        dict(family("olmoe", "stack", 24, L=4, logits="router", down="bf16"), name="olmoe stack decode 24"),
        # the always-on shared expert alone at a decode-size batch
        dict(kind="dense", T=48, H=2048, shared_F=5632, dtype="bf16", down="f16",
             name="shared expert batch 48"),
        # the router's GEMM and top-k, as a layer's first step at prefill
        dict(kind="router", T=8192, H=2048, n=64, k=8, dtype="bf16", name="router gemm 8192"),
    ]


def spread(rng, lo, hi):
    """An integer of [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "scored", "generic", "f32", "dense", "router", "stack"])
    down = rng.choice(["bf16", "f16"])
    if kind in ("layer", "scored"):
        name = rng.choice(sorted(FAMILIES))
        return family(name, kind, spread(rng, 1, FAMILIES[name][7]), down=down,
                      beta=rng.choice([0, 0, 1, 2]) if kind == "layer" else 0)
    if kind in ("generic", "f32"):
        f32 = kind == "f32"
        n = spread(rng, 2, 32 if f32 else 128)
        return dict(kind=rng.choice(["layer", "layer", "scored"]), T=spread(rng, 8, 1024 if f32 else 4096),
                    H=64 * spread(rng, 3, 12 if f32 else 48), n=n, F=64 * spread(rng, 3, 16 if f32 else 40),
                    k=rng.randint(1, min(n, 4 if f32 else 8)), dtype="f32" if f32 else "bf16",
                    density=round(rng.uniform(0.1, 0.8), 2), logits=rng.choice(["normal", "zipf"]), shared_F=0,
                    down="f32" if f32 else down, beta=0)
    if kind == "dense":
        return dict(kind="dense", T=spread(rng, 1, 8192), H=64 * spread(rng, 8, 48), shared_F=64 * spread(rng, 8, 100),
                    dtype="bf16", down=down)
    if kind == "router":
        n = spread(rng, 4, 256)
        return dict(kind="router", T=spread(rng, 1, 16384), H=64 * spread(rng, 4, 112), n=n,
                    k=rng.randint(1, min(n, 8)), dtype="bf16")
    return family("olmoe", "stack", spread(rng, 1, 256), L=rng.randint(1, 4), logits="router", down="bf16",
                  k=rng.randint(2, 8))


# ------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype).mul_(std)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _logits(case, g):
    T, n = case["T"], case["n"]
    l = _randn(g, (T, n), 1.0, torch.float32)
    if case["logits"] == "normal_bias":
        l = l + _randn(g, (n,), 0.5, torch.float32)
    elif case["logits"] == "zipf":
        rank = torch.randperm(n, generator=g, device=DEV) + 1
        l = l - 1.1 * torch.log(rank.to(torch.float32))
    return l.contiguous()


def _inputs(case, seed):
    """The tensors of a case, by name."""
    g, dt = _gen(seed), _dtype(case)
    d = {"x": _randn(g, (case["T"], case["H"]), 1.0, dt)}
    H, Fs = case["H"], case.get("shared_F", 0)
    if case["kind"] == "router":
        d["wr"] = _randn(g, (case["n"], H), 0.02, dt)
        return d
    if Fs:
        d["shared"] = (_randn(g, (Fs, H), 0.02, dt), _randn(g, (Fs, H), 0.02, dt), _randn(g, (H, Fs), 0.02, dt))
    if case["kind"] == "dense":
        return d
    n, F = case["n"], case["F"]
    d["logits"] = _logits(case, g)
    mask = (torch.rand((n, n), generator=g, device=DEV) < case["density"]).to(torch.uint8)
    d["mask"] = mask.fill_diagonal_(1)
    if case["kind"] == "scored":   # the initialisation of the compatibility bias and the target prior
        bias = torch.rand((n, n), generator=g, device=DEV) - 1.5
        d["bias"] = bias.fill_diagonal_(0.0)
        d["g_tgt"] = _randn(g, (case["T"], n), 1.0, torch.float32)
        d["lam"] = 0.5
    d["w_gate"] = _randn(g, (n, F, H), 0.02, dt)
    d["w_up"] = _randn(g, (n, F, H), 0.02, dt)
    d["w_down"] = _randn(g, (n, H, F), 0.02, dt)
    return d


def _stack(case, seed):
    st = random_stack(case["L"], case["T"], case["H"], case["F"], case["n"], case["k"], case["density"],
                      seed, DEV, native_layers=1)
    return st, _randn(_gen(seed + 1), (case["T"], case["H"]), 1.0, torch.bfloat16)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "stack":
        st, x = _stack(case, seed)
        return {"kind": kind, "stack": st, "x": x, "h": torch.empty_like(x)}
    d = _inputs(case, seed)
    s = {"kind": kind, "case": case, "d": d}
    if kind == "router":
        T, n, k = case["T"], case["n"], case["k"]
        s["ids"] = torch.empty((T, k), dtype=torch.int32, device=DEV)
        s["w"] = torch.empty((T, k), dtype=torch.float32, device=DEV)
        s["logits"] = torch.empty((T, n), dtype=torch.float32, device=DEV)
        s["ws"] = torch.empty((pcm.workspace_bytes(binding.OP_ROUTE_LOGITS, T, case["H"], 0, n, k, pcm.PCM_BF16),),
                              dtype=torch.uint8, device=DEV)
        return s
    if case["down"] == "f16":      # projection weights widened once per layer
        if "w_down" in d:
            d["w_down"] = pcm.pcm_widen_f16(d["w_down"])
        if "shared" in d:
            d["shared"] = d["shared"][:2] + (pcm.pcm_widen_f16(d["shared"][2]),)
    T, H = case["T"], case["H"]
    if kind == "dense":
        s["y"] = torch.empty((T, H), dtype=torch.float32, device=DEV)
        s["ws"] = torch.empty((pcm.workspace_bytes(binding.OP_DENSE_SWIGLU, T, H, case["shared_F"], 1, 1, pcm.PCM_BF16),),
                              dtype=torch.uint8, device=DEV)
        return s
    sizes = (T, H, case["F"], case["n"], case["k"], _dtype(case), DEV, case["shared_F"])
    if kind == "scored":
        s["plan"] = pcm.ScoredLayerPlan(*sizes)
        s["plan"].build_layout(d["mask"], d["bias"])   # once per layer
    else:
        s["plan"] = pcm.LayerPlan(*sizes, beta_mode=case["beta"])
        s["packed"] = pcm.pcm_mask_pack(d["mask"])     # once per layer
    return s


def run(s):
    kind = s["kind"]
    if kind == "stack":
        return s["stack"].forward(s["h"].copy_(s["x"]))
    d = s["d"]
    if kind == "router":
        ids, w, logits = pcm.pcm_route_logits(d["x"], d["wr"], s["case"]["k"], s["logits"], s["ids"], s["w"],
                                              want_logits=True, ws=s["ws"])
        return {"ids": ids, "w": w, "logits": logits}
    if kind == "dense":
        return pcm.pcm_dense_swiglu(d["x"], *d["shared"], y=s["y"], ws=s["ws"])
    if kind == "scored":
        return s["plan"].forward(d["x"], d["logits"], d["g_tgt"], d["lam"], d["w_gate"], d["w_up"],
                                 d["w_down"], d.get("shared"))
    return s["plan"].forward(d["x"], d["logits"], s["packed"], d["w_gate"], d["w_up"], d["w_down"],
                             d.get("shared"))


# ------------------------------------------------------------ work and tolerance
def _touched(n, k, T):
    """Experts that T tokens with k of n each are expected to reach."""
    return n * (1.0 - (1.0 - k / n) ** T)


def work(case):
    kind, T, H = case["kind"], case["T"], case["H"]
    size = 2 if case["dtype"] == "bf16" else 4
    if kind == "router":
        n, k = case["n"], case["k"]
        return {"bytes": size * (T * H + n * H) + 4 * T * n + 8 * T * k, "flops": 2 * T * n * H}
    Fs = case.get("shared_F", 0)
    b, f = size * T * H + 4 * T * H + size * 3 * H * Fs, 6 * T * H * Fs   # x, y, the shared expert
    if kind == "dense":
        return {"bytes": b, "flops": f}
    n, F, k = case["n"], case["F"], case["k"]
    layers = case.get("L", 1)
    b += layers * (size * 3 * H * F * _touched(n, k, T) + n * n)
    b += layers * size * n * H if kind == "stack" else 4 * T * n * (2 if kind == "scored" else 1)
    f += layers * 6 * T * k * H * F
    if kind == "scored":
        # distinct sources are fewer than paths by an amount that the inputs decide: count half
        # of the expansion
        f -= 2 * T * k * H * F
    return {"bytes": int(b), "flops": int(f)}


def tolerance(case):
    # about four times the error measured against exact(): bf16 layers carry the projection input
    # as float16 (2.1e-4 at every shape), float32 layers 6e-7 to 9e-7, the router 4e-7, with near
    # ties of its logits in another order. The stack rounds its hidden states to bf16 between
    # layers, where one different rounding can move a near-tie of the next router.
    if case["kind"] == "stack":
        return {"rel": 1e-2}
    if case["kind"] == "router":
        return {"rel": 2e-6, "differ": 5e-4}
    return {"rel": 8e-4, "max": 1e-2} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 1e-4}


# -------------------------------------------------------------- float64 reference
def _swiglu64(x, wg, wu):
    g = x @ wg.double().T
    return torch.nn.functional.silu(g) * (x @ wu.double().T)


def _topk64(logits, k):
    v, i = torch.sort(logits, dim=1, descending=True, stable=True)   # ties to the lower expert
    return i[:, :k], torch.softmax(v[:, :k].double(), dim=1)


def _beta64(p, on, mode):
    """Path weights [T, k, k] of allowed paths `on` from the slot weights p [T, k]."""
    pair = p[:, :, None] * p[:, None, :] * on
    if mode == 1:
        return pair
    den = (p[:, None, :] * on).sum(2, keepdim=True) if mode == 0 else pair.sum((1, 2), keepdim=True)
    return pair / den


def _experts64(x, d, ids, beta, y, sources=None):
    """y[t] += sum over (a, b) of beta[t, a, b] D_(ids[t, b]) U_(sources[t, a]) x_t."""
    T, k = ids.shape
    sources = ids if sources is None else sources
    U = x.new_empty((T, k, d["w_gate"].shape[1]))
    for e in range(d["w_gate"].shape[0]):
        t, a = (sources == e).nonzero(as_tuple=True)
        if t.numel():
            U[t, a] = _swiglu64(x[t], d["w_gate"][e], d["w_up"][e])
    z = torch.empty_like(U)
    for b in range(k):
        z[:, b] = (beta[:, :, b, None] * U).sum(1)
    del U
    for e in range(d["w_down"].shape[0]):
        t, b = (ids == e).nonzero(as_tuple=True)
        if t.numel():
            y.index_put_((t,), z[t, b] @ d["w_down"][e].double().T, accumulate=True)


def _scored64(case, d):
    """Per selected path: source, target and weight [T, k]. Scores are compared in float32, as the
    router forms them: one rounding of g_base + bias, one of the fused multiply-add."""
    n, k = case["n"], case["k"]
    flat = torch.nonzero(d["mask"].reshape(-1)).reshape(-1)   # active pairs in ascending order
    src, tgt, w = [], [], []
    for t0 in range(0, case["T"], 256):
        gb, gt = d["logits"][t0:t0 + 256], d["g_tgt"][t0:t0 + 256]
        base = gb[:, flat // n] + d["bias"].reshape(-1)[flat]
        s = (d["lam"] * gt[:, flat % n].double() + base.double()).float()
        v, i = torch.sort(s, dim=1, descending=True, stable=True)
        p = flat[i[:, :k]]
        src.append(p // n)
        tgt.append(p % n)
        w.append(torch.softmax(v[:, :k].double(), dim=1))
    return torch.cat(src), torch.cat(tgt), torch.cat(w)


def exact(case, seed):
    kind = case["kind"]
    if kind == "stack":
        return None     # hidden states are rounded to bf16 between its layers
    d = _inputs(case, seed)
    x = d["x"].double()
    if kind == "router":
        logits = x @ d["wr"].double().T
        return {"ids": None, "w": _topk64(logits, case["k"])[1], "logits": logits}
    y = torch.zeros_like(x)
    if "shared" in d:
        wg, wu, wd = d["shared"]
        for t0 in range(0, case["T"], 4096):
            y[t0:t0 + 4096] = _swiglu64(x[t0:t0 + 4096], wg, wu) @ wd.double().T
    if kind == "dense":
        return y
    if kind == "scored":
        src, tgt, w = _scored64(case, d)
        _experts64(x, d, tgt, torch.diag_embed(w), y, sources=src)
    else:
        ids, p = _topk64(d["logits"], case["k"])
        on = d["mask"][ids[:, :, None], ids[:, None, :]] != 0
        _experts64(x, d, ids, _beta64(p, on, case["beta"]), y)
    return y
