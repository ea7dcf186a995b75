"""Tile kernels at the sizes where they can go wrong (tile edges, remainders, one K slice, the
line between two tile shapes) against the CPU oracle and float64 products (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_01024_amd as pcm
from workloads import CONFIGS, make_inputs, scaled

from test_gpu_parity import assert_y_close, dev, poison, run_layer, say

pytestmark = pytest.mark.gpu
DEV = "cuda"


# float32: 64 x 64 tiles from 768 expected tiles on, 32 x 64 below; K slices of 32 values
@pytest.mark.parametrize("T,H,n,F,k", [(1, 64, 1, 64, 1), (31, 64, 1, 192, 1), (33, 128, 3, 64, 2),
                                       (130, 192, 5, 448, 3), (700, 320, 6, 2112, 4),
                                       (64, 4160, 32, 1024, 8), (9, 64, 12, 1088, 8)])
def test_f32_layer_tiles(T, H, n, F, k):
    cfg = scaled(CONFIGS["tiny"], T=T, H=H, n=n, F=F, k=k, x_std=1.0, logits="normal", name=f"f32_{T}_{H}")
    say(f"float32 tiles {cfg.name}")
    inp = make_inputs(cfg, seed=41)
    d = dev(inp)
    plan = pcm.LayerPlan(T, H, F, n, k, torch.float32, DEV)
    poison(plan)
    y = plan.forward(d["x"], d["logits"], d["mask"], d["w_gate"], d["w_up"], d["w_down"])
    torch.cuda.synchronize()
    assert_y_close(y.cpu().numpy(), oracle.layer_inputs(inp), "f32", cfg.name)


@pytest.mark.parametrize("T", [1, 63, 65, 3000])
def test_f32_dense_swiglu_accumulate(T):
    """One group of rows, and accumulation into y: exactly the stored values added."""
    cfg = scaled(CONFIGS["finegrained_shared"], T=T, H=192, F=64, shared_F=1088, dtype="f32", name=f"dense{T}")
    say(f"float32 dense {T}")
    inp = make_inputs(cfg, seed=42)
    d = dev(inp)
    base = torch.randn((T, cfg.H), device=DEV)
    y0 = pcm.pcm_dense_swiglu(d["x"], *d["shared"])
    y = pcm.pcm_dense_swiglu(d["x"], *d["shared"], y=base.clone(), accumulate=True)
    torch.cuda.synchronize()
    assert_y_close(y0.cpu().numpy(), oracle.dense_swiglu(inp.x, inp.s_gate, inp.s_up, inp.s_down), "f32", cfg.name)
    assert torch.equal(y, base + y0)


# router GEMM: one launch (32-token workgroups, all experts) or two (16 x 16 blocks, K slices);
# token and expert remainders, every count of 64-expert groups, one 64-wide K slice, and tokens on
# both sides of the line between the two forms
@pytest.mark.parametrize("T,H,n,k", [(2048, 2048, 64, 8), (1024, 2048, 64, 8), (4129, 64, 33, 3),
                                     (5001, 192, 100, 8), (4097, 832, 130, 5), (3001, 1024, 256, 8),
                                     (17, 7168, 256, 8), (5, 64, 1, 1), (1, 4096, 8, 2)])
def test_router_forms(T, H, n, k):
    from test_gpu_parity import check_route_logits
    say(f"router T={T} H={H} n={n}")
    g = torch.Generator().manual_seed(T + n)
    x = torch.randn((T, H), generator=g).to(torch.bfloat16)
    wr = (torch.randn((n, H), generator=g) * 0.02).to(torch.bfloat16)
    check_route_logits(x, wr, k, f"T={T} H={H} n={n} k={k}")


# The two-launch router adds in one order: chains of `steps` 32-wide K steps (about 2048 waves share the
# steps), then their sums in ascending order. Each step here holds one non-zero product, an integer below
# 2^14 times its chain's power of two, so that a chain of up to 2^9 steps is exact and float32 additions
# of the chains, whose scales differ, give every bit.
@pytest.mark.parametrize("T,H,n", [(24, 2048, 64), (1, 4096, 8), (17, 7168, 256), (200, 2048, 64), (256, 1088, 33),
                                   (40, 192, 130), (700, 2048, 64)])
def test_router_sum_order(T, H, n):
    say(f"router order T={T} H={H} n={n}")
    g = torch.Generator().manual_seed(T + H)
    KT = H // 32
    want = min(max(-(-2048 // (-(-n // 16) * -(-T // 16))), 1), KT)
    steps = -(-KT // want)
    wr = torch.randint(-127, 128, (n, H), generator=g).float()
    at = torch.arange(KT) * 32 + torch.randint(0, 32, (T, KT), generator=g)
    scale = 2.0 ** -torch.randint(0, 24, (T, KT), generator=g)[:, torch.arange(KT) // steps * steps].float()
    v = torch.randint(-127, 128, (T, KT), generator=g).float() * scale
    x = torch.zeros((T, H)).scatter_(1, at, v)
    lg = pcm.pcm_route_logits(x.to(DEV, torch.bfloat16), wr.to(DEV, torch.bfloat16), 1, want_logits=True)[2]
    torch.cuda.synchronize()
    prod = v.numpy()[:, :, None] * wr.numpy().T[at.numpy()]     # [T, KT, n]
    ref = np.zeros((T, n), np.float32)
    for s in range(0, KT, steps):
        ref += prod[:, s:s + steps].sum(1, dtype=np.float32)    # exact in any order
    assert (lg.cpu().numpy() == ref).all(), int((lg.cpu().numpy() != ref).sum())


# The one-launch router folds its sums every few K slices, so its rounding error against 64 bits stays at
# that of the two launches, which add partial sums of K slices (chains of 51 MFMA steps at H 6528, 1000
# tokens: error about sqrt(51 / 2); folded, chains of 14 steps and 15 of them, sqrt(14 / 2 + 15 / 2); one
# chain of 204 steps would show twice the two launches' error). A quarter is left for the sample. H = 256
# and 320: one slice per chain, the fewest.
@pytest.mark.parametrize("T,H,n", [(2018, 6528, 181), (2400, 4096, 64), (4129, 320, 100), (4129, 256, 256)])
def test_router_fold_error(T, H, n):
    say(f"router fold T={T} H={H} n={n}")
    g = torch.Generator().manual_seed(H)
    x = torch.randn((T, H), generator=g).to(torch.bfloat16)
    wr = (torch.randn((n, H), generator=g) * 0.02).to(torch.bfloat16)
    ref = x.double() @ wr.double().T
    xd, wd = x.to(DEV), wr.to(DEV)
    one = pcm.pcm_route_logits(xd, wd, 1, want_logits=True)[2]
    two = pcm.pcm_route_logits(xd[:1000].contiguous(), wd, 1, want_logits=True)[2]
    torch.cuda.synchronize()

    def error(lg):
        r = ref[:lg.shape[0]]
        return float((lg.cpu().double() - r).norm() / r.norm())
    e1, e2 = error(one), error(two)
    print(f"  one launch {e1:.2e}, two {e2:.2e}", flush=True)
    # (24 bits: results that are all exact up to their last rounding leave 2^-24 / sqrt(3))
    assert e1 <= max(1.25 * e2, 2.0 ** -24), (e1, e2)


# one group of rows (the shared expert) on the shapes that pick_shape chooses between: streaming with
# slices shared by the waves (rows 1 to 64 per tile, 17 and 33 and 49 start another block; several row tiles where N is small), 64-row ring tiles (row and
# column remainders), large tiles; K = 512 and 448 are the two sides of the split's line
@pytest.mark.parametrize("T,H,Fs", [(1, 512, 512), (16, 448, 576), (17, 576, 1088), (33, 1024, 640), (49, 1024, 1600),
                                    (64, 2048, 512), (40, 2112, 2176), (64, 2112, 2176), (65, 2048, 512), (128, 1024, 1984), (300, 1024, 2112),
                                    (1000, 576, 2048), (2500, 320, 320)])
def test_dense_swiglu_shapes(T, H, Fs):
    cfg = scaled(CONFIGS["finegrained_shared"], T=T, H=H, F=64, shared_F=Fs, name=f"dense{T}")
    say(f"dense T={T} H={H} Fs={Fs}")
    inp = make_inputs(cfg, seed=43)
    d = dev(inp)
    sg, su, sd = d["shared"]
    ws = torch.full((pcm.workspace_bytes(3, T, H, Fs, 1, 1, 1),), 0xFF, dtype=torch.uint8, device=DEV)
    base = torch.randn((T, H), device=DEV)
    ref = oracle.dense_swiglu(inp.x, inp.s_gate, inp.s_up, inp.s_down)
    y0 = torch.full((T, H), float("nan"), device=DEV)
    for down in (sd, pcm.pcm_widen_f16(sd)):
        pcm.pcm_dense_swiglu(d["x"], sg, su, down, y=y0, ws=ws)
        y = pcm.pcm_dense_swiglu(d["x"], sg, su, down, y=base.clone(), accumulate=True, ws=ws)
        torch.cuda.synchronize()
        assert_y_close(y0.cpu().numpy(), ref, "bf16", cfg.name)
        assert torch.equal(y, base + y0), "accumulate adds the stored values"


# grouped rows: streaming with slices shared by the waves (below 16 rows per expert; 16-row tiles, 32-row from a mean of
# 4 on, several tiles in one expert), ring tiles, and a K split of the projection on the ring; the last
# three: top-8 mixes whose last wave has few columns (path weights are read from lanes past them)
@pytest.mark.parametrize("T,H,n,F,k,logits", [(1, 1024, 64, 2048, 8, "normal"), (3, 4096, 8, 2112, 2, "normal"),
                                              (40, 1024, 8, 2048, 2, "normal+one_expert"),
                                              (200, 1088, 60, 2048, 4, "zipf"), (130, 512, 16, 576, 4, "zipf"),
                                              (70, 320, 4, 4096, 1, "normal"), (257, 192, 5, 1088, 2, "normal"),
                                              (900, 256, 3, 1536, 2, "normal"), (5, 128, 16, 1088, 8, "normal"),
                                              (7, 64, 10, 4160, 8, "normal"), (6, 64, 9, 8256, 8, "normal")])
def test_layer_shapes(T, H, n, F, k, logits):
    cfg = scaled(CONFIGS["olmoe"], T=T, H=H, n=n, F=F, k=k, logits=logits, zipf_s=1.1, name=f"shape{T}_{H}")
    say(f"layer shapes {cfg.name}")
    inp = make_inputs(cfg, seed=44)
    d = dev(inp)
    plan = pcm.LayerPlan(T, H, F, n, k, torch.bfloat16, DEV)
    ref = oracle.layer_inputs(inp)
    ys = []
    for down in (d["w_down"], pcm.pcm_widen_f16(d["w_down"])):
        poison(plan)
        y = plan.forward(d["x"], d["logits"], d["mask"], d["w_gate"], d["w_up"], down)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy().copy())
        assert_y_close(ys[-1], ref, "bf16", cfg.name)
    assert np.array_equal(ys[0], ys[1]), "bf16 and widened projection weights give the same bits"
    if R_mean(cfg) >= 16:   # no split of K beyond the large tiles' own: the same sums in the same order
        y = run_layer(d, k, tuning=pcm.Tuning(tile="L"))
        assert np.array_equal(y, ys[0]), "the default and the large tiles"


# Whatever the default kernels are, every sum over K runs in one order: that of the streaming kernel whose
# waves keep to themselves and of the register ring. Expansions share slices from H = 4096, projections
# from F = 2048 (16-row tiles, 32-row from a mean of 4 on; K slices that the four waves share out unevenly).
@pytest.mark.parametrize("T,H,n,F,k", [(1, 1024, 64, 2048, 8), (3, 4096, 8, 2112, 2), (40, 1088, 8, 2176, 2),
                                       (24, 2048, 64, 1024, 8), (17, 1152, 12, 2240, 8), (2, 1216, 3, 2048, 1),
                                       (2, 4160, 3, 2112, 1), (9, 4224, 3, 2048, 2), (17, 4288, 12, 64, 8)])
def test_streaming_sum_order(T, H, n, F, k):
    cfg = scaled(CONFIGS["olmoe"], T=T, H=H, n=n, F=F, k=k, logits="normal", name=f"order{T}_{H}")
    say(f"streaming sum order {cfg.name}")
    d = dev(make_inputs(cfg, seed=45))
    y = run_layer(d, k)
    for depth in (0, 2):
        assert np.array_equal(y, run_layer(d, k, tuning=pcm.Tuning(tile="S", stream_depth=depth))), depth


# The same for one group of rows, by the medium tiles: every row count per tile of one and of two column
# blocks per workgroup (two from 257 workgroups on: N = 4160; 2112: rows in tiles of 16 to 64), in the expansion (Fs) and in the projection
# (H), K slices shared out unevenly; the oracle and accumulation too.
@pytest.mark.parametrize("T", [1, 16, 17, 33, 48, 49, 64])
@pytest.mark.parametrize("H,Fs", [(512, 4160), (576, 4160), (640, 2112), (2112, 704), (4160, 512), (4160, 704), (704, 832)])
def test_dense_swiglu_sum_order(T, H, Fs):
    cfg = scaled(CONFIGS["finegrained_shared"], T=T, H=H, F=64, shared_F=Fs, name=f"dense{T}")
    say(f"dense sum order T={T} H={H} Fs={Fs}")
    inp = make_inputs(cfg, seed=46)
    d = dev(inp)
    base = torch.randn((T, H), device=DEV)
    y0 = torch.full((T, H), float("nan"), device=DEV)
    pcm.pcm_dense_swiglu(d["x"], *d["shared"], y=y0)
    y = pcm.pcm_dense_swiglu(d["x"], *d["shared"], y=base.clone(), accumulate=True)
    m = pcm.pcm_dense_swiglu(d["x"], *d["shared"], tuning=pcm.Tuning(tile="M"))
    torch.cuda.synchronize()
    assert_y_close(y0.cpu().numpy(), oracle.dense_swiglu(inp.x, inp.s_gate, inp.s_up, inp.s_down), "bf16", cfg.name)
    assert torch.equal(y, base + y0), "accumulate adds the stored values"
    assert torch.equal(y0, m), "the default and the medium tiles"


def R_mean(cfg):
    return cfg.T * cfg.k // cfg.n


# Weights of more than half of the 256 MB MALL are read non-temporally by the groups of a single row tile:
# the large tiles on four and eight waves and the 64-row ring tiles (means of 20, 50 and 100 rows; skewed,
# with groups of one and of several row tiles in a call). One order of the sums (F / 2 is no multiple of 64,
# so the projection takes one slice of K).
@pytest.mark.parametrize("T,logits", [(80, "normal"), (200, "zipf"), (400, "normal")])
def test_nontemporal_weights(T, logits):
    H, n, F, k = 2048, 8, 4160, 2
    assert 2 * n * F * H * 2 > 128 << 20 and n * F * H * 2 > 128 << 20   # gate and up, down
    cfg = scaled(CONFIGS["mixtral"], T=T, H=H, n=n, F=F, k=k, logits=logits, zipf_s=1.1, name=f"nt{T}")
    say(f"non-temporal weights {cfg.name}")
    inp = make_inputs(cfg, seed=47)
    d = dev(inp)
    y = run_layer(d, k)
    assert_y_close(y, oracle.layer_inputs(inp), "bf16", cfg.name)
    for tile in ("S", "M", "L", "W"):
        say(f"tile {tile}")
        assert np.array_equal(y, run_layer(d, k, tuning=pcm.Tuning(tile=tile))), tile


# path build of up to 256 tokens: one thread per (token, slot), at most two each
@pytest.mark.parametrize("beta_mode", [0, 1, 2])
@pytest.mark.parametrize("T,n,k", [(1, 8, 8), (128, 256, 8), (129, 9, 8), (255, 64, 5), (256, 256, 8), (200, 1, 1)])
def test_build_paths_small(T, n, k, beta_mode):
    from test_gpu_parity import check_paths
    rng = np.random.default_rng(T + n)
    lg = torch.from_numpy(rng.standard_normal((T, n)).astype(np.float32)).to(DEV)
    ids, w = pcm.pcm_route(lg, k)
    check_paths(ids, w, (rng.random((n, n)) < 0.4).astype(np.uint8), n, beta_mode)


# scored route: every score equal (more than a wave of pairs reach the bound), more than 256 pairs per
# lane, 4 and 16 waves per token, and dispatches that sum the count table themselves (up to 16384
# tokens) or scan it
@pytest.mark.parametrize("T,n,K,d,equal", [(600, 64, 8, 1.0, True), (40, 64, 8, 1.0, True), (520, 256, 8, 1.0, False),
                                           (33, 256, 8, 1.0, False), (512, 96, 7, 0.5, False), (512, 97, 7, 0.5, False),
                                           (16384, 8, 2, 0.5, False), (16400, 8, 2, 0.5, False)])
def test_route_scored_branches(T, n, K, d, equal):
    from test_gpu_scored import check_route
    rng = np.random.default_rng(T + n)
    z = (lambda *s: np.zeros(s, np.float32)) if equal else (lambda *s: rng.standard_normal(s).astype(np.float32))
    mask = (rng.random((n, n)) < d).astype(np.uint8)
    check_route(z(T, n), z(T, n), 0.5, z(n, n), mask, K, f"T={T} n={n} K={K}")
