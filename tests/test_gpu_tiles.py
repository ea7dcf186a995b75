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
                                       (64, 4160, 32, 1024, 8)])
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
