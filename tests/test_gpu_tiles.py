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
