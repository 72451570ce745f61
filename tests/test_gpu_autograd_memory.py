"""The differentiable render keeps no step's buffers once its outputs are dropped (no cycle through the
autograd node that only the garbage collector would free)."""
from __future__ import annotations

import gc

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import custom_scene, make_scene

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


def test_outputs_are_freed_with_their_last_reference():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_14737_amd as fmb
    sc, cams = custom_scene(12, [(32, 32)], seed=3)
    scene, _ = make_scene(fmb, torch, sc, cams, np.array([W.BETA1, W.BETA2], np.float32), 1.0, DEV)
    ps = [torch.as_tensor(a, device=DEV).clone().requires_grad_() for a in
          (sc.means, sc.prec, sc.weights, np.array([W.BETA1, W.BETA2], np.float32))]

    def step():
        depth, alpha, *_ = fmb.render(scene, *ps)
        torch.autograd.grad(depth.sum() + alpha.sum(), ps)

    step()
    torch.cuda.synchronize()
    gc.collect()
    gc.disable()
    try:
        before = torch.cuda.memory_allocated()
        for _ in range(3):
            step()
        assert torch.cuda.memory_allocated() <= before
    finally:
        gc.enable()
