"""The compositing forward's outputs to the last bit: the sign of an L1 loss follows it, so a render that
moves by rounding turns a cotangent of a ray whose value meets its target, and with it a gradient.

tests/golden/composite_forward.npz holds depth, alpha, normals and colours of two small scenes (40 Gaussians;
128 dense ones, whose tiles take several depth windows) as the first one-wave-per-item form of the kernel
rendered them; weights are sums of logarithms in scene order there, whatever the cut of the work, so
every later form of the kernel for scenes of at most 128 Gaussians gives the same bits."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import custom_scene, make_scene

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "composite_forward.npz")


@pytest.mark.parametrize("n,view,scales", [(40, (24, 24), (0.05, 0.2)), (128, (16, 24), (0.1, 0.3))], ids=["n40", "n128"])
def test_forward_bits(n, view, scales):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_14737_amd as fmb
    sc, cams = custom_scene(n, [view], seed=900 + n, s_range=scales)
    scene, _ = make_scene(fmb, torch, sc, cams, np.array([W.BETA1, W.BETA2], np.float32), 1.0, DEV)
    scene.set_model("composite")
    q = (1.5 * np.random.Generator(np.random.PCG64(n)).standard_normal((n, 3))).astype(np.float32)
    colors = torch.as_tensor(q, device=DEV)
    scene.set_colors(colors)
    out = scene.render(normals=True, color=True)
    torch.cuda.synchronize()
    with np.load(GOLDEN) as golden:
        for k in ("depth", "alpha", "normal", "color"):
            want = golden[f"n{n}_{k}"]
            got = out[k].cpu().numpy()
            differ = int((got.view(np.int32) != want.view(np.int32)).sum())
            assert differ == 0, (k, differ, float(np.abs(got - want).max()))
