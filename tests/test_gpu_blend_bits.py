"""The blend forward's depths to the last bit: the sign of an L1 depth loss, and the flow, follow it.

tests/golden/blend_forward.npz holds the depths of two scenes of 100 Gaussians, four crops of a 640 x 480 frame
each, as the first tiled form of the kernel rendered them: per ray a running maximum that starts at the
first weight, sums in scene order.  (Rays that see nothing denser than 2^-48 may add their pairs in another
order; these crops hold none that it changes.)"""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import custom_scene, make_scene

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "blend_forward.npz")


@pytest.mark.parametrize("seed", [0, 1])
def test_depth_bits(seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_14737_amd as fmb
    sc, cams = custom_scene(100, [(32, 40)] * 4, seed=seed, s_range=(0.05, 0.2))
    for v, (x, y) in enumerate(((0, 0), (60, -40), (-90, 70), (120, 100))):
        cams.intr[v] = [480.0, 480.0, 20.0 - x, 16.0 - y]
    scene, _ = make_scene(fmb, torch, sc, cams, np.array([W.BETA1, W.BETA2], np.float32), 1.0, DEV)
    got = scene.render(normals=True)["depth"].cpu().numpy()
    with np.load(GOLDEN) as golden:
        want = golden[f"seed{seed}"]
    assert int((got.view(np.int32) != want.view(np.int32)).sum()) == 0, float(np.abs(got - want).max())
