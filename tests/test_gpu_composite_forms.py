"""The compositing kernels' two forms (four waves sharing a staged scene of at most 128 Gaussians; one
wave per tile with the tile's survivors staged) at the sizes where they meet, alone and mixed in one
batch: each scene of the batch equals its own launches bit for bit and the FP64 oracle to the
contract's tolerances."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import assert_forward, assert_grads, compare_forward, compare_grads, custom_scene, hit_mask_cot

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
BETAS = np.array([W.BETA1, W.BETA2], np.float32)


@pytest.fixture(scope="module")
def fmb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_14737_amd as m
    return m


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV).contiguous()


# (Gaussians, views, scale range): the two forms' meeting point; survivors below and above one staged tile
SETS = {
    "edge": [(127, [(40, 33)], (0.05, 0.2)), (128, [(17, 24), (8, 8)], (0.05, 0.2)), (129, [(24, 31)], (0.05, 0.2))],
    "survivors": [(33, [(64, 64)], (0.05, 0.2)), (500, [(48, 40)], (0.01, 0.05)), (260, [(16, 24)], (0.1, 0.3))],
}


@pytest.mark.parametrize("label", list(SETS))
def test_forms_alone_and_mixed(fmb, label):
    parts = [custom_scene(n, views, seed=400 + n, s_range=s) for n, views, s in SETS[label]]
    scenes, camsl = [p[0] for p in parts], [p[1] for p in parts]
    cat = lambda k: _t(np.concatenate([getattr(s, k) for s in scenes]))  # noqa: E731
    means, prec, weights = cat("means"), cat("prec"), cat("weights")
    betas = _t(np.tile(BETAS, (len(scenes), 1)))
    cams = [fmb.Cameras.from_numpy(c.w2c, c.intr, c.hw, device=DEV) for c in camsl]
    b = fmb.Batch(means, prec, weights, betas, [1.0] * len(scenes), [s.n for s in scenes], cams)
    b.set_model("composite")
    print(f"[forms] {label}: N={[s.n for s in scenes]} P={b.n_rays}", flush=True)
    outs = b.forward(b.alloc_outputs(normals=True))
    refs = [O.render_workload_view(s, c, BETAS, 1.0, model="composite")[0] for s, c in zip(scenes, camsl)]
    gc = hit_mask_cot(W.random_cotangents(b.n_rays, 31, flow=False), np.concatenate([r["alpha"] for r in refs]))
    for normals in (True, False):
        cot = {"depth": _t(gc["depth"]), "alpha": _t(gc["alpha"]), "normal": _t(gc["normal"]) if normals else None}
        grads = b.backward(outs, cot, b.alloc_grads())
        lbar = b.split_statistic(torch.ones(b.n_rays, device=DEV), outs)
        torch.cuda.synchronize()
        for i, (sc, cm) in enumerate(zip(scenes, camsl)):
            r0, r1, g0, g1 = b.ray_off[i], b.ray_off[i + 1], b.gauss_off[i], b.gauss_off[i + 1]
            one = fmb.Scene(means[g0:g1], prec[g0:g1], weights[g0:g1], betas[i], 1.0, cams[i])
            one.set_model("composite")
            o = one.render(normals=True)
            g = one.backward(o, cot["depth"][r0:r1], cot["alpha"][r0:r1], cot["normal"][r0:r1] if normals else None)
            na = one.backward(o, cot["depth"][r0:r1], cot["alpha"][r0:r1], cot["normal"][r0:r1] if normals else None, noalloc=True)
            torch.cuda.synchronize()
            for k in ("depth", "alpha", "normal", "stash"):
                assert torch.equal(o[k], outs[k][r0:r1]), (i, k)
            for k in ("means", "prec", "weights"):
                assert torch.equal(g[k], grads[k][g0:g1]), (i, k)
                assert torch.equal(na[k], g[k]), (i, k, "noalloc")
            # the weights of a ray sum to one
            assert abs(float(lbar[g0:g1].double().sum()) - 1.0) < 1e-5
            cot_np = {k: None if gc[k] is None or (k == "normal" and not normals) else gc[k][r0:r1] for k in gc}
            _, gref, _ = O.render_workload_view(sc, cm, BETAS, 1.0, cot=cot_np, model="composite")
            assert_forward(compare_forward(o, refs[i]), f"{label} N={sc.n}")
            assert_grads(compare_grads(g, gref), f"{label} N={sc.n} normals={normals}")
