"""The tiled backward with a normal cotangent (8 ray tiles per item) at its edges: one Gaussian, a full
and an overfull staged tile, pre-culled rounds, views that fill no tile row, with and without colour and
flow cotangents -- against the FP64 oracle, and a batch of such scenes against their own launches bit
for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import assert_grads, compare_grads, custom_scene, hit_mask_cot, normwise, to_np

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"
BETAS = np.array([W.BETA1, W.BETA2], np.float32)


def _t(a):
    return None if a is None else torch.as_tensor(np.ascontiguousarray(a), device=DEV).contiguous()


@pytest.mark.parametrize("extras", [False, True], ids=["normals", "normals_colour_flow"])
def test_normal_cotangent_edges(extras):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_14737_amd as fmb
    sizes = [(1, [(8, 8)]), (64, [(33, 71), (5, 3)]), (65, [(64, 64)]), (300, [(40, 24)])]
    parts = [custom_scene(n, v, seed=500 + n, flow=True) for n, v in sizes]
    scenes, camsl = [p[0] for p in parts], [p[1] for p in parts]
    g = np.random.Generator(np.random.PCG64(5))
    cat = lambda k: _t(np.concatenate([getattr(s, k) for s in scenes]))  # noqa: E731
    means, prec, weights, betas = cat("means"), cat("prec"), cat("weights"), _t(np.tile(BETAS, (len(scenes), 1)))
    cams = [fmb.Cameras.from_numpy(c.w2c, c.intr, c.hw, c.w2c_b, c.intr_b, device=DEV) for c in camsl]
    b = fmb.Batch(means, prec, weights, betas, [1.0] * len(scenes), [s.n for s in scenes], cams)
    q = (1.5 * g.standard_normal((means.shape[0], 3))).astype(np.float32) if extras else None
    if extras:
        qt = _t(q)
        b.set_colors(qt)
    outs = b.forward(b.alloc_outputs(normals=True, color=extras))
    qs = [q[b.gauss_off[i]:b.gauss_off[i + 1]] if extras else None for i in range(len(scenes))]
    refs = [O.render_workload_view(s, c, BETAS, 1.0, colors=k)[0] for s, c, k in zip(scenes, camsl, qs)]
    cot = W.random_cotangents(b.n_rays, 51, flow=extras)
    cot["color"] = g.standard_normal((b.n_rays, 3)).astype(np.float32) if extras else None
    cot = hit_mask_cot(cot, np.concatenate([r["alpha"] for r in refs]))
    grads = b.backward(outs, {k: _t(v) for k, v in cot.items()}, b.alloc_grads(colors=extras))
    torch.cuda.synchronize()
    for i, (sc, cm) in enumerate(zip(scenes, camsl)):
        r0, r1, g0, g1 = b.ray_off[i], b.ray_off[i + 1], b.gauss_off[i], b.gauss_off[i + 1]
        cut = {k: None if v is None else v[r0:r1] for k, v in cot.items()}
        one = fmb.Scene(means[g0:g1], prec[g0:g1], weights[g0:g1], betas[i], 1.0, cams[i])
        if extras:
            one.set_colors(qt[g0:g1])
        o = one.render(normals=True)
        gi = one.backward(o, _t(cut["depth"]), _t(cut["alpha"]), _t(cut["normal"]), _t(cut["flow"]), g_color=_t(cut["color"]))
        torch.cuda.synchronize()
        for k in ("means", "prec", "weights") + (("colors",) if extras else ()):
            assert torch.equal(gi[k], grads[k][g0:g1]), (sc.n, k)
        _, gref, _ = O.render_workload_view(sc, cm, BETAS, 1.0, cot=cut, colors=qs[i])
        eg = compare_grads(gi, gref)
        if extras:
            eg["colors"] = normwise(to_np(gi["colors"]), gref["colors"])
        print(f"[normals] N={sc.n}: {eg}", flush=True)
        # one Gaussian: the blend has one weight of 1, so the gradients of betas are zero up to rounding
        assert_grads({k: v for k, v in eg.items() if sc.n > 1 or k != "betas"}, f"N={sc.n}")
