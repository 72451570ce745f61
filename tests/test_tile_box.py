"""The bounds over a tile's box of rays that decide which (ray tile, Gaussian) pairs a kernel takes.

CPU: the bounds restated in FP64 (tile_bounds in csrc/fmb_device.h, without its rounding slack)
against the exact peak of every ray on random tiles and anisotropic Gaussians: the squared
Mahalanobis distance m and the peak depth t of every ray lie inside them.  GPU: scenes at the edges
of the staged tiles (one tile, one Gaussian more, pre-culled rounds) render an alpha that is
relatively exact down to densities far below one, which the cutoffs relative to the tile's density sum
must not disturb.
"""
from __future__ import annotations

import numpy as np
import pytest


def _rotation(g):
    q, r = np.linalg.qr(g.standard_normal((3, 3)))
    return q * np.sign(np.diag(r))


def _bounds(U, mu, c, ex, ey, X, Y, Z):
    """(m_lo, m_hi, t_lo, t_hi) over the box, the depths None where they are not bounded."""
    a, b = U @ c, U @ mu
    na, nb, vc = np.linalg.norm(a), np.linalg.norm(b), a @ b
    p, q = U @ ex, U @ ey
    f = np.sqrt(X * X * (p @ p) + Y * Y * (q @ q) + 2 * X * Y * abs(p @ q)) + Z * na
    s = min(f / na, 1.0)
    co = np.sqrt(1 - s * s)
    t, root = vc / na ** 2, np.sqrt(max(nb ** 2 - (vc / na) ** 2, 0.0))
    gs, gc = abs(t) * min(f, na), abs(t) * na * co
    lo = max(0.0, root * co - gs)
    hi = root * co + gs if root * s < gc and s < 0.999 else nb
    if s >= 0.999:
        return lo ** 2, hi ** 2, None, None
    nlo, nhi = gc - root * s, gc + root * s if lo > 0 else nb
    lt, ht = (nlo / (na + f) if nlo >= 0 else nlo / (na - f)), nhi / (na - f)
    return (lo ** 2, hi ** 2) + ((lt, ht) if vc >= 0 else (-ht, -lt))


def test_bounds_hold_on_every_ray():
    g = np.random.Generator(np.random.PCG64(21))
    tight = bounded = 0
    for _ in range(600):
        s = np.exp(g.uniform(np.log(0.005), np.log(0.5), 3))
        r = _rotation(g)
        U = np.linalg.cholesky(r @ np.diag(s ** -2.0) @ r.T).T
        mu = g.uniform(-1, 1, 3) + np.array([0.0, 0.0, g.choice([3.0, 0.5, -2.0])])
        c = g.standard_normal(3) + np.array([0.0, 0.0, 3.0])
        c /= np.linalg.norm(c)
        ex = _rotation(g)[0]
        ex -= (ex @ c) * c
        ex /= np.linalg.norm(ex)
        ey = np.cross(c, ex)
        h = g.uniform(0.001, 0.03) * g.choice([1.0, 1.0, 20.0])
        v = c + g.uniform(-h, h, (64, 1)) * ex + g.uniform(-h, h, (64, 1)) * ey
        v /= np.linalg.norm(v, axis=1, keepdims=True)
        e = v - c
        m_lo, m_hi, t_lo, t_hi = _bounds(U, mu, c, ex, ey, *(np.abs(e @ k).max() for k in (ex, ey, c)))
        a, b = v @ U.T, U @ mu
        t = (a @ b) / (a * a).sum(1)
        m = ((t[:, None] * a - b) ** 2).sum(1)
        tol = 1e-10 * (b @ b)
        assert m_lo - tol <= m.min() and m.max() <= m_hi + tol, (m_lo, m.min(), m.max(), m_hi)
        if t_lo is not None:
            assert t_lo - 1e-10 <= t.min() and t.max() <= t_hi + 1e-10, (t_lo, t.min(), t.max(), t_hi)
            bounded += 1
        tight += m_lo > 0.5 * m.min()
    assert bounded > 400 and tight > 200, (bounded, tight)  # not vacuous


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 128, 129, 256, 257, 300])
def test_alpha_is_relatively_exact(n):
    """alpha = 1 - exp(-sum delta) of every ray with alpha >= 1e-9, relative to the oracle.  A pair's
    density errs by half of m's error, sqrt(m) |U|_2 |t| 2^-23 for m <= 2 ln(1e9) = 41.4, |U|_2 <= 20 and
    |t| <= 5: below 8e-5; the cutoffs leave out 2^-26 of the sum and every density below 2^-48 (n of
    them: 1e-3 of 1e-9 for n = 300)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as O
    import paper_2308_14737_amd as fmb
    import workloads as W
    from tests.gpu_util import custom_scene, make_scene, to_np
    sc, cams = custom_scene(n, [(40, 56), (9, 130)], seed=300 + n)
    betas = np.array([W.BETA1, W.BETA2], np.float32)
    print(f"[alpha] N={n} P={cams.n_rays}", flush=True)
    scene, _ = make_scene(fmb, torch, sc, cams, betas, 1.0, "cuda:0")
    out = scene.render(normals=True)
    ref, _, _ = O.render_workload_view(sc, cams, betas, 1.0)
    a, r = to_np(out["alpha"]), ref["alpha"]
    at = r >= 1e-9
    err = np.abs(a[at] / r[at] - 1.0).max()
    print(f"[alpha] N={n}: {at.sum()} rays, relative error {err:.2e}", flush=True)
    assert err <= 8e-5 + n * 2.0 ** -48 / 1e-9 + 1e-6, err
