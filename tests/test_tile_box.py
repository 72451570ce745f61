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


def _f32_bounds(u, mu, lam, box, hm):
    """tile_bounds' log2 density bounds in FP32, from the FP32 entry that the pre-culls use
    (make_bound_entry): u the packed factor, mu the mean relative to the camera, box (c, Z, ex, X, ey, Y)."""
    f = np.float32
    u00, u01, u02, u11, u12, u22 = (f(x) for x in u)
    m = mu.astype(f)
    c, Z, ex, X, ey, Y = [np.asarray(k, dtype=f) for k in box]

    def mul(a):
        return np.array([u00 * a[0] + u01 * a[1] + u02 * a[2], u11 * a[1] + u12 * a[2], u22 * a[2]], f)

    b, n = mul(m), np.abs(m)
    a0 = abs(u00) * n[0] + abs(u01) * n[1] + abs(u02) * n[2]
    ab = np.array([a0, abs(u11) * n[1] + abs(u12) * n[2], abs(b[2])], f)
    cc = np.array([u00 * b[0], u01 * b[0] + u11 * b[1], u02 * b[0] + u12 * b[1] + u22 * b[2]], f)
    est_x, est_z = (b * b).sum(dtype=f), (ab * ab).sum(dtype=f)
    est_y = (abs(u00) + abs(u01) + abs(u02)) * ab[0] + (abs(u11) + abs(u12)) * ab[1] + abs(u22) * ab[2]
    err, up, down = f(2.0 ** -17), f(1 + 2e-5), f(1 - 2e-5)
    a = mul(c)
    aa, vc = (a * a).sum(dtype=f), (c * cc).sum(dtype=f)
    t = vc / aa
    na = np.sqrt(aa)
    p, q = mul(ex), mul(ey)
    fr = (Z * na + np.sqrt(X * X * (p @ p) + Y * Y * (q @ q) + f(2) * X * Y * abs(p @ q))) * up
    s = min(fr / na, f(1))
    co = np.sqrt(f(1) - s * s)
    terr = err * est_y / aa
    at, atl = abs(t) + terr, abs(t) - terr
    mid, e = est_x - vc * t, err * (est_y * at + est_z)
    sl, sh, nb = np.sqrt(max(mid - e, f(0))), np.sqrt(max(mid + e, f(0))), np.sqrt(est_x + err * est_z)
    gs, gl = at * min(fr, na), atl * na * co
    lo = max(sl * co * down - gs * up, f(0))
    hi = (sh * co + gs if sh * s < gl and s < 0.999 else nb) * up
    l2l = f(np.log2(lam))
    return float(hm * lo * lo + l2l) + 1e-3, float(hm * hi * hi + l2l) - 1e-3


def test_single_precision_bounds_hold():
    """The FP32 entry and bounds with their slack terms, needles and discs seen edge on included."""
    g = np.random.Generator(np.random.PCG64(23))
    hm = -0.5 * np.log2(np.e)
    near = 0
    for k in range(500):
        s = np.exp(g.uniform(np.log(0.003), np.log(0.6), 3))
        r = _rotation(g)
        U = np.linalg.cholesky(r @ np.diag(s ** -2.0) @ r.T).T
        u = np.array([U[0, 0], U[0, 1], U[0, 2], U[1, 1], U[1, 2], U[2, 2]]).astype(np.float32)
        U = np.array([[u[0], u[1], u[2]], [0, u[3], u[4]], [0, 0, u[5]]], dtype=np.float64)
        c = g.standard_normal(3)
        c /= np.linalg.norm(c)
        ex = _rotation(g)[0]
        ex -= (ex @ c) * c
        ex /= np.linalg.norm(ex)
        ey = np.cross(c, ex)
        mu = g.uniform(0.3, 8.0) * c + s.max() * g.uniform(0, 6) * g.standard_normal(3)
        h = np.exp(g.uniform(np.log(2e-4), np.log(0.05)))
        v = c + g.uniform(-h, h, (64, 1)) * ex + g.uniform(-h, h, (64, 1)) * ey
        v /= np.linalg.norm(v, axis=1, keepdims=True)
        X, Y, Z = (np.abs((v - c) @ d).max() * (1 + 1e-5) + 5e-7 for d in (ex, ey, c))
        lam = g.uniform(0.1, 2.0)
        hi, lo = _f32_bounds(u, mu, lam, (c, Z, ex, X, ey, Y), hm)
        a, b = v @ U.T, U @ mu
        t = (a @ b) / (a * a).sum(1)
        d2 = np.log2(lam) + hm * ((t[:, None] * a - b) ** 2).sum(1)
        assert d2.max() <= hi and d2.min() >= lo, (k, lo, d2.min(), d2.max(), hi)
        near += hi < d2.max() + 5
    assert near > 200, near
