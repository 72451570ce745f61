"""The kernels' own tile boxes and bounds (csrc/fmb_device.h), compiled for the CPU with a wave of 64 lanes in
step: every ray of a tile lies in its box and in its item's box, and on every ray each Gaussian's log2
density and log2 weight, exact in FP64 and as the kernels evaluate them in FP32, lie within the bounds that
decide which pairs are skipped.  No tolerance: the bounds hold their own slack.  A NaN bound bounds
nothing (the kernels keep the pair)."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LOG2E = 1.0 / np.log(2.0)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("bounds") / "bounds.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-w", "-fPIC", "-shared",
                    "-I" + os.path.join(HERE, "c", "host_shim"), "-I" + os.path.join(ROOT, "paper_2308_14737_amd", "csrc"),
                    os.path.join(HERE, "c", "device_bounds.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _rotation(g):
    q, r = np.linalg.qr(g.standard_normal((3, 3)))
    return q * np.sign(np.diag(r))


def _camera(g):
    """Centre (FP64, as the kernels form it) and the world-to-camera matrix of a random pose."""
    r = _rotation(g)
    r[0] *= np.sign(np.linalg.det(r))
    e = np.concatenate([r, (-r @ g.uniform(-3, 3, 3))[:, None]], 1).astype(np.float32)
    ed = e.astype(np.float64)
    return e, np.ascontiguousarray(-ed[:, :3].T @ ed[:, 3])


def _unit(d):
    d = np.asarray(d, np.float64)
    return (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)


def _tiles(g, kind, e, count):
    """`count` tiles of one view: (directions [64,3] float32, mask [64]) each."""
    rot = e[:, :3].astype(np.float64)
    res = []
    if kind in ("pixels", "edge", "coarse"):
        f = {"pixels": 256.0, "edge": 150.0, "coarse": 12.0}[kind]  # (coarse: a tile spans some 40 degrees)
        row0, col0 = g.integers(-8, 8) * 8, g.integers(-8, 8) * 8
        if kind == "coarse":
            row0, col0 = -4, -4
        for k in range(count):
            lane = np.arange(64)
            x, y = (col0 + 8 * k + (lane & 7) + 0.5) / f, (row0 + (lane >> 3) + 0.5) / f
            ok = np.ones(64, bool)
            if kind == "edge":
                ok = ((lane & 7) < g.integers(1, 8)) & ((lane >> 3) < g.integers(1, 9))
            res.append((_unit(np.stack([x, y, np.ones(64)], 1) @ rot), ok))
    else:
        # explicit rays: a strip of random ones in image order, a wide cone, one ray, any direction
        for k in range(count):
            if kind == "strip":
                d = np.stack([g.uniform(-0.5, 0.5, 64), np.full(64, -0.4 + 0.02 * k) + g.uniform(0, 0.02, 64), np.ones(64)], 1)
            elif kind == "cone":
                d = np.concatenate([g.uniform(-1.7, 1.7, (64, 2)), np.ones((64, 1))], 1)
            else:
                d = g.standard_normal((64, 3))
            ok = np.ones(64, bool)
            if kind == "any" and k == 0:
                ok = np.arange(64) == 17
            res.append((_unit(d @ rot), ok))
    if kind == "edge" and count > 1:
        res[-1] = (res[-1][0], np.zeros(64, bool))  # a tile without rays
    return res


def _gaussians(g, n, o, rays, needles):
    lo, hi = (np.log(5e-4), np.log(0.5)) if needles else (np.log(0.005), np.log(0.3))
    s = np.exp(g.uniform(lo, hi, (n, 3)))
    u = np.stack([np.linalg.cholesky(r @ np.diag(k ** -2.0) @ r.T).T for k, r in ((k, _rotation(g)) for k in s)])
    prec = np.stack([u[:, 0, 0], u[:, 0, 1], u[:, 0, 2], u[:, 1, 1], u[:, 1, 2], u[:, 2, 2]], 1).astype(np.float32)
    # around points on the rays, near and far, some behind the camera, one at it
    on = rays[g.integers(0, len(rays), n)].astype(np.float64) * (g.choice([0.3, 2.0, 3.0, 30.0, -2.0], n))[:, None]
    means = (o + on + g.standard_normal((n, 3)) * np.exp(g.uniform(-6, 0.5, (n, 1)))).astype(np.float32)
    means[0] = o
    weights = np.exp(g.uniform(-3, 1, n)).astype(np.float32)
    weights[1] = 1e-20
    return means, prec, weights


def _exact(means, prec, weights, o, v, b1, nc2):
    """FP64 log2 density and log2 weight [n, rays]."""
    p = prec.astype(np.float64)
    u = np.zeros((len(p), 3, 3))
    u[:, 0, 0], u[:, 0, 1], u[:, 0, 2], u[:, 1, 1], u[:, 1, 2], u[:, 2, 2] = p.T
    b = np.einsum("nij,nj->ni", u, means.astype(np.float64) - o)
    a = np.einsum("nij,rj->nri", u, v.astype(np.float64))
    t = np.einsum("nri,ni->nr", a, b) / (a * a).sum(2)
    r = t[:, :, None] * a - b[:, None, :]
    d2 = -0.5 * LOG2E * (r * r).sum(2) + np.log2(weights.astype(np.float64))[:, None]
    return d2, b1 * d2 + nc2 * t


def _box(lib, v, ok, e):
    out = np.zeros(12, np.float32)
    assert lib.db_wave_box(_p(v), _p(ok.astype(np.uint8)), _p(e), _p(out)) == 1
    return out


def _in_box(box, v):
    """The rays' offsets from the box's centre along its axes, against its half extents."""
    b = box.astype(np.float64).reshape(3, 4)
    off = np.abs((v.astype(np.float64) - b[0, :3]) @ b[:, :3].T)
    assert (off <= b[:, 3]).all(), (off.max(0), b[:, 3])


KINDS = ["pixels", "edge", "coarse", "strip", "cone", "any"]


@pytest.mark.parametrize("kind", KINDS)
def test_bounds_hold(lib, kind):
    g = np.random.Generator(np.random.PCG64(KINDS.index(kind)))
    taken = total = 0
    for trial in range(24):
        e, o = _camera(g)
        tiles = _tiles(g, kind, e, 16)
        boxes = [_box(lib, v, ok, e) for v, ok in tiles]
        item = np.zeros(12, np.float32)
        cat = np.concatenate(boxes)
        assert lib.db_item_box(_p(cat), len(boxes), _p(e), _p(item)) == 1
        rays = [v[ok] for v, ok in tiles]
        for box, v in zip(boxes, rays):
            if len(v) == 0:
                assert box[3] == -1.0
                continue
            axes = box.astype(np.float64).reshape(3, 4)[:, :3]
            assert np.abs(axes @ axes.T - np.eye(3)).max() < 1e-5
            _in_box(box, v)
        every = np.concatenate(rays)
        _in_box(item, every)
        n = 24
        means, prec, weights = _gaussians(g, n, o, every, needles=trial % 2 == 1)
        b1, nc2 = [(21.4, -3.14 * LOG2E), (21.4, -3.14 * LOG2E), (2.0, 5.0), (0.0, -1.0)][trial % 4]
        for box, v in [(boxes[0], rays[0]), (boxes[5], rays[5]), (item, every)]:
            if len(v) == 0:
                continue
            v = np.ascontiguousarray(v)
            out = np.zeros((n, 2, 4), np.float32)
            c = ctypes.c_float
            lib.db_bounds(n, _p(means), _p(prec), _p(weights), _p(o), _p(box), c(b1), c(nc2), _p(out))
            d2, z2 = (np.zeros((n, len(v)), np.float32) for _ in range(2))
            lib.db_pairs(n, _p(means), _p(prec), _p(weights), _p(o), len(v), _p(v), c(b1), c(nc2), _p(d2), _p(z2))
            d2x, z2x = _exact(means, prec, weights, o, v, b1, nc2)
            for i in range(n):
                for form in range(2):  # bounds of the FP64 entry, of the FP32 one
                    d_hi, d_lo, z_hi, z_lo = out[i, form].astype(np.float64)
                    what = (kind, trial, i, form, means[i] - o, prec[i], box)
                    for d, z in ((d2x[i], z2x[i]), (d2[i], z2[i])):
                        assert not (d.max() > d_hi) and not (d.min() < d_lo), what + (d.min(), d.max(), d_lo, d_hi)
                        assert not (z.max() > z_hi) and not (z.min() < z_lo), what + (z.min(), z.max(), z_lo, z_hi)
                total += 1
                taken += not out[i, 0, 0] < -48.0
    assert 0 < taken < total, (taken, total)  # (the cutoff decides both ways over these inputs)


def test_no_lower_bound_where_no_density(lib):
    """A zero precision factor has no peak on a ray (0 / 0): the kernels' density is NaN and the Gaussian is
    passed over, so it may not promise a density to the cutoffs that are relative to one."""
    g = np.random.Generator(np.random.PCG64(4))
    e, o = _camera(g)
    v, ok = _tiles(g, "pixels", e, 1)[0]
    box = _box(lib, v, ok, e)
    means, prec, weights = _gaussians(g, 4, o, v, False)
    prec[:] = 0.0
    out = np.zeros((4, 2, 4), np.float32)
    c = ctypes.c_float
    for b1, nc2 in ((0.0, 0.0), (21.4, -4.5)):
        lib.db_bounds(4, _p(means), _p(prec), _p(weights), _p(o), _p(box), c(b1), c(nc2), _p(out))
        assert not (out[:, :, 1] > -np.inf).any() and not (out[:, :, 3] > -np.inf).any(), out


def test_unusable_camera_axes_bound_nothing(lib):
    """A rank-deficient camera matrix has no frame: nothing may be skipped by its boxes."""
    g = np.random.Generator(np.random.PCG64(3))
    e = np.zeros((3, 4), np.float32)
    v = _unit(g.standard_normal((64, 3)) * 0.1 + np.array([0.0, 0.0, 1.0]))
    box = _box(lib, v, np.ones(64, bool), e)
    o = np.zeros(3)
    means, prec, weights = _gaussians(g, 16, o, v, False)
    out = np.zeros((16, 2, 4), np.float32)
    c = ctypes.c_float
    lib.db_bounds(16, _p(means), _p(prec), _p(weights), _p(o), _p(box), c(21.4), c(-4.5), _p(out))
    d2x, z2x = _exact(means, prec, weights, o, v, 21.4, -4.5)
    for form in range(2):
        assert not (d2x.max(1) > out[:, form, 0]).any() and not (z2x.max(1) > out[:, form, 2]).any()
        assert not (d2x.min(1) < out[:, form, 1]).any() and not (z2x.min(1) < out[:, form, 3]).any()
