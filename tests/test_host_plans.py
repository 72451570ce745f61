"""The host library's work plans, workspaces and uploads on a recording runtime, without a GPU: each check
runs in a process of its own (tests/host_runtime.py)."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
if __name__ == "__main__":
    sys.path.insert(0, os.path.dirname(HERE))

from tests.host_runtime import OOM, Runtime, Scene  # noqa: E402


def _tiles(h, w):
    return ((w + 7) // 8) * ((h + 7) // 8) if w >= 8 else (h * w + 63) // 64


def _covered(items, tiles, lane_tiles=True):
    """Per view, the ray tiles that the items of one backward launch take; fails on a view or tile past the end."""
    got = [0] * len(tiles)
    for view, ray0, span, *_ in items:
        assert 0 <= view < len(tiles) and 0 <= ray0 < tiles[view], (view, ray0, tiles)
        got[view] += min(span, tiles[view] - ray0)
    return got


def noalloc_plan_follows_the_cameras():
    """fmb_backward_noalloc after other cameras or rays: fewer views, more views, explicit rays."""
    rt = Runtime()
    for composite in (False, True):
        sc = Scene(rt, 40)
        sc.set_model(composite)
        steps = [("cams", [(64, 64)] * 3), ("cams", [(32, 24)]), ("cams", [(40, 64)] * 5), ("rays", [100, 0, 70]), ("cams", [(9, 5)])]
        for kind, arg in steps:
            if kind == "cams":
                sc.set_cameras(arg)
                tiles = [_tiles(h, w) for h, w in arg]
            else:
                sc.set_rays(arg)
                tiles = [(c + 63) // 64 for c in arg]
            sc.check(sc.render())
            rt.launches()
            sc.check(sc.backward(noalloc=True))
            items = [i for name, _, i in rt.launches() if "bwd" in name][0]
            assert _covered(items, tiles) == tiles, (composite, kind, arg)


def reduction_of_many_gaussians():
    """A chunk of a whole scene of few items is reduced in one stage up to 65535 slices of 3 Gaussians (2 with
    colour), and in two above: none of them is refused, nor is an autotuner that meets one."""
    rt = Runtime()
    for n, colour, one in ((196605, False, True), (196606, False, False), (131070, True, True), (131071, True, False)):
        for variant in (None, 3):  # the compositing model; the ray-lane variant of the blend
            sc = Scene(rt, n)
            sc.set_model(variant is None)
            sc.set_cameras([(16, 16)])
            sc.set_colors(colour)
            if variant is not None:
                sc.set_variants(0, variant)
            rt.launches()
            sc.check(sc.backward(color=colour))
            names = [name for name, _, _ in rt.launches()]
            assert any("fin_one" in k for k in names) == one and any("fin2" in k for k in names) != one, (n, colour, names)
            sc.check(rt.lib.fmb_scene_destroy(sc.h))
    sc = Scene(rt, 200000)
    sc.set_cameras([(16, 16)])
    sc.check(sc.autotune())


def lists_are_not_overwritten_under_a_kernel():
    """On a stream of the caller's: a list that an earlier pass may still read is replaced only after a wait;
    new rays cost one wait a step, and a repeated step none."""
    rt = Runtime()
    for composite in (False, True):
        sc = Scene(rt, 300, stream=0x770)
        sc.set_model(composite)
        sc.set_colors()

        def step(**kw):
            sc.check(sc.render(normal=True, color=True))
            sc.check(sc.backward(**kw))

        sc.set_rays([200, 90])
        step()
        for kw in ({"normal": True}, {"color": True}, {"normal": True, "color": True}, {}):
            step(**kw)  # other cotangents: another plan
            sc.check(sc.split())
        for counts in ([100, 190], [290, 0], [1, 2], [500, 900]):
            before = rt.count("syncs")
            sc.set_rays(counts)
            step()
            sc.check(sc.split())
            assert rt.count("syncs") - before <= 1, (composite, counts)
        before = rt.count("syncs")
        step()
        assert rt.count("syncs") == before
        sc.set_cameras([(64, 64)])
        step()
        sc.set_variants(3, 2)
        step()
        sc.check(sc.backward(noalloc=True))
        sc.set_cameras([(24, 24)])
        assert rt.count("overwrites") == 0, (composite, rt.count("overwrites"))


def failed_build_is_not_taken_for_built():
    """A backward that runs out of memory leaves no half-replaced lists behind: the earlier configuration
    is built again, with its own items, once there is room."""
    rt = Runtime()
    sc = Scene(rt, 700)
    sc.set_cameras([(200, 200)])
    sc.set_variants(1, 8)
    tiles = [_tiles(200, 200)]
    sc.check(sc.render())
    sc.check(sc.backward())
    rt.rr.rr_set_limit(rt.rr.rr_in_use() + (1 << 10))
    sc.set_variants(1, 0)  # Gaussian lanes: more records than the room left
    assert sc.backward() == OOM
    rt.rr.rr_set_limit(-1)
    sc.set_variants(1, 8)
    rt.launches()
    sc.check(sc.render())
    sc.check(sc.backward())
    items = [i for name, _, i in rt.launches() if "bwdt" in name][0]
    whole = [i for i in items if i[3] == 0]  # the first part of each record
    assert _covered(whole, tiles) == tiles and all(i[4] == 700 for i in items)


def coarser_cuts_where_memory_is_short():
    """Records of the finer cuts that do not fit give way to 16-tile ones (the tiled form of a normal cotangent
    to the Gaussian-lane variant), which fit; the whole view is still taken once."""
    rt = Runtime()
    for n, hw, composite, normal in ((20000, (400, 400), False, False), (5000, (480, 640), True, False), (10000, (1080, 1920), False, True)):
        def passes(limit):
            rt.rr.rr_set_limit(-1)
            sc = Scene(rt, n)
            sc.set_model(composite)
            sc.set_cameras([hw])
            base = rt.rr.rr_in_use()
            if limit is not None:
                rt.rr.rr_set_limit(base + limit)
            sc.check(sc.render())
            rt.launches()
            rc = sc.backward(normal=normal)
            items = [i for name, _, i in rt.launches() if "bwd" in name]
            need = rt.rr.rr_in_use() - base
            rt.lib.fmb_scene_destroy(sc.h)
            return rc, need, items[0] if items else None

        rc, fine, _ = passes(None)
        assert rc == 0
        rc, coarse, items = passes(fine - 1)
        assert rc == 0 and coarse < fine, (n, rc, fine, coarse)
        if not normal:
            assert _covered([i for i in items if i[3] == 0], [_tiles(*hw)]) == [_tiles(*hw)] and (items[:, 2] == 16).all()
        rc, _, _ = passes(coarse // 2)
        assert rc == OOM, (n, rc)


def split_statistic_uploads_what_its_kernel_reads():
    """First split statistic on new cameras: items, tasks, ray counts and (compositing, whose kernel has two
    forms) the items' order."""
    rt = Runtime()
    for composite, copies in ((False, 3), (True, 4)):
        sc = Scene(rt, 40)
        sc.set_model(composite)
        sc.set_cameras([(64, 64)] * 4)
        sc.check(sc.render())
        before = rt.count("copies")
        sc.check(sc.split())
        assert rt.count("copies") - before == copies, (composite, rt.count("copies") - before)


def variant_tables():
    """Each backward variant has one of the three sizes, the others are 0 (no table is read past its end)."""
    rt = Runtime()
    for v in range(10):  # 9: the tiled form of a normal cotangent
        of = [getattr(rt.lib, "_ZN3fmb%d%sEi" % (len(f), f))(v) for f in ("bwd_variant_rt", "bwd_variant_ray_tile", "bwd_variant_tiles")]
        assert [x > 0 for x in of] == [v < 3, 3 <= v < 6, v >= 6], (v, of)


# (composite, variant or None, colour, normal cotangent, views of H x W, Gaussians): the largest views of their
# width whose backward fitted the fixed workspace when the items were 32 bytes and one stage of the reduction
# more was needed
NOALLOC_FITS = [
    (False, None, False, False, 1, (322848, 64), 40), (False, None, False, True, 7, (2285, 203), 128),
    (False, None, True, True, 1, (31728, 1000), 100), (False, 2, False, False, 1, (1536, 64), 2000),
    (False, 2, True, False, 7, (4485, 1000), 200), (False, 3, False, False, 7, (920, 1000), 129),
    (True, None, False, False, 1, (322848, 64), 40), (True, None, True, True, 7, (912, 1000), 100),
    (True, None, False, True, 1, (100720, 64), 129),
]


def noalloc_takes_what_it_took():
    """Views at the limit of fmb_backward_noalloc's workspace."""
    rt = Runtime()
    for composite, variant, colour, normal, v, hw, n in NOALLOC_FITS:
        sc = Scene(rt, n)
        sc.set_model(composite)
        sc.set_cameras([hw] * v)
        sc.set_colors(colour)
        if variant is not None:
            sc.set_variants(0, variant)
        sc.check(sc.backward(normal=normal, color=colour, noalloc=True))
        rt.launches()


def compositing_step_is_recorded_after_one_forward():
    """A capture allows no allocation and no synchronous copy: after one eager compositing forward with a
    stash, a forward and a backward need neither (nor does a forward without one plan a backward)."""
    rt = Runtime()
    for colour in (False, True):
        sc = Scene(rt, 40, stream=0x770)
        sc.set_model(True)
        sc.set_colors(colour)
        sc.set_cameras([(64, 64)])
        sc.check(sc.render(color=colour))
        rt.rr.rr_set_capturing(1)
        sc.check(sc.render(color=colour))
        sc.check(sc.backward(color=colour))
        rt.rr.rr_set_capturing(0)
        assert rt.count("refused") == 0


def compositing_parts_by_the_measured_rule():
    """Blocks of the compositing forward: 16, 4 or 1 a tile of a larger scene, as measured best for these."""
    rt = Runtime()
    for n, hw, parts in ((1200, (200, 200), 16), (1200, (150, 300), 16), (1000, (128, 128), 16), (600, (200, 200), 4),
                         (700, (270, 480), 4), (1000, (270, 480), 4), (400, (270, 480), 1), (1000, (540, 960), 1)):
        sc = Scene(rt, n)
        sc.set_model(True)
        sc.set_cameras([hw])
        rt.launches()
        sc.check(sc.render())
        grid = [g for name, g, _ in rt.launches() if "fwdc" in name][0]
        assert grid[0] == parts * _tiles(*hw), (n, hw, grid)


def host_memory_exhausted_is_a_status():
    """A plan that the host cannot hold ends in FMB_ERR_OOM, not in an exception through the C interface, and
    the scene works again once there is room."""
    import resource
    rt = Runtime()
    sc = Scene(rt, 40)
    big, small = [(16384, 16384)] * 4, [(64, 64)]  # 1.7e7 ray tiles

    def limited(f):
        with open("/proc/self/statm") as st:
            now = int(st.read().split()[0]) * resource.getpagesize()
        old = resource.getrlimit(resource.RLIMIT_AS)
        resource.setrlimit(resource.RLIMIT_AS, (now + (16 << 20), old[1]))
        try:
            return f()
        finally:
            resource.setrlimit(resource.RLIMIT_AS, old)

    for composite in (False, True):
        sc.set_model(composite)
        sc.set_cameras(big)
        assert limited(sc.render) == OOM
        assert limited(sc.backward) == OOM
        assert limited(sc.split) == OOM
        assert limited(lambda: sc.backward(noalloc=True)) == OOM
        sc.set_cameras(small)
        rt.launches()
        sc.check(sc.render())
        sc.check(sc.backward())
        sc.check(sc.backward(noalloc=True))
        for name, _, items in rt.launches():
            assert len(items) == 0 or _covered(items, [64]) == [64], name


CHECKS = [host_memory_exhausted_is_a_status, compositing_parts_by_the_measured_rule, compositing_step_is_recorded_after_one_forward, noalloc_takes_what_it_took, variant_tables, split_statistic_uploads_what_its_kernel_reads, coarser_cuts_where_memory_is_short, failed_build_is_not_taken_for_built, lists_are_not_overwritten_under_a_kernel, noalloc_plan_follows_the_cameras, reduction_of_many_gaussians]


@pytest.mark.parametrize("check", [c.__name__ for c in CHECKS])
def test_host(check):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), check], capture_output=True, text=True, timeout=300,
                       cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


if __name__ == "__main__":
    globals()[sys.argv[1]]()
