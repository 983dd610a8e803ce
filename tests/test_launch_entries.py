"""How launches of one workgroup per entry deal their tiles, by the library's own
functions (tr_debug_entries): every part of every tile once, whatever the
frames' sizes, and as many workgroups as a render launches."""
import ctypes as C

import numpy as np
import pytest

import hip_model
import scenegen


def entries(lib, sizes, ranges=False):
    """int32 [workgroups, 5]: job, column, row, part, parts."""
    tx, ty = (np.ascontiguousarray([s[k] for s in sizes], dtype=np.int32) for k in (0, 1))
    call = lambda cap, out: lib.tr_debug_entries(len(sizes), tx.ctypes.data, ty.ctypes.data, int(ranges), cap, out)
    n = call(0, None)
    assert n > 0
    out = np.full((n, 5), -7, dtype=np.int32)
    assert call(n, out.ctypes.data) == n
    return out


@pytest.fixture(scope="module")
def lib():
    import paper_0801_1500_amd as tr
    return tr.lib()


@pytest.mark.parametrize("sizes", [[(1, 1)], [(7, 1)], [(8, 1)], [(3, 3)], [(1023, 1)], [(32, 32)], [(1025, 1)],
                                   [(1, 1030)], [(33, 32)], [(37, 29)], [(60, 60)], [(13, 277)], [(64, 64)],
                                   [(32, 128)], [(32, 131)], [(121, 143)], [(483, 569)], [(241, 285)] * 2,
                                   [(130, 127)] * 3, [(129, 131), (1, 1), (200, 300)], [(20, 20)] * 5,
                                   [(5, 1000), (1000, 5), (64, 77)], [(16, 1137)] * 4])
@pytest.mark.parametrize("ranges", [False, True])
def test_every_part_once(lib, sizes, ranges):
    e = entries(lib, sizes, ranges)
    assert len(e) % 8 == 0 and ((e[:, 0] >= -1) & (e[:, 0] < len(sizes))).all()
    for k, (w, h) in enumerate(sizes):
        _, tx, ty, part, parts = e[e[:, 0] == k].T
        assert (tx >= 0).all() and (tx < w).all() and (ty >= 0).all() and (ty < h).all()
        assert np.isin(parts, (1, 4, 8)).all() and (part >= 0).all() and (part < parts).all()
        seen = np.zeros((h, w, 8), dtype=np.int32)
        for q in range(8):
            np.add.at(seen, (ty, tx, q), (q // (8 // parts) == part).astype(np.int32))
        assert (seen == 1).all()


@pytest.mark.parametrize("jobs,ranges", [(1, False), (2, False), (4, True)])
def test_dealing_is_even(lib, jobs, ranges):
    """Workgroup b runs on XCD b mod 8, which deals its workgroups out in turn.
    Frames whose rays lie in a disk (a pixel there costs what 17 others do): no
    XCD, and no eighth of one, may have a quarter more than its fair part,
    whatever the frames' width.  (An XCD had 1.5 times its part at rows of 64
    tiles; of ranges, an eighth had up to four times at rows of 32 and 64.)"""
    for w in list(range(8, 36)) + [48, 57, 64, 73, 96, 128]:
        h = 1100
        y, x = np.mgrid[0:h, 0:64 * w]
        disk = (x - 35.2 * w) ** 2 + (y - 0.525 * h) ** 2 < (0.42 * min(h, 64 * w)) ** 2
        cost = 64.0 + 16.0 * disk.reshape(h, w, 64).sum(2)
        if ranges:  # the middle half of the tiles, as rows of a frame of their own
            cost = cost[h // 4:h // 4 + h // 2]
        e = entries(lib, [(w, len(cost))] * jobs, ranges)
        b = np.flatnonzero(e[:, 0] >= 0)
        _, tx, ty, _, parts = e[b].T
        c = cost[ty, tx] / parts
        for unit in (b % 8, b % 64):
            load = np.bincount(unit, c)
            assert load.max() <= 1.25 * load.mean(), (w, load.max() / load.mean())


def renders_launch_as_many(model, tr):
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for sizes, fp64 in (([(130, 67)], False), ([(700, 431)], False), ([(700, 431), (65, 9), (2048, 300)], False),
                        ([(700, 431)], True)):
        jobs = [(s, tr.make_camera(scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, w, h)),
                 tr.make_params(scenegen.Params(), "fp64" if fp64 else "fp32"),
                 tr.Frame(0x1000000, None, None, None, None)) for w, h in sizes]
        n = len(jobs)
        sc = (C.c_void_p * n)(*[j[0].handle for j in jobs])
        cm, pr, fr = ((t * n)(*[j[k] for j in jobs]) for k, t in ((1, tr.Camera), (2, tr.Params), (3, tr.Frame)))
        assert tr.lib().tr_render_batch(n, sc, cm, pr, fr, None) == 0
        tiles = [((w + 7) // 8, (h + 7) // 8) if fp64 else ((w + 63) // 64, h) for w, h in sizes]
        assert hip_model.launches(model)[-1][1] == len(entries(tr.lib(), tiles)), sizes


def test_renders_launch_as_many():
    hip_model.run("test_launch_entries", "renders_launch_as_many")
