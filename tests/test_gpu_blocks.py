"""Launches dealt to the XCDs in blocks of tiles: every tile of a frame taken
once whatever its size (the host's rule and the kernels' decoding in plain
integers), and frames bit-identical to the same kernel's row order (persistent
waves; for FP64 the counted walk) with blocks cut by the frame's edges, several
frames in a launch, and ranges of tiles, which keep row order."""
import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

OUT = ("rgb", "hit_id", "ao_mask", "light_mask")


def _tiles(sizes, one_scene):
    """(job, tx, ty, part, parts) of every workgroup of a launch of whole
    frames of the given sizes in tiles."""
    begin = np.concatenate([[0], np.cumsum([w * h for w, h in sizes])])
    total, jobs = int(begin[-1]), len(sizes)
    pl = 3 if total <= 1024 else 2
    cl = 0 if total <= 1024 else (7 if one_scene and jobs > 2 and total // jobs >= 16384 else 3)
    split, group = int((20.0 if jobs > 1 else 60.0) * np.sqrt(float(total))), 8 << cl
    whole = ((total - split) // group) << cl if total > 1024 and total > split else 0
    groups = ((total + group - 1) // group) << cl
    b = np.arange((whole + ((groups - whole) << pl)) * 8, dtype=np.int64)
    e = b // 8
    sp = np.where(e < whole, 0, e - whole)
    i = np.where(e < whole, e, whole + (sp >> pl))
    j = i >> cl
    q = (b + (j if cl else ((j * 0x9E3779B1) & 0xFFFFFFFF) >> 29)) % 8
    tile = ((j * 8 + q) << cl) + (i & ((1 << cl) - 1))
    ok = tile < total
    tile, part, parts = tile[ok], np.where(e < whole, 0, sp & ((1 << pl) - 1))[ok], np.where(e < whole, 1, 1 << pl)[ok]
    job = np.searchsorted(begin, tile, side="right") - 1
    t = tile - begin[job]
    w, h = np.array(sizes).T[0][job], np.array(sizes).T[1][job]
    if not cl:
        return job, t % w, t // w, part, parts
    band = 1 << ((cl + 1) >> 1)
    k = t // (band * w)
    r = t - k * band * w
    rows = np.minimum(band, h - k * band)
    return job, r // rows, k * band + r - (r // rows) * rows, part, parts


@pytest.mark.parametrize("sizes", [[(1025, 1)], [(1, 1030)], [(33, 32)], [(37, 29)], [(121, 143)], [(483, 569)],
                                   [(241, 285)] * 2, [(130, 127)] * 3, [(129, 131), (1, 1), (200, 300)],
                                   [(20, 20)] * 5])
@pytest.mark.parametrize("one_scene", [False, True])
def test_every_tile_once(sizes, one_scene):
    job, tx, ty, part, parts = _tiles(sizes, one_scene)
    for n, (w, h) in enumerate(sizes):
        seen = np.zeros((h, w, 8), dtype=np.int32)
        m = job == n
        assert (tx[m] >= 0).all() and (tx[m] < w).all() and (ty[m] >= 0).all() and (ty[m] < h).all()
        for k in range(8):
            p = parts[m]
            np.add.at(seen, (ty[m], tx[m], k), (k // (8 // p) == part[m]).astype(np.int32))
        assert (seen == 1).all()


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


def _cam(w, h):
    return scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, w, h)


def _same(a, b):
    for k in OUT:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("size", [(8200, 8), (7, 8240), (264, 256), (290, 230), (965, 1137), (1030, 517)])
def test_blocks_equal_rows(tr, size):
    gs = tr.Scene(scenegen.tiny_scene(seed=6))
    p = scenegen.Params(ao_samples=3, seed=5)
    got = [frame_to_numpy(tr.render(gs, _cam(*size), p, outputs=OUT, tune=t)) for t in ({}, {"waves_per_cu": 19})]
    _same(*got)
    got = [frame_to_numpy(tr.render(gs, _cam(*size), p, precision="fp64", outputs=OUT, stats=st))
           for st in (False, True)]
    _same(*got)


@pytest.mark.gpu
def test_large_blocks_and_ranges(tr):
    gs = tr.Scene(scenegen.tiny_scene(seed=6))
    p = scenegen.Params(ao_samples=2, seed=5)
    cams = [_cam(1029, 1030), _cam(9, 5), _cam(1600, 1337)]
    ref = [frame_to_numpy(tr.render(gs, c, p, outputs=OUT, tune={"waves_per_cu": 19})) for c in cams]
    frames = [tr.alloc_frame(c, OUT) for c in cams]
    tr.render_batch_into([gs] * 3, cams, [p] * 3, frames)
    for f, r in zip(frames, ref):
        _same(frame_to_numpy(f), r)
    other = tr.Scene(scenegen.tiny_scene(seed=6))  # (equal, so another scene of the launch)
    tr.render_batch_into([gs, other, gs], cams, [p] * 3, frames)
    for f, r in zip(frames, ref):
        _same(frame_to_numpy(f), r)
    n = [tr.tile_count(c.width, c.height) for c in cams]
    frames = [tr.alloc_frame(c, OUT) for c in cams]
    for part in ([(0, 7001), (0, 0), (13, n[2])], [(7001, n[0]), (0, n[1]), (0, 13)]):
        tr.render_batch_tiles_into([gs] * 3, cams, [p] * 3, frames, *zip(*part))
    for f, r in zip(frames, ref):
        _same(frame_to_numpy(f), r)
