"""Launches of one workgroup per tile or part of a tile (the default shape)
against the persistent waves of the same kernel (any other number of waves):
bit-identical frames at the edges of the split -- frames narrower than a part,
rows that end inside one, one tile more than all are split in eight at, the
first tiles whole and the rest split, several frames in one launch -- for
every tile width and kernel variant."""
import numpy as np
import pytest

import scenegen
from parity_util import assert_fp32_parity, compare, frame_to_numpy

OUT = ("rgb", "hit_id", "ao_mask", "light_mask")


def _entries(total, jobs):
    """The launch's workgroups as (tile, part, parts): the host's rule and the
    kernel's decoding, in plain integers."""
    split = int((20.0 if jobs > 1 else 60.0) * np.sqrt(float(total)))
    pl = 3 if total <= 1024 else 2
    whole = (total - split) // 8 if total > 1024 and total > split else 0
    groups = (total + 7) // 8
    out = []
    for b in range((whole + ((groups - whole) << pl)) * 8):
        e = b // 8
        sp = 0 if e < whole else e - whole
        j = e if e < whole else whole + (sp >> pl)
        q = (b + (((j * 0x9E3779B1) & 0xFFFFFFFF) >> 29)) % 8
        tile = j * 8 + q
        if tile < total:
            out.append((tile, 0, 1) if e < whole else (tile, sp & ((1 << pl) - 1), 1 << pl))
    return out


@pytest.mark.parametrize("jobs", [1, 2])
@pytest.mark.parametrize("total", [1, 7, 8, 9, 1023, 1024, 1025, 3600, 3601, 4096, 18192])
def test_every_part_once(total, jobs):
    seen = np.zeros((total, 8), dtype=np.int64)
    for tile, part, parts in _entries(total, jobs):
        seen[tile, part * (8 // parts):(part + 1) * (8 // parts)] += 1
    assert (seen == 1).all()


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


def _cam(w, h):
    return scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, w, h)


def _same(a, b):
    for k in a:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("tile_w", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("size", [(1, 1), (5, 3), (63, 2), (65, 9), (130, 67), (256, 256), (257, 257),
                                  (700, 431)])
def test_equals_persistent(tr, size, tile_w):
    gs = tr.Scene(scenegen.mixed_tiny_scene())
    p = scenegen.Params(ao_samples=5, seed=3)
    got = [frame_to_numpy(tr.render(gs, _cam(*size), p, outputs=OUT, tune=t))
           for t in ({"tile_w": tile_w}, {"tile_w": tile_w, "waves_per_cu": 19})]
    _same(*got)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["spheres", "triangles", "layers", "bvh", "fp32"])
def test_variants_equal_persistent(tr, variant):
    scene = scenegen.mixed_tiny_scene() if variant == "triangles" else scenegen.tiny_scene(seed=4)
    if variant == "layers":
        scene.sph_opacity = np.full(scene.n_spheres, 0.5, np.float32)
    gs = tr.Scene(scene)
    if variant == "bvh":
        gs.build_bvh()
    p = scenegen.Params(ao_samples=9, seed=3, max_layers=4 if variant == "layers" else 0)
    prec = "fp32" if variant == "fp32" else "fp32_resolve"
    for size in ((97, 61), (640, 480)):
        got = [frame_to_numpy(tr.render(gs, _cam(*size), p, precision=prec, outputs=OUT,
                                        tune={"accel": int(variant == "bvh"), **t}))
               for t in ({}, {"waves_per_cu": 19})]
        _same(*got)


@pytest.mark.gpu
def test_batch_and_oracle(tr, oracle_mod):
    scene = scenegen.tiny_scene(seed=4)
    gs, other = tr.Scene(scene), tr.Scene(scenegen.mixed_tiny_scene())
    p = scenegen.Params(ao_samples=7, seed=11)
    cams = [_cam(33, 21), _cam(500, 300), _cam(1, 64)]
    frames = [tr.alloc_frame(c, OUT) for c in cams]
    tr.render_batch_into([gs, other, gs], cams, [p] * 3, frames)
    for s, c, f in zip((gs, other, gs), cams, frames):
        _same(frame_to_numpy(f), frame_to_numpy(tr.render(s, c, p, outputs=OUT, tune={"waves_per_cu": 19})))
    ref = oracle_mod.render(scene, cams[0], p, grid=None)
    assert_fp32_parity(compare(frame_to_numpy(frames[0]), ref, p.ao_samples, scene.n_lights))
