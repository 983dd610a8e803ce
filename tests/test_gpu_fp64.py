"""The queued FP64 renderer (no stats buffer) against the counting FP64
kernel, one thread per pixel over a plain 3D-DDA (with one): bit-identical
frames for every primitive kind and option, at frames narrower than a tile,
with rays along the axes, from inside the scene and from far away, with and
without lights and AO rays, and for an empty scene."""
import math

import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

pytestmark = pytest.mark.gpu

OUT = ("rgb", "hit_id", "ao_mask", "light_mask")


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


def _scene(kind):
    if kind == "empty":
        return scenegen.tiny_scene(n=0)
    if kind == "dark":
        return scenegen.tiny_scene(seed=3, n_lights=0)
    if kind == "sparse":  # long empty stretches between small clusters
        s = scenegen.tiny_scene(seed=5, n=40, ball_radius=2.0)
        s.sph_center[20:] += (60.0, -45.0, 30.0)
        return s
    if kind == "walk":
        return scenegen.random_walk_scene(400, 9.0, seed=6)
    s = scenegen.mixed_tiny_scene()
    if kind == "layers":
        s.sph_opacity = np.full(s.n_spheres, 0.5, np.float32)
        s.tri_opacity = np.full(s.n_triangles, 0.25, np.float32)
    return s


@pytest.mark.parametrize("kind", ["empty", "dark", "sparse", "walk", "mixed", "layers"])
@pytest.mark.parametrize("eye,size", [((0.0, 0.0, 30.0), (67, 45)), ((0.0, 0.0, 30.0), (1, 9)),
                                      ((0.3, -0.2, 0.1), (130, 97)), ((40.0, 25.0, -60.0), (311, 203)),
                                      ((0.0, 6000.0, 0.5), (64, 64))])
def test_equals_counting_kernel(tr, kind, eye, size):
    gs = tr.Scene(_scene(kind))
    fovy = 50.0 if math.dist(eye, (0, 0, 0)) < 1000.0 else 0.4
    cam = scenegen.Camera(eye, (0.0, 0.0, 0.0), (0.0, 0.1, 1.0) if eye[1] > 1000 else (0.0, 1.0, 0.0), fovy, *size)
    for p in (scenegen.Params(ao_samples=9, seed=5, specular=0.4, max_layers=5 if kind == "layers" else 0),
              scenegen.Params(ao_samples=3, seed=7, ao_maxdist=2.5, aa_samples=3),
              scenegen.Params(ao_samples=0, seed=7, background=(0.25, 0.5, 0.75))):
        got = [frame_to_numpy({k: v for k, v in tr.render(gs, cam, p, precision="fp64", outputs=OUT,
                                                          stats=st).items() if k in OUT})
               for st in (False, True)]
        for k in got[0]:
            assert np.array_equal(got[0][k], got[1][k]), k
