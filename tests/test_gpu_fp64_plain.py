"""FP64 frames with little to trace, which one thread per pixel renders without
counting: bit-identical to the counting kernel."""
import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

pytestmark = pytest.mark.gpu

OUT = ("rgb", "hit_id", "ao_mask", "light_mask")


@pytest.mark.parametrize("n,size,ao,away,layers", [(1, (640, 361), 0, False, 0), (1, (641, 360), 16, False, 0),
                                                   (64, (965, 301), 0, False, 0), (64, (400, 500), 9, True, 0),
                                                   (0, (333, 222), 4, False, 0), (64, (800, 601), 0, False, 4)])
def test_equals_counting_kernel(n, size, ao, away, layers):
    import paper_0801_1500_amd as tr
    scene = scenegen.tiny_scene(seed=4, n=n)
    if layers:
        scene.sph_opacity = np.full(n, 0.5, np.float32)
    gs = tr.Scene(scene)
    cam = scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 60.0 if away else 0.0), (0.0, 1.0, 0.0), 50.0, *size)
    p = scenegen.Params(ao_samples=ao, seed=5, max_layers=layers, background=(0.25, 0.5, 0.75))
    got = [tr.render(gs, cam, p, precision="fp64", outputs=OUT, stats=st) for st in (False, True)]
    a, b = (frame_to_numpy({k: f[k] for k in OUT}) for f in got)
    for k in OUT:
        assert np.array_equal(a[k], b[k]), k
