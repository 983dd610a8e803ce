"""FP32 frames from far away, where the walk's times round by as much as the
grid's margins: against the FP64 frames of the same view.  A hit may differ where
an edge passes within the rounding of a pixel's centre.  The camera's position
and direction and the distance each round by 2^-24 of the distance D at most, so
by 3 x 2^-24 D / p of a pixel of size p together; with an edge or two in
each direction within a pixel, 4 times that share of the pixels."""
import math

import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["balls", "mixed", "protein"])
@pytest.mark.parametrize("log2", [4, 6, 8, 9, 10])
def test_far_camera(kind, log2):
    import paper_0801_1500_amd as tr
    scene = {"balls": lambda: scenegen.tiny_scene(seed=4), "mixed": scenegen.mixed_tiny_scene,
             "protein": scenegen.protein_scene}[kind]()
    gs = tr.Scene(scene)
    lo, hi, _, _ = gs.grid_info()
    centre, ext = (lo + hi) / 2, float((hi - lo).max())
    dist, n = ext * 2.0 ** log2, 300
    for d in ((0.0, 0.0, 1.0), (1.0, 0.3, 0.2), (-0.5, 0.7, -0.4)):
        d = np.array(d) / np.linalg.norm(d)
        cam = scenegen.Camera(tuple(centre + dist * d), tuple(centre), (0.0, 1.0, 0.1),
                              2.0 * math.degrees(math.atan(0.6 * ext / dist)), n, n)
        a, b = (frame_to_numpy(tr.render(gs, cam, scenegen.Params(ao_samples=8, seed=3), precision=p))
                for p in ("fp32_resolve", "fp64"))
        wrong = np.mean(a["hit_id"] != b["hit_id"])
        assert (b["hit_id"] >= 0).sum() > 1000
        assert wrong <= 4 * 3 * 2.0 ** -24 * dist / (1.2 * ext / n), (kind, log2, wrong)
