"""The linear BVH at the sizes where its build changes: one and two box chunks
(512 leaves), several sort tiles (1024 keys), the last small tree and the first
large one (131,072 leaves); and walks whose stack grows past the entries that
LDS holds."""
import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy
from test_gpu_bvh import OUT, check_bvh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


def _spheres(c, r):
    z3 = np.zeros((0, 3))
    ld = np.array([[0.3, 0.4, 1.0]])
    return scenegen.Scene(np.asarray(c, np.float64), np.asarray(r, np.float64),
                          np.full((len(r), 3), 0.6, np.float32), z3, z3.copy(), np.zeros(0),
                          np.zeros((0, 3), np.float32), ld, np.ones_like(ld))


@pytest.mark.parametrize("n", [3, 512, 513, 514, 1024, 1025, 1537, 131072, 131073])
def test_tree_at_chunk_edges(tr, n):
    rng = np.random.default_rng(n)
    # a third of the centres on few points, so codes repeat across chunk ends
    c = rng.uniform(-20.0, 20.0, (n, 3))
    c[: n // 3] = np.repeat(c[:8], (n // 3 + 7) // 8, axis=0)[: n // 3]
    s = _spheres(c, rng.uniform(0.05, 0.3, n))
    print("bvh build", n, flush=True)
    gs = tr.Scene(s)
    gs.build_bvh()
    nodes = check_bvh(gs, s)
    # every inner child's box is the union of its own children's, exactly:
    # the outward rounding of the records is monotone
    lo = np.minimum(nodes[:, 0:3], nodes[:, 6:9])
    hi = np.maximum(nodes[:, 3:6], nodes[:, 9:12])
    kids = nodes[:, 12:14].copy().view(np.int32)
    for side in (0, 1):
        k = kids[:, side]
        q = k >= 0
        assert np.array_equal(nodes[q, 6 * side:6 * side + 3], lo[k[q]])
        assert np.array_equal(nodes[q, 6 * side + 3:6 * side + 6], hi[k[q]])


def _largest_stack(nodes, org, d):
    # entries that a near-first walk of the ray holds at most, nothing hit
    kids = nodes[:, 12:14].copy().view(np.int32)
    stack, best, item = [], 0, 0
    while True:
        if item >= 0:
            t = []
            for side in (0, 1):
                b = nodes[item, 6 * side:6 * side + 6].astype(np.float64)
                t0, t1 = (b[:3] - org) / d, (b[3:] - org) / d
                a, z = np.minimum(t0, t1).max(), np.maximum(t0, t1).min()
                t.append(max(a, 0.0) if z >= max(a, 0.0) else None)
            hit = [(t[q], int(kids[item, q])) for q in (0, 1) if t[q] is not None]
            hit.sort(key=lambda x: x[0])
            if len(hit) == 2:
                stack.append(hit[1][1])
                best = max(best, len(stack))
            if hit:
                item = hit[0][1]
                continue
        if not stack:
            return best
        item = stack.pop()


@pytest.mark.parametrize("side", [-1.0, 1.0])
def test_deep_stack_walk_equals_grid(tr, side):
    # spheres closing in by halves on a corner that holds 4096 equal ones: a
    # chain of splits, then 12 levels whose boxes are all the same; a ray along
    # the diagonal from the corner's side meets both children at every level
    p = [[32.0 * 0.5 ** k] * 3 for k in range(8)] + [[0.0, 0.0, 0.0]] * 4096
    s = _spheres(p, np.full(len(p), 0.06))
    gs = tr.Scene(s)
    gs.build_bvh()
    nodes = check_bvh(gs, s)
    lo, hi, _, _ = gs.grid_info()
    d = np.ones(3)
    d /= np.linalg.norm(d)
    depth = _largest_stack(nodes, -200.0 * d - 0.5 * (lo + hi), d)
    eye = tuple(side * 60.0 * d)
    c = scenegen.Camera(eye, (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 0.25, 64, 64)
    prm = scenegen.Params(ao_samples=16, seed=3)
    print("bvh deep", side, gs.bvh_depth(), depth, flush=True)
    assert depth > 16
    import torch
    res = []
    for accel in (1, 0):
        fr = tr.render(gs, c, prm, precision="fp32_resolve", outputs=OUT, tune={"accel": accel})
        torch.cuda.synchronize()
        res.append(frame_to_numpy(fr))
    assert (res[0]["hit_id"] >= 0).sum() > 200
    for k in OUT:
        assert np.array_equal(res[0][k], res[1][k]), k
