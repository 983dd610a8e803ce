"""Scenes whose arrays lie in blocks that other scenes had before: grids and
frames the same as those of the first scenes, whatever the blocks held, for
sizes in turn (one past the 8 MB staging block), on another stream, and with
several builders at once."""
import threading

import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

pytestmark = pytest.mark.gpu

CAM = scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, 130, 67)
PARAMS = scenegen.Params(ao_samples=4, seed=3)


def _hosts():
    mixed = scenegen.mixed_tiny_scene()
    return [scenegen.tiny_scene(seed=4), mixed, scenegen.tiny_scene(seed=5, n=3000),
            scenegen.tiny_scene(seed=6, n=200000, ball_radius=100.0), scenegen.tiny_scene(seed=7, n=3100)]


def _state(tr, host, stream=None, bvh=False):
    s = tr.Scene(host, stream=stream)
    if bvh:
        s.build_bvh(stream=stream)
    frames = [tr.render(s, CAM, PARAMS, precision=p, stream=stream) for p in ("fp32_resolve", "fp64")]
    if bvh:
        frames.append(tr.render(s, CAM, PARAMS, tune={"accel": 1}, stream=stream))
    out = list(s.grid_arrays(stream=stream)) + list(s.walk_arrays(stream=stream))
    for f in frames:
        f = frame_to_numpy(f)
        out += [f[k] for k in sorted(f)]
    return s, out


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


@pytest.fixture(scope="module")
def first(tr):
    """Every scene built while all the others are held: blocks of their own."""
    got = [_state(tr, h, bvh=True) for h in _hosts()]
    for s, _ in got:
        s.destroy()
    return [g for _, g in got]


def test_sizes_in_turn(tr, first):
    import torch
    hosts = _hosts()
    other = torch.cuda.Stream()
    for k in (3, 0, 4, 1, 2, 2, 4, 0, 3, 1):
        for stream in (None, other):
            with torch.cuda.stream(other) if stream else torch.cuda.stream(torch.cuda.default_stream()):
                s, got = _state(tr, hosts[k], stream=stream, bvh=True)
            _same(got, first[k])
            s.destroy()


def test_destroyed_under_way(tr, first):
    """A scene destroyed with its render still enqueued, and the next one, of
    its size, built on another stream at once."""
    import torch
    hosts = _hosts()
    streams = [torch.cuda.Stream() for _ in range(2)]
    out = []
    for n in range(8):
        with torch.cuda.stream(streams[n % 2]):
            s = tr.Scene(hosts[2 if n % 4 < 2 else 4])
            out.append((2 if n % 4 < 2 else 4, tr.render(s, CAM, PARAMS)))
            s.destroy()
    torch.cuda.synchronize()
    for k, f in out:
        f = frame_to_numpy(f)
        _same([f[q] for q in sorted(f)], first[k][4:4 + len(f)])


def test_builders_at_once(tr, first):
    import torch
    hosts = _hosts()
    got = [[] for _ in range(4)]

    def work(n):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in [(n + q) % 5 for q in range(5)] * 2:
                s, out = _state(tr, hosts[k])
                got[n].append((k, out))
                s.destroy()
    threads = [threading.Thread(target=work, args=(n,)) for n in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for rows in got:
        assert len(rows) == 10
        for k, out in rows:
            _same(out, first[k][:len(out)])
