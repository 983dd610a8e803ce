"""Scene memory on a model of the HIP runtime (no GPU): freed blocks are kept
for the next scene only when nothing can still be using them, they are given
back when memory runs out, and one builder at a time has the staging block."""
import ctypes as C
import threading

import pytest

import hip_model
import scenegen
from test_host_launch import _job, _render


def _scene(tr, seed=4, n=64):
    return tr.Scene(scenegen.tiny_scene(seed=seed, n=n))


def other_device(model, tr):
    """A scene destroyed or rebuilt while another device is current: its own
    device is waited for before its blocks can go to another scene."""
    hip = C.CDLL(hip_model.LIB)
    for what in ("destroy", "rebuild", "bvh"):
        hip.hipSetDevice(0)
        s = _scene(tr)
        s.build_bvh()
        assert _render(tr, "render", [_job(tr, s, 64, 64)]) == 0
        assert model.model_pending(0) > 0
        hip.hipSetDevice(1)
        if what == "destroy":
            s.destroy()
        elif what == "rebuild":
            s.rebuild(cells_per_prim=200000.0)  # (a larger grid: its old blocks are freed)
        else:
            s.build_bvh()
        assert model.model_pending(0) == 0, what
        now = C.c_int(-1)
        hip.hipGetDevice(C.byref(now))
        assert now.value == 1
        hip.hipSetDevice(0)
        s.destroy()


def failed_wait(model, tr):
    """Where the device cannot be waited for (a capture under way), blocks are
    given to the runtime, which waits by itself, and none are kept."""
    s = _scene(tr)
    s.destroy()
    held, frees = model.model_used(0), model.model_frees()
    s = _scene(tr)
    assert model.model_used(0) == held  # (the same blocks again)
    model.model_fail_sync(1)
    s.destroy()
    model.model_fail_sync(0)
    assert model.model_frees() - frees >= 20  # (what is left: the upload's block, idle since)
    assert model.model_used(0) < held / 8, model.model_used(0)
    assert model.model_misuse() == 0


def out_of_memory(model, tr):
    """Every device allocation of the library gets the kept blocks back when
    the device has nothing left."""
    L = tr.lib()
    s = _scene(tr)

    def aa():
        return _render(tr, "render", [_job(tr, s, 300, 300, aa_samples=4)], 0x5000)

    def table():
        return _render(tr, "batch", [_job(tr, s, 64, 64)] * 300, 0x6000)

    def graph():
        return _render(tr, "graph", [_job(tr, s, 64, 64)] * 30)

    def targa():
        size = C.c_int64()
        img, out = (C.c_uint8 * 48)(), (C.c_uint8 * 256)()
        return L.tr_frame_encode_tga(img, 4, 4, out, 256, C.byref(size), 0x7000)

    def scene():
        _scene(tr, n=700)
        return 0

    for op in (aa, table, graph, targa, scene):
        _scene(tr, n=40000).destroy()
        held = model.model_used(0)
        assert held > 4 << 20
        model.model_capacity(0, held)
        assert op() == 0, (op.__name__, L.tr_last_error())
        assert model.model_used(0) < held
        model.model_capacity(0, 1 << 50)
    assert model.model_misuse() == 0


def host_out_of_memory(model, tr):
    """No C++ exception leaves a scene call when the host runs out of memory
    while a block is taken or given back."""
    _scene(tr).destroy()
    for k in range(2000):
        model.model_fail_new(k + 1)  # (the scene itself is made)
        try:
            s = _scene(tr)
        except tr.TRError as e:
            assert e.status == tr.TR_ENOMEM, str(e)
            s = None
        done = not model.model_failed_new()
        model.model_fail_new(-1)
        if s:
            s.destroy()
        if done:
            break
    assert done and k > 20
    for k in range(2000):
        s = _scene(tr)
        model.model_fail_new(k)
        s.destroy()
        done = not model.model_failed_new()
        model.model_fail_new(-1)
        if done:
            break
    assert done and model.model_misuse() == 0


def failed_bvh(model, tr):
    """A BVH build that fails leaves no tree to walk, also where there was one."""
    s = _scene(tr, n=2000)
    s.build_bvh()
    def walk():
        scene, cam, p, f = _job(tr, s, 64, 64)
        return tr.lib().tr_render_tuned(scene.handle, C.byref(cam), C.byref(p), C.byref(f),
                                        C.byref(tr.make_tune({"accel": 1})), None)
    assert walk() == 0
    model.model_capacity(0, model.model_used(0))
    with pytest.raises(Exception):
        _scene(tr, n=300000)  # (the kept blocks are given back)
    model.model_capacity(0, model.model_used(0))
    with pytest.raises(Exception):
        s.build_bvh()
    assert walk() != 0


def changing_sizes(model, tr):
    """Blocks of sizes that do not come back make room for later ones: after
    any mix of scenes the next of a size finds the last one's blocks, and no
    more is kept than the limit."""
    for k in range(40):  # some 500 blocks of different sizes, 300 MB
        _scene(tr, n=1000 + 1700 * k).destroy()
        assert model.model_used(0) <= 256 << 20
    for _ in range(2):
        _scene(tr, n=20000).destroy()
    n = model.model_mallocs()
    for _ in range(3):
        s = _scene(tr, n=20000)
        s.destroy()
    assert model.model_mallocs() == n, model.model_mallocs() - n
    assert model.model_misuse() == 0


def footprint(model, tr):
    """tr_scene_footprint is what the scene takes from the device."""
    for n, cells in ((1, 0.0), (64, 0.0), (5000, 0.0), (5000, 3.0)):
        for bvh in (False, True):
            s = tr.Scene(scenegen.tiny_scene(seed=4, n=n), cells_per_prim=cells)
            if bvh:
                s.build_bvh()
            used, held = model.model_used(0), s.footprint()
            model.model_fail_sync(1)  # (so that its blocks are freed, not kept)
            s.destroy()
            model.model_fail_sync(0)
            assert held == used - model.model_used(0), (n, bvh, held, used - model.model_used(0))


def two_builders(model, tr):
    """A build whose upload is under way keeps the staging block: others copy
    array by array, and neither sees the other's arrays.  Nor does a build of
    more than the block's 8 MB wait for it."""
    _scene(tr).destroy()
    model.model_hold_copy()
    t = threading.Thread(target=lambda: _scene(tr, seed=1, n=3000))
    t.start()
    model.model_await_held()
    _scene(tr, seed=2, n=3000)
    _scene(tr, seed=3, n=300000)
    model.model_release_copy()
    t.join()
    assert model.model_staged_changed() == 0 and model.model_misuse() == 0


def test_two_builders():
    hip_model.run("test_host_memory", "two_builders")


def test_footprint():
    hip_model.run("test_host_memory", "footprint")


def test_kept_blocks_follow_the_scenes():
    hip_model.run("test_host_memory", "changing_sizes")


def test_no_exception_leaves():
    hip_model.run("test_host_memory", "host_out_of_memory")


@pytest.mark.parametrize("test", ["out_of_memory", "failed_bvh"])
def test_kept_blocks_are_given_back(test):
    hip_model.run("test_host_memory", test)


@pytest.mark.parametrize("test", ["other_device", "failed_wait"])
def test_blocks_wait_for_their_device(test):
    hip_model.run("test_host_memory", test)
