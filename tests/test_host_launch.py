"""Host side of the render launches, on a model of the HIP runtime (no GPU):
launch sizes at the runtime's limit of 2^32 work-items per dimension, and the
order of the accesses to the job tables when equal stream handles are not one
stream, under capture and with tables that grow."""
import ctypes as C
import threading

import numpy as np
import pytest

import hip_model
import scenegen

LIMIT = 2 ** 26  # one-wave workgroups the runtime no longer launches


def _job(tr, scene, width, height, precision="fp32_resolve", **params):
    """One job's arguments; the frame's address is never read here."""
    cam = scenegen.Camera((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, width, height)
    p = scenegen.Params(ao_samples=4, seed=3, **params)
    f = tr.Frame(0x1000000, None, None, None, None)
    return scene, tr.make_camera(cam), tr.make_params(p, precision), f


def _render(tr, entry, jobs, stream=None):
    n = len(jobs)
    sc = (C.c_void_p * n)(*[j[0].handle for j in jobs])
    cm, pr, fr = ((t * n)(*[j[k] for j in jobs]) for k, t in ((1, tr.Camera), (2, tr.Params), (3, tr.Frame)))
    L = tr.lib()
    if entry == "render":
        return L.tr_render(sc[0], cm, pr, fr, stream)
    if entry == "batch":
        return L.tr_render_batch(n, sc, cm, pr, fr, stream)
    if entry == "noalloc":
        return L.tr_render_batch_noalloc(n, sc, cm, pr, fr, None, stream)
    g = C.c_void_p()
    return L.tr_graph_create(n, sc, cm, pr, fr, None, stream, C.byref(g))


def large_fp32(model, tr):
    """Frames up to the limit in one workgroup per entry, larger ones on
    persistent waves, through every entry point."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for entry in ("render", "batch", "noalloc", "graph"):
        # (one-pixel rows: a tile each; the last tiles are split in four)
        for tiles in (LIMIT // 2, LIMIT - 2000000, LIMIT - 600000, LIMIT - 1, LIMIT, 2 * LIMIT - 1, 2 * LIMIT + 1):
            assert _render(tr, entry, [_job(tr, s, 1, tiles)]) == 0, (entry, tiles, tr.lib().tr_last_error())
            name, grid, block = hip_model.launches(model)[-1]
            assert "k_render_wave" in name and grid * block < 2 ** 32
            assert (grid < tiles) == (tiles >= LIMIT - 600000), (entry, tiles, grid)
    assert _render(tr, "render", [_job(tr, s, 3860, 4548, aa_samples=256)]) == 0, tr.lib().tr_last_error()
    assert _render(tr, "batch", [_job(tr, s, 1024, 1024)] * 4096) == 0, tr.lib().tr_last_error()


def wide(model, tr):
    """Rows and columns of up to 2^31 - 2 pixels (a tile of the default shape is
    64 x 1)."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for w, h, tiles in ((2 ** 31 - 65, 1, 2 ** 25 - 1), (2 ** 31 - 2, 1, 2 ** 25), (1, 2 ** 31 - 2, 2 ** 31 - 2)):
        assert tr.tile_count(w, h) == tiles
        assert _render(tr, "render", [_job(tr, s, w, h)]) == 0, (w, h, tr.lib().tr_last_error())
        name, grid, _ = hip_model.launches(model)[-1]
        assert "k_render_wave" in name
        assert (tiles <= grid < 1.05 * tiles) if tiles < LIMIT else ("ILi2E" in name), (w, h, name, grid)


def large_fp64(model, tr):
    """Narrow FP64 frames of 2^26 tiles and more: all entries in launches that
    the runtime takes."""
    model.model_radius(10.0)
    s = tr.Scene(scenegen.tiny_scene(seed=4, n=20000))  # (objects enough for the queued kernel)
    for height in (8 * 5000, 8 * (LIMIT - 1), 8 * LIMIT, 2 ** 31 - 2):
        before = len(hip_model.launches(model))
        job = _job(tr, s, 1, height, "fp64")
        job[2].ao_samples = 16
        assert _render(tr, "render", [job]) == 0, (height, tr.lib().tr_last_error())
        grids = [g for n, g, b in hip_model.launches(model)[before:] if "k_render_f64" in n]
        tiles = (height + 7) // 8
        split = int(60.0 * tiles ** 0.5)
        assert tiles <= sum(grids) <= tiles + 3 * split + 4096, (height, grids)
        assert all(g % 8 == 0 for g in grids)  # (a workgroup's XCD is its number mod 8)


def tables_per_thread_stream(model, tr):
    """hipStreamPerThread is one handle and another stream in every thread."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for n in (1, 3, 5, 20):
        for rounds in (1, 9, 2):
            def work():
                for _ in range(rounds):
                    assert _render(tr, "batch", [_job(tr, s, 64, 64)] * n, 2) == 0
            t = threading.Thread(target=work)
            t.start()
            t.join()
    assert model.model_races() == 0, model.model_races()


def planes_per_thread_stream(model, tr):
    """The workspace of antialiased frames, on the stream that is another one in
    every thread, at one size and while it grows."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for w in (64, 32, 65, 64):
        for entry, precision in (("render", "fp32_resolve"), ("batch", "fp32_resolve"), ("batch", "fp64")):
            def work():
                for _ in range(2):
                    assert _render(tr, entry, [_job(tr, s, w, 64, precision, aa_samples=3)], 2) == 0
            t = threading.Thread(target=work)
            t.start()
            t.join()
    assert model.model_races() == 0 and model.model_misuse() == 0


def rows_per_thread_stream(model, tr):
    """The Targa encoder's row offsets, on the stream that is another one in
    every thread."""
    size = C.c_int64()
    for height in (64, 32, 65, 64):
        def work():
            for _ in range(2):
                assert tr.lib().tr_frame_encode_tga(0x1000000, 64, height, 0x2000000, 1 << 20, C.byref(size), 2) == 0
        t = threading.Thread(target=work)
        t.start()
        t.join()
    assert model.model_races() == 0


def planes_of_two_threads(model, tr):
    """A frame whose sample jobs are under way keeps the workspace until its
    folds are enqueued: a larger frame of another thread on the stream waits."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    def frame(w):
        assert _render(tr, "render", [_job(tr, s, w, 64, aa_samples=8)], 0x5000) == 0
    frame(64)
    model.model_hold_copy()  # (of the first frame's 8 jobs)
    threads = [threading.Thread(target=frame, args=(w,)) for w in (64, 128)]
    threads[0].start()
    model.model_await_held()
    threads[1].start()
    threads[1].join(0.5)
    model.model_release_copy()
    for t in threads:
        t.join()
    assert model.model_misuse() == 0


def tables_under_capture(model, tr):
    """Captured renders wait for nothing on the host and leave nothing behind
    that a later render could not wait for."""
    s = tr.Scene(scenegen.tiny_scene(seed=4))
    for n in (1, 3, 5):
        for _ in range(5):  # the slots' memory
            assert _render(tr, "batch", [_job(tr, s, 64, 64)] * 5, 0x5000) == 0
        model.model_capture(0x5000, 1)
        for _ in range(5):
            assert _render(tr, "batch", [_job(tr, s, 64, 64)] * n, 0x5000) == 0, tr.lib().tr_last_error()
        model.model_capture(0x5000, 0)
        for _ in range(9):
            assert _render(tr, "batch", [_job(tr, s, 64, 64)] * n, 0x5000) == 0, tr.lib().tr_last_error()
    assert model.model_bad_waits() == 0 and model.model_races() == 0
    model.model_capture(0x6000, 1)  # another stream's capture, as another thread may have under way
    for _ in range(9):
        assert _render(tr, "batch", [_job(tr, s, 64, 64)], 0x5000) == 0, tr.lib().tr_last_error()
    assert model.model_races() == 0


def few_rays(model, tr):
    """Launches of few rays over many objects take persistent waves (two banks),
    others one workgroup per entry (one bank), through every entry point."""
    model.model_radius(10.0)  # (seen from 30 away: 0.74 of the height)
    scenes = {n: tr.Scene(scenegen.tiny_scene(seed=4, n=n)) for n in (64, 20000, 200000)}
    for n, jobs, w, h, ao, waves in (
            (200000, 1, 965, 1137, 0, True), (200000, 1, 965, 1137, 16, False), (64, 1, 965, 1137, 0, False),
            (200000, 64, 256, 256, 4, True), (64, 64, 256, 256, 4, False), (200000, 1, 128, 128, 0, False),
            (200000, 1, 3860, 4548, 0, True), (64, 1, 3860, 4548, 0, False), (20000, 64, 256, 256, 0, True), (20000, 1, 965, 1137, 0, False)):
        for entry in ("render", "batch", "noalloc", "graph"):
            if (entry == "render" and jobs > 1) or (entry == "noalloc" and jobs > 16):
                continue
            job = list(_job(tr, scenes[n], w, h))
            job[2].ao_samples = ao
            assert _render(tr, entry, [tuple(job)] * jobs) == 0
            name, grid, _ = hip_model.launches(model)[-1]
            assert ("k_render_waveILi2E" in name) == waves, (n, jobs, w, h, ao, entry, name)
    glass = scenegen.tiny_scene(seed=4, n=200000)
    glass.sph_opacity = np.full(200000, 0.5, np.float32)
    corners = np.random.default_rng(1).normal(size=(200000, 3, 3))
    kinds = {"layers": tr.Scene(glass), "triangles": tr.Scene(scenegen.with_triangles(scenegen.tiny_scene(n=0), corners))}
    for kind, jobs, w, h, ao, waves in (
            ("layers", 64, 256, 256, 0, True), ("layers", 64, 256, 256, 8, False), ("layers", 1, 965, 1137, 0, False),
            ("triangles", 64, 256, 256, 8, True), ("triangles", 64, 256, 256, 32, False),
            ("triangles", 1, 965, 1137, 0, True), ("triangles", 1, 965, 1137, 16, False)):
        job = list(_job(tr, kinds[kind], w, h))
        job[2].ao_samples, job[2].max_layers = ao, 4
        assert _render(tr, "batch", [tuple(job)] * jobs) == 0
        name = hip_model.launches(model)[-1][0]
        assert ("k_render_waveILi2E" in name) == waves, (kind, jobs, w, h, ao, name)
    away = list(_job(tr, scenes[200000], 965, 1137))
    away[2].ao_samples = 0
    away[1].lookat[2] = 60.0
    assert _render(tr, "render", [tuple(away)]) == 0  # (nothing to be seen)
    assert "k_render_waveILi1E" in hip_model.launches(model)[-1][0]


def fp64_kernels(model, tr):
    """FP64 frames with little to trace go to one thread per pixel, others to
    the queued kernel."""
    model.model_radius(10.0)
    scenes = {n: tr.Scene(scenegen.tiny_scene(seed=4, n=n)) for n in (1, 64, 20000)}
    for n, w, h, ao, away, plain in (
            (1, 1920, 1080, 0, False, True), (1, 1920, 1080, 16, False, True), (1, 128, 128, 16, False, False),
            (64, 965, 1137, 0, False, True), (64, 965, 1137, 16, False, False), (64, 128, 128, 8, False, False),
            (20000, 965, 1137, 0, False, False), (20000, 965, 1137, 16, False, False),
            (20000, 965, 1137, 16, True, True)):
        job = _job(tr, scenes[n], w, h, "fp64")
        job[2].ao_samples = ao
        if away:
            job[1].lookat[2] = 60.0
        for entry in ("render", "batch", "noalloc"):
            assert _render(tr, entry, [job]) == 0
            name = hip_model.launches(model)[-1][0]
            assert ("k_render_plain_f64ILb0ELb0E" in name) == plain, (n, w, h, ao, away, entry, name)
    glass = scenegen.tiny_scene(seed=4)
    glass.sph_opacity = np.full(64, 0.5, np.float32)
    for ao, plain in ((0, True), (16, False)):
        job = _job(tr, tr.Scene(glass), 965, 1137, "fp64")
        job[2].ao_samples, job[2].max_layers = ao, 4
        for entry in ("render", "batch", "noalloc"):
            assert _render(tr, entry, [job]) == 0
            name = hip_model.launches(model)[-1][0]
            assert ("k_render_plain_f64ILb0ELb1E" in name) == plain, (ao, entry, name)


@pytest.mark.parametrize("test", ["few_rays", "fp64_kernels"])
def test_kernel_choice(test):
    hip_model.run("test_host_launch", test)


@pytest.mark.parametrize("test", ["tables_per_thread_stream", "tables_under_capture",
                                  "planes_per_thread_stream", "rows_per_thread_stream",
                                  "planes_of_two_threads"])
def test_job_tables(test):
    hip_model.run("test_host_launch", test)


@pytest.mark.parametrize("test", ["large_fp32", "large_fp64", "wide"])
def test_launch_sizes(test):
    hip_model.run("test_host_launch", test)
