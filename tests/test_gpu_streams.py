"""Renders on the per-thread default stream from several threads at once (one
stream handle, another stream in each): every frame as rendered alone."""
import threading

import numpy as np
import pytest

import scenegen
from parity_util import frame_to_numpy

HIP_STREAM_PER_THREAD = 2


@pytest.mark.gpu
@pytest.mark.parametrize("jobs,aa", [(1, 1), (5, 1), (1, 4)])
def test_threads_on_the_per_thread_stream(jobs, aa):
    import torch
    import paper_0801_1500_amd as tr
    scenes = [tr.Scene(scenegen.tiny_scene(seed=4 + k)) for k in range(2)]
    cams = [scenegen.Camera((2.0 * k, 1.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 50.0, 150 + 37 * k, 90)
            for k in range(4)]
    p = scenegen.Params(ao_samples=8, seed=3, aa_samples=aa)
    want = [frame_to_numpy(tr.render(scenes[k % 2], c, p)) for k, c in enumerate(cams)]
    frames = [[[tr.alloc_frame(c) for _ in range(jobs)] for _ in range(12)] for c in cams]
    torch.cuda.synchronize()

    def work(k):
        for row in frames[k]:
            tr.render_batch_into([scenes[k % 2]] * jobs, [cams[k]] * jobs, [p] * jobs, row,
                                 stream=HIP_STREAM_PER_THREAD)
        torch.cuda.ExternalStream(HIP_STREAM_PER_THREAD).synchronize()
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for k in range(4):
        for row in frames[k]:
            for f in row:
                assert np.array_equal(frame_to_numpy(f)["rgb"], want[k]["rgb"]), k
