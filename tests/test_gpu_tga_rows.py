"""The Targa writer's rows at the edges of its workgroups, byte for byte
against the oracle: widths about whole waves and whole steps (8 pixels a
thread, 1,024 threads: 8,192 pixels), runs and raw stretches across the step,
and images and files at every byte alignment."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tr():
    import paper_0801_1500_amd as tr
    tr.lib()
    return tr


def _image(kind, h, w, seed):
    rng = np.random.default_rng(seed)
    if kind == "noise":
        return rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
    if kind == "flat":
        return np.full((h, w, 3), seed % 251, np.uint8)
    run = rng.integers(1, 200, size=h * w)  # runs of every length, some of one pixel
    val = rng.integers(0, 256, (h * w, 3), dtype=np.uint8)
    run[rng.random(h * w) < 0.5] = 1
    return np.repeat(val, run, axis=0)[:h * w].reshape(h, w, 3)


@pytest.mark.parametrize("w", [7, 8, 9, 511, 512, 513, 3860, 8191, 8192, 8193, 8320, 16385])
def test_widths(tr, oracle_mod, w):
    import torch
    for kind in ("noise", "flat", "runs"):
        img = _image(kind, 5, w, w)
        print("tga rows", kind, w, flush=True)
        got = tr.encode_tga(torch.from_numpy(img).cuda()).cpu().numpy().tobytes()
        assert got == oracle_mod.tga_encode(img), kind


@pytest.mark.parametrize("shift", range(4))
def test_alignments(tr, oracle_mod, shift):
    import torch
    for w in (1, 2, 21, 777, 8195):
        img = _image("runs", 3, w, w + shift)
        n = img.size
        src = torch.zeros(n + 8, dtype=torch.uint8, device="cuda")
        src[shift:shift + n] = torch.from_numpy(img.reshape(-1)).cuda()
        buf = torch.full((tr.tga_max_bytes(w, 3) + 8,), 9, dtype=torch.uint8, device="cuda")
        out = tr.encode_tga(src[shift:shift + n].reshape(3, w, 3), out=buf[3 - shift:-4])
        want = oracle_mod.tga_encode(img)
        assert out.cpu().numpy().tobytes() == want
        rest = buf.cpu().numpy()
        assert (rest[:3 - shift] == 9).all() and (rest[3 - shift + len(want):] == 9).all()
