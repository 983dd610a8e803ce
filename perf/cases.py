"""Timed cases of the ray caster's public entry points.

Each case is one thing a program does with the library over and over: a small
interactive still, a step of a render service, a frame of a moving molecule
(grid rebuilt, then rendered) at the two resolutions of the paper's renders,
an orbit through a captured graph, the double-precision frame, the BVH walk,
triangle surfaces, transparency, antialiasing, the whole way from host arrays
to an image file, and the 8-bit image output alone.

Scenes are chains of atoms (spheres) and bonds (cylinders) folded into a ball
at a protein's density (26,318 objects in a ball of radius 40; the orbit's a million in one of radius
250), or closed icosphere blobs in such a ball; the camera looks at the ball
from three radii.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_0801_1500_amd as tr

LIGHTS = [(-0.5, 0.5, 1.0), (1.0, 2.0, 0.5)]
PALETTE = np.array([[0.80, 0.30, 0.30], [0.30, 0.75, 0.35], [0.30, 0.45, 0.80], [0.80, 0.75, 0.30]],
                   dtype=np.float32)
CHAIN = 128     # atoms of one chain
STEP = 1.5      # distance between the atoms of a chain
EPS = 1e-4      # where a secondary ray starts


# ------------------------------------------------------------------ cases

def _case(name, path, objects, width, height, samples, **more):
    c = {"path": path, "objects": objects, "width": width, "height": height, "samples": samples,
         "kind": "chains", "precision": "fp32_resolve", "jobs": 1, "aa": 1, "layers": 0,
         "specular": 0.0, "masks": False}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: an interactive still of a few atoms, with the hit
        # ids and masks that picking reads
        _case("still_128", "render", 64, 128, 128, 8, kind="balls", masks=True),
        # one step of a render service: requests of mixed sizes over resident
        # scenes of 2,000 to 200,000 objects, one launch
        _case("service_step", "batch", 20000, 1920, 1080, 16, jobs=6),
        # a frame of a moving molecule at the paper's lower resolution ...
        _case("frame_965x1137", "frame", 26318, 965, 1137, 16),
        # ... and at its higher one: the headline frame
        _case("frame_3860x4548", "frame", 26318, 3860, 4548, 16),
        # views around a very large scene, replayed from a captured graph with
        # new cameras
        _case("orbit_8x1080p", "graph", 1000000, 1920, 1080, 32, kind="sparse", jobs=8),
        # the frame in double precision, as the paper renders
        _case("double_965x1137", "render", 26318, 965, 1137, 16, precision="fp64"),
        # the alternative acceleration structure: built, then walked
        _case("bvh_965x1137", "bvh", 26318, 965, 1137, 16),
        # a molecular surface: triangles
        _case("surface_1930x2274", "render", 26560, 1930, 2274, 16, kind="surface", masks=True),
        # atoms drawn half transparent, up to four surfaces a pixel
        _case("glass_965x1137", "render", 26318, 965, 1137, 16, kind="glass", layers=4),
        # a picture for print: four primary samples a pixel and a highlight
        _case("print_965x1137", "render", 26318, 965, 1137, 16, aa=4, specular=0.3),
        # host arrays to the bytes of an image file, once per scene
        _case("arrays_to_tga", "pipeline", 26318, 965, 1137, 16),
        # image output of a large frame: 8-bit conversion and the Targa file
        _case("image_3860x4548", "image", 26318, 3860, 4548, 16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["render", "render", "render", "frame", "frame", "batch", "graph", "bvh",
                       "pipeline", "image"])
    px = _log(rng, 12000, 2200000)
    aspect = rng.uniform(0.6, 1.8)
    w, h = max(16, int(math.sqrt(px * aspect))), max(16, int(math.sqrt(px / aspect)))
    n = _log(rng, 64, 200000)
    c = _case("", path, n, w, h, rng.randint(4, 32))
    if path == "render":
        c["kind"] = rng.choice(["balls", "chains", "surface", "glass"])
        c["masks"] = rng.random() < 0.5
        c["precision"] = rng.choice(["fp32_resolve", "fp32_resolve", "fp32", "fp64"])
        if c["kind"] == "glass":
            c["layers"] = rng.randint(2, 8)
        elif rng.random() < 0.3 and px < 1100000:
            c["aa"] = rng.randint(2, 8)
            c["specular"] = rng.choice([0.0, 0.3])
        if c["precision"] == "fp64":  # the slow path: frames of up to a megapixel
            c["width"], c["height"], c["aa"] = min(w, 965), min(h, 1137), 1
    elif path == "bvh":
        c["kind"] = rng.choice(["chains", "surface"])
    elif path == "batch":
        c["jobs"] = rng.randint(2, 8)
    elif path == "graph":
        c["jobs"] = rng.randint(1, 6)
        c["objects"] = _log(rng, 2000, 500000)
        c["kind"] = rng.choice(["chains", "sparse"])
    elif path == "image":
        px = _log(rng, 12000, 17500000)
        c["width"] = max(16, int(math.sqrt(px * aspect)))
        c["height"] = max(16, int(math.sqrt(px / aspect)))
    return c


# ----------------------------------------------------------------- inputs

def _unit(rng, n):
    v = rng.standard_normal((n, 3))
    return v / np.maximum(np.sqrt((v * v).sum(axis=1)), 1e-12)[:, None]


def _in_ball(rng, n, radius):
    return _unit(rng, n) * (radius * np.cbrt(rng.random(n)))[:, None]


def _radius(case, objects=None):
    n = case["objects"] if objects is None else objects
    if case["kind"] == "balls":
        return 10.0 * (n / 64.0) ** (1.0 / 3.0)
    if case["kind"] == "sparse":
        return 250.0 * (n / 1e6) ** (1.0 / 3.0)
    return 40.0 * (n / 26318.0) ** (1.0 / 3.0)


def _chains(rng, n, radius):
    """n spheres and n bonds: chains of CHAIN atoms folded into the ball, a
    bond from each atom to the next place of its chain."""
    m = -(-n // CHAIN)
    p = _in_ball(rng, m, radius)
    places = [p]
    for _ in range(CHAIN):
        p = p + STEP * _unit(rng, m)
        r = np.sqrt((p * p).sum(axis=1))
        out = r > radius
        p[out] *= ((2.0 * radius - r[out]) / r[out])[:, None]
        places.append(p)
    at = np.stack(places, axis=1)
    return at[:, :-1].reshape(-1, 3)[:n].copy(), at[:, 1:].reshape(-1, 3)[:n].copy()


def _icosphere():
    """Unit icosphere of 320 faces, as vertices [320, 3, 3]."""
    g = (1.0 + math.sqrt(5.0)) / 2.0
    v = np.array([(-1, g, 0), (1, g, 0), (-1, -g, 0), (1, -g, 0), (0, -1, g), (0, 1, g), (0, -1, -g),
                  (0, 1, -g), (g, 0, -1), (g, 0, 1), (-g, 0, -1), (-g, 0, 1)]) / math.sqrt(1.0 + g * g)
    f = np.array([(0, 11, 5), (0, 5, 1), (0, 1, 7), (0, 7, 10), (0, 10, 11), (1, 5, 9), (5, 11, 4),
                  (11, 10, 2), (10, 7, 6), (7, 1, 8), (3, 9, 4), (3, 4, 2), (3, 2, 6), (3, 6, 8), (3, 8, 9),
                  (4, 9, 5), (2, 4, 11), (6, 2, 10), (8, 6, 7), (9, 8, 1)])
    t = v[f]
    for _ in range(2):
        m = t + np.roll(t, -1, axis=1)
        m /= np.sqrt((m * m).sum(axis=2, keepdims=True))
        t = np.concatenate([np.stack([t[:, 0], m[:, 0], m[:, 2]], 1), np.stack([t[:, 1], m[:, 1], m[:, 0]], 1),
                            np.stack([t[:, 2], m[:, 2], m[:, 1]], 1), m])
    return t


def _scene(case, seed, objects=None):
    """Host arrays of one scene, from the seed."""
    rng = np.random.default_rng(seed)
    n = case["objects"] if objects is None else objects
    radius = _radius(case, n)
    zero3, zero = np.zeros((0, 3)), np.zeros(0)
    s = SimpleNamespace(
        sph_center=zero3, sph_radius=zero, sph_rgb=np.zeros((0, 3), np.float32), cyl_a=zero3, cyl_b=zero3,
        cyl_radius=zero, cyl_rgb=np.zeros((0, 3), np.float32), light_dir=np.array(LIGHTS),
        light_rgb=np.ones((len(LIGHTS), 3)), sph_opacity=None, cyl_opacity=None, tri_v=None, tri_rgb=None,
        tri_opacity=None)
    if case["kind"] == "surface":  # closed blobs of 320 triangles, each turned its own way
        unit = _icosphere()
        m = max(1, n // unit.shape[0])
        q, r = np.linalg.qr(rng.normal(size=(m, 3, 3)))
        q = q * np.sign(np.diagonal(r, axis1=1, axis2=2))[:, None, :]
        turned = np.matmul(unit.reshape(1, -1, 3), q.transpose(0, 2, 1)).reshape(m, -1, 3, 3)
        s.tri_v = (_in_ball(rng, m, radius)[:, None, None, :] + 4.0 * turned).reshape(-1, 3, 3)
        s.tri_rgb = PALETTE[(np.arange(s.tri_v.shape[0]) // unit.shape[0]) % 4]
        return s
    if case["kind"] == "balls":
        s.sph_center = _in_ball(rng, n, radius)
        s.sph_radius = rng.uniform(0.5, 1.5, n)
    else:
        k = max(1, n // 2)
        s.sph_center, end = _chains(rng, k, radius)
        s.sph_radius = rng.uniform(1.2, 1.9, k)
        s.cyl_a, s.cyl_b, s.cyl_radius = s.sph_center, end, np.full(k, 0.3)
        s.cyl_rgb = PALETTE[np.arange(k) % 4]
        if case["kind"] == "glass":
            s.sph_opacity = np.full(k, 0.5, np.float32)
    s.sph_rgb = PALETTE[np.arange(s.sph_radius.shape[0]) % 4]
    return s


def _camera(case, angle, radius, width=None, height=None):
    d = 3.0 * radius
    return SimpleNamespace(eye=(d * math.sin(angle), 0.0, d * math.cos(angle)), lookat=(0.0, 0.0, 0.0),
                           up=(0.0, 1.0, 0.0), fovy_deg=50.0, width=width or case["width"],
                           height=height or case["height"])


def _params(case, seed, view=0, samples=None):
    return SimpleNamespace(light_rescale=0.3, skylight=1.0, ao_samples=samples or case["samples"],
                           ao_maxdist=math.inf, seed=seed, view_id=view, background=(0.0, 0.0, 0.0),
                           aa_samples=case["aa"], specular=case["specular"], shininess=20.0,
                           max_layers=case["layers"])


def _requests(case):
    """The requests of a batch: the largest is the case's own size, the others
    smaller (objects from a tenth to ten times the case's)."""
    rng = np.random.default_rng(case["objects"] + 77)
    out = []
    for j in range(case["jobs"]):
        n = int(min(200000, max(64, case["objects"] * math.exp(rng.uniform(-2.3, 2.3)))))
        k = 1.0 if j == 0 else float(rng.uniform(0.15, 1.0))
        out.append((n, max(16, int(case["width"] * k)), max(16, int(case["height"] * k)),
                    int(rng.integers(4, case["samples"] + 1)) if j else case["samples"],
                    float(rng.uniform(0.0, 2.0 * math.pi))))
    return out


def _angle(seed):
    return float(np.random.default_rng(seed + 55).uniform(0.0, 2.0 * math.pi))


def prepare(case, seed):
    s = SimpleNamespace(case=case, path=case["path"], precision=case["precision"])
    outs = ("rgb", "hit_id", "ao_mask", "light_mask") if case["masks"] else ("rgb",)
    radius = _radius(case)
    if s.path == "batch":
        req = _requests(case)
        s.scenes = [tr.Scene(_scene(case, seed + 1000 * j, r[0])) for j, r in enumerate(req)]
        s.cams = [_camera(case, r[4], _radius(case, r[0]), r[1], r[2]) for r in req]
        s.params = [_params(case, seed + j, 0, r[3]) for j, r in enumerate(req)]
        s.frames = [tr.alloc_frame(c, outs) for c in s.cams]
        return s
    if s.path == "graph":
        s.scene = tr.Scene(_scene(case, seed))
        k, a = case["jobs"], _angle(seed)
        s.cams = [_camera(case, a + 2.0 * math.pi * j / k, radius * 2.5 / 3.0) for j in range(k)]
        s.params = [_params(case, seed, j) for j in range(k)]
        s.frames = [tr.alloc_frame(c, outs) for c in s.cams]
        s.graph = tr.Graph([s.scene] * k, s.cams, s.params, s.frames, s.precision)
        return s
    s.cam = _camera(case, _angle(seed), radius)
    s.params = _params(case, seed)
    s.host = _scene(case, seed)
    if s.path in ("pipeline", "image"):  # room for the longest file, on the GPU and on the host
        n = tr.tga_max_bytes(s.cam.width, s.cam.height)
        s.file = torch.zeros(n, dtype=torch.uint8, device="cuda")
    if s.path == "pipeline":
        s.bytes = torch.zeros(n, dtype=torch.uint8, pin_memory=True)
        return s
    s.scene = tr.Scene(s.host)
    s.frame = tr.alloc_frame(s.cam, outs)
    if s.path == "image":  # a rendered frame waits to be written out
        tr.render_into(s.scene, s.cam, s.params, s.frame, s.precision)
    return s


# -------------------------------------------------------------------- run

def run(s):
    if s.path == "batch":
        return tr.render_batch_into(s.scenes, s.cams, s.params, s.frames, s.precision)
    if s.path == "graph":
        s.graph.update(cams=s.cams)
        s.graph.launch()
        return s.frames
    if s.path == "pipeline":
        scene = tr.Scene(s.host)
        frame = tr.render(scene, s.cam, s.params, s.precision, outputs=("rgb",))
        tga = tr.encode_tga(tr.quantize_rgb8(frame["rgb"]), out=s.file)
        s.bytes[:tga.numel()].copy_(tga)
        return s.bytes, tga.numel()
    if s.path == "image":
        image = tr.quantize_rgb8(s.frame["rgb"])
        tga = tr.encode_tga(image, out=s.file)
        return image, s.file, tga.numel()
    if s.path == "frame":
        s.scene.rebuild()
        return tr.render_into(s.scene, s.cam, s.params, s.frame, s.precision)
    if s.path == "bvh":
        s.scene.build_bvh()
        return tr.render_into(s.scene, s.cam, s.params, s.frame, s.precision, tune={"accel": 1})
    return tr.render_into(s.scene, s.cam, s.params, s.frame, s.precision)


# ------------------------------------------------------------------- work

def _cover(case, width, height):
    """Share of the pixels that hit the ball of objects."""
    r = math.tan(math.asin(1.0 / 3.0)) / math.tan(math.radians(25.0))
    share = 0.35 if case["kind"] == "sparse" else 0.75
    return min(1.0, share * math.pi * r * r / (4.0 * width / height))


def _frame_work(case, width, height, samples, objects):
    px = width * height
    hits = px * _cover(case, width, height) * case["aa"] * max(1, min(case["layers"], 3))
    rays = px * case["aa"] + hits * (samples + 1.5)
    # a ray meets about seven primitives at 30 operations, and is set up, drawn
    # and shaded with about as many
    flops = 250.0 * rays
    return {"bytes": px * (12 + (9 if case["masks"] else 0)) + objects * 64, "flops": flops}


def work(case):
    px = case["width"] * case["height"]
    if case["path"] == "image":  # the floats in, the 8-bit image and about 40% of it as a file out
        return {"bytes": px * (12 + 3 + 1.2), "flops": px * 6.0}
    if case["path"] == "batch":
        w = [_frame_work(case, r[1], r[2], r[3], r[0]) for r in _requests(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    w = _frame_work(case, case["width"], case["height"], case["samples"], case["objects"])
    if case["path"] == "graph":
        return {k: v * case["jobs"] for k, v in w.items()}
    if case["path"] in ("frame", "pipeline", "bvh"):  # the structure: FP64 primitives in, lists out
        w["bytes"] += case["objects"] * 200
    if case["path"] == "pipeline":
        w["bytes"] += px * 4.2
    return w


# ------------------------------------------------------------------ exact

def _philox(c0, c1, c2, c3, k0, k1):
    """Words 0 and 1 of Philox4x32-10, int64 tensors holding 32-bit words."""
    low = 0xFFFFFFFF

    def mul(m, x):
        a, b = m * (x & 0xFFFF), m * (x >> 16)
        lo = (a + ((b & 0xFFFF) << 16))
        return ((b >> 16) + (lo >> 32)) & low, lo & low

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c0, c1


class _Brute:
    """Every ray against every primitive, in 64 bits."""

    def __init__(self, s, dev):
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
        self.c, self.r = t(s.sph_center), t(s.sph_radius)
        self.a, b, self.rho = t(s.cyl_a), t(s.cyl_b), t(s.cyl_radius)
        self.len = (b - self.a).norm(dim=1)
        self.w = (b - self.a) / self.len[:, None]
        v = t(s.tri_v if s.tri_v is not None else np.zeros((0, 3, 3)))
        self.v0, self.e1, self.e2 = v[:, 0], v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
        self.rgb = torch.cat([t(s.sph_rgb), t(s.cyl_rgb),
                              t(s.tri_rgb if s.tri_rgb is not None else np.zeros((0, 3)))])
        self.n = [self.c.shape[0], self.a.shape[0], self.v0.shape[0]]

    def times(self, o, d, tmin):
        """Hit times [rays, primitives], infinite without a hit past tmin."""
        inf = torch.tensor(math.inf, dtype=torch.float64, device=o.device)
        pick = lambda t, ok: torch.where(ok & (t > tmin), t, inf)
        out = []
        if self.n[0]:
            q = self.c[None] - o[:, None]
            b = (q * d[:, None]).sum(2)
            l = q - b[..., None] * d[:, None]
            disc = self.r ** 2 - (l * l).sum(2)
            sq = disc.clamp(min=0).sqrt()
            out.append(torch.minimum(pick(b - sq, disc >= 0), pick(b + sq, disc >= 0)))
        if self.n[1]:
            D = o[:, None] - self.a[None]
            dw, Dw = d @ self.w.T, (D * self.w[None]).sum(2)
            dp, Dp = d[:, None] - dw[..., None] * self.w[None], D - Dw[..., None] * self.w[None]
            A, B = (dp * dp).sum(2), (dp * Dp).sum(2)
            disc = B * B - A * ((Dp * Dp).sum(2) - self.rho ** 2)
            sq, A = disc.clamp(min=0).sqrt(), A.clamp(min=1e-300)
            best = inf
            for t in ((-B - sq) / A, (-B + sq) / A):
                h = Dw + t * dw
                best = torch.minimum(best, pick(t, (disc >= 0) & (A > 1e-12) & (h >= 0) & (h <= self.len)))
            out.append(best)
        if self.n[2]:
            P = torch.linalg.cross(d[:, None].expand(-1, self.n[2], -1), self.e2[None].expand(d.shape[0], -1, -1))
            det = (P * self.e1[None]).sum(2)
            T = o[:, None] - self.v0[None]
            Q = torch.linalg.cross(T, self.e1[None].expand_as(T))
            u, v, t = (T * P).sum(2) / det, (Q * d[:, None]).sum(2) / det, (Q * self.e2[None]).sum(2) / det
            out.append(pick(t, (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1)))
        return torch.cat(out, 1)

    def trace(self, o, d, tmin, skip=None):
        t, k = [], []
        chunk = max(1, 8000000 // max(1, sum(self.n)))
        for i in range(0, o.shape[0], chunk):
            x = self.times(o[i:i + chunk], d[i:i + chunk], tmin)
            if skip is not None:  # a ray that leaves a surface outward never meets it again
                x.scatter_(1, skip[i:i + chunk].clamp(min=0)[:, None],
                           torch.where(skip[i:i + chunk] >= 0, math.inf, x.gather(
                               1, skip[i:i + chunk].clamp(min=0)[:, None])[:, 0])[:, None])
            m = x.min(1)
            t.append(m.values)
            k.append(m.indices)
        return torch.cat(t), torch.cat(k)

    def normal(self, k, o, d, t):
        P = o + t[:, None] * d
        n = torch.zeros_like(P)
        s, c = k < self.n[0], (k >= self.n[0]) & (k < self.n[0] + self.n[1])
        if s.any():
            n[s] = P[s] - self.c[k[s]]
        if c.any():
            j = k[c] - self.n[0]
            D = P[c] - self.a[j]
            n[c] = D - (D * self.w[j]).sum(1, keepdim=True) * self.w[j]
        q = ~(s | c)
        if q.any():
            j = k[q] - self.n[0] - self.n[1]
            n[q] = torch.linalg.cross(self.e1[j], self.e2[j])
        return n / n.norm(dim=1, keepdim=True)


def exact(case, seed):
    """The frame's colours in 64 bits by brute force, where that is quick."""
    w, h, S = case["width"], case["height"], case["samples"]
    pairs = w * h * case["aa"] * (1 + _cover(case, w, h) * (S + 2)) * case["objects"]
    if case["path"] not in ("render", "frame", "bvh") or case["layers"] > 1 or pairs > 1e10:
        return None
    dev = torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")
    V = lambda x: torch.tensor(x, dtype=torch.float64, device=dev)
    host, cam, p = _scene(case, seed), _camera(case, _angle(seed), _radius(case)), _params(case, seed)
    B = _Brute(host, dev)
    key = (seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF)
    eye = V(cam.eye)
    f = (V(cam.lookat) - eye) / (V(cam.lookat) - eye).norm()
    r = torch.linalg.cross(f, V(cam.up))
    r = r / r.norm()
    u = torch.linalg.cross(r, f)
    th = math.tan(math.radians(cam.fovy_deg / 2.0))
    pix = torch.arange(w * h, device=dev)
    total = torch.zeros((w * h, 3), dtype=torch.float64, device=dev)
    for a in range(case["aa"]):
        px, py = (pix % w).double() + 0.5, (pix // w).double() + 0.5
        if a:
            x = _philox(pix, torch.full_like(pix, a), torch.zeros_like(pix), torch.full_like(pix, 0xFFFFFFFF), *key)
            px, py = (pix % w) + (x[0] >> 8).double() * 2.0 ** -24, (pix // w) + (x[1] >> 8).double() * 2.0 ** -24
        d = f + ((2.0 * px / w - 1.0) * th * w / h)[:, None] * r + ((1.0 - 2.0 * py / h) * th)[:, None] * u
        d = d / d.norm(dim=1, keepdim=True)
        o = eye.expand_as(d)
        t, k = B.trace(o, d, 0.0)
        hit = torch.isfinite(t).nonzero()[:, 0]
        o, d, t, k, id_ = o[hit], d[hit], t[hit], k[hit], pix[hit]
        N, P = B.normal(k, o, d, t), o + t[:, None] * d
        front = (N * d).sum(1) < 0
        N = torch.where(front[:, None], N, -N)
        skip = torch.where(front, k, -1)
        diffuse, shine = torch.zeros_like(N), torch.zeros_like(N)
        for q in range(len(LIGHTS)):
            L = V(LIGHTS[q]) / V(LIGHTS[q]).norm()
            cl = N @ L
            ts, _ = B.trace(P, L.expand_as(P), EPS, skip)
            on = ((cl > 2.0 ** -40) & ~torch.isfinite(ts)).double()
            diffuse += (p.light_rescale * on * cl)[:, None]
            if p.specular > 0:
                rv = -((2.0 * cl[:, None] * N - L) * d).sum(1)
                shine += (p.light_rescale * on * p.specular * rv.clamp(min=0) ** p.shininess)[:, None]
        sg = torch.where(N[:, 2] < 0, -1.0, 1.0).double()
        ca = -1.0 / (sg + N[:, 2])
        cb = N[:, 0] * N[:, 1] * ca
        tx = torch.stack([1.0 + sg * N[:, 0] ** 2 * ca, sg * cb, -sg * N[:, 0]], 1)
        bx = torch.stack([cb, sg + N[:, 1] ** 2 * ca, -N[:, 1]], 1)
        free = torch.zeros_like(t)
        for s in range(S):
            x = _philox(id_, torch.full_like(id_, s), torch.zeros_like(id_), torch.full_like(id_, a), *key)
            u1, u2 = (x[0] >> 8).double() * 2.0 ** -24, (x[1] >> 8).double() * 2.0 ** -24
            lx, ly = u1.sqrt() * torch.cos(2.0 * math.pi * u2), u1.sqrt() * torch.sin(2.0 * math.pi * u2)
            wd = lx[:, None] * tx + ly[:, None] * bx + (1.0 - u1).sqrt()[:, None] * N
            ts, _ = B.trace(P, wd, EPS, skip)
            free += (~torch.isfinite(ts)).double()
        ao = free / S
        total[hit] += (B.rgb[k] * (diffuse + (p.skylight * ao)[:, None]) + shine).clamp(0.0, 1.0)
    out = {"rgb": (total / case["aa"]).reshape(h, w, 3)}
    if case["masks"]:  # whole numbers: compared as they are
        out.update(hit_id=None, ao_mask=None, light_mask=None)
    return out
