"""Workloads of the library's public entry points, from one camera frame to a full gallery.

Each case is a dict of plain values. `prepare` makes what a caller has in hand (planes or
features on the GPU, boxes, a context, a batch, weights, a pipeline), `run` makes the one call
and returns everything it computes, `work` gives the bytes and operations the result cannot do
without, and `exact` the same result from plain torch in 64 bits.

Kinds of work, by entry point:

* features  -- `Context.features` (host boxes over camera frames), `Context.features_batch`
               (a device-resident box table), `Context.features_warped` (boxes resized);
* scores    -- `Context.score` in every precision of the weights;
* pipeline  -- the captured serving step: features, scores and identities of a batch;
* enrol     -- `Context.train`: one-vs-rest SVMs from enrolment features.
"""
import math

import numpy as np
import torch

from paper_1504_01883_amd import lbpf

DEV = "cuda"
FRAME_W, FRAME_H = 640, 480  # a Kinect-shaped frame
MAPPINGS = {"u59": lbpf.MAP_U59, "full256": lbpf.MAP_FULL256}
MODALITIES = {"both": lbpf.MOD_BOTH, "grey": lbpf.MOD_GREY, "depth": lbpf.MOD_DEPTH}
EXACT_STEPS = 100_000  # coordinate steps the plain trainer can take in a few seconds


# --- the cases -------------------------------------------------------------------------


def listed():
    return [
        # One camera frame's faces, the smallest call of a live recogniser.
        {"name": "frame_features", "kind": "frame", "faces": 5, "lo": 48, "hi": 256},
        # A batch of equal crops kept as one tall image (4096 crops of 128 x 128).
        {"name": "uniform_features", "kind": "batch", "n": 4096, "w": 128, "h": 128},
        # An archive of face crops of all sizes, each its own tightly packed image.
        {"name": "ragged_features", "kind": "ragged", "n": 16384, "lo": 48, "hi": 256},
        # Close-up faces of a high-resolution camera, up to the largest side accepted.
        {"name": "closeup_features", "kind": "ragged", "n": 128, "lo": 257, "hi": 1024},
        # The paper's own form: every box resized to 200 x 200, 256-bin histograms of one
        # modality (its accuracy table reports the modalities separately).
        {"name": "literal_features", "kind": "literal", "n": 1024, "side": 200, "grid": 8,
         "mapping": "full256", "modality": "grey", "window": 150},
        # The resize of the paper's Sec. 3 in front of the default features.
        {"name": "resized_features", "kind": "warped", "frames": 256, "per_frame": 8, "side": 200},
        # One frame's faces against the enrolled identities.
        {"name": "frame_scores", "kind": "scores", "n": 5, "k": 1024, "precision": "fp32"},
        # The uniform batch against 256 identities, the ragged one against 1024.
        {"name": "uniform_scores", "kind": "scores", "n": 4096, "k": 256, "precision": "fp32"},
        {"name": "ragged_scores", "kind": "scores", "n": 16384, "k": 1024, "precision": "fp32"},
        # A large gallery in the smallest operand type.
        {"name": "gallery_scores", "kind": "scores", "n": 16384, "k": 8192, "precision": "fp8"},
        # One batch of the serving loop: up to 64 frames' faces, BF16 scores, 1024 identities.
        {"name": "serving_batch", "kind": "pipeline", "frames": 64, "per_frame": 4, "k": 1024,
         "precision": "bf16"},
        # Enrolment: 256 people, 20 crops each.
        {"name": "enrolment", "kind": "enrol", "k": 256, "per": 20, "side": 128},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["frame", "batch", "ragged", "closeup", "literal", "warped", "scores",
                       "scores", "scores", "pipeline", "enrol"])
    if kind == "frame":
        lo = rng.randint(40, 120)
        return {"kind": kind, "faces": rng.randint(1, 8), "lo": lo, "hi": rng.randint(lo, 320)}
    if kind == "batch":
        w, h = rng.randint(24, 256), rng.randint(24, 256)
        return {"kind": kind, "n": _log_int(rng, 16, 4096), "w": w, "h": h}
    if kind == "ragged":
        lo = rng.randint(3, 120)
        return {"kind": kind, "n": _log_int(rng, 16, 8192), "lo": lo, "hi": rng.randint(lo + 8, 300)}
    if kind == "closeup":
        lo = rng.randint(257, 800)
        return {"kind": "ragged", "n": _log_int(rng, 1, 128), "lo": lo, "hi": rng.randint(lo, 1024)}
    if kind == "literal":
        return {"kind": kind, "n": _log_int(rng, 4, 1024), "side": rng.randint(60, 256),
                "grid": rng.choice([1, 4, 7, 8]), "mapping": rng.choice(["u59", "full256"]),
                "modality": rng.choice(["both", "grey", "depth"]),
                "window": rng.choice([0, 100, 150, 400])}
    if kind == "warped":
        return {"kind": kind, "frames": _log_int(rng, 1, 256), "per_frame": rng.randint(1, 8),
                "side": rng.randint(64, 256)}
    if kind == "scores":
        return {"kind": kind, "n": _log_int(rng, 1, 16384), "k": _log_int(rng, 10, 8192),
                "precision": rng.choice(["fp32", "fp32", "f16x3", "bf16", "fp16", "fp8"])}
    if kind == "pipeline":
        return {"kind": kind, "frames": _log_int(rng, 1, 64), "per_frame": rng.randint(1, 8),
                "k": _log_int(rng, 16, 2048),
                "precision": rng.choice(["fp32", "bf16", "fp16", "fp8", "f16x3"])}
    return {"kind": kind, "k": _log_int(rng, 2, 256), "per": rng.randint(3, 20),
            "side": rng.randint(48, 128)}


# --- inputs ----------------------------------------------------------------------------


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1504_01883 * 1_000_003 + 7919 * int(seed) + stream)
    return g


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device=DEV)


def _sides(case, seed):
    """(w, h) of every crop: w uniform in [lo, hi], aspect 0.8 to 1.25, h clamped to the range."""
    rng = np.random.default_rng([case["n"], case["lo"], case["hi"], int(seed) & 0x7FFFFFFF])
    w = rng.integers(case["lo"], case["hi"] + 1, size=case["n"])
    h = np.rint(w * rng.uniform(0.8, 1.25, size=case["n"])).astype(np.int64)
    return np.stack([w, np.clip(h, case["lo"], case["hi"])], 1).astype(np.int64)


class Faces:
    """Face-like crops: per crop (or per identity) a grey base with 12 blobs, a depth ellipsoid
    with relief bumps before a far background, integer noise and 2% invalid depth."""

    def __init__(self, seed, n, identities=None):
        g = _gen(seed, 1)
        m = n if identities is None else int(identities.max()) + 1
        of = slice(None) if identities is None else torch.from_numpy(identities).to(DEV)
        self.base = _uniform(g, 90, 160, m, 1, 1)[of]
        self.cen = _uniform(g, 0.2, 0.8, m, 2, 12)[of]
        self.sig = _uniform(g, 0.06, 0.18, m, 12)[of]
        self.amp = _uniform(g, -80, 80, m, 12)[of]
        self.bcen = _uniform(g, 0.3, 0.7, m, 2, 6)[of]
        self.bsig = _uniform(g, 0.05, 0.12, m, 6)[of]
        self.bamp = _uniform(g, -25, 25, m, 6)[of]
        self.jit = 3 * torch.randn((n, 2), generator=g, device=DEV)
        self.z0 = _uniform(g, 500, 1500, n, 1, 1)
        self.far = _uniform(g, 2500, 4000, n, 1, 1)
        self.g = g

    def chunk(self, a, b, sizes):
        """Crops a .. b-1 padded to their largest sides: grey u8, depth i32 [n, H, W], and which
        pixels are inside."""
        wh = torch.from_numpy(sizes[a:b]).to(DEV).float()
        w, h = wh[:, :1], wh[:, 1:]
        H, W = int(sizes[a:b, 1].max()), int(sizes[a:b, 0].max())
        ys = torch.arange(H, device=DEV, dtype=torch.float32)[None]
        xs = torch.arange(W, device=DEV, dtype=torch.float32)[None]
        inside = (ys < h)[:, :, None] & (xs < w)[:, None, :]
        short = torch.minimum(w, h)
        jy, jx = self.jit[a:b, :1], self.jit[a:b, 1:]

        def bumps(cen, sig, amp):
            s = 2 * (sig * short) ** 2
            cy, cx = cen[:, 0] * h + jy, cen[:, 1] * w + jx
            gy = torch.exp(-(ys[:, :, None] - cy[:, None, :]) ** 2 / s[:, None, :])
            gx = torch.exp(-(xs[:, None, :] - cx[:, :, None]) ** 2 / s[:, :, None])
            return torch.bmm(gy * amp[:, None, :], gx)

        def noise(k):
            return torch.randint(-k, k + 1, (b - a, H, W), generator=self.g, device=DEV,
                                 dtype=torch.int32)

        grey = torch.round(self.base[a:b] + bumps(self.cen[a:b], self.sig[a:b], self.amp[a:b]))
        grey = (grey.int() + noise(8)).clamp_(0, 255).to(torch.uint8)
        ey = (ys - ((h - 1) / 2 + jy)) / (0.47 * h)
        ex = (xs - ((w - 1) / 2 + jx)) / (0.45 * w)
        r2 = ey[:, :, None] ** 2 + ex[:, None, :] ** 2
        z = self.z0[a:b] + 200 * (1 - torch.sqrt((1 - r2).clamp(0, 1)))
        z = z + bumps(self.bcen[a:b], self.bsig[a:b], self.bamp[a:b])
        z = torch.where(r2 < 1, torch.round(z).int(), self.far[a:b].int() + noise(5))
        bad = torch.rand((b - a, H, W), generator=self.g, device=DEV) < 0.02
        return grey, z.masked_fill_(bad, 0), inside


def _chunks(sizes):
    """Ranges of crops whose padded area is at most about 16 million pixels."""
    a, n = 0, len(sizes)
    while a < n:
        b, W, H = a, 0, 0
        while b < n and b - a < 512:
            W, H = max(W, sizes[b, 0]), max(H, sizes[b, 1])
            if b > a and (b + 1 - a) * W * H > 1 << 24:
                break
            b += 1
        yield a, b
        a = b


def _pool(case, seed, identities=None):
    """Crops packed one after another: grey u8 [P], depth u16 [P], offsets, sizes."""
    sizes = (_sides(case, seed) if case["kind"] == "ragged" else
             np.tile(np.array([[case["w"], case["h"]]], np.int64), (case["n"], 1)))
    faces = Faces(seed, len(sizes), identities)
    grey, depth = [], []
    for a, b in _chunks(sizes):
        g, z, inside = faces.chunk(a, b, sizes)
        grey.append(g[inside])
        depth.append(z[inside].to(torch.int16).view(torch.uint16))
    area = sizes[:, 0] * sizes[:, 1]
    return torch.cat(grey), torch.cat(depth), np.concatenate([[0], np.cumsum(area)[:-1]]), sizes


def _frames(seed, n_frames, per_frame, lo, hi):
    """Camera frames with faces pasted at boxes: [(grey, depth)], boxes [n, 5]."""
    rng = np.random.default_rng([n_frames, per_frame, lo, hi, int(seed) & 0x7FFFFFFF])
    n = n_frames * per_frame
    w = rng.integers(lo, hi + 1, size=n)
    h = np.clip(np.rint(w * rng.uniform(0.8, 1.25, size=n)).astype(np.int64), lo, min(hi, FRAME_H))
    x, y = rng.integers(0, FRAME_W - w + 1), rng.integers(0, FRAME_H - h + 1)
    boxes = np.stack([np.arange(n) // per_frame, x, y, w, h], 1).astype(np.int32)
    g = _gen(seed, 2)
    grey = torch.randint(100, 117, (n_frames, FRAME_H, FRAME_W), generator=g, device=DEV).to(torch.uint8)
    depth = torch.randint(3000, 3011, (n_frames, FRAME_H, FRAME_W), generator=g, device=DEV,
                          dtype=torch.int32)
    depth.masked_fill_(torch.rand(depth.shape, generator=g, device=DEV) < 0.02, 0)
    depth = depth.to(torch.int16)
    sizes = np.stack([w, h], 1).astype(np.int64)
    faces = Faces(seed, n)
    for a, b in _chunks(sizes):
        fg, fz, _ = faces.chunk(a, b, sizes)
        fz = fz.to(torch.int16)
        for i in range(a, b):
            im, bx, by, bw, bh = (int(v) for v in boxes[i])
            grey[im, by:by + bh, bx:bx + bw] = fg[i - a, :bh, :bw]
            depth[im, by:by + bh, bx:bx + bw] = fz[i - a, :bh, :bw]
    depth = depth.view(torch.uint16)
    return [(grey[i], depth[i]) for i in range(n_frames)], boxes


def _gallery(case, seed, D, rows):
    """Enrolled weights [k, D], biases [k] and `rows` features of those identities: histograms
    with a common skew and an identity's own, so that a row's best identity stands out."""
    g = _gen(seed, 3)
    k = case["k"]
    common = torch.exp(1.2 * torch.randn((1, D), generator=g, device=DEV))
    own = common * torch.exp(0.4 * torch.randn((k, D), generator=g, device=DEV))
    own /= own.sum(1, keepdim=True)
    who = torch.randint(0, k, (rows,), generator=g, device=DEV)
    pixels = _uniform(g, 3000, 40000, rows, 1)
    X = torch.empty((rows, D), device=DEV)
    for a in range(0, rows, 2048):
        X[a:a + 2048] = torch.poisson(own[who[a:a + 2048]] * pixels[a:a + 2048], generator=g)
    X /= X.sum(1, keepdim=True).clamp_(min=1)
    W = own - own.mean(0, keepdim=True)
    W *= 60 / W.norm(dim=1, keepdim=True).clamp_(min=1e-12)
    W += 0.1 * torch.randn(W.shape, generator=g, device=DEV)
    b = -0.9 + 0.01 * torch.randn((k,), generator=g, device=DEV)
    return X, W, b


def _enrol_inputs(case, seed):
    """Default features (FP32) and labels of k people with `per` crops each."""
    k, per, side = case["k"], case["per"], case["side"]
    ident = np.repeat(np.arange(k), per)
    c = {"kind": "batch", "n": k * per, "w": side, "h": side}
    grey, depth, offs, sizes = _pool(c, seed, ident)
    cfg = _config(case)
    X = torch.cat([_plain_features(*_crops(grey, depth, offs, sizes, a, b), cfg)
                   for a, b in _chunks(sizes)]).float()
    return X, torch.from_numpy(ident.astype(np.int32)).to(DEV)


# --- plain 64-bit results ----------------------------------------------------------------


def _config(case):
    """(grid, bins, use grey, use depth, window) of a case's context."""
    m = case.get("modality", "both")
    return (case.get("grid", 8), 59 if case.get("mapping", "u59") == "u59" else 256,
            m != "depth", m != "grey", case.get("window", 150))


def _dim(case):
    grid, bins, ug, ud, _ = _config(case)
    return grid * grid * bins * (ug + ud)


def _crops(grey, depth, offs, sizes, a, b):
    """Crops a .. b-1 of a pool, padded: grey i32, depth i32 [n, H, W], sizes."""
    w, h = (torch.from_numpy(sizes[a:b, i].copy()).to(DEV) for i in (0, 1))
    H, W = int(sizes[a:b, 1].max()), int(sizes[a:b, 0].max())
    ys, xs = torch.arange(H, device=DEV)[None, :, None], torch.arange(W, device=DEV)[None, None]
    at = torch.from_numpy(offs[a:b].copy()).to(DEV)[:, None, None] + ys * w[:, None, None] + xs
    at = torch.where((ys < h[:, None, None]) & (xs < w[:, None, None]), at, 0)
    z = depth.view(torch.int16)[at].int() & 0xFFFF
    return grey[at].int(), z, w, h


def _plain_features(grey, depth, w, h, cfg):
    """count / T in 64 bits for padded crops [n, H, W] of sizes w, h."""
    grid, bins, ug, ud, window = cfg
    n, H, W = depth.shape
    ys, xs = torch.arange(H, device=DEV)[None, :, None], torch.arange(W, device=DEV)[None, None]
    w, h = w[:, None, None], h[:, None, None]
    seen = (ys < h) & (xs < w) & (depth > 0)
    count = seen.flatten(1).sum(1)
    ranked = torch.where(seen, depth, 1 << 20).flatten(1).sort(1).values
    m = ranked.gather(1, ((count - 1).clamp(min=0) // 2)[:, None])[:, :, None]
    ok = (ys >= 1) & (xs >= 1) & (ys <= h - 2) & (xs <= w - 2)
    if window > 0:
        ok = ok & (depth > 0) & ((depth - m).abs() < window) & (count > 0)[:, None, None]
    cell = (((ys + 1) * grid - 1) // h) * grid + ((xs + 1) * grid - 1) // w
    table = torch.arange(256)
    if bins == 59:
        flips = [bin(c ^ ((c >> 1) | ((c & 1) << 7))).count("1") for c in range(256)]
        uniform = [c for c in range(256) if flips[c] <= 2]
        table = torch.tensor([uniform.index(c) if flips[c] <= 2 else 58 for c in range(256)])
    table = table.to(DEV)
    per = grid * grid * bins
    dim = per * (ug + ud)
    out = torch.zeros(n * dim, dtype=torch.float64, device=DEV)
    base = torch.arange(n, device=DEV)[:, None, None] * dim + cell * bins
    hoods = [(-1, -1), (-1, 0), (-1, 1), (0, 1), (1, 1), (1, 0), (1, -1), (0, -1)]
    for ch, plane in enumerate([p for p, use in ((grey, ug), (depth, ud)) if use]):
        code = torch.zeros_like(plane)
        for p, (dy, dx) in enumerate(hoods):
            code |= (torch.roll(plane, (-dy, -dx), (1, 2)) >= plane).int() << p
        at = (base + ch * per + table[code.long()])[ok]
        out += torch.bincount(at, minlength=n * dim)
    total = (ug + ud) * ok.flatten(1).sum(1)
    return out.view(n, dim) / total.clamp(min=1).double()[:, None]


def _frame_features(planes, boxes, cfg, resize=None):
    """_plain_features of boxes over frames, each resized to resize x resize when given."""
    grey = torch.stack([g for g, _ in planes])
    depth = torch.stack([z.view(torch.int16) for _, z in planes])
    out = []
    for a in range(0, len(boxes), 128):
        im, x, y, w, h = (torch.from_numpy(boxes[a:a + 128, i].astype(np.int64)).to(DEV)
                          for i in range(5))
        if resize:  # nearest sample at each output pixel's centre, 16.16 fixed point
            ux, uy = (w << 16) // resize, (h << 16) // resize
            at = torch.arange(resize, device=DEV)[None]
            xs = ((ux[:, None] * at + ((x << 16) + ux // 2)[:, None]) >> 16)[:, None, :]
            ys = ((uy[:, None] * at + ((y << 16) + uy // 2)[:, None]) >> 16)[:, :, None]
            w = h = torch.full_like(w, resize)
        else:
            xs = (x[:, None] + torch.arange(int(w.max()), device=DEV)[None]).clamp(max=FRAME_W - 1)[:, None, :]
            ys = (y[:, None] + torch.arange(int(h.max()), device=DEV)[None]).clamp(max=FRAME_H - 1)[:, :, None]
        im = im[:, None, None]
        out.append(_plain_features(grey[im, ys, xs].int(), depth[im, ys, xs].int() & 0xFFFF, w, h, cfg))
    return torch.cat(out)


def _splitmix(state, m):
    z = (state + (m + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15))
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _plain_train(X, labels, k, C=1.0, eps=1e-6, epochs=200, seed=150401883):
    """Dual coordinate descent of every class at once on the Gram matrix, in 64 bits."""
    X, labels = X.double().cpu().numpy(), labels.cpu().numpy()
    n = len(X)
    if n * epochs > EXACT_STEPS:
        return None
    norm = np.sort(np.linalg.norm(X, axis=1))[(n - 1) // 2]
    X = X / norm if norm > 0 else X
    G = X @ X.T + 1.0
    y = np.where(labels[None, :] == np.arange(k)[:, None], 1.0, -1.0)
    alpha, g = np.zeros((k, n)), np.zeros((k, n))
    took, live, rows = np.full(k, epochs), np.ones(k, bool), np.arange(k)
    with np.errstate(over="ignore"):
        state = np.uint64(seed) ^ (np.uint64(0x5851F42D4C957F2D) * (rows.astype(np.uint64) + np.uint64(1)))
    for e in range(epochs):
        order = np.tile(np.arange(n), (k, 1))
        for i in range(n - 1, 0, -1):
            with np.errstate(over="ignore"):
                r = _splitmix(state, np.uint64(e * (n - 1) + n - 1 - i))
            j = (r % np.uint64(i + 1)).astype(np.int64)
            order[rows, i], order[rows, j] = order[rows, j], order[rows, i].copy()
        worst = np.zeros(k)
        for s in range(n):
            i = order[:, s]
            grad, a, yi = y[rows, i] * g[rows, i] - 1.0, alpha[rows, i], y[rows, i]
            pg = np.where(a <= 0, np.minimum(grad, 0), np.where(a >= C, np.maximum(grad, 0), grad))
            worst = np.maximum(worst, np.abs(pg))
            new = np.clip(a - grad / G[i, i], 0, C)
            step = np.where(live & (pg != 0), new - a, 0.0)
            alpha[rows, i] += step
            moved = np.nonzero(step)[0]
            g[moved] += (step * yi)[moved, None] * G[i[moved]]
        ended = live & (worst < eps)
        took[ended] = e + 1
        live &= ~ended
        if not live.any():
            break
    W = (alpha * y) @ X / (norm if norm > 0 else 1.0)
    return {"W": W, "b": (alpha * y).sum(1), "epochs": None}


# --- the functions --------------------------------------------------------------------


def _context(case):
    grid, _, _, _, window = _config(case)
    return lbpf.Context(grid=(grid, grid), mapping=MAPPINGS[case.get("mapping", "u59")],
                        window=window, modality=MODALITIES[case.get("modality", "both")])


def _tall(case, seed):
    """Equal crops as one image: grey, depth [n h, w], boxes."""
    n, w, h = case["n"], case.get("w", case.get("side")), case.get("h", case.get("side"))
    grey, depth, _, _ = _pool({"kind": "batch", "n": n, "w": w, "h": h}, seed)
    boxes = np.zeros((n, 5), np.int32)
    boxes[:, 2], boxes[:, 3], boxes[:, 4] = np.arange(n) * h, w, h
    return grey.view(n * h, w), depth.view(n * h, w), boxes


def _warp_boxes(boxes, side):
    return [(int(i), side, side, *(2 * (lbpf.resize_frame(int(x), int(y), int(w), int(h), side, side),)))
            for i, x, y, w, h in boxes]


def prepare(case, seed):
    kind = case["kind"]
    ctx = _context(case)
    st = {"kind": kind, "ctx": ctx}
    if kind == "frame":
        st["planes"], st["boxes"] = _frames(seed, 1, case["faces"], case["lo"], case["hi"])
    elif kind in ("batch", "literal"):
        grey, depth, boxes = _tall(case, seed)
        st["batch"] = ctx.batch([(grey, depth)], boxes)
        st["out"] = torch.empty((case["n"], ctx.dim), device=DEV)
    elif kind == "ragged":
        grey, depth, offs, sizes = _pool(case, seed)
        planes = [(grey[o:o + w * h].view(h, w), depth[o:o + w * h].view(h, w))
                  for o, (w, h) in zip(offs.tolist(), sizes.tolist())]
        boxes = np.zeros((case["n"], 5), np.int32)
        boxes[:, 0], boxes[:, 3:] = np.arange(case["n"]), sizes
        st["batch"] = ctx.batch(planes, boxes)
        st["out"] = torch.empty((case["n"], ctx.dim), device=DEV)
    elif kind == "warped":
        planes, boxes = _frames(seed, case["frames"], case["per_frame"], 48, 256)
        st["images"] = lbpf.ImageTable(planes)
        st["table"] = lbpf.WarpBoxTable(_warp_boxes(boxes, case["side"]))
        st["workspace"] = torch.empty(st["table"].workspace_bytes, dtype=torch.uint8, device=DEV)
        st["out"] = torch.empty((len(boxes), ctx.dim), device=DEV)
    elif kind == "scores":
        st["X"], W, b = _gallery(case, seed, ctx.dim, case["n"])
        st["weights"] = ctx.weights(W, b, precision=case["precision"])
    elif kind == "pipeline":
        planes, st["boxes"] = _frames(seed, case["frames"], case["per_frame"], 48, 256)
        _, W, b = _gallery(case, seed, ctx.dim, 1)
        st["weights"] = ctx.weights(W, b, precision=case["precision"])
        st["images"] = lbpf.ImageTable(planes)
        st["pipeline"] = ctx.pipeline(st["weights"], 512)  # 64 frames of up to 8 faces
    else:
        st["X"], st["labels"] = _enrol_inputs(case, seed)
        st["k"] = case["k"]
    return st


def run(st):
    kind, ctx = st["kind"], st["ctx"]
    if kind == "frame":
        return ctx.features(st["planes"], st["boxes"])[0]
    if kind in ("batch", "literal", "ragged"):
        return ctx.features_batch(st["batch"], st["out"])
    if kind == "warped":
        return ctx.features_warped(st["images"], st["table"], out=st["out"],
                                   workspace=st["workspace"])[0]
    if kind == "scores":
        scores, identity = ctx.score(st["X"], st["weights"])
        return {"scores": scores, "identity": identity}
    if kind == "pipeline":
        p = st["pipeline"]
        n = p.launch(st["images"], st["boxes"])
        return {"hist": p.hist[:n], "scores": p.scores[:n], "identity": p.argmax[:n]}
    out = ctx.train(st["X"], st["labels"], st["k"])
    return {"W": out["W"], "b": out["b"], "epochs": out["epochs"]}


def _pixels(case):
    """Expected pixels of a case's crops (their mean side squared; aspects average to 1)."""
    if case["kind"] in ("batch",):
        return case["n"] * case["w"] * case["h"]
    if case["kind"] in ("literal",):
        return case["n"] * case["side"] ** 2
    lo, hi, n = {"frame": (case.get("lo"), case.get("hi"), case.get("faces")),
                 "ragged": (case.get("lo"), case.get("hi"), case.get("n"))}.get(
                     case["kind"], (48, 256, case.get("frames", 0) * case.get("per_frame", 0)))
    return n * (lo * lo + lo * hi + hi * hi) / 3


def work(case):
    kind, D = case["kind"], _dim(case)
    _, _, grey, depth, window = _config(case)
    per_px = grey + 2 * (depth or window > 0)  # u8 grey, u16 depth (the mask needs it too)
    if kind in ("frame", "batch", "literal", "ragged"):
        n = case.get("n", case.get("faces"))
        return {"bytes": per_px * _pixels(case) + 4 * n * D, "flops": 0}
    if kind == "warped":
        n, px = case["frames"] * case["per_frame"], case["side"] ** 2
        return {"bytes": n * (min(px, _pixels(case) / n) * 3 + 4 * D), "flops": 0}
    size = {"fp32": 4, "f16x3": 4, "bf16": 2, "fp16": 2, "fp8": 1}.get(case.get("precision"), 4)
    if kind == "scores":
        n, k = case["n"], case["k"]
        return {"bytes": 4 * n * D + size * k * D + 4 * n * k + 4 * n, "flops": 2 * n * k * D}
    if kind == "pipeline":
        n, k = case["frames"] * case["per_frame"], case["k"]
        return {"bytes": 3 * _pixels(case) + 4 * n * D + size * k * D + 4 * n * k + 4 * n,
                "flops": 2 * n * k * D}
    n, k = case["k"] * case["per"], case["k"]
    return {"bytes": 4 * n * D + 4 * k * D, "flops": n * n * D + 2 * n * k * D}


def exact(case, seed):
    kind, cfg = case["kind"], _config(case)
    if kind == "frame":
        planes, boxes = _frames(seed, 1, case["faces"], case["lo"], case["hi"])
        return _frame_features(planes, boxes, cfg)
    if kind in ("batch", "literal", "ragged"):
        c = case if kind == "ragged" else {"kind": "batch", "n": case["n"],
                                           "w": case.get("w", case.get("side")),
                                           "h": case.get("h", case.get("side"))}
        pool = _pool(c, seed)
        return torch.cat([_plain_features(*_crops(*pool, a, b), cfg) for a, b in _chunks(pool[3])])
    if kind == "warped":
        planes, boxes = _frames(seed, case["frames"], case["per_frame"], 48, 256)
        return _frame_features(planes, boxes, cfg, resize=case["side"])
    if kind == "scores":
        X, W, b = _gallery(case, seed, _dim(case), case["n"])
        W, b = W.double(), b.double()
        return {"scores": torch.cat([x.double() @ W.T + b for x in X.split(4096)]), "identity": None}
    if kind == "pipeline":
        planes, boxes = _frames(seed, case["frames"], case["per_frame"], 48, 256)
        _, W, b = _gallery(case, seed, _dim(case), 1)
        hist = _frame_features(planes, boxes, cfg)
        return {"hist": hist, "scores": hist @ W.double().T + b.double(), "identity": None}
    return _plain_train(*_enrol_inputs(case, seed), case["k"])
