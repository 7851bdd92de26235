"""The work a user of the library has it do, as cases that can be timed.

`listed()` names twelve cases over the library's public entry points, from one
small image to a structure-from-motion batch; `draw(rng)` gives more of the
same ranges.  `prepare(case, seed)` makes on the GPU what a program holds
before the call, `run(state)` is one pass through the binding, `work(case)`
the bytes and operations that pass cannot do without, and `exact(case, seed)`
the floating-point outputs in 64 bits (the others are whole numbers).

Kinds of case:
  extract   descriptors of one image's keypoints (48 x 48 / 7 x 7, or the
            64 x 64 / 8 x 8 weighted geometry)
  match     one query set against one train set, 2-NN and ratio test
  batch     keypoints of many images in one call, then the matching of the
            consecutive image pairs, as two eager calls or one captured plan
  detect    FAST keypoints of one or several images, optionally followed by
            the batched extraction of what was found, with no host round trip
  dense     descriptors of every pixel of a region
  window    2-NN of two descriptor grids within a radius
"""
import functools
import math

import numpy as np
import torch

from paper_1609_03986_amd import synth
from paper_1609_03986_amd.binding import Latch, image_table, pair_table

UNEVEN_SIZES = synth.UNEVEN_SIZES


def listed():
    return [
        # The smallest call: one 640x480 frame, 2,000 upright keypoints.
        dict(name="extract_640x480", kind="extract", height=480, width=640, pad=0, n=2000,
             upright=True, geometry="default"),
        # A full-HD frame whose rows are padded, 10,000 oriented and scaled keypoints.
        dict(name="extract_1920x1080", kind="extract", height=1080, width=1920, pad=64, n=10000,
             upright=False, geometry="default"),
        # The paper's own geometry (64 x 64 windows, 8 x 8 patches, Gaussian weights).
        dict(name="extract_weighted", kind="extract", height=1080, width=1920, pad=0, n=20000,
             upright=False, geometry="gaussian"),
        # Two frames' descriptors against each other: small, then ordinary and ragged.
        dict(name="match_2000x2000", kind="match", nq=2000, nt=2000, k=2, path="auto"),
        dict(name="match_9973x10007", kind="match", nq=9973, nt=10007, k=2, path="auto"),
        # One serving request against a resident database.
        dict(name="match_8000x1000000", kind="match", nq=8000, nt=1000000, k=2, path="auto"),
        # Structure from motion: 64 overlapping 3000x2000 images, 63 pairs, a captured plan.
        dict(name="sfm_plan", kind="batch", images=64, sizes="3000x2000", kps=20000, spread=0.0,
             plan=True),
        # Images of five sizes with log-normal keypoint counts, as two eager calls.
        dict(name="uneven_batch", kind="batch", images=48, sizes="uneven", kps=5000, spread=1.0,
             plan=False),
        # Corner detection of one frame, and of three odd-sized ones with their descriptors.
        dict(name="detect_1920x1080", kind="detect", height=1080, width=1920, images=1,
             threshold=20, describe=False),
        dict(name="detect_describe_3", kind="detect", height=719, width=1277, images=3,
             threshold=30, describe=True),
        # Dense descriptors of a whole frame, and the matching of two such grids.
        dict(name="dense_1920x1080", kind="dense", height=1080, width=1920, x0=0, y0=0, gw=1920,
             gh=1080),
        dict(name="window_1920x1080_r4", kind="window", gw=1920, gh=1080, radius=4, k=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("extract", "extract", "match", "match", "match", "batch", "detect", "dense",
                       "window"))
    if kind == "extract":
        geometry = rng.choice(("default", "default", "default", "gaussian", "clatch7"))
        return dict(kind=kind, height=_log_int(rng, 120, 3000), width=_log_int(rng, 160, 4000),
                    pad=rng.choice((0, 0, rng.randint(1, 64))), n=_log_int(rng, 100, 50000),
                    upright=rng.random() < 0.3, geometry=geometry)
    if kind == "match":
        path = rng.choice(("auto", "auto", "auto", "auto", "mfma", "popcount"))
        most = {"auto": 2.0e10, "mfma": 8.0e9, "popcount": 3.0e9}[path]
        nq = _log_int(rng, 1, 50000)
        return dict(kind=kind, nq=nq, nt=_log_int(rng, 2, max(2, min(1000000, most / nq))),
                    k=rng.choice((2, 2, 2, 1)), path=path)
    if kind == "batch":
        return dict(kind=kind, images=rng.randint(2, 48),
                    sizes=rng.choice(("uneven", "uneven", "1280x720")),
                    kps=_log_int(rng, 500, 8000), spread=rng.choice((0.0, 0.5, 1.0)),
                    plan=rng.random() < 0.5)
    if kind == "detect":
        return dict(kind=kind, height=_log_int(rng, 120, 2160), width=_log_int(rng, 160, 3840),
                    images=rng.randint(1, 4), threshold=rng.randint(10, 50),
                    describe=rng.random() < 0.5)
    gw, gh = _log_int(rng, 64, 2048), _log_int(rng, 48, 1200)
    if kind == "dense":
        height, width = gh + rng.randint(0, 200), gw + rng.randint(0, 200)
        return dict(kind=kind, height=height, width=width, x0=rng.randint(-20, width - gw),
                    y0=rng.randint(-20, height - gh), gw=gw, gh=gh)
    return dict(kind=kind, gw=gw, gh=gh, radius=rng.randint(1, 8), k=rng.choice((2, 2, 1)))


# --- inputs ---------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _handle(geometry):
    """A program keeps one handle per geometry."""
    if geometry == "default":
        return Latch(synth.triplet_table())
    weights = synth.gaussian_weights(8) if geometry == "gaussian" else synth.clatch_7x7_weights()
    return Latch(synth.triplet_table_geom(64, 8), window=64, patch=8, weights=weights)


def _blur(x, sigma, radius):
    """Separable Gaussian of a float image, edges reflected."""
    i = np.arange(-radius, radius + 1)
    w = np.exp(-i ** 2 / (2.0 * sigma ** 2))
    w = (w / w.sum()).tolist()
    for dim in (0, 1):
        n = x.shape[dim]
        at = torch.arange(-radius, n + radius, device=x.device).abs()
        at = torch.where(at >= n, 2 * (n - 1) - at, at)
        p = x.index_select(dim, at)
        x = sum(w[j] * p.narrow(dim, j, n) for j in range(2 * radius + 1))
    return x, sum(v * v for v in w)


def _texture(gen, g, height, width, shapes=150):
    """A textured u8 image: smoothed noise of mean 128 and deviation 48 with
    half-blended rectangles and Gaussian blobs."""
    noise = torch.rand((height, width), generator=gen, device="cuda") - 0.5
    img, energy = _blur(noise, 1.5, 5)
    img = img * (48.0 * math.sqrt(12.0) / energy) + 128.0
    for _ in range(shapes):
        h, w = (int(v) for v in g.integers(8, 201, 2))
        y, x = int(g.integers(0, max(1, height - h))), int(g.integers(0, max(1, width - w)))
        img[y:y + h, x:x + w] = 0.5 * img[y:y + h, x:x + w] + 0.5 * float(g.integers(0, 256))
        sig, amp = float(g.uniform(3.0, 30.0)), float(g.uniform(-80.0, 80.0))
        cy, cx, r = int(g.integers(0, height)), int(g.integers(0, width)), int(3 * sig) + 1
        y0, y1, x0, x1 = max(0, cy - r), min(height, cy + r), max(0, cx - r), min(width, cx + r)
        ey = torch.exp(-((torch.arange(y0, y1, device="cuda") - cy) ** 2) / (2 * sig * sig))
        ex = torch.exp(-((torch.arange(x0, x1, device="cuda") - cx) ** 2) / (2 * sig * sig))
        img[y0:y1, x0:x1] += amp * ey[:, None] * ex[None, :]
    return img.round().clamp(0, 255).to(torch.uint8)


def _noisy(gen, img, most=4):
    """Another exposure of an image: +-`most` per pixel."""
    d = torch.randint(-most, most + 1, img.shape, generator=gen, device="cuda", dtype=torch.int16)
    return (img.to(torch.int16) + d).clamp(0, 255).to(torch.uint8)


def _keypoints(g, n, height, width, upright):
    kps = synth.random_keypoints(g, n, height, width)
    if upright:
        kps[:, 2], kps[:, 3] = 0.0, 1.0
    return kps


def _words(bits):
    """[n, 512] truth values to [n, 16] int32 words."""
    place = torch.ones(32, dtype=torch.int64, device="cuda") << torch.arange(32, device="cuda")
    return (bits.view(-1, 16, 32) * place).sum(-1).to(torch.int32)


def _descriptors(gen, n):
    w = torch.randint(-2 ** 31, 2 ** 31, (n, 16), generator=gen, device="cuda", dtype=torch.int64)
    return w.to(torch.int32)


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed), np.random.default_rng(seed)


def _prepare_extract(case, gen, g):
    h, w = case["height"], case["width"]
    img = _texture(gen, g, h, w)
    if case["pad"]:
        rows = torch.zeros((h, w + case["pad"]), dtype=torch.uint8, device="cuda")
        rows[:, :w] = img
        img = rows[:, :w]
    kps = torch.from_numpy(_keypoints(g, case["n"], h, w, case["upright"])).cuda()
    return dict(lat=_handle(case["geometry"]), img=img, kps=kps)


def _prepare_match(case, gen, g):
    """Half of the queries are seen again in the train set with one bit in
    ten flipped, as far as both sets go; the rest are unrelated."""
    nq, nt = case["nq"], case["nt"]
    query, train = _descriptors(gen, nq), _descriptors(gen, nt)
    m = (min(nq, nt) + 1) // 2
    flips = _words(torch.rand((m, 512), generator=gen, device="cuda") < 0.1)
    qi = torch.randperm(nq, generator=gen, device="cuda")[:m]
    ti = torch.randperm(nt, generator=gen, device="cuda")[:m]
    query[qi] = train[ti] ^ flips
    return dict(lat=_handle("default"), query=query, train=train)


def _batch_shape(case, g):
    """Image sizes and keypoint counts of a batch (for `work`, of any seed alike
    on average)."""
    sizes = []
    for _ in range(case["images"]):
        if case["sizes"] == "uneven":
            sizes.append(UNEVEN_SIZES[int(g.integers(0, len(UNEVEN_SIZES)))])
        else:
            w, h = (int(v) for v in case["sizes"].split("x"))
            sizes.append((h, w))
    counts = [int(np.clip(np.rint(g.lognormal(math.log(case["kps"]), case["spread"])), 200, 50000))
              for _ in range(case["images"])]
    return sizes, counts


def _prepare_batch(case, gen, g):
    # Sizes and counts come from the case: another seed is another scene of
    # the same cameras.
    sizes, counts = _batch_shape(case, np.random.default_rng(160903986))
    mh, mw = max(h for h, _ in sizes), max(w for _, w in sizes)
    n = case["images"]
    scene = _texture(gen, g, mh + 8 * (n - 1), mw + 16 * (n - 1))
    images = [_noisy(gen, scene[8 * i:8 * i + h, 16 * i:16 * i + w])
              for i, (h, w) in enumerate(sizes)]
    kps = torch.from_numpy(np.concatenate(
        [_keypoints(g, c, h, w, False) for c, (h, w) in zip(counts, sizes)])).cuda()
    ids = torch.from_numpy(np.repeat(np.arange(n, dtype=np.int32), counts)).cuda()
    first = np.concatenate([[0], np.cumsum(counts)[:-1]])
    pairs = pair_table([(first[i], counts[i], first[i + 1], counts[i + 1], first[i])
                        for i in range(n - 1)])
    total = int(sum(counts))
    lat = _handle("default")
    state = dict(lat=lat, images=images, table=image_table(images), n=n, ids=ids, kps=kps,
                 pairs=pairs, total=total)
    if case["plan"]:
        desc = torch.zeros((total, 16), dtype=torch.int32, device="cuda")
        idx = torch.full((total, 2), -2, dtype=torch.int32, device="cuda")
        dist = torch.full((total, 2), -2, dtype=torch.int32, device="cuda")
        accept = torch.full((total,), 255, dtype=torch.uint8, device="cuda")
        plan = lat.plan(state["table"], n, ids, kps, desc, pairs, idx, dist, accept)
        state.update(plan=plan, out=(desc, idx, dist, accept))
    return state


def _detect_images(case, gen, g):
    return [_texture(gen, g, case["height"], case["width"]) for _ in range(case["images"])]


def _detect_cap(case):
    return case["images"] * case["height"] * case["width"] // 16 + 64


def _prepare_detect(case, gen, g):
    cap = _detect_cap(case)
    images = _detect_images(case, gen, g)
    state = dict(lat=_handle("default"), images=images, cap=cap, threshold=case["threshold"],
                 kps=torch.zeros((cap, 4), dtype=torch.float32, device="cuda"),
                 ids=torch.zeros((cap,), dtype=torch.int32, device="cuda"))
    if case["describe"]:
        state.update(table=image_table(images),
                     desc=torch.zeros((cap, 16), dtype=torch.int32, device="cuda"))
    return state


def _prepare_dense(case, gen, g):
    return dict(lat=_handle("default"), img=_texture(gen, g, case["height"], case["width"]),
                region=(case["x0"], case["y0"], case["gw"], case["gh"]))


def _prepare_window(case, gen, g):
    """The dense descriptors of a frame and of its twin, moved by (1, 2) and
    re-exposed."""
    gw, gh, lat = case["gw"], case["gh"], _handle("default")
    scene = _texture(gen, g, gh + 2, gw + 2)
    query = lat.extract_dense(scene[:gh, :gw], 0, 0, gw, gh)
    train = lat.extract_dense(_noisy(gen, scene[1:gh + 1, 2:gw + 2]), 0, 0, gw, gh)
    return dict(lat=lat, query=query, train=train, gw=gw, gh=gh, radius=case["radius"])


_PREPARE = dict(extract=_prepare_extract, match=_prepare_match, batch=_prepare_batch,
                detect=_prepare_detect, dense=_prepare_dense, window=_prepare_window)


def prepare(case, seed):
    state = _PREPARE[case["kind"]](case, *_rng(seed))
    state["case"] = case
    return state


# --- one pass -------------------------------------------------------------

def _run_batch(s):
    if "plan" in s:
        s["plan"].run()
        return s["out"]
    lat = s["lat"]
    desc = lat.extract_batch(s["table"], s["n"], s["ids"], s["kps"])
    return (desc,) + lat.knn_batch(desc, desc, s["pairs"], s["total"])


def _run_detect(s):
    lat, count = s["lat"], None
    for i, img in enumerate(s["images"]):
        _, count = lat.detect(img, s["threshold"], s["cap"], kps=s["kps"], n_kps=count,
                              image_id=s["ids"], image_index=i)
    if "desc" not in s:
        return s["kps"], count, s["ids"]
    desc = lat.extract_batch(s["table"], len(s["images"]), s["ids"], s["kps"], desc=s["desc"],
                             n_kps=count)
    return s["kps"], count, s["ids"], desc


def run(state):
    case, lat = state["case"], state["lat"]
    kind = case["kind"]
    if kind == "extract":
        return lat.extract(state["img"], state["kps"])
    if kind == "match":
        return lat.knn(state["query"], state["train"], k=case["k"], path=case["path"])
    if kind == "batch":
        return _run_batch(state)
    if kind == "detect":
        return _run_detect(state)
    if kind == "dense":
        return lat.extract_dense(state["img"], *state["region"])
    return lat.knn_window(state["query"], state["train"], state["gw"], state["gh"],
                          state["radius"], k=case["k"])


# --- what a pass cannot do without -----------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "extract":
        patch = 49 * 2 if case["geometry"] == "default" else 64 * 4
        return dict(bytes=case["height"] * case["width"] + case["n"] * 80,
                    flops=case["n"] * 512 * 2 * patch)
    if kind == "match":
        nq, nt = case["nq"], case["nt"]
        return dict(bytes=(nq + nt) * 64 + nq * (8 * case["k"] + 1), flops=nq * nt * 1024)
    if kind == "batch":
        sizes, counts = _batch_shape(case, np.random.default_rng(160903986))
        total = sum(counts)
        return dict(bytes=sum(h * w for h, w in sizes) + total * (16 + 4 + 64 + 64 + 17),
                    flops=total * 512 * 2 * 98 +
                    1024 * sum(a * b for a, b in zip(counts, counts[1:])))
    if kind == "detect":
        px = case["images"] * case["height"] * case["width"]
        found = px // 60 if case["threshold"] < 25 else px // 150
        return dict(bytes=px + found * (20 + (84 if case["describe"] else 0)),
                    flops=px * 32 + found * (709 * 4 + (512 * 2 * 98 if case["describe"] else 0)))
    n = case["gw"] * case["gh"]
    if kind == "dense":
        return dict(bytes=n + n * 64, flops=n * 512 * 9)
    side = 2 * case["radius"] + 1
    return dict(bytes=n * (128 + 8 * case["k"] + 1), flops=n * side * side * 1024)


# --- 64 bits ----------------------------------------------------------------

_CIRCLE = ((0, -3), (1, -3), (2, -2), (3, -1), (3, 0), (3, 1), (2, 2), (1, 3), (0, 3), (-1, 3),
           (-2, 2), (-3, 1), (-3, 0), (-3, -1), (-2, -2), (-1, -3))


def _exact_detect(img, threshold):
    """Keypoints (x, y, angle, 1) of one image in raster order: FAST-9 scores,
    strict suppression among 8 neighbours, intensity-centroid angle rounded
    to 1/4096 of a turn."""
    h, w = img.shape
    border = 16
    if h <= 2 * border or w <= 2 * border:
        return np.zeros((0, 4))
    a = img.astype(np.int16)
    c = a[border:h - border, border:w - border]
    ih, iw = c.shape
    d = np.stack([a[border + dy:border + dy + ih, border + dx:border + dx + iw] - c
                  for dx, dy in _CIRCLE])
    lo, hi = d, d
    lo9 = functools.reduce(np.minimum, [np.roll(lo, -i, 0) for i in range(9)])
    hi9 = functools.reduce(np.maximum, [np.roll(hi, -i, 0) for i in range(9)])
    score = np.maximum(lo9.max(0), -hi9.min(0))
    score = np.pad(np.where(score > threshold, score, 0), 1)
    mid = score[1:-1, 1:-1]
    keep = mid > 0
    for dy in range(3):
        for dx in range(3):
            if (dy, dx) != (1, 1):
                keep &= mid > score[dy:dy + ih, dx:dx + iw]
    ys, xs = np.nonzero(keep)
    ys, xs = ys + border, xs + border
    m10, m01 = np.zeros(len(ys), np.int64), np.zeros(len(ys), np.int64)
    for dy in range(-15, 16):
        for dx in range(-15, 16):
            if dx * dx + dy * dy <= 225:
                v = a[ys + dy, xs + dx].astype(np.int64)
                m10 += dx * v
                m01 += dy * v
    turn = np.arctan2(m01.astype(np.float64), m10.astype(np.float64)) / (2.0 * math.pi)
    angle = (np.rint(turn * 4096.0).astype(np.int64) & 4095) * (360.0 / 4096.0)
    return np.stack([xs.astype(np.float64), ys.astype(np.float64), angle, np.ones(len(ys))], 1)


def exact(case, seed):
    """The floating-point outputs: only detection has any (keypoint records);
    every other output is a whole number."""
    if case["kind"] != "detect":
        return None
    images = _detect_images(case, *_rng(seed))
    found = np.concatenate([_exact_detect(i.cpu().numpy(), case["threshold"]) for i in images])
    kps = np.zeros((_detect_cap(case), 4))
    m = min(len(found), len(kps))
    kps[:m] = found[:m]
    return (kps, None, None, None) if case["describe"] else (kps, None, None)
