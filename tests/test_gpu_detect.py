"""GPU parity of keypoint detection (latch_detect): FAST-9 corners, strict
3x3 suppression, raster order and the intensity-centroid angle bin, each
keypoint exactly equal to the oracle's; counts beyond max_kps, image ids,
row pitch, small images, and detection feeding batched extraction."""
import numpy as np
import pytest

import oracle
from paper_1609_03986_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def lat(torch_cuda, triplets):
    from paper_1609_03986_amd.binding import Latch
    L = Latch(triplets)
    L.check_errors(clear=True)
    yield L
    L.close()


def run(torch, lat, img, t, max_kps, **kw):
    kps, n = lat.detect(torch.from_numpy(img).cuda(), t, max_kps, **kw)
    torch.cuda.synchronize()
    return kps.cpu().numpy(), int(n.cpu().item())


@pytest.mark.parametrize("shape", [(33, 33), (34, 97), (131, 77), (480, 640)])
@pytest.mark.parametrize("t", [5, 20, 45])
def test_matches_oracle(torch_cuda, lat, shape, t):
    g = np.random.default_rng(shape[0] * 1000 + shape[1] + t)
    img = synth.smoothed_noise(g, *shape)
    want, wn = oracle.detect(img, t)
    kps, n = run(torch_cuda, lat, img, t, max(wn, 1) + 5)
    print(shape, t, wn)
    assert n == wn
    assert np.array_equal(kps[:n], want)


def test_textured_image_all_bins(torch_cuda, lat):
    """A larger textured image: thousands of keypoints, angles over the whole circle."""
    g = np.random.default_rng(41)
    img = synth.textured_image(g, 720, 1280)
    img = np.clip(img.astype(int) + g.integers(-20, 21, img.shape), 0, 255).astype(np.uint8)
    want, wn = oracle.detect(img, 20)
    kps, n = run(torch_cuda, lat, img, 20, wn)
    assert n == wn and wn > 2000
    assert np.array_equal(kps, want)
    assert len(np.unique(want[:, 2])) > 1000


@pytest.mark.parametrize("shape", [(40, 4500), (300, 4160), (2200, 160)])
def test_wide_and_tall_images(torch_cuda, lat, shape):
    """Rows of more than 64 tiles (several count chunks per row, the emit
    kernel's left sum over two lane passes, a partial last chunk) and more than
    2048 rows (a second scan pass carrying the running total)."""
    g = np.random.default_rng(shape[0] + 7 * shape[1])
    img = synth.textured_image(g, *shape)
    want, wn = oracle.detect(img, 20)
    kps, n = run(torch_cuda, lat, img, 20, max(wn, 1))
    print(shape, wn)
    assert n == wn and wn > 0
    assert np.array_equal(kps[:n], want)


@pytest.mark.parametrize("shape", [(1000, 4093), (1031, 4093), (1100, 4096)])
def test_sizes_around_the_scan_limit(torch_cuda, lat, shape):
    """Images of just under and over 4,096 tiles (slots from the per-tile
    totals, or from the row scan), by bytes and by dwords."""
    g = np.random.default_rng(shape[0])
    img = g.integers(0, 256, shape, dtype=np.uint8)
    want, wn = oracle.detect(img, 100)
    kps, n = run(torch_cuda, lat, img, 100, wn + 5)
    assert n == wn and wn > 10000
    assert np.array_equal(kps[:n], want)


@pytest.mark.parametrize("t", [0, 1, 254, 255])
@pytest.mark.parametrize("levels", [2, 3, 256])
def test_extreme_scores(torch_cuda, lat, t, levels):
    """Scores from 1 to 255 at the ends of the threshold's range: random
    images of 2, 3 and 256 levels between 0 and 255, and isolated dots."""
    g = np.random.default_rng(17 * t + levels)
    img = (g.integers(0, levels, (97, 145)) * 255 // (levels - 1)).astype(np.uint8)
    img[40:60, 30:110] = 255 * (levels % 2)
    img[50, 40:100:7] = 255 - 255 * (levels % 2)
    want, wn = oracle.detect(img, t)
    kps, n = run(torch_cuda, lat, img, t, wn + 5)
    assert n == wn
    assert np.array_equal(kps[:n], want)


def test_truncation_keeps_raster_prefix_and_full_count(torch_cuda, lat):
    g = np.random.default_rng(3)
    img = synth.smoothed_noise(g, 300, 400)
    want, wn = oracle.detect(img, 10)
    assert wn > 500
    for m in (0, 1, 63, 257, wn - 1):
        kps, n = run(torch_cuda, lat, img, 10, m)
        assert n == wn
        assert kps.shape == (m, 4) and np.array_equal(kps, want[:m])


def test_pitch_and_image_id(torch_cuda, lat):
    torch = torch_cuda
    g = np.random.default_rng(4)
    big = synth.smoothed_noise(g, 200, 320)
    img = big[:, 20:270]                            # row stride 320, width 250
    want, wn = oracle.detect(np.ascontiguousarray(img), 15)
    dev = torch.from_numpy(big).cuda()[:, 20:270]
    assert dev.stride(0) == 320
    ids = torch.full((wn + 10,), -7, dtype=torch.int32, device="cuda")
    kps, n = lat.detect(dev, 15, wn + 10, image_id=ids, image_index=5)
    torch.cuda.synchronize()
    assert int(n.item()) == wn
    assert np.array_equal(kps.cpu().numpy()[:wn], want)
    ids = ids.cpu().numpy()
    assert np.all(ids[:wn] == 5) and np.all(ids[wn:] == -7)


def test_small_and_flat_images(torch_cuda, lat):
    for shape in ((1, 1), (32, 500), (500, 32), (40, 40)):
        img = np.full(shape, 100, np.uint8)
        kps, n = run(torch_cuda, lat, img, 0, 4)
        assert n == 0
    g = np.random.default_rng(5)
    img = g.integers(0, 256, (32, 200)).astype(np.uint8)    # no row 16 px from both edges
    assert run(torch_cuda, lat, img, 0, 8)[1] == 0


def test_bad_arguments(torch_cuda, lat):
    from paper_1609_03986_amd.binding import LATCH_EINVAL, LATCH_ERANGE, LatchError
    img = torch_cuda.zeros((64, 64), dtype=torch_cuda.uint8, device="cuda")
    with pytest.raises(LatchError) as e:
        lat.detect(img, 256, 4)
    assert e.value.code == LATCH_ERANGE
    with pytest.raises(LatchError) as e:
        lat.detect(img, -1, 4)
    assert e.value.code == LATCH_ERANGE
    with pytest.raises(LatchError) as e:
        lat.detect(img, 10, -1, kps=torch_cuda.empty((1, 4), device="cuda"))
    assert e.value.code == LATCH_EINVAL


def test_detect_then_batched_extract(torch_cuda, lat, triplets):
    """Three images detected in turn into one keypoint array (appended, with
    image ids), the device count handed to batched extraction: no host round
    trip; keypoints and descriptors equal to the oracle's."""
    from paper_1609_03986_amd.binding import image_table
    torch = torch_cuda
    g = np.random.default_rng(6)
    imgs = [synth.smoothed_noise(g, 240, 320), synth.smoothed_noise(g, 200, 300),
            synth.smoothed_noise(g, 90, 150)]
    dimgs = [torch.from_numpy(im).cuda() for im in imgs]
    cap = 12000
    kps = torch.tensor([[50.0, 50.0, 0.0, 1.0]], device="cuda").repeat(cap, 1)
    ids = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    n = torch.zeros((1,), dtype=torch.int64, device="cuda")
    for i, d in enumerate(dimgs):
        lat.detect(d, 20, cap, kps=kps, n_kps=n, image_id=ids, image_index=i)
    desc = torch.zeros((cap, 16), dtype=torch.int32, device="cuda")
    lat.extract_batch(image_table(dimgs), 3, ids, kps, desc, n_kps=n)
    torch.cuda.synchronize()
    D, K, I = desc.cpu().numpy().view(np.uint32), kps.cpu().numpy(), ids.cpu().numpy()
    first = 0
    for i, im in enumerate(imgs):
        want_k, wn = oracle.detect(im, 20)
        assert wn > 0
        sl = slice(first, first + wn)
        assert np.array_equal(K[sl], want_k) and np.all(I[sl] == i)
        want_d, _ = oracle.extract(im, want_k, triplets)
        assert np.array_equal(D[sl], want_d)
        first += wn
    assert int(n.item()) == first < cap
    assert np.all(D[first:] == 0) and np.all(I[first:] == -1)
    assert lat.check_errors(clear=True) == 0


def test_append_past_capacity(torch_cuda, lat):
    """Appending to an array that fills up: the keypoints that fit are written,
    the count keeps the full total."""
    torch = torch_cuda
    g = np.random.default_rng(8)
    a, b = synth.smoothed_noise(g, 150, 200), synth.smoothed_noise(g, 160, 180)
    ka, na = oracle.detect(a, 12)
    kb, nb = oracle.detect(b, 12)
    cap = na + nb // 2
    kps = torch.zeros((cap, 4), dtype=torch.float32, device="cuda")
    n = torch.zeros((1,), dtype=torch.int64, device="cuda")
    lat.detect(torch.from_numpy(a).cuda(), 12, cap, kps=kps, n_kps=n)
    lat.detect(torch.from_numpy(b).cuda(), 12, cap, kps=kps, n_kps=n)
    lat.detect(torch.from_numpy(a).cuda(), 12, cap, kps=kps, n_kps=n)    # nothing fits
    torch.cuda.synchronize()
    assert int(n.item()) == 2 * na + nb
    K = kps.cpu().numpy()
    assert np.array_equal(K[:na], ka) and np.array_equal(K[na:], kb[:cap - na])


def dot_image(shape, pts, background=30):
    img = np.full(shape, background, np.uint8)
    for x, y, v in pts:
        img[y, x] = v
    return img


@pytest.mark.parametrize("shape,pts", [
    ((64, 70), [(33, 40, 230), (34, 40, 230)]),                  # equal plateau: none kept
    ((64, 70), [(33, 40, 230), (34, 41, 200)]),                  # diagonal, weaker dropped
    ((64, 70), [(33, 40, 230), (32, 41, 230)]),                  # equal diagonal: none kept
    ((64, 70), [(33, 40, 230), (35, 40, 200)]),                  # two apart: both kept
    ((64, 70), [(16, 24, 230), (15, 44, 230), (53, 30, 230), (54, 50, 230)]),   # left/right border
    ((64, 70), [(24, 16, 230), (44, 15, 230), (30, 47, 230), (50, 48, 230)]),   # top/bottom border
    ((33, 33), [(16, 16, 230)]),
    ((32, 32), [(16, 16, 230)]),
])
def test_suppression_and_border_cases(torch_cuda, lat, shape, pts):
    img = dot_image(shape, pts)
    want, wn = oracle.detect(img, 10)
    kps, n = run(torch_cuda, lat, img, 10, 8)
    assert n == wn
    assert np.array_equal(kps[:n], want)
