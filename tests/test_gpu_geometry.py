"""GPU parity of extraction with the paper's CLATCH geometry and per-pixel
patch weights (latch_create_geometry): descriptors bit-exactly equal to the
oracle's weighted extraction, single-image and batched, with ragged counts,
clamped borders, all angles and scales, and out-of-domain keypoints."""
import numpy as np
import pytest

import oracle
from paper_1609_03986_amd import synth

pytestmark = pytest.mark.gpu

GEOMETRIES = {
    "64x8_gauss": (64, 8, lambda: synth.gaussian_weights(8, 2.0, 128)),
    "64x8_7x7": (64, 8, synth.clatch_7x7_weights),
    "64x8_ones": (64, 8, lambda: None),
    "64x7_rand": (64, 7, lambda: np.random.default_rng(1).integers(0, 129, (7, 7)).astype(np.uint8)),
    "48x8_rand": (48, 8, lambda: np.random.default_rng(2).integers(0, 129, (8, 8)).astype(np.uint8)),
    "48x7_weighted": (48, 7, lambda: synth.gaussian_weights(7, 1.5, 100)),
}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def keypoints(g, n, H, W):
    kps = synth.random_keypoints(g, n, H, W, margin=0)
    kps[:6] = [[0, 0, 45, 1], [W - 1, H - 1, 200, 2.0], [-5, 10, 0, 1], [W / 2, H / 2, 0, 4.0],
               [10.5, 20.5, 90, 1], [W / 3, H / 3, 359.9, 0.5]]
    kps[6] = [np.nan, 5, 0, 1]                              # outside the rule: zero + flag
    kps[7] = [20, 20, 0, 0.001]                             # sq = 0: outside
    return kps


@pytest.mark.parametrize("name", sorted(GEOMETRIES))
def test_single_image_matches_oracle(torch_cuda, name):
    from paper_1609_03986_amd.binding import FLAG_BAD_KEYPOINT, Latch
    torch = torch_cuda
    window, patch, wf = GEOMETRIES[name]
    w = wf()
    trip = synth.triplet_table_geom(window, patch)
    g = np.random.default_rng(hash(name) % 1000)
    H, W = 300, 410
    img = synth.textured_image(g, H, W, n_rect=40, n_blob=40)
    kps = keypoints(g, 1037, H, W)
    lat = Latch(trip, window=window, patch=patch, weights=w)
    try:
        lat.check_errors(clear=True)
        d = lat.extract(torch.from_numpy(img).cuda(), torch.from_numpy(kps).cuda())
        torch.cuda.synchronize()
        got = d.cpu().numpy().view(np.uint32)
        want, f = oracle.extract_geom(img, kps, trip, window, patch, w)
        assert f == FLAG_BAD_KEYPOINT
        bad = np.nonzero((got != want).any(1))[0]
        assert bad.size == 0, (name, bad[:10])
        assert lat.check_errors(clear=True) == FLAG_BAD_KEYPOINT
    finally:
        lat.close()


def test_batched_images_match_oracle(torch_cuda):
    from paper_1609_03986_amd.binding import Latch, image_table
    torch = torch_cuda
    window, patch = 64, 8
    w = synth.gaussian_weights(8, 2.5, 90)
    trip = synth.triplet_table_geom(window, patch)
    g = np.random.default_rng(21)
    shapes = [(240, 320), (97, 130), (480, 640)]
    imgs = [synth.smoothed_noise(g, h, wd) for h, wd in shapes]
    counts = [700, 65, 1300]
    kps = np.concatenate([synth.random_keypoints(g, c, h, wd, margin=0) for c, (h, wd) in zip(counts, shapes)])
    ids = np.repeat(np.arange(3, dtype=np.int32), counts)
    lat = Latch(trip, window=window, patch=patch, weights=w)
    try:
        dimgs = [torch.from_numpy(im).cuda() for im in imgs]
        d = lat.extract_batch(image_table(dimgs), 3, torch.from_numpy(ids).cuda(), torch.from_numpy(kps).cuda())
        torch.cuda.synchronize()
        got = d.cpu().numpy().view(np.uint32)
        first = 0
        for im, c in zip(imgs, counts):
            want, _ = oracle.extract_geom(im, kps[first:first + c], trip, window, patch, w)
            assert np.array_equal(got[first:first + c], want)
            first += c
        assert lat.check_errors(clear=True) == 0
    finally:
        lat.close()


def test_7x7_weights_equal_7x7_patches_on_gpu(torch_cuda):
    """The paper's statement on the GPU path: zero weights on the first row and
    column of the 8 x 8 patch give the 7 x 7 descriptor exactly."""
    from paper_1609_03986_amd.binding import Latch
    torch = torch_cuda
    trip = synth.triplet_table_geom(64, 8)
    g = np.random.default_rng(22)
    img = torch.from_numpy(synth.textured_image(g, 256, 256, n_rect=30, n_blob=30)).cuda()
    kps = torch.from_numpy(synth.random_keypoints(g, 500, 256, 256)).cuda()
    a, b = Latch(trip, 64, 8, synth.clatch_7x7_weights()), Latch(trip, 64, 7)
    try:
        da, db = a.extract(img, kps), b.extract(img, kps)
        torch.cuda.synchronize()
        assert torch.equal(da, db)
    finally:
        a.close()
        b.close()


def test_hd_sampled(torch_cuda):
    """20,000 keypoints on a 1920 x 1080 image in one launch; every 40th
    descriptor checked against the oracle."""
    from paper_1609_03986_amd.binding import Latch
    torch = torch_cuda
    w = synth.gaussian_weights(8, 2.0, 128)
    trip = synth.triplet_table_geom(64, 8)
    wl = synth.workload_hd()
    kps = np.concatenate([wl["query_kps"], wl["train_kps"]])
    lat = Latch(trip, 64, 8, w)
    try:
        d = lat.extract(torch.from_numpy(wl["query_image"]).cuda(), torch.from_numpy(kps).cuda())
        torch.cuda.synchronize()
        got = d.cpu().numpy().view(np.uint32)
        sel = np.arange(0, len(kps), 40)
        want, _ = oracle.extract_geom(wl["query_image"], kps[sel], trip, 64, 8, w)
        assert np.array_equal(got[sel], want)
    finally:
        lat.close()


def test_plan_with_geometry_handle(torch_cuda):
    """A captured plan (batched extraction + matching in one HIP graph) of a
    weighted-geometry handle: replays equal the oracle's weighted descriptors
    and its 2-NN."""
    from paper_1609_03986_amd.binding import Latch, image_table
    torch = torch_cuda
    w = synth.gaussian_weights(8, 2.0, 128)
    trip = synth.triplet_table_geom(64, 8)
    g = np.random.default_rng(23)
    imgs = [synth.smoothed_noise(g, 200, 260), synth.smoothed_noise(g, 150, 300)]
    counts = [900, 700]
    kps = np.concatenate([synth.random_keypoints(g, c, *im.shape, margin=-5) for c, im in zip(counts, imgs)])
    ids = np.repeat(np.arange(2, dtype=np.int32), counts)
    pairs = np.array([[0, counts[0], counts[0], counts[1], 0]], np.int64)
    lat = Latch(trip, 64, 8, w)
    try:
        dimgs = [torch.from_numpy(im).cuda() for im in imgs]
        table = image_table(dimgs)
        dk, di = torch.from_numpy(kps).cuda(), torch.from_numpy(ids).cuda()
        desc = torch.zeros((len(kps), 16), dtype=torch.int32, device="cuda")
        dp = torch.from_numpy(pairs).cuda()
        idx = torch.zeros((len(kps), 2), dtype=torch.int32, device="cuda")
        dist = torch.zeros_like(idx)
        acc = torch.zeros(len(kps), dtype=torch.uint8, device="cuda")
        plan = lat.plan(table, 2, di, dk, desc, dp, idx, dist, acc)
        try:
            for rep in range(3):
                desc.fill_(-1)
                idx.fill_(-7)
                torch.cuda.synchronize()
                plan.run()
                torch.cuda.synchronize()
                D = desc.cpu().numpy().view(np.uint32)
                for i, im in enumerate(imgs):
                    sel = np.nonzero(ids == i)[0]
                    want, _ = oracle.extract_geom(im, kps[sel], trip, 64, 8, w)
                    assert np.array_equal(D[sel], want), (rep, i)
                wi, wd, wa = oracle.knn(D[:counts[0]], D[counts[0]:])
                assert np.array_equal(idx.cpu().numpy()[:counts[0]], wi), rep
                assert np.array_equal(acc.cpu().numpy()[:counts[0]], wa), rep
        finally:
            plan.close()
    finally:
        lat.close()


@pytest.mark.parametrize("sq", [4, 64, 256, 307, 512, 1024])
@pytest.mark.parametrize("window", [48, 64])
def test_every_fourth_angle_bin_by_scale(torch_cuda, window, sq):
    """Windows sampled along image rows at every fourth angle bin (all octants, exact diagonals
    and axes) and scales with and without offsets halfway between two pixels, from an interior
    centre, and every 64th bin at a corner (clamped)."""
    from paper_1609_03986_amd.binding import Latch
    torch = torch_cuda
    g = np.random.default_rng(window * 10_000 + sq)
    img = g.integers(0, 256, (311, 337), dtype=np.uint8)
    kps = np.zeros((1024 + 64, 4), np.float32)
    kps[:, 0], kps[:, 1], kps[:, 3] = 168, 155, sq / 256.0
    kps[:1024, 2] = np.arange(1024) * (360.0 / 1024.0)
    kps[1024:, 2] = kps[:1024:16, 2]
    kps[1024:, :2] = 4, 300
    trip, w = synth.triplet_table_geom(window, 8), synth.gaussian_weights(8, 2.0, 128)
    lat = Latch(trip, window=window, patch=8, weights=w)
    try:
        got = lat.extract(torch.from_numpy(img).cuda(), torch.from_numpy(kps).cuda())
        want, f = oracle.extract_geom(img, kps, trip, window, 8, w)
        assert f == 0 and lat.check_errors(clear=True) == 0
        assert np.array_equal(got.cpu().numpy().view(np.uint32), want)
    finally:
        lat.close()
