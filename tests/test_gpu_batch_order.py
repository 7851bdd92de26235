"""GPU parity of batched extraction with the spatial order (batches of at
least 2^18 keypoints are counting-sorted by image and band of rows before
extraction): every descriptor lands in its own keypoint's row, bit-exact
against the single-image call and, on a sample, the oracle; malformed
keypoints and image entries still give zero rows and their flags; a device
count limits the order as it limits the extraction; the order's workspace is
reserved like any other."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1609_03986_amd import synth

pytestmark = pytest.mark.gpu

ORDER_MIN = 1 << 18
SENTINEL = -0x55555556


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def make_batch(seed, sizes, n):
    """n keypoints over images of the given sizes, interleaved at random, with
    some windows clamping at the borders and some malformed entries."""
    g = np.random.default_rng(seed)
    imgs = [synth.smoothed_noise(g, h, w) for h, w in sizes]
    ids = g.integers(0, len(sizes), n).astype(np.int32)
    kps = np.zeros((n, 4), np.float32)
    for i, (h, w) in enumerate(sizes):
        sel = np.nonzero(ids == i)[0]
        kps[sel] = synth.random_keypoints(g, len(sel), h, w, margin=-8)
    bad_id = g.choice(n, 40, replace=False)
    ids[bad_id[:20]] = -1
    ids[bad_id[20:]] = len(sizes) + 3
    bad_y = g.choice(np.setdiff1d(np.arange(n), bad_id), 20, replace=False)
    kps[bad_y, 1] = np.nan
    return imgs, kps, ids


def single_calls(torch, lat, dev_imgs, kps, ids):
    """Each image's keypoints through the single-image call (never ordered)."""
    want = np.zeros((len(kps), 16), np.uint32)
    for i, im in enumerate(dev_imgs):
        sel = np.nonzero(ids == i)[0]
        if len(sel):
            d = lat.extract(im, torch.from_numpy(kps[sel]).cuda())
            torch.cuda.synchronize()
            want[sel] = d.cpu().numpy().view(np.uint32)
    return want


def test_order_workspace_size(torch_cuda, triplets):
    from paper_1609_03986_amd.binding import Latch
    lat = Latch(triplets)
    try:
        assert lat.extract_batch_workspace_size(5, ORDER_MIN - 1) == 0
        assert lat.extract_batch_workspace_size(5, 0) == 0
        need = lat.extract_batch_workspace_size(5, ORDER_MIN)
        assert 12 * ORDER_MIN <= need <= 12 * ORDER_MIN + 5 * 4096
        assert lat.extract_batch_workspace_size(1 << 16, ORDER_MIN) > need
        assert lat.extract_batch_workspace_size((1 << 16) + 1, ORDER_MIN) == 0   # too many images
    finally:
        lat.close()


def test_ordered_batch_equals_single_calls(torch_cuda, triplets):
    torch = torch_cuda
    from paper_1609_03986_amd import binding
    from paper_1609_03986_amd.binding import FLAG_BAD_IMAGE, FLAG_BAD_KEYPOINT, Latch, image_table
    sizes = [(480, 640), (2000, 300), (37, 2500), (3000, 40), (1, 1), (1100, 1900), (64, 64)]
    n = ORDER_MIN + 37_000                      # ragged: not a multiple of any tile
    imgs, kps, ids = make_batch(11, sizes, n)
    dev_imgs = [torch.from_numpy(im).cuda() for im in imgs]
    table = image_table(dev_imgs)
    table[24 * 6:24 * 6 + 8] = 0                # image 6: a NULL pointer entry
    k = torch.from_numpy(kps).cuda()
    idt = torch.from_numpy(ids).cuda()
    lat = Latch(triplets)
    try:
        # A fresh handle holds no workspace: the call fails and writes nothing.
        out = torch.full((n, 16), SENTINEL, dtype=torch.int32, device="cuda")
        lib = binding.load_library()
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())
        rc = lib.latch_extract_batch(lat.h, ptr(table), len(sizes), ptr(idt), ptr(k), n, None,
                                     ptr(out), None)
        assert rc == binding.LATCH_EWORKSPACE
        assert b"latch_reserve" in lib.latch_last_error(lat.h)
        torch.cuda.synchronize()
        assert (out == SENTINEL).all()

        lat.reserve(lat.extract_batch_workspace_size(len(sizes), n))
        lat.timing(True)
        lat.extract_batch(table, len(sizes), idt, k, desc=out)
        torch.cuda.synchronize()
        assert lat.timing_read("extract_order")[0] == 1          # the order ran
        lat.timing(False)
        got = out.cpu().numpy().view(np.uint32)
        flags = lat.check_errors(clear=True)
        assert flags == FLAG_BAD_IMAGE | FLAG_BAD_KEYPOINT

        bad_image = (ids < 0) | (ids >= len(sizes)) | (ids == 6)
        assert not got[bad_image].any()
        want = single_calls(torch, lat, dev_imgs[:6], kps, np.where(bad_image, -1, ids))
        lat.check_errors(clear=True)
        assert np.array_equal(got, want)

        # The oracle on a sample of the well-formed rows.
        good = np.nonzero(~bad_image & np.isfinite(kps[:, 1]))[0][::97]
        for i in range(6):
            sel = good[ids[good] == i]
            if len(sel):
                d, f = oracle.extract(imgs[i], kps[sel], triplets)
                assert f == 0
                assert np.array_equal(got[sel], d)
    finally:
        lat.close()


def test_device_count_limits_the_order(torch_cuda, triplets):
    torch = torch_cuda
    from paper_1609_03986_amd.binding import Latch, image_table
    sizes = [(900, 1200), (300, 2800), (2200, 500)]
    n = ORDER_MIN + 5000
    imgs, kps, ids = make_batch(12, sizes, n)
    ids = np.clip(ids, 0, len(sizes) - 1)
    kps[:, 1] = np.nan_to_num(kps[:, 1], nan=5.0)
    dev_imgs = [torch.from_numpy(im).cuda() for im in imgs]
    table = image_table(dev_imgs)
    k = torch.from_numpy(kps).cuda()
    idt = torch.from_numpy(ids).cuda()
    lat = Latch(triplets)
    try:
        full = lat.extract_batch(table, len(sizes), idt, k).cpu().numpy().view(np.uint32)
        m = n - 12_345
        out = torch.full((n, 16), SENTINEL, dtype=torch.int32, device="cuda")
        lat.extract_batch(table, len(sizes), idt, k, desc=out,
                          n_kps=torch.tensor([m], dtype=torch.int64, device="cuda"))
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint32)
        assert np.array_equal(got[:m], full[:m])
        assert np.all(got[m:] == 0xAAAAAAAA)     # untouched past the device count
        assert lat.check_errors(clear=True) == 0
        want = single_calls(torch, lat, dev_imgs, kps, ids)
        assert np.array_equal(full, want)
    finally:
        lat.close()


def test_interleaved_tall_images(torch_cuda, triplets):
    """100 images of 2048 rows (64 bands each), keypoints interleaved at random:
    a chunk of consecutive keypoints spans more buckets than the per-chunk
    LDS count holds, so ranks come from one global atomic per keypoint."""
    torch = torch_cuda
    from paper_1609_03986_amd.binding import Latch, image_table
    g = np.random.default_rng(13)
    sizes = [(2048, 24 + (i % 5)) for i in range(100)]
    n = ORDER_MIN + 1234
    imgs = [synth.smoothed_noise(g, h, w) for h, w in sizes]
    ids = g.integers(0, len(sizes), n).astype(np.int32)
    kps = np.zeros((n, 4), np.float32)
    for i, (h, w) in enumerate(sizes):
        sel = np.nonzero(ids == i)[0]
        kps[sel] = synth.random_keypoints(g, len(sel), h, w, margin=-8)
    dev_imgs = [torch.from_numpy(im).cuda() for im in imgs]
    lat = Latch(triplets)
    try:
        got = lat.extract_batch(image_table(dev_imgs), len(sizes), torch.from_numpy(ids).cuda(),
                                torch.from_numpy(kps).cuda())
        torch.cuda.synchronize()
        assert lat.check_errors(clear=True) == 0
        want = single_calls(torch, lat, dev_imgs, kps, ids)
        assert np.array_equal(got.cpu().numpy().view(np.uint32), want)
    finally:
        lat.close()


def test_plan_with_order_and_device_count(torch_cuda, triplets):
    """A captured plan over 2^18 + 3,000 keypoints (so the order runs inside the
    graph) replayed with the full count, a smaller one and the full one again:
    descriptors equal the single-image calls up to the count and are untouched
    past it, and matches equal eager batched matching of those descriptors."""
    torch = torch_cuda
    from paper_1609_03986_amd.binding import Latch, image_table, pair_table
    g = np.random.default_rng(14)
    sizes = [(1200, 1600), (900, 1000), (1500, 700)]
    counts = [100_000, 90_000, ORDER_MIN + 3000 - 190_000]
    imgs = [synth.smoothed_noise(g, h, w) for h, w in sizes]
    kps = np.concatenate([synth.random_keypoints(g, n, h, w, margin=-8)
                          for (h, w), n in zip(sizes, counts)]).astype(np.float32)
    ids = np.repeat(np.arange(3, dtype=np.int32), counts)
    n = len(kps)
    first = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.int64)
    pairs_np = np.array([(first[i], counts[i], first[i + 1], counts[i + 1], first[i])
                         for i in range(2)], np.int64)
    dev_imgs = [torch.from_numpy(im).cuda() for im in imgs]
    lat = Latch(triplets)
    try:
        table = image_table(dev_imgs)
        k = torch.from_numpy(kps).cuda()
        idt = torch.from_numpy(ids).cuda()
        nk = torch.tensor([n], dtype=torch.int64, device="cuda")
        desc = torch.full((n, 16), SENTINEL, dtype=torch.int32, device="cuda")
        idx = torch.full((n, 2), -7, dtype=torch.int32, device="cuda")
        dist = torch.full((n, 2), -7, dtype=torch.int32, device="cuda")
        acc = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
        pairs = pair_table(pairs_np)
        plan = lat.plan(table, 3, idt, k, desc, pairs, idx, dist, acc, n_kps=nk)
        want = single_calls(torch, lat, dev_imgs, kps, ids)
        try:
            for count in (n, n - 50_001, n):
                nk.fill_(count)
                desc.fill_(SENTINEL)
                plan.run()
                torch.cuda.synchronize()
                got = desc.cpu().numpy().view(np.uint32)
                assert np.array_equal(got[:count], want[:count])
                assert np.all(got[count:] == 0xAAAAAAAA)
            # The last replay matched the whole set: same as eager batched matching.
            e_idx, e_dist, e_acc = lat.knn_batch(desc, desc, pairs, n)
            torch.cuda.synchronize()
            q = counts[0] + counts[1]                 # the query rows of the two pairs
            assert torch.equal(idx[:q], e_idx[:q]) and torch.equal(dist[:q], e_dist[:q])
            assert torch.equal(acc[:q], e_acc[:q])
            assert lat.check_errors(clear=True) == 0
        finally:
            plan.close()
    finally:
        lat.close()


@pytest.mark.parametrize("n_images,shuffled", [(1, False), (16, True), (17, True), (64, False), (65, False),
                                               (200, True)])
def test_order_over_many_buckets(torch_cuda, triplets, n_images, shuffled):
    """Bucket counts on both sides of a chunk's span and of the scan's 4096 entries, keypoints image
    by image and shuffled: the ordered batch equals unordered parts of it."""
    torch = torch_cuda
    from paper_1609_03986_amd.binding import Latch, image_table
    g = np.random.default_rng(n_images)
    n = ORDER_MIN + 1025
    imgs = [torch.from_numpy(g.integers(0, 256, (2048, 64), dtype=np.uint8)).cuda() for _ in range(n_images)]
    ids = np.sort(g.integers(0, n_images, n)).astype(np.int32)
    if shuffled:
        g.shuffle(ids)
    kps = np.zeros((n, 4), np.float32)
    kps[:, 0], kps[:, 1] = g.uniform(0, 64, n), g.uniform(-3, 2051, n)
    kps[:, 2], kps[:, 3] = g.uniform(0, 360, n), g.uniform(0.5, 2, n)
    idt, k = torch.from_numpy(ids).cuda(), torch.from_numpy(kps).cuda()
    table = image_table(imgs)
    lat = Latch(triplets)
    try:
        got = lat.extract_batch(table, n_images, idt, k)
        half = n // 2
        for part in (slice(0, half), slice(half, n)):
            want = lat.extract_batch(table, n_images, idt[part].contiguous(), k[part].contiguous())
            assert torch.equal(got[part], want)
        assert lat.check_errors(clear=True) == 0
    finally:
        lat.close()


def test_order_in_several_launches(torch_cuda, triplets):
    """A batch that runs in three launches, with a device count inside the last: the descriptors
    before the count equal unordered parts, those after it stay untouched."""
    torch = torch_cuda
    from paper_1609_03986_amd.binding import Latch, image_table
    g = np.random.default_rng(5)
    n, count = 1_200_001, 1_100_003
    imgs = [torch.from_numpy(g.integers(0, 256, (300, 200), dtype=np.uint8)).cuda() for _ in range(3)]
    ids = torch.from_numpy(g.integers(0, 3, n).astype(np.int32)).cuda()
    kps = np.zeros((n, 4), np.float32)
    kps[:, 0], kps[:, 1] = g.uniform(0, 200, n), g.uniform(0, 300, n)
    kps[:, 2], kps[:, 3] = g.uniform(0, 360, n), 1
    k = torch.from_numpy(kps).cuda()
    table = image_table(imgs)
    lat = Latch(triplets)
    try:
        got = torch.full((n, 16), -7, dtype=torch.int32, device="cuda")
        lat.extract_batch(table, 3, ids, k, desc=got,
                          n_kps=torch.tensor([count], dtype=torch.int64, device="cuda"))
        assert bool((got[count:] == -7).all())
        for first in range(0, count, 200_000):
            part = slice(first, min(count, first + 200_000))
            assert torch.equal(got[part], lat.extract_batch(table, 3, ids[part].contiguous(),
                                                            k[part].contiguous()))
        assert lat.check_errors(clear=True) == 0
    finally:
        lat.close()
