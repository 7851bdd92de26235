"""GPU test of captured plans (latch_plan_*): one HIP graph holding batched
extraction + batched matching, replayed several times with eager work and
synchronisations in between and with new batch contents written into the
same buffers; every replay must equal the eager calls (and the oracle)."""
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


MAX_IMAGES, MAX_KPS, MAX_PAIRS = 6, 6000, 5


def batch_contents(seed):
    """Images, keypoints (grouped by image), ids, and consecutive pairs."""
    g = np.random.default_rng(seed)
    n_img = int(g.integers(3, MAX_IMAGES + 1))
    sizes = [(int(g.integers(60, 400)), int(g.integers(60, 500))) for _ in range(n_img)]
    counts = [int(g.integers(0, MAX_KPS // MAX_IMAGES)) for _ in range(n_img)]
    imgs = [synth.smoothed_noise(g, h, w) for h, w in sizes]
    kps = np.concatenate([synth.random_keypoints(g, c, h, w, margin=-5)
                          for (h, w), c in zip(sizes, counts)])
    ids = np.repeat(np.arange(n_img, dtype=np.int32), counts)
    first = np.concatenate([[0], np.cumsum(counts)[:-1]])
    pairs = np.array([(first[i], counts[i], first[i + 1], counts[i + 1], first[i])
                      for i in range(n_img - 1)], np.int64)
    return imgs, kps.astype(np.float32), ids, pairs


def write_contents(torch, bufs, imgs, kps, ids, pairs):
    from paper_1609_03986_amd.binding import image_table
    dimgs = [torch.from_numpy(im).cuda() for im in imgs]
    table = image_table(dimgs + [dimgs[0]] * (MAX_IMAGES - len(dimgs)))
    bufs["table"].copy_(table)
    n = len(kps)
    bufs["kps"][:n].copy_(torch.from_numpy(kps))
    bufs["ids"][:n].copy_(torch.from_numpy(ids))
    bufs["n"].fill_(n)
    p = np.zeros((MAX_PAIRS, 5), np.int64)      # unused pairs: nq = nt = 0
    p[:len(pairs)] = pairs
    bufs["pairs"].copy_(torch.from_numpy(p))
    torch.cuda.synchronize()
    return dimgs


def test_plan_replays_equal_eager_and_oracle(torch_cuda, lat, triplets):
    torch = torch_cuda
    bufs = {
        "table": torch.zeros(MAX_IMAGES * 24, dtype=torch.uint8, device="cuda"),
        "kps": torch.zeros((MAX_KPS, 4), dtype=torch.float32, device="cuda"),
        "ids": torch.zeros(MAX_KPS, dtype=torch.int32, device="cuda"),
        "n": torch.zeros(1, dtype=torch.int64, device="cuda"),
        "desc": torch.zeros((MAX_KPS, 16), dtype=torch.int32, device="cuda"),
        "pairs": torch.zeros((MAX_PAIRS, 5), dtype=torch.int64, device="cuda"),
        "idx": torch.zeros((MAX_KPS, 2), dtype=torch.int32, device="cuda"),
        "dist": torch.zeros((MAX_KPS, 2), dtype=torch.int32, device="cuda"),
        "acc": torch.zeros(MAX_KPS, dtype=torch.uint8, device="cuda"),
    }
    imgs, kps, ids, pairs = batch_contents(0)
    keep = write_contents(torch, bufs, imgs, kps, ids, pairs)
    plan = lat.plan(bufs["table"], MAX_IMAGES, bufs["ids"], bufs["kps"], bufs["desc"],
                    bufs["pairs"], bufs["idx"], bufs["dist"], bufs["acc"], n_kps=bufs["n"])
    try:
        for rep in range(4):
            if rep in (1, 3):                          # new contents, same buffers
                imgs, kps, ids, pairs = batch_contents(rep)
                keep = write_contents(torch, bufs, imgs, kps, ids, pairs)
            for t in ("desc", "idx", "dist"):
                bufs[t].fill_(-7)
            torch.cuda.synchronize()
            plan.run()
            torch.cuda.synchronize()
            n = len(kps)
            got_desc = bufs["desc"][:n].cpu().numpy().view(np.uint32)
            got_idx = bufs["idx"][:n].cpu().numpy()
            got_dist = bufs["dist"][:n].cpu().numpy()
            got_acc = bufs["acc"][:n].cpu().numpy()
            # eager work between replays, and the eager result of the same batch
            eager = lat.extract_batch(bufs["table"], MAX_IMAGES, bufs["ids"][:n], bufs["kps"][:n])
            ei, ed, ea = lat.knn_batch(eager, eager, bufs["pairs"], n)
            torch.cuda.synchronize()
            assert np.array_equal(got_desc, eager.cpu().numpy().view(np.uint32)), rep
            nq_total = int(pairs[:, 1].sum()) if len(pairs) else 0
            rows = np.concatenate([np.arange(p[4], p[4] + p[1]) for p in pairs]) if nq_total else []
            assert np.array_equal(got_idx[rows], ei.cpu().numpy()[rows]), rep
            assert np.array_equal(got_dist[rows], ed.cpu().numpy()[rows]), rep
            assert np.array_equal(got_acc[rows], ea.cpu().numpy()[rows]), rep
            # and the oracle, for the descriptors of one image and one pair
            i = len(imgs) // 2
            sel = np.nonzero(ids == i)[0]
            want, _ = oracle.extract(imgs[i], kps[sel], triplets)
            assert np.array_equal(got_desc[sel], want), rep
            qf, nq, tf, nt, of = pairs[0]
            wi, wd, wa = oracle.knn(got_desc[qf:qf + nq], got_desc[tf:tf + nt])
            assert np.array_equal(got_idx[of:of + nq], wi), rep
            assert lat.check_errors(clear=True) == 0
    finally:
        plan.close()
        del keep


@pytest.mark.parametrize("path", ["fp4", "mfma", "popcount"])
def test_plan_of_every_path_with_a_long_pair(torch_cuda, lat, path):
    """A plan holds the memory for dividing train ranges on the FP4 path and none on the others; a
    pair long enough to be divided, with short ones, gives what the eager calls give, replay after
    replay, while an eager batch on the handle divides ranges of its own in between."""
    from paper_1609_03986_amd.binding import image_table, pair_table
    torch = torch_cuda
    g = np.random.default_rng(17)
    counts = [500, 9000, 40, 700]
    imgs = [torch.from_numpy(synth.smoothed_noise(g, 200, 260)).cuda() for _ in counts]
    kps = torch.from_numpy(np.concatenate([synth.random_keypoints(g, c, 200, 260) for c in counts])
                           .astype(np.float32)).cuda()
    ids = torch.from_numpy(np.repeat(np.arange(4, dtype=np.int32), counts)).cuda()
    first = np.concatenate([[0], np.cumsum(counts)[:-1]])
    pairs = pair_table([(first[i], counts[i], first[i + 1], counts[i + 1], first[i]) for i in range(3)])
    total, table = sum(counts), image_table(imgs)
    desc = lat.extract_batch(table, 4, ids, kps)
    want = (desc,) + lat.knn_batch(desc, desc, pairs, total, path=path)
    out = [torch.zeros_like(x) for x in want]
    plan = lat.plan(table, 4, ids, kps, out[0], pairs, out[1], out[2], out[3], path=path)
    try:
        for _ in range(3):
            out[0].zero_()
            for x, w in zip(out[1:], want[1:]):
                x.copy_(w)                                   # rows that no pair writes
                x[:total - counts[3]] = 5
            plan.run()
            torch.cuda.synchronize()
            for x, w in zip(out, want):
                assert bool((x == w).all())
            again = lat.knn_batch(desc, desc, pairs, total, path="fp4")
            assert all(bool((a == w).all()) for a, w in zip(again, want[1:]))
    finally:
        plan.close()
