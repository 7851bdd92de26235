"""GPU parity of batched matching (hamming_knn_batch): many query/train pairs
in one persistent launch, each pair exactly equal to the oracle's brute-force
2-NN on its ranges and to the single hamming_knn call."""
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


def dev(torch, d):
    return torch.from_numpy(np.ascontiguousarray(d, np.uint32).view(np.int32)).cuda()


def consecutive_pairs(counts):
    """Pairs (i, i + 1) of images with `counts` descriptors each, in one array."""
    first = np.concatenate([[0], np.cumsum(counts)[:-1]])
    rows, out = [], 0
    for i in range(len(counts) - 1):
        rows.append((first[i], counts[i], first[i + 1], counts[i + 1], out))
        out += counts[i]
    return rows, out


def check_pairs(torch, lat, D, rows, out_rows, k, ratio, path):
    from paper_1609_03986_amd.binding import pair_table
    Dd = dev(torch, D)
    idx, dist, acc = lat.knn_batch(Dd, Dd, pair_table(rows), out_rows, k=k, ratio=ratio, path=path)
    torch.cuda.synchronize()
    idx, dist, acc = idx.cpu().numpy(), dist.cpu().numpy(), acc.cpu().numpy()
    for qf, nq, tf, nt, of in rows:
        wi, wd, wa = oracle.knn(D[qf:qf + nq], D[tf:tf + nt], k=k, ratio=ratio)
        assert np.array_equal(idx[of:of + nq], wi), (path, qf, nq, tf, nt)
        assert np.array_equal(dist[of:of + nq], wd), (path, qf, nq, tf, nt)
        assert np.array_equal(acc[of:of + nq], wa), (path, qf, nq, tf, nt)
    return idx, dist, acc


@pytest.mark.parametrize("path", ["mfma", "fp4", "popcount"])
def test_uneven_consecutive_pairs(torch_cuda, lat, path):
    g = np.random.default_rng(7)
    counts = [300, 0, 257, 1, 2, 511, 33, 1000, 640, 5]
    D = synth.random_descriptors(g, sum(counts), 0.3)
    D[100:140] = D[400:440]                       # cross-image duplicates: ties
    rows, out_rows = consecutive_pairs(counts)
    for k in (1, 2):
        check_pairs(torch_cuda, lat, D, rows, out_rows, k, 0.8, path)
    assert lat.check_errors(clear=True) == 0


def test_batch_equals_single_calls(torch_cuda, lat):
    g = np.random.default_rng(8)
    counts = [700, 900, 650, 1200]
    D = synth.random_descriptors(g, sum(counts))
    rows, out_rows = consecutive_pairs(counts)
    idx, dist, acc = check_pairs(torch_cuda, lat, D, rows, out_rows, 2, 0.8, "auto")
    for qf, nq, tf, nt, of in rows:
        si, sd, sa = lat.knn(dev(torch_cuda, D[qf:qf + nq]), dev(torch_cuda, D[tf:tf + nt]))
        torch_cuda.cuda.synchronize()
        assert np.array_equal(si.cpu().numpy(), idx[of:of + nq])
        assert np.array_equal(sd.cpu().numpy(), dist[of:of + nq])
        assert np.array_equal(sa.cpu().numpy(), acc[of:of + nq])


def test_out_of_range_pair_is_flagged_and_skipped(torch_cuda, lat):
    from paper_1609_03986_amd.binding import FLAG_BAD_PAIR, pair_table
    g = np.random.default_rng(9)
    D = synth.random_descriptors(g, 400)
    rows = [(0, 100, 100, 100, 0), (200, 100, 350, 100, 100), (300, 50, 0, 200, 200)]  # 2nd: train past the end
    Dd = dev(torch_cuda, D)
    idx, dist, acc = lat.knn_batch(Dd, Dd, pair_table(rows), 250)
    torch_cuda.cuda.synchronize()
    assert lat.check_errors(clear=True) & FLAG_BAD_PAIR
    idx = idx.cpu().numpy()
    assert np.all(idx[100:200] == -2)             # untouched
    wi, _, _ = oracle.knn(D[0:100], D[100:200])
    assert np.array_equal(idx[0:100], wi)
    wi, _, _ = oracle.knn(D[300:350], D[0:200])
    assert np.array_equal(idx[200:250], wi)


def test_sfm_shaped_batch_sampled(torch_cuda, lat, triplets):
    """Eight overlapping crops of one mosaic, 3,000 keypoints each, extracted in
    one batched launch and matched as 7 consecutive pairs in one batched launch;
    every 9th query of every pair checked against the oracle."""
    from paper_1609_03986_amd.binding import image_table, pair_table
    torch = torch_cuda
    g = np.random.default_rng(64)
    H, W, n_img, n_kp = 600, 800, 8, 3000
    mosaic = synth.textured_image(g, H + 16 * n_img, W + 16 * n_img, n_rect=60, n_blob=60)
    imgs = [np.clip(mosaic[8 * i:8 * i + H, 16 * i:16 * i + W].astype(int)
                    + g.integers(-4, 5, (H, W)), 0, 255).astype(np.uint8) for i in range(n_img)]
    kps = np.concatenate([synth.random_keypoints(g, n_kp, H, W) for _ in range(n_img)])
    ids = np.repeat(np.arange(n_img, dtype=np.int32), n_kp)
    dimgs = [torch.from_numpy(im).cuda() for im in imgs]
    desc = lat.extract_batch(image_table(dimgs), n_img, torch.from_numpy(ids).cuda(),
                             torch.from_numpy(kps).cuda())
    rows, out_rows = consecutive_pairs([n_kp] * n_img)
    idx, dist, acc = lat.knn_batch(desc, desc, pair_table(rows), out_rows)
    torch.cuda.synchronize()
    D = desc.cpu().numpy().view(np.uint32)
    want_d, f = oracle.extract(imgs[3], kps[3 * n_kp:4 * n_kp], triplets)
    assert np.array_equal(D[3 * n_kp:4 * n_kp], want_d)
    idx, dist, acc = idx.cpu().numpy(), dist.cpu().numpy(), acc.cpu().numpy()
    for qf, nq, tf, nt, of in rows:
        sel = np.arange(0, nq, 9)
        wi, wd, wa = oracle.knn(D[qf + sel], D[tf:tf + nt])
        assert np.array_equal(idx[of + sel], wi)
        assert np.array_equal(dist[of + sel], wd)
        assert np.array_equal(acc[of + sel], wa)
    assert lat.check_errors(clear=True) == 0


@pytest.mark.parametrize("path", ["fp4", "mfma"])
def test_long_train_ranges(torch_cuda, lat, path):
    """Pairs whose train range exceeds 2^14 rows: the MXFP4 batch matcher scans
    such a range in pieces of 2^14 rows and merges them in registers; ties
    across piece boundaries resolve to the lowest index."""
    g = np.random.default_rng(12)
    counts = [70, 16385, 300, 40000, 5]
    D = synth.random_descriptors(g, sum(counts), 0.05)
    D[70 + 16384] = D[70]                         # tie across the 2^14 boundary of pair 0
    D[70 + 16385 + 300 + 20000] = D[70 + 16385 + 5]
    rows, out_rows = consecutive_pairs(counts)
    check_pairs(torch_cuda, lat, D, rows, out_rows, 2, 0.8, path)
    assert lat.check_errors(clear=True) == 0


@pytest.mark.parametrize("path", ["fp4", "mfma"])
def test_many_pairs_across_cost_classes(torch_cuda, lat, path):
    """700 pairs (more than the setup block's 256 threads) in random order,
    train lengths log-uniform over 0..20,000 rows (work items laid out over
    several dozen cost classes, longest first), query counts 0..300, train
    ranges overlapping anywhere in the array: every pair's rows equal the
    single hamming_knn call on its ranges, and a sample equals the oracle."""
    from paper_1609_03986_amd.binding import pair_table
    torch = torch_cuda
    g = np.random.default_rng(21)
    n_rows = 30_000
    D = synth.random_descriptors(g, n_rows, 0.2)
    n_pairs = 700
    nt = np.floor(np.exp(g.uniform(0, np.log(20_001), n_pairs))).astype(np.int64) - 1
    nt[g.choice(n_pairs, 20, replace=False)] = 0
    nq = g.integers(0, 301, n_pairs)
    rows, out = [], 0
    for i in range(n_pairs):
        qf = int(g.integers(0, n_rows - nq[i] + 1))
        tf = int(g.integers(0, n_rows - nt[i] + 1))
        rows.append((qf, int(nq[i]), tf, int(nt[i]), out))
        out += int(nq[i])
    Dd = dev(torch, D)
    idx, dist, acc = lat.knn_batch(Dd, Dd, pair_table(rows), out, path=path)
    torch.cuda.synchronize()
    assert lat.check_errors(clear=True) == 0
    idx, dist, acc = idx.cpu().numpy(), dist.cpu().numpy(), acc.cpu().numpy()
    for i, (qf, q, tf, t, of) in enumerate(rows):
        if q == 0:
            continue
        si, sd, sa = lat.knn(Dd[qf:qf + q], Dd[tf:tf + t], path=path)
        torch.cuda.synchronize()
        assert np.array_equal(idx[of:of + q], si.cpu().numpy()), (i, q, t)
        assert np.array_equal(dist[of:of + q], sd.cpu().numpy()), (i, q, t)
        assert np.array_equal(acc[of:of + q], sa.cpu().numpy()), (i, q, t)
        if i % 7 == 0:
            sel = np.arange(0, q, 37)
            wi, wd, wa = oracle.knn(D[qf + sel], D[tf:tf + t])
            assert np.array_equal(idx[of + sel], wi), (i, q, t)
            assert np.array_equal(dist[of + sel], wd), (i, q, t)
            assert np.array_equal(acc[of + sel], wa), (i, q, t)
    assert lat.check_errors(clear=True) == 0


# Train rows around the least part of a divided train range (80 tiles of 32 rows) and its
# multiples, several 2^14-row ranges within a part, and short pairs beside long ones.
DIVIDED = [[(300, 2560), (5, 2561)], [(300, 3072), (5, 3073)], [(600, 5121)], [(385, 6145), (1, 3104)], [(768, 9_000), (384, 33), (0, 9_000)],
           [(40, 300_000)], [(1500, 20_000), (100, 0), (100, 1), (3000, 500), (64, 40_001)]]


@pytest.mark.parametrize("p", [0.5, 0.01])
@pytest.mark.parametrize("blocks", [2, 3])
@pytest.mark.parametrize("sizes", DIVIDED)
def test_divided_train_ranges(torch_cuda, lat, triplets, sizes, blocks, p):
    """Pairs whose train rows several workgroups share: parts merge to the oracle's results, with
    random and heavily tied descriptors, on every call, and with a workspace that holds no room
    for dividing."""
    import ctypes
    from paper_1609_03986_amd.binding import Latch, Tuning, load_library, pair_table
    g = np.random.default_rng(sum(a * 31 + b for a, b in sizes))
    Q = synth.random_descriptors(g, sum(a for a, _ in sizes), p)
    T = synth.random_descriptors(g, max(b for _, b in sizes) + 7, p)
    rows, first = [], 0
    for i, (nq, nt) in enumerate(sizes):
        rows.append((first, nq, i, nt, first))
        first += nq
    want = [oracle.knn(Q[a:a + nq], T[t:t + nt], k=2, ratio=0.8) for a, nq, t, nt, _ in rows]
    dq, dt, table = dev(torch_cuda, Q), dev(torch_cuda, T), pair_table(rows)
    small = Latch(triplets)
    try:
        # The pairs' state (16 bytes each), the header and the unit map alone.
        up = lambda n: (n + 255) // 256 * 256
        small.reserve(up(16 * len(rows)) + 256 + up(4 * (len(Q) // 256 + len(rows) + 1)))
        for L in (lat, small):
            L.set_tuning(Tuning.from_dict(dict(L.get_tuning().to_dict(), fp4_query_blocks=blocks)))
            for k in (1, 2, 2):
                if L is lat:
                    got = L.knn_batch(dq, dt, table, len(Q), k=k, ratio=0.8, path="fp4")
                else:
                    new = lambda *s, t=torch_cuda.int32: torch_cuda.zeros(s, dtype=t, device="cuda")
                    got = new(len(Q), k), new(len(Q), k), new(len(Q), t=torch_cuda.uint8)
                    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
                    assert load_library().hamming_knn_batch(
                        L.h, ptr(dq), len(Q), ptr(dt), len(T), ptr(table), len(rows), k, 0.8,
                        ptr(got[0]), ptr(got[1]), ptr(got[2]), len(Q), 3,
                        ctypes.c_void_p(torch_cuda.cuda.current_stream().cuda_stream)) == 0
                got = [a.cpu().numpy() for a in got]
                for (a, nq, _, _, _), (wi, wd, wa) in zip(rows, want):
                    assert np.array_equal(got[0][a:a + nq], wi[:, :k])
                    assert np.array_equal(got[1][a:a + nq], wd[:, :k])
                    assert np.array_equal(got[2][a:a + nq], wa)
    finally:
        lat.set_tuning(Tuning.from_dict(dict(lat.get_tuning().to_dict(), fp4_query_blocks=3)))
        small.close()


def test_more_divided_groups_than_slots(torch_cuda, lat):
    """Pairs enough for twice the slots of divided query groups: some are divided, the others not."""
    from paper_1609_03986_amd.binding import pair_table
    g = np.random.default_rng(77)
    n, nq, nt = 40, 40_000, 3200
    D = dev(torch_cuda, synth.random_descriptors(g, n * nq // 16))
    D = torch_cuda.cat([D ^ i for i in range(16)])
    rows = [(i * nq, nq, i * nq, nt, i * nq) for i in range(n)]
    idx, dist, acc = lat.knn_batch(D, D, pair_table(rows), n * nq, path="fp4")
    for i in range(n):
        part = slice(i * nq, (i + 1) * nq)
        want = lat.knn(D[part], D[i * nq:i * nq + nt], path="mfma")
        for got, w in zip((idx[part], dist[part], acc[part]), want):
            assert bool((got == w).all()), i


def test_batch_leaves_a_sufficient_workspace_alone(torch_cuda, triplets):
    """On a handle whose workspace holds what the call needs, a batch with a divided pair keeps that
    workspace, so that a graph captured over it stays valid; and a call on a stream that is capturing
    and is not the current one is captured like any other."""
    from paper_1609_03986_amd.binding import Latch, pair_table
    torch = torch_cuda
    g = np.random.default_rng(11)
    Q, T = synth.random_descriptors(g, 700, 0.3), synth.random_descriptors(g, 9000, 0.3)
    q, t = dev(torch, Q), dev(torch, T)
    rows = [(0, 600, 0, 9000, 0), (600, 100, 40, 33, 600)]
    table = pair_table(rows)
    want = [np.concatenate(x) for x in zip(*(oracle.knn(Q[a:a + n], T[f:f + m]) for a, n, f, m, _ in rows))]
    outputs = lambda: (torch.zeros((700, 2), dtype=torch.int32, device="cuda"),
                       torch.zeros((700, 2), dtype=torch.int32, device="cuda"),
                       torch.zeros((700,), dtype=torch.uint8, device="cuda"))
    lat = Latch(triplets)
    try:
        single = lat.knn_workspace_size(8, 9000, "fp4")
        held = lat.reserve(max(single, lat.knn_batch_workspace_size(len(rows), 700)))
        # Less than the batch's three query groups and the rest would take with room for dividing.
        assert 0 < single <= held < 3 * 6144 + 2048
        one = oracle.knn(Q[:8], T)
        out = [x[:8] for x in outputs()]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            lat.knn(q[:8], t, path="fp4", idx=out[0], dist=out[1], accept=out[2])
        batch_out, side = outputs(), torch.cuda.Stream()
        batch_graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(batch_graph, stream=stream):
            with torch.cuda.stream(side):
                lat.knn_batch(q, t, table, 700, path="fp4", idx=batch_out[0], dist=batch_out[1],
                              accept=batch_out[2], stream=stream)
        for rep in range(3):
            for path in ("fp4", "mfma", "popcount"):
                got = lat.knn_batch(q, t, table, 700, path=path)
                assert lat.reserve(0) == held
                for x, w in zip(got, want):
                    assert np.array_equal(x.cpu().numpy(), w), path
            for replay, to, ref in ((graph, out, one), (batch_graph, batch_out, want)):
                for x in to:
                    x.fill_(7)
                replay.replay()
                torch.cuda.synchronize()
                for x, w in zip(to, ref):
                    assert np.array_equal(x.cpu().numpy(), w), rep
        del graph, batch_graph
    finally:
        torch.cuda.synchronize()
        lat.close()


@pytest.mark.parametrize("p", [0.5, 0.02])
def test_pairs_refused_a_division(torch_cuda, lat, p):
    """31 pairs of 78 query groups with train tiles falling by a quarter octave from 16,384: every
    pair's train range is to be divided (the host test of the rule holds the same sizes), and their
    2,418 groups want more than the 2,048 slots, so that some pairs stay undivided."""
    from paper_1609_03986_amd.binding import pair_table
    g = np.random.default_rng(31)
    groups, n = 78, 31
    nq = groups * 384
    tiles = [int(np.floor(16384 * 2 ** (-i / 4) + 0.5)) for i in range(n)]
    D = dev(torch_cuda, synth.random_descriptors(g, 32 * tiles[0] // 8, p))
    D = torch_cuda.cat([D ^ i for i in range(8)])
    Q = dev(torch_cuda, synth.random_descriptors(g, nq, p))
    rows = [(0, nq, 5 * i, 32 * t, i * nq) for i, t in enumerate(tiles)]
    idx, dist, acc = lat.knn_batch(Q, D, pair_table(rows), n * nq, path="fp4")
    for i, (_, _, first, nt, out) in enumerate(rows):
        want = lat.knn(Q, D[first:first + nt], path="mfma")
        for got, w in zip((idx, dist, acc), want):
            assert bool((got[out:out + nq] == w).all()), i
