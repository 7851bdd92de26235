"""Descriptor and result arrays that are aligned as their 32-bit elements and no better: the kernels
move them 8 and 16 bytes at a time, and give what they give for aligned arrays."""
import ctypes

import numpy as np
import pytest

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
    yield L
    L.close()


def shifted(torch, t):
    """A contiguous copy of t one element past a 16-byte boundary."""
    flat = torch.empty((t.numel() + 4,), dtype=t.dtype, device="cuda")
    out = flat[1:1 + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.is_contiguous() and out.data_ptr() % 16 == t.element_size()
    return out


def same(a, b):
    return all(bool((x == y).all()) for x, y in zip(a, b))


def words(torch, seed, n):
    return torch.from_numpy(synth.random_descriptors(np.random.default_rng(seed), n, 0.3).view(np.int32)).cuda()


@pytest.mark.parametrize("path", ["fp4", "mfma", "popcount"])
@pytest.mark.parametrize("nq,nt", [(130, 200), (1000, 9001)])
def test_matching(torch_cuda, lat, nq, nt, path):
    from paper_1609_03986_amd.binding import pair_table
    torch = torch_cuda
    q, t = words(torch, 1, nq), words(torch, 2, nt)
    new = lambda *s: shifted(torch, torch.zeros(s, dtype=torch.int32, device="cuda"))
    want = lat.knn(q, t, path=path)
    assert same(want, lat.knn(shifted(torch, q), shifted(torch, t), path=path, idx=new(nq, 2), dist=new(nq, 2)))
    pairs = pair_table([(0, nq, 0, nt, 0)])
    assert same(want, lat.knn_batch(shifted(torch, q), shifted(torch, t), pairs, nq, path=path,
                                    idx=new(nq, 2), dist=new(nq, 2)))


@pytest.mark.parametrize("radius", [1, 2, 4, 8])
@pytest.mark.parametrize("k", [1, 2])
def test_window_matching(torch_cuda, lat, radius, k):
    from paper_1609_03986_amd import binding
    torch = torch_cuda
    gw, gh = 45, 37
    n = gw * gh
    q, t = words(torch, 3, n), words(torch, 4, n)
    want = lat.knn_window(q, t, gw, gh, radius, k=k)
    new = lambda: shifted(torch, torch.zeros((n, k), dtype=torch.int32, device="cuda"))
    qs, ts, idx, dist = shifted(torch, q), shifted(torch, t), new(), new()
    acc = torch.zeros((n,), dtype=torch.uint8, device="cuda")
    ptr = lambda x: ctypes.c_void_p(x.data_ptr())
    assert binding.load_library().hamming_knn_window(
        lat.h, ptr(qs), ptr(ts), gw, gh, radius, k, 0.8, ptr(idx), ptr(dist), ptr(acc),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert same(want, (idx, dist, acc))


def test_dense_extraction(torch_cuda, lat):
    torch = torch_cuda
    img = torch.from_numpy(synth.smoothed_noise(np.random.default_rng(5), 90, 150)).cuda()
    want = lat.extract_dense(img, 3, -5, 140, 70)
    out = shifted(torch, torch.zeros_like(want))
    assert bool((lat.extract_dense(img, 3, -5, 140, 70, desc=out) == want).all())
