"""The binding's calls without a GPU: the library is replaced by a record of what was called."""
import pytest

from paper_1609_03986_amd import binding


class Library:
    """hamming_knn_batch answers from `results`; every call is recorded."""

    def __init__(self, results):
        self.results, self.calls = list(results), []

    def hamming_knn_batch(self, *args):
        self.calls.append("hamming_knn_batch")
        return self.results.pop(0)

    def hamming_knn_batch_workspace_size(self, h, n_pairs, out_rows, out):
        self.calls.append("size")
        out._obj.value = 4096
        return binding.LATCH_OK

    def latch_reserve(self, h, nbytes, held):
        self.calls.append("reserve %d" % nbytes)
        held._obj.value = nbytes
        return binding.LATCH_OK


@pytest.mark.parametrize("path", ["fp4", "mfma", "popcount", "auto"])
@pytest.mark.parametrize("results,calls", [
    ([binding.LATCH_OK], ["hamming_knn_batch"]),
    ([binding.LATCH_EWORKSPACE, binding.LATCH_OK],
     ["hamming_knn_batch", "size", "reserve 4096", "hamming_knn_batch"])])
def test_batch_reserves_only_when_the_call_needs_it(monkeypatch, results, calls, path):
    """A workspace that the call accepts is left alone (a reservation may wait for the device and
    free what captured graphs use), whatever the state of any stream."""
    import torch
    lib = Library(results)
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(binding, "_dev", lambda t, dtype, name: 0)
    monkeypatch.setattr(binding, "_stream_ptr", lambda stream: 0)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    d, pairs = torch.zeros((4, 16), dtype=torch.int32), torch.zeros((1, 5), dtype=torch.int64)
    binding.hamming_knn_batch(None, d, d, pairs, 4, path=path)
    assert lib.calls == calls
