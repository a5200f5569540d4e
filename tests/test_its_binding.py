"""Marshalling of the ITS binding, on the CPU: the library call is replaced by
one that records the structures and reports tracklet counts."""
import ctypes as C

import pytest
import torch

from paper_1712_09434_amd import _abi as A
from paper_1712_09434_amd import its


class Library:
    """Stands for the loaded library: every event gets `counts` tracklets whose
    tl0 entries are 100 e + k (on the CPU; other devices are not written)."""

    def __init__(self, counts):
        self.counts, self.calls = counts, []

    def tpcca_its_track_batch(self, ctx, n, cls, sts):
        self.calls.append([(cls[e].n, sts[e].cap) for e in range(n)])
        for e in range(n):
            sts[e].n_tracklets = self.counts[e]
            assert sts[e].n_tracklets <= sts[e].cap
            if sts[e].tl0:
                p = C.cast(sts[e].tl0, C.POINTER(C.c_int32))
                for k in range(self.counts[e]):
                    p[k] = 100 * e + k
        return A.TPCCA_OK

    def tpcca_its_track(self, ctx, cl, st):
        return self.tpcca_its_track_batch(ctx, 1, C.cast(cl, C.POINTER(A.tpcca_its_clusters)),
                                          C.cast(st, C.POINTER(A.tpcca_its_tracks)))


def tracker(counts):
    t = its.ItsTracker.__new__(its.ItsTracker)
    t.L, t.ctx, t.nbins = Library(counts), None, 400
    return t


def event(n, device="cpu"):
    """n clusters, every sixth of them on layer 0."""
    f = torch.zeros(n, device=device)
    return f, f, f, (torch.arange(n) % 6).to(torch.int8).to(device), torch.zeros(n, dtype=torch.int16, device=device)


@pytest.mark.parametrize("devices", [["cpu"] * 3, ["cpu", "meta", "cpu"]])
@pytest.mark.parametrize("form", [list, tuple, iter])
def test_batches_of_any_iterable(devices, form):
    """Sequences and iterators of events, on one device (one array per field)
    and on several (arrays of each event's own)."""
    t = tracker([2, 0, 3])
    out = t.track_batch(form([event(n, d) for n, d in zip((12, 1, 30), devices)]), hist=True)
    assert t.L.calls == [[(12, 12), (1, 1), (30, 30)]]
    assert [r.tl0.shape[0] for r in out] == [2, 0, 3]
    assert [r.tl0.device.type for r in out] == devices and all(r.hist.numel() == 400 for r in out)
    assert out[0].tl0.tolist() == [0, 1] and out[2].tl0.tolist() == [200, 201, 202]
    assert out[2].in_cov.shape == (3, 15) and out[2].in_cov.is_contiguous()
    shared = out[0].tl0.untyped_storage().data_ptr() == out[2].tl0.untyped_storage().data_ptr()
    assert shared == (devices[1] == "cpu")


def test_empty_batch():
    t = tracker([])
    assert t.track_batch([]) == [] and t.track_batch(iter([])) == [] and t.L.calls == []


def test_large_calls_count_their_layer_0_clusters(monkeypatch):
    """Up to the limit a call holds an entry per cluster, beyond it one per
    layer-0 cluster."""
    monkeypatch.setattr(its, "_COUNT_ABOVE", 60)
    t = tracker([3, 4])
    t.track(*event(60))
    t.track(*event(61))
    t.track_batch([event(30), event(30)])
    out = t.track_batch([event(30), event(31)])
    assert t.L.calls == [[(60, 60)], [(61, 11)], [(30, 30), (30, 30)], [(30, 5), (31, 6)]]
    assert out[1].tl0.tolist() == [100, 101, 102, 103]
    assert out[0].in_cov.untyped_storage().nbytes() == 2 * 16 * 15 * 4
