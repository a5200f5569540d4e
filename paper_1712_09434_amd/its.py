"""Binding of the ITS standalone tracker (tpcca_its_* in include/tpcca.h).

Argument marshalling only: every step (vertexer, tracklets, following,
inward fit, vertex fit) runs in the library's kernels.
"""
from __future__ import annotations

import ctypes as C
from dataclasses import dataclass
from typing import Optional

import numpy as np
import torch

from . import _abi as A
from .tracker import _ptr, _stream_handle, pieces, struct_dtype, struct_ptr, used_pieces

# per-tracklet arrays: type and values per tracklet
_FIELDS = {k: (torch.float32 if k in ("chi2", "out_x", "out_p", "out_cov", "in_p", "in_cov") else torch.int32,
               {"cls": (6,), "out_p": (5,), "out_cov": (15,), "in_p": (5,), "in_cov": (15,)}.get(k, ()))
           for k in A.ITS_TRACK_ARRAYS}
_CLUSTERS_DT = struct_dtype(A.tpcca_its_clusters)
_TRACKS_DT = struct_dtype(A.tpcca_its_tracks)
# The tracklets are at most the layer-0 clusters, but counting those waits for
# the device: calls of up to this many clusters hold an entry per cluster (224
# bytes, about six times what they need) instead (one small event 313 us with
# the wait, 283 without).  Beyond, where the wait no longer shows, the
# layer-0 clusters are counted, so that the surplus stays below 200 MB a call.
_COUNT_ABOVE = 1 << 20


def _check(L, ctx, rc):
    if rc != A.TPCCA_OK:
        msg = L.tpcca_its_last_error(ctx).decode() if ctx else ""
        raise A.TpccaError(rc, msg)


@dataclass
class ItsResult:
    """One event: per-tracklet tensors (device, sliced to the count) and the
    vertexer / vertex-fit scalars."""
    tl0: torch.Tensor
    tl1: torch.Tensor
    ok: torch.Tensor
    cls: torch.Tensor          # [T, 6]
    ncls: torch.Tensor
    chi2: torch.Tensor
    out_layer: torch.Tensor
    out_stave: torch.Tensor
    out_x: torch.Tensor
    out_p: torch.Tensor        # [T, 5]
    out_cov: torch.Tensor      # [T, 15]
    in_ok: torch.Tensor
    in_stave: torch.Tensor
    in_p: torch.Tensor         # [T, 5]
    in_cov: torch.Tensor       # [T, 15]
    hist: Optional[torch.Tensor]
    n_pairs: int
    peak: int
    vz_ok: bool
    vz: float
    vfit_ok: bool
    vfit_n: int
    vertex: tuple
    vfit_sumw: float


class ItsTracker:
    def __init__(self, geom, params: Optional[A.tpcca_its_params] = None):
        self.L = A.load()
        g = A.tpcca_its_geometry()
        g.n_layers = int(geom.n_layers)
        for i in range(g.n_layers):
            g.radius[i] = float(geom.radius[i]); g.half_z[i] = float(geom.half_z[i])
            g.x_over_x0[i] = float(geom.x_over_x0[i]); g.sigma_y[i] = float(geom.sigma_y[i])
            g.sigma_z[i] = float(geom.sigma_z[i]); g.n_staves[i] = int(geom.n_staves[i])
        g.bz = float(geom.bz)
        ctx = C.c_void_p()
        rc = self.L.tpcca_its_create(C.byref(g), C.byref(ctx))
        if rc != A.TPCCA_OK:
            raise A.TpccaError(rc, "tpcca_its_create")
        self.ctx = ctx
        self.nbins = 400
        if params is not None:
            self.set_params(params)

    @staticmethod
    def default_params() -> A.tpcca_its_params:
        p = A.tpcca_its_params()
        A.load().tpcca_its_default_params(C.byref(p))
        return p

    def set_params(self, p: A.tpcca_its_params):
        _check(self.L, self.ctx, self.L.tpcca_its_set_params(self.ctx, C.byref(p)))
        self.nbins = int(round(2.0 * p.vtx_range / p.vtx_bin))

    def _event(self, x, y, z, layer, stave, hist):
        """Marshals one event: the cluster struct, the output struct and the
        tensors behind both (kept alive by the caller until the call ends)."""
        dev = x.device
        cl = A.tpcca_its_clusters()
        cl.n = int(x.shape[0])
        keep = [t.contiguous() for t in (x, y, z, layer, stave)]
        cl.x, cl.y, cl.z, cl.layer, cl.stave = (_ptr(t) for t in keep)
        cl.stream = _stream_handle(dev)
        cap = max(cl.n if cl.n <= _COUNT_ABOVE else int((layer == 0).sum()), 1)
        o = {k: torch.empty((cap, *shape), dtype=dtype, device=dev) for k, (dtype, shape) in _FIELDS.items()}
        h = torch.empty(self.nbins, dtype=torch.int32, device=dev) if hist else None
        st = A.tpcca_its_tracks()
        st.cap = cap
        for k in A.ITS_TRACK_ARRAYS:
            setattr(st, k, _ptr(o[k]))
        st.hist = _ptr(h)
        return cl, st, o, h, keep

    @staticmethod
    def _result(st, o, h) -> ItsResult:
        T = int(st.n_tracklets)
        sl = {k: v[:T] for k, v in o.items()}
        return ItsResult(**sl, hist=h, n_pairs=int(st.n_pairs), peak=int(st.peak), vz_ok=bool(st.vz_ok),
                         vz=float(st.vz), vfit_ok=bool(st.vfit_ok), vfit_n=int(st.vfit_n),
                         vertex=tuple(st.vertex), vfit_sumw=float(st.vfit_sumw))

    def track(self, x, y, z, layer, stave, hist: bool = False) -> ItsResult:
        """One event (device tensors).  The result's tensors are the used parts
        of arrays of one entry per cluster (per layer-0 cluster in events of
        more than 2^20 clusters); clone them to keep them without the rest."""
        cl, st, o, h, keep = self._event(x, y, z, layer, stave, hist)
        _check(self.L, self.ctx, self.L.tpcca_its_track(self.ctx, C.byref(cl), C.byref(st)))
        return self._result(st, o, h)

    def prepare_batch(self, events, hist: bool = False):
        """Marshals a batch once (output tensors, structs) and returns
        run(results=True): one tpcca_its_track_batch call on it, for repeated
        calls on the same inputs.  The result tensors of the events are slices
        of one array per field (clone those of an event to keep it without the
        others), overwritten by the next run."""
        events = list(events)
        E = len(events)
        if E == 0:
            return lambda results=True: []
        dev = events[0][0].device
        if any(e[0].device != dev for e in events):
            return self._prepare_apart(events, hist)
        stream = _stream_handle(dev)
        stream = (stream.value or 0) if stream is not None else 0
        keep = [[t.contiguous() for t in e] for e in events]
        cls = np.array([(e[0].shape[0], *(t.data_ptr() for t in e), stream) for e in keep], dtype=_CLUSTERS_DT)
        cap = cls["n"]
        if int(cap.sum()) > _COUNT_ABOVE:
            cap = torch.stack([(e[3] == 0).sum() for e in keep]).cpu().numpy()
        cap = np.maximum(cap, 1)
        size, at = pieces(cap)
        total = int(size.sum())
        o = {k: torch.empty((total, *shape), dtype=dtype, device=dev) for k, (dtype, shape) in _FIELDS.items()}
        h = torch.empty(E, self.nbins, dtype=torch.int32, device=dev) if hist else None
        sts = np.zeros(E, _TRACKS_DT)
        sts["cap"] = cap
        for k, v in o.items():
            sts[k] = v.data_ptr() + v[0].numel() * 4 * at
        if hist:
            sts["hist"] = h.data_ptr() + 4 * self.nbins * np.arange(E)

        def run(results: bool = True):
            _check(self.L, self.ctx, self.L.tpcca_its_track_batch(self.ctx, len(keep),
                                                                  struct_ptr(cls, A.tpcca_its_clusters),
                                                                  struct_ptr(sts, A.tpcca_its_tracks)))
            if not results:
                return None
            n = sts["n_tracklets"]
            cut = zip(*(used_pieces(v, n, size) for v in o.values()))
            hs = h.unbind(0) if hist else [None] * E
            col = [sts[k].tolist() for k in ("n_pairs", "peak", "vz_ok", "vz", "vfit_ok", "vfit_n", "vertex",
                                             "vfit_sumw")]
            return [ItsResult(**dict(zip(o, f)), hist=hh, n_pairs=a, peak=b, vz_ok=bool(c), vz=d, vfit_ok=bool(e),
                              vfit_n=g, vertex=tuple(v), vfit_sumw=w)
                    for f, hh, a, b, c, d, e, g, v, w in zip(cut, hs, *col)]
        return run

    def _prepare_apart(self, events, hist: bool):
        """prepare_batch with each event's outputs in tensors of its own
        (events on several devices)."""
        ev = [self._event(*e, hist) for e in events]
        n = len(ev)
        cls = (A.tpcca_its_clusters * n)(*[e[0] for e in ev])
        sts = (A.tpcca_its_tracks * n)(*[e[1] for e in ev])

        def run(results: bool = True):
            _check(self.L, self.ctx, self.L.tpcca_its_track_batch(self.ctx, n, cls, sts))
            return [self._result(sts[i], e[2], e[3]) for i, e in enumerate(ev)] if results else None
        return run

    def track_batch(self, events, hist: bool = False) -> list:
        """events: sequence of (x, y, z, layer, stave) device tensors, one
        tuple per event, all on one device and stream; one library call.  The
        results as of prepare_batch."""
        return self.prepare_batch(events, hist)()

    def close(self):
        if self.ctx:
            self.L.tpcca_its_destroy(self.ctx)
            self.ctx = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass
