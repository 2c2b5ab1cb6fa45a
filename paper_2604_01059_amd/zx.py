"""ctypes binding of libzx (include/zx.h): argument marshalling only.

Device buffers are torch tensors on a ROCm device (their data_ptr() is passed
through); host arrays are numpy.  Every computation happens in the HIP
library; if libzx.so is missing this module raises instead of falling back.
"""
from __future__ import annotations

import ctypes as C
import os

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libzx.so")

ZX_OK, ZX_EINVAL, ZX_ENOMATCH, ZX_ECAPACITY, ZX_EDEVICE, ZX_EBUSY = 0, -1, -2, -3, -4, -5
ZX_GRAPH_ONLY = 0x1
ZX_RESUME = 0x2
ZX_FALLBACK = 0x4
ZX_SYNC = 0x100
ZX_POLICY_GREEDY, ZX_POLICY_LEARNED = 0, 1
ZX_GATE_H, ZX_GATE_RZ, ZX_GATE_CZ, ZX_GATE_CNOT = 0, 1, 2, 3
MLP_IN, MLP_HID = 16, 256
MLP_NPARAM = MLP_IN * MLP_HID + 2 * MLP_HID + 1
MLP_NBF16 = MLP_IN * MLP_HID + MLP_HID
STATUS_NAMES = {0: "ZX_OK", -1: "ZX_EINVAL", -2: "ZX_ENOMATCH", -3: "ZX_ECAPACITY",
                -4: "ZX_EDEVICE", -5: "ZX_EBUSY"}


class ZxError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__("%s: %s" % (STATUS_NAMES.get(code, code), msg))
        self.code = code


class GraphInfo(C.Structure):
    _fields_ = [("pow_sqrt2", C.c_int64), ("phase8", C.c_int32), ("status", C.c_int32),
                ("n", C.c_int32), ("n_alive", C.c_int32), ("n_edges", C.c_int64),
                ("n_trace", C.c_int32), ("rounds", C.c_int32), ("fill_in", C.c_int64),
                ("rank", C.c_int32), ("policy", C.c_int32), ("rowops", C.c_int64)]


class MlpHandle(C.Structure):
    _fields_ = [("param", C.c_void_p), ("wbf16", C.c_void_p)]


class SimplifyOpts(C.Structure):
    _fields_ = [("policy", C.c_int32), ("extract", C.c_int32), ("tune_id", C.c_int32),
                ("flags", C.c_uint32), ("max_rounds", C.c_int32), ("pad", C.c_int32),
                ("mlp", C.POINTER(MlpHandle))]


class Request(C.Structure):
    _fields_ = [("n", C.c_int32), ("n_in", C.c_int32), ("n_out", C.c_int32), ("pad", C.c_int32),
                ("adj", C.c_void_p), ("phase", C.c_void_p), ("inputs", C.c_void_p), ("outputs", C.c_void_p),
                ("bnd_is_h", C.c_void_p), ("tag", C.c_int64)]


class Result(C.Structure):
    _fields_ = [("ticket", C.c_int64), ("tag", C.c_int64), ("status", C.c_int32), ("n_alive", C.c_int32),
                ("rounds", C.c_int32), ("n_trace", C.c_int32), ("rank", C.c_int32), ("phase8", C.c_int32),
                ("n_edges", C.c_int64), ("rowops", C.c_int64), ("pow_sqrt2", C.c_int64), ("fill_in", C.c_int64),
                ("policy", C.c_int32), ("pad", C.c_int32),
                ("t_submit", C.c_double), ("t_launch", C.c_double), ("t_done", C.c_double),
                ("t_device", C.c_double), ("t_claim_dev", C.c_double), ("t_end_dev", C.c_double)]


class ServerStats(C.Structure):
    _fields_ = [("submitted", C.c_int64), ("refused", C.c_int64), ("completed", C.c_int64),
                ("batches", C.c_int64), ("pending", C.c_int64), ("running", C.c_int64),
                ("pool_bytes", C.c_size_t), ("pool_used", C.c_size_t), ("pool_peak", C.c_size_t)]


ZX_SERVE_TRUSTED = 0x1

_lib = None


def load():
    """Load libzx.so (built by ``python -m paper_2604_01059_amd.build``)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError("libzx.so is not built (%s); run __graft_entry__.build()" % LIB_PATH)
    lib = C.CDLL(LIB_PATH)
    P, i32, i64, u32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_uint32, C.c_size_t
    sigs = {
        "zx_version": ([], i32),
        "zx_last_error": ([], C.c_char_p),
        "zx_device_info": ([C.c_char_p, i32, C.POINTER(i32)], i32),
        "zx_graph_bytes": ([i32, i32, i32], sz),
        "zx_graph_create": ([C.POINTER(P), P, sz, i32, P, P, P, i32, P, i32, P, P], i32),
        "zx_graph_attach": ([C.POINTER(P), P, sz], i32),
        "zx_graph_bytes_ex": ([i32, i32, i32, i32], sz),
        "zx_graph_create_ex": ([C.POINTER(P), P, sz, i32, P, P, P, i32, P, i32, P, i32, P, P], i32),
        "zx_graph_read_params": ([P, P, C.POINTER(i32), P, P, P, i32, P], i32),
        "zx_gf2_basis": ([P, i32, i32, i64, P, P, P, P, i64, P, sz, P], i32),
        "zx_graph_destroy": ([P], None),
        "zx_graph_arena": ([P], P),
        "zx_graph_read": ([P, P, P, P, C.POINTER(GraphInfo), P], i32),
        "zx_graph_read_trace": ([P, P, i32, C.POINTER(i32), P], i32),
        "zx_graph_read_frontier": ([P, P, P, P], i32),
        "zx_graph_status": ([P, P], i32),
        "zx_graph_reset": ([P, P], i32),
        "zx_local_comp": ([P, i32, u32, P], i32),
        "zx_pivot": ([P, i32, i32, u32, P], i32),
        "zx_simplify_variants": ([], i32),
        "zx_simplify_variant_name": ([i32], C.c_char_p),
        "zx_simplify_workspace_bytes": ([i32], sz),
        "zx_simplify": ([P, i32, C.POINTER(SimplifyOpts), P, sz, P], i32),
        "zx_batch_prepare": ([C.POINTER(P), P, i32, P, sz, P], i32),
        "zx_batch_simplify": ([P, C.POINTER(SimplifyOpts), P], i32),
        "zx_batch_status": ([P, P], i32),
        "zx_batch_autotune": ([P, i32, i32, C.POINTER(i32), C.POINTER(C.c_float), P], i32),
        "zx_batch_destroy": ([P], None),
        "zx_gf2_workspace_bytes": ([i32, i32], sz),
        "zx_gf2_eliminate": ([P, P, i32, i32, i64, P, P, P, i64, P, sz, P], i32),
        "zx_gf2_eliminate_noalloc": ([P, P, i32, i32, i64, P, P, P, i64, P], i32),
        "zx_gf2_status": ([P, P], i32),
        "zx_gf2_profile_read": ([P, i32, P, i32, P], i32),
        "zx_pauli_commute": ([P, P, i64, i32, i64, P, i64, u32, P], i32),
        "zx_gf2_matmul": ([P, i64, i64, P, i64, i64, i32, P, i64, u32, P], i32),
        "zx_phase_pair_product": ([P, P, i64, i32, i64, P, P, i32, i64, P, P, P], i32),
        "zx_detector_workspace_bytes": ([i32], sz),
        "zx_detector_sample": ([P, P, i64, P, i32, i32, C.c_uint64, i64, i64, P, i64, P, sz, P], i32),
        "zx_detector_status": ([P, P], i32),
        "zx_gflow_workspace_bytes": ([i32], sz),
        "zx_gflow": ([P, i32, P, P, P, sz, P], i32),
        "zx_extract_workspace_bytes": ([i32], sz),
        "zx_extract": ([P, i32, i32, P, P, P, P, P, sz, P], i32),
        "zx_mlp_sync": ([C.POINTER(MlpHandle), P], i32),
        "zx_mlp_forward": ([C.POINTER(MlpHandle), P, i64, P, P], i32),
        "zx_mlp_loss": ([P, P, P, i32, P, P, P], i32),
        "zx_mlp_workspace_bytes": ([i64], sz),
        "zx_mlp_backward": ([C.POINTER(MlpHandle), P, P, i64, P, P, sz, P], i32),
        "zx_mlp_adam": ([C.POINTER(MlpHandle), P, P, P, C.c_float, C.c_float, C.c_float, C.c_float, i32, P],
                        i32),
        "zx_rollout_workspace_bytes": ([P, i32], sz),
        "zx_rollout": ([P, i32, i32, P, P, P, P, P, sz, P], i32),
        "zx_policy_features": ([P, P, P, i32, P, P], i32),
        "zx_server_create": ([C.POINTER(P), P, sz, i32, C.POINTER(SimplifyOpts), u32], i32),
        "zx_server_submit": ([P, C.POINTER(Request), C.POINTER(i64)], i32),
        "zx_server_poll": ([P, P, i32, C.POINTER(i32)], i32),
        "zx_server_stats_read": ([P, C.POINTER(ServerStats)], i32),
        "zx_server_destroy": ([P], None),
    }
    for name, (args, res) in sigs.items():
        f = getattr(lib, name)
        f.argtypes = args
        f.restype = res
    _lib = lib
    return lib


def exported_symbols():
    return ["zx_version", "zx_last_error", "zx_device_info", "zx_graph_bytes", "zx_graph_create",
            "zx_graph_attach", "zx_graph_bytes_ex", "zx_graph_create_ex", "zx_graph_read_params",
            "zx_gf2_basis", "zx_graph_destroy", "zx_graph_arena", "zx_graph_read",
            "zx_graph_read_trace", "zx_graph_read_frontier", "zx_graph_status", "zx_graph_reset",
            "zx_local_comp", "zx_pivot", "zx_simplify_variants", "zx_simplify_variant_name",
            "zx_simplify_workspace_bytes", "zx_simplify", "zx_batch_prepare", "zx_batch_simplify",
            "zx_batch_status", "zx_batch_autotune", "zx_batch_destroy", "zx_gf2_workspace_bytes",
            "zx_gf2_eliminate", "zx_gf2_eliminate_noalloc", "zx_gf2_status", "zx_gf2_profile_read", "zx_pauli_commute",
            "zx_gf2_matmul", "zx_phase_pair_product", "zx_detector_workspace_bytes",
            "zx_detector_sample", "zx_detector_status", "zx_gflow_workspace_bytes", "zx_gflow",
            "zx_extract_workspace_bytes", "zx_extract", "zx_mlp_sync", "zx_mlp_forward", "zx_mlp_loss", "zx_mlp_workspace_bytes", "zx_mlp_backward",
            "zx_mlp_adam", "zx_rollout_workspace_bytes", "zx_rollout", "zx_policy_features", "zx_server_create",
            "zx_server_submit", "zx_server_poll", "zx_server_stats_read", "zx_server_destroy"]


def _check(rc):
    if rc < 0:
        raise ZxError(rc, load().zx_last_error().decode())
    return rc


def _stream(stream=None):
    import torch
    s = torch.cuda.current_stream() if stream is None else stream
    return C.c_void_p(s.cuda_stream)


def _ptr(t):
    return C.c_void_p(t.data_ptr()) if t is not None else None


def _np(a):
    return a.ctypes.data_as(C.c_void_p) if a is not None else None


def version():
    return load().zx_version()


def device_info():
    buf = C.create_string_buffer(128)
    cu = C.c_int32(0)
    _check(load().zx_device_info(buf, 128, C.byref(cu)))
    return buf.value.decode(), cu.value


# ---------------------------------------------------------------- graphs --

class Graph:
    """Host handle of a diagram arena (torch uint8 device tensor)."""

    def __init__(self, handle, arena, n, n_in, n_out, n_params=0):
        self.h = handle
        self.arena = arena
        self.n, self.n_in, self.n_out = n, n_in, n_out
        self.W = (n + 63) // 64
        self.n_params = int(n_params)
        self.pw = (self.n_params + 63) // 64

    def __del__(self):
        if getattr(self, "h", None) and _lib is not None:
            _lib.zx_graph_destroy(self.h)
            self.h = None

    @staticmethod
    def bytes_for(n, n_in, n_out):
        return load().zx_graph_bytes(n, n_in, n_out)

    @staticmethod
    def bytes_for_params(n, n_in, n_out, n_params):
        return load().zx_graph_bytes_ex(n, n_in, n_out, n_params)

    @classmethod
    def create(cls, adj, phase, inputs, outputs, bnd_is_h=None, arena=None, stream=None, n_params=0,
               params=None):
        """params: n x ceil(n_params/64) uint64 parameter rows (with n_params > 0)."""
        import torch
        adj = np.ascontiguousarray(adj, dtype=np.uint64)
        phase = np.ascontiguousarray(phase, dtype=np.int8)
        inputs = np.ascontiguousarray(inputs, dtype=np.int32)
        outputs = np.ascontiguousarray(outputs, dtype=np.int32)
        n = int(adj.shape[0])
        nb = cls.bytes_for_params(n, len(inputs), len(outputs), n_params)
        if arena is None:
            arena = torch.empty(nb, dtype=torch.uint8, device="cuda")
        bh = None if bnd_is_h is None else np.ascontiguousarray(bnd_is_h, dtype=np.uint8)
        prm = None if not n_params else np.ascontiguousarray(params, dtype=np.uint64)
        h = C.c_void_p()
        _check(load().zx_graph_create_ex(C.byref(h), _ptr(arena), arena.numel(), n, _np(adj), _np(phase),
                                         _np(inputs), len(inputs), _np(outputs), len(outputs), _np(bh),
                                         int(n_params), _np(prm), _stream(stream)))
        return cls(h, arena, n, len(inputs), len(outputs), n_params)

    def params(self, stream=None):
        """(rows (n x pw), k_ab (m x 2), u (m x pw), v (m x pw)): CURRENT
        parameter rows and the recorded phase-pair terms."""
        pw = max(self.pw, 1)
        rows = np.zeros((self.n, pw), np.uint64)
        cap = self.n + 1
        kab = np.zeros((cap, 2), np.int32)
        u = np.zeros((cap, pw), np.uint64)
        v = np.zeros((cap, pw), np.uint64)
        nt = C.c_int32(0)
        _check(load().zx_graph_read_params(self.h, _np(rows), C.byref(nt), _np(kab), _np(u), _np(v), cap,
                                           _stream(stream)))
        m = nt.value
        return rows[:, : self.pw], kab[:m].copy(), u[:m, : self.pw].copy(), v[:m, : self.pw].copy()

    @classmethod
    def from_diagram(cls, d, arena=None, stream=None):
        return cls.create(d.adj, d.phase, d.inputs, d.outputs, d.bnd_is_h, arena=arena, stream=stream)

    @classmethod
    def attach(cls, arena):
        """Handle for an arena that already holds a diagram (synchronous)."""
        h = C.c_void_p()
        _check(load().zx_graph_attach(C.byref(h), _ptr(arena), arena.numel()))
        import torch
        hdr = arena[:192].cpu().numpy().view(np.int32)
        return cls(h, arena, int(hdr[1]), int(hdr[2]), int(hdr[3]), int(hdr[46]))

    def snapshot(self):
        """Independent copy of the arena (SOURCE, CURRENT, trace, header)."""
        return Graph.attach(self.arena.clone())

    def read(self, stream=None):
        adj = np.zeros((self.n, self.W), np.uint64)
        ph = np.zeros(self.n, np.int8)
        al = np.zeros(self.W, np.uint64)
        info = GraphInfo()
        _check(load().zx_graph_read(self.h, _np(adj), _np(ph), _np(al), C.byref(info), _stream(stream)))
        return adj, ph, al, info

    def info(self, stream=None):
        info = GraphInfo()
        _check(load().zx_graph_read(self.h, None, None, None, C.byref(info), _stream(stream)))
        return info

    def trace(self, stream=None):
        cap = self.n + 1
        tr = np.zeros((cap, 4), np.int32)
        nt = C.c_int32(0)
        _check(load().zx_graph_read_trace(self.h, _np(tr), cap, C.byref(nt), _stream(stream)))
        return tr[: nt.value].copy()

    def frontier(self, stream=None):
        rows = np.zeros((self.n_out, self.W), np.uint64)
        piv = np.zeros(max(self.n_out, 1), np.int32)
        _check(load().zx_graph_read_frontier(self.h, _np(rows), _np(piv), _stream(stream)))
        return rows, piv[: self.n_out].copy()

    def status(self, stream=None):
        return load().zx_graph_status(self.h, _stream(stream))

    def reset(self, stream=None):
        _check(load().zx_graph_reset(self.h, _stream(stream)))

    def local_comp(self, u, graph_only=False, stream=None):
        _check(load().zx_local_comp(self.h, int(u), ZX_GRAPH_ONLY if graph_only else 0, _stream(stream)))

    def pivot(self, u, v, graph_only=False, stream=None):
        _check(load().zx_pivot(self.h, int(u), int(v), ZX_GRAPH_ONLY if graph_only else 0, _stream(stream)))


def simplify_workspace_bytes(n_graphs):
    return load().zx_simplify_workspace_bytes(n_graphs)


def _graph_array(graphs):
    arr = (C.c_void_p * len(graphs))(*[g.h.value if isinstance(g.h, C.c_void_p) else g.h for g in graphs])
    return arr


def _opts(extract, tune_id, policy, mlp, max_rounds, resume, fallback=False):
    flags = (ZX_RESUME if resume else 0) | (ZX_FALLBACK if fallback else 0)
    o = SimplifyOpts(policy, 1 if extract else 0, tune_id, flags, int(max_rounds), 0, None)
    if mlp is not None:
        o.mlp = C.pointer(mlp.handle)
    return o


def simplify(graphs, extract=True, tune_id=-1, ws=None, stream=None, policy=ZX_POLICY_GREEDY, mlp=None,
             max_rounds=0, resume=False, fallback=False):
    """fallback (learned policy): keep the greedy result where its gate2q is lower (ZX_FALLBACK)."""
    import torch
    n = len(graphs)
    nb = simplify_workspace_bytes(n)
    if ws is None:
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    opts = _opts(extract, tune_id, policy, mlp, max_rounds, resume, fallback)
    _check(load().zx_simplify(_graph_array(graphs), n, C.byref(opts), _ptr(ws), ws.numel(), _stream(stream)))
    return ws


class Batch:
    """A prepared batch: the launches of its plan per ``run`` (capturable)."""

    def __init__(self, graphs, stream=None):
        import torch
        self.graphs = list(graphs)
        n = len(self.graphs)
        self.ws = torch.empty(simplify_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        h = C.c_void_p()
        _check(load().zx_batch_prepare(C.byref(h), _graph_array(self.graphs), n, _ptr(self.ws),
                                       self.ws.numel(), _stream(stream)))
        self.h = h

    def run(self, extract=True, tune_id=-1, stream=None, policy=ZX_POLICY_GREEDY, mlp=None, max_rounds=0,
            resume=False, fallback=False):
        self._opts = _opts(extract, tune_id, policy, mlp, max_rounds, resume, fallback)
        _check(load().zx_batch_simplify(self.h, C.byref(self._opts), _stream(stream)))

    def status(self, stream=None):
        return load().zx_batch_status(self.h, _stream(stream))

    def autotune(self, extract=True, reps=3, stream=None):
        best = C.c_int32(-1)
        ms = C.c_float(0)
        _check(load().zx_batch_autotune(self.h, 1 if extract else 0, reps, C.byref(best), C.byref(ms),
                                        _stream(stream)))
        return best.value, ms.value

    def __del__(self):
        if getattr(self, "h", None) and _lib is not None:
            _lib.zx_batch_destroy(self.h)
            self.h = None


# ------------------------------------------------------- learned proposal --

class MLP:
    """Scoring network in device memory: fp32 master ``param`` (W1 | b1 | w2 |
    b2), bf16 copy ``wbf16`` (W1 transposed | w2), Adam moments ``m``, ``v``."""

    def __init__(self, param):
        import torch
        assert param.numel() == MLP_NPARAM and param.dtype == torch.float32
        self.param = param.contiguous().cuda()
        self.wbf16 = torch.zeros(MLP_NBF16, dtype=torch.int16, device=self.param.device)
        self.m = torch.zeros_like(self.param)
        self.v = torch.zeros_like(self.param)
        self.grad = torch.zeros_like(self.param)
        self.step = 0
        self.handle = MlpHandle(self.param.data_ptr(), self.wbf16.data_ptr())
        self.sync()

    def sync(self, stream=None):
        _check(load().zx_mlp_sync(C.byref(self.handle), _stream(stream)))

    def forward(self, x, score=None, stream=None):
        import torch
        rows = x.shape[0]
        if score is None:
            score = torch.empty(rows, dtype=torch.float32, device=x.device)
        _check(load().zx_mlp_forward(C.byref(self.handle), _ptr(x), rows, _ptr(score), _stream(stream)))
        return score

    @staticmethod
    def loss(score, cost, seg_off, stream=None):
        import torch
        n_seg = seg_off.numel() - 1
        dscore = torch.empty_like(score)
        loss = torch.empty(max(n_seg, 1), dtype=torch.float32, device=score.device)
        _check(load().zx_mlp_loss(_ptr(score), _ptr(cost), _ptr(seg_off), n_seg, _ptr(dscore), _ptr(loss),
                                  _stream(stream)))
        return dscore, loss[:n_seg]

    def backward(self, x, dscore, ws=None, stream=None):
        import torch
        rows = x.shape[0]
        nb = load().zx_mlp_workspace_bytes(rows)
        if ws is None or ws.numel() < nb:
            ws = torch.empty(nb, dtype=torch.uint8, device=x.device)
        _check(load().zx_mlp_backward(C.byref(self.handle), _ptr(x), _ptr(dscore), rows, _ptr(self.grad),
                                      _ptr(ws), ws.numel(), _stream(stream)))
        return self.grad

    def adam(self, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, grad=None, stream=None):
        self.step += 1
        g = self.grad if grad is None else grad
        _check(load().zx_mlp_adam(C.byref(self.handle), _ptr(g), _ptr(self.m), _ptr(self.v), lr, beta1, beta2,
                                  eps, self.step, _stream(stream)))


class Server:
    """Continuous-batching simplification service over a device pool."""

    def __init__(self, pool_bytes, max_batch=1024, policy=ZX_POLICY_GREEDY, mlp=None, extract=True,
                 trusted=False, fallback=False):
        import torch
        self.pool = torch.empty(pool_bytes, dtype=torch.uint8, device="cuda")
        self.mlp = mlp
        self._opts = _opts(extract, -1, policy, mlp, 0, False, fallback)
        h = C.c_void_p()
        _check(load().zx_server_create(C.byref(h), _ptr(self.pool), pool_bytes, max_batch, C.byref(self._opts),
                                       ZX_SERVE_TRUSTED if trusted else 0))
        self.h = h
        self._out = (Result * 4096)()

    def submit(self, d, tag=0):
        """Submit a workloads.Diagram; returns the ticket, or None when the
        pool is full (ZX_EBUSY)."""
        adj = np.ascontiguousarray(d.adj, dtype=np.uint64)
        ph = np.ascontiguousarray(d.phase, dtype=np.int8)
        ins = np.ascontiguousarray(d.inputs, dtype=np.int32)
        outs = np.ascontiguousarray(d.outputs, dtype=np.int32)
        bh = None if d.bnd_is_h is None else np.ascontiguousarray(d.bnd_is_h, dtype=np.uint8)
        r = Request(int(d.n), len(ins), len(outs), 0, adj.ctypes.data, ph.ctypes.data,
                    ins.ctypes.data if len(ins) else None, outs.ctypes.data if len(outs) else None,
                    bh.ctypes.data if bh is not None else None, int(tag))
        t = C.c_int64(-1)
        rc = load().zx_server_submit(self.h, C.byref(r), C.byref(t))
        if rc == ZX_EBUSY:
            return None
        _check(rc)
        return t.value

    def poll(self):
        n = C.c_int32(0)
        _check(load().zx_server_poll(self.h, C.cast(self._out, C.c_void_p), len(self._out), C.byref(n)))
        return [Result.from_buffer_copy(self._out[i]) for i in range(n.value)]

    def stats(self):
        st = ServerStats()
        _check(load().zx_server_stats_read(self.h, C.byref(st)))
        return st

    def close(self):
        if getattr(self, "h", None) and _lib is not None:
            _lib.zx_server_destroy(self.h)
            self.h = None

    def __del__(self):
        self.close()


def rollout(states, per_state, stream=None):
    """Candidate rollouts of CURRENT diagrams: (cost, fill, move, feats) device
    tensors of n_states * per_state rows (synchronous)."""
    import torch
    n = len(states)
    arr = _graph_array(states)
    nb = load().zx_rollout_workspace_bytes(arr, n)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    items = n * per_state
    cost = torch.empty(items, dtype=torch.int64, device="cuda")
    fill = torch.empty(items, dtype=torch.int64, device="cuda")
    move = torch.empty((items, 3), dtype=torch.int32, device="cuda")
    feats = torch.empty((items, MLP_IN), dtype=torch.int16, device="cuda")
    _check(load().zx_rollout(arr, n, per_state, _ptr(cost), _ptr(fill), _ptr(move), _ptr(feats), _ptr(ws),
                             ws.numel(), _stream(stream)))
    return cost, fill, move, feats


def policy_features(graph, max_cand=None, stream=None):
    """Candidates of the next round of graph's CURRENT state as the learned
    schedule lists them, and their learned-proposal features: (cand int32
    tensor [C, 2] of (u, v), v = -1 for LC; feats int16 tensor [C, MLP_IN]
    holding bf16 bits), C the full count (synchronous)."""
    import torch
    if max_cand is None:  # the list capacity of a round: a power of two >= max(64, n)
        cap = 64
        while cap < graph.n:
            cap *= 2
    else:
        cap = max_cand
    cand = torch.empty((max(cap, 1), 2), dtype=torch.int32, device="cuda")
    feats = torch.empty((max(cap, 1), MLP_IN), dtype=torch.int16, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    _check(load().zx_policy_features(graph.h, _ptr(cand), _ptr(feats), cap, _ptr(cnt), _stream(stream)))
    C = int(cnt.item())
    k = min(C, cap)
    return cand[:k], feats[:k], C


def simplify_variants():
    lib = load()
    return [lib.zx_simplify_variant_name(i).decode() for i in range(lib.zx_simplify_variants())]


# ------------------------------------------------------------------ GF(2) --

def gf2_workspace_bytes(m, n_cols):
    return load().zx_gf2_workspace_bytes(m, n_cols)


def gf2_eliminate(A, R=None, n_cols=None, rank=None, pivots=None, ws=None, stream=None, T=None):
    """RREF of A (torch int64/uint64-view device tensor, m x ld words).
    T: optional device tensor (m x >= ceil(m/64) words) that receives the
    transform with T A = R.  Returns (R, rank tensor, pivots tensor, ws)."""
    import torch
    m, ld = A.shape
    n_cols = 64 * ld if n_cols is None else n_cols
    if R is None:
        R = torch.empty_like(A)
    if rank is None:
        rank = torch.zeros(1, dtype=torch.int32, device=A.device)
    if pivots is None:
        pivots = torch.zeros(m, dtype=torch.int32, device=A.device)
    if ws is None:
        ws = torch.empty(gf2_workspace_bytes(m, n_cols), dtype=torch.uint8, device=A.device)
    ldt = T.shape[1] if T is not None else 0
    _check(load().zx_gf2_eliminate(_ptr(A), _ptr(R), m, n_cols, ld, _ptr(rank), _ptr(pivots),
                                   _ptr(T) if T is not None else None, ldt, _ptr(ws), ws.numel(),
                                   _stream(stream)))
    return R, rank, pivots, ws


def gf2_eliminate_noalloc(A, R, rank, pivots, n_cols=None, stream=None, T=None):
    """RREF of A into the caller's R, rank and pivots tensors through the
    allocation-free entry point (workspace: the library's static device
    array).  Returns R."""
    m, ld = A.shape
    n_cols = 64 * ld if n_cols is None else n_cols
    ldt = T.shape[1] if T is not None else 0
    _check(load().zx_gf2_eliminate_noalloc(_ptr(A), _ptr(R), m, n_cols, ld, _ptr(rank), _ptr(pivots),
                                           _ptr(T) if T is not None else None, ldt, _stream(stream)))
    return R


def gf2_basis(D, n_cols, stream=None):
    """Minimal basis of the rows of D (device word tensor m x ld): returns
    (R, rank tensor, pivots tensor, coeff) with the first rank rows of R the
    basis and D = coeff . basis."""
    import torch
    m, ld = D.shape
    R = torch.empty_like(D)
    rank = torch.zeros(1, dtype=torch.int32, device=D.device)
    piv = torch.zeros(m, dtype=torch.int32, device=D.device)
    ldc = (min(m, n_cols) + 63) // 64
    coeff = torch.empty((m, ldc), dtype=torch.int64, device=D.device)
    ws = torch.empty(gf2_workspace_bytes(m, n_cols), dtype=torch.uint8, device=D.device)
    _check(load().zx_gf2_basis(_ptr(D), m, n_cols, ld, _ptr(R), _ptr(rank), _ptr(piv), _ptr(coeff), ldc, _ptr(ws),
                               ws.numel(), _stream(stream)))
    return R, rank, piv, coeff


def gf2_status(ws, stream=None):
    return load().zx_gf2_status(_ptr(ws), _stream(stream))


def gf2_profile(ws, m, max_strips=8192, stream=None):
    """Per-strip timestamps (n x 8, 100 MHz ticks) if ZX_RREF_PROFILE=1 was set."""
    out = np.zeros((max_strips, 8), np.int64)
    _check(load().zx_gf2_profile_read(_ptr(ws), m, _np(out), max_strips, _stream(stream)))
    return out


# ------------------------------------------------------------------ Pauli --

ZX_PAULI_AUTO, ZX_PAULI_FORCE_VALU, ZX_PAULI_FORCE_MFMA = 0x0, 0x1, 0x2


def pauli_commute(X, Z, n_qubits, C_out=None, stream=None, flags=ZX_PAULI_AUTO):
    import torch
    n, ldq = X.shape
    ldc = (n + 63) // 64
    if C_out is None:
        C_out = torch.empty((n, ldc), dtype=X.dtype, device=X.device)
    _check(load().zx_pauli_commute(_ptr(X), _ptr(Z), n, n_qubits, ldq, _ptr(C_out), C_out.shape[1], flags,
                                   _stream(stream)))
    return C_out


# ------------------------------------------------ parameterized evaluation --

def gf2_matmul(A, B, k_bits, C_out=None, stream=None):
    """C[i][j] = parity of A_i & B_j over the first k_bits bits (device tensors
    of words, rows A: m, B: n).  Returns C (m x ceil(n/64) words)."""
    import torch
    m, lda = A.shape
    n, ldb = B.shape
    if C_out is None:
        C_out = torch.empty((m, (n + 63) // 64), dtype=torch.int64, device=A.device)
    _check(load().zx_gf2_matmul(_ptr(A), m, lda, _ptr(B), n, ldb, int(k_bits), _ptr(C_out), C_out.shape[1], 0,
                                _stream(stream)))
    return C_out


def phase_pair_product(A, B, k_alpha, k_beta, n_settings, phase8=0, pow_sqrt2=0, mant=None, expo=None,
                       stream=None):
    """Per setting: omega^phase8 sqrt(2)^pow prod_k h(...).  A, B: n_terms x
    ld word tensors; k_alpha, k_beta: int8 device tensors.  Returns (mant
    float32 [n, 2], expo int32 [n])."""
    import torch
    n_terms = int(k_alpha.numel())
    ld = A.shape[1] if n_terms else (n_settings + 63) // 64
    dev = k_alpha.device
    if mant is None:
        mant = torch.empty((n_settings, 2), dtype=torch.float32, device=dev)
    if expo is None:
        expo = torch.empty(n_settings, dtype=torch.int32, device=dev)
    _check(load().zx_phase_pair_product(_ptr(A) if n_terms else None, _ptr(B) if n_terms else None, ld,
                                        n_terms, n_settings, _ptr(k_alpha) if n_terms else None,
                                        _ptr(k_beta) if n_terms else None, int(phase8), int(pow_sqrt2),
                                        _ptr(mant), _ptr(expo), _stream(stream)))
    return mant, expo


def to_device_words(a: np.ndarray):
    """numpy uint64 array -> torch int64 device tensor with the same bits."""
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint64).view(np.int64)).cuda()


def to_host_words(t) -> np.ndarray:
    return t.cpu().numpy().view(np.uint64)


# ------------------------------------------------------- detector sampling --

def gflow(graphs, stream=None):
    """Generalised-flow layers of the CURRENT diagrams (zx_gflow): returns
    (exists, layers) with exists[i] in {1, 0, ZX_ECAPACITY} and layers[i] the
    int32 layer of each spider of graph i (-1: none)."""
    import torch
    n = len(graphs)
    total = sum(g.n for g in graphs)
    res = torch.empty(n + max(total, 1), dtype=torch.int32, device="cuda")  # one copy back
    exists, layers = res[:n], res[n:]
    nb = load().zx_gflow_workspace_bytes(n)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    _check(load().zx_gflow(_graph_array(graphs), n, _ptr(layers), _ptr(exists), _ptr(ws), nb, _stream(stream)))
    res = res.cpu().numpy()
    lay = res[n:]
    out, off = [], 0
    for g in graphs:
        out.append(lay[off:off + g.n].copy())
        off += g.n
    return res[:n].copy(), out


def decode_gates(words):
    """uint32 gate words -> ("H", q) / ("RZ", q, k) / ("CZ", a, b) / ("CNOT", c, t)."""
    out = []
    for w in np.asarray(words, np.uint32).tolist():
        t, a, b = w >> 30, (w >> 15) & 0x7FFF, w & 0x7FFF
        if t == ZX_GATE_H:
            out.append(("H", a))
        elif t == ZX_GATE_RZ:
            out.append(("RZ", a, b))
        elif t == ZX_GATE_CZ:
            out.append(("CZ", a, b))
        else:
            out.append(("CNOT", a, b))
    return out


def extract(graphs, max_gates=None, stream=None, raw=False):
    """Circuits of the CURRENT diagrams (zx_extract).  Returns one
    (status, gates, perm) per graph: gates decoded (``raw``: the uint32
    words), perm[q] = input wire of qubit q.  max_gates defaults to a bound
    on what a diagram of that size can emit."""
    import torch
    n = len(graphs)
    if max_gates is None:
        max_gates = max(64, max((g.n + 2 * g.n_in) * (g.n_out + 4) for g in graphs))
    gates = torch.empty(n * max_gates, dtype=torch.int32, device="cuda")
    res = torch.empty(2 * n + max(1, sum(g.n_out for g in graphs)), dtype=torch.int32, device="cuda")
    n_gates, status, perm = res[:n], res[n:2 * n], res[2 * n:]
    nb = load().zx_extract_workspace_bytes(n)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    _check(load().zx_extract(_graph_array(graphs), n, int(max_gates), _ptr(gates), _ptr(n_gates), _ptr(perm),
                             _ptr(status), _ptr(ws), nb, _stream(stream)))
    res = res.cpu().numpy()
    ng, st, pm = res[:n], res[n:2 * n], res[2 * n:]
    need = int(ng[st == ZX_ECAPACITY].max()) if (st == ZX_ECAPACITY).any() else 0
    if need > max_gates:  # the buffer was short: once more with the counted size
        return extract(graphs, max_gates=need, stream=stream, raw=raw)
    # only as many columns as the longest list: the bound is several times what is emitted
    used = min(int(ng.max(initial=0)), max_gates)
    G = gates.view(n, max_gates)[:, :used].contiguous().cpu().numpy().view(np.uint32)
    out, off = [], 0
    for i, g in enumerate(graphs):
        words = G[i, :min(int(ng[i]), max_gates)].copy()
        out.append((int(st[i]), words if raw else decode_gates(words), pm[off:off + g.n_out].copy()))
        off += g.n_out
    return out


class DetectorSampler:
    """Device copy of a detector error model (T as CSC, probabilities) and a
    workspace; sample() fills rows of f bits for a range of shots."""

    def __init__(self, col_ptr, col_idx, prob, n_f, device="cuda"):
        import torch
        self.n_err = int(len(prob))
        self.n_f = int(n_f)
        self.nnz = int(len(col_idx))
        self.col_ptr = torch.from_numpy(np.ascontiguousarray(col_ptr, np.int32)).to(device)
        self.col_idx = torch.from_numpy(np.ascontiguousarray(col_idx, np.int32)).to(device)
        if self.nnz == 0:
            self.col_idx = torch.zeros(1, dtype=torch.int32, device=device)
        self.prob = torch.from_numpy(np.ascontiguousarray(prob, np.float64)).to(device)
        self.ws = torch.empty(load().zx_detector_workspace_bytes(self.n_err), dtype=torch.uint8, device=device)

    def sample(self, seed, shot0, n_shots, out=None, stream=None):
        import torch
        fw = (self.n_f + 63) // 64
        if out is None:
            out = torch.empty((n_shots, fw), dtype=torch.int64, device=self.ws.device)
        _check(load().zx_detector_sample(_ptr(self.col_ptr), _ptr(self.col_idx), self.nnz, _ptr(self.prob),
                                         self.n_err, self.n_f, int(seed) & (2 ** 64 - 1), int(shot0), int(n_shots),
                                         _ptr(out), out.shape[1], _ptr(self.ws), self.ws.numel(), _stream(stream)))
        return out

    def status(self, stream=None):
        return load().zx_detector_status(_ptr(self.ws), _stream(stream))
