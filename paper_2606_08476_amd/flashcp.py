"""Python binding of the C ABI in ``include/flashcp.h``.

Argument marshalling only: every planner, view and kernel call goes to the
native library ``libflashcp.so`` built in this directory. Torch supplies
device memory and the current HIP stream; tensor shapes, dtypes and
devices are checked here so that no kernel is handed a buffer smaller than
the view implies. There is no fallback: if the library is missing, loading
fails with an error.
"""
from __future__ import annotations

import ctypes as C
import os

import numpy as np

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libflashcp.so")

FC_TWO_PASS = 0
FC_FUSED = 1

ERRORS = {
    -1: "FC_ERR_INVALID_ARG", -2: "FC_ERR_PLAN", -3: "FC_ERR_SHAPE", -4: "FC_ERR_UNSUPPORTED",
    -5: "FC_ERR_WORKSPACE", -6: "FC_ERR_HIP", -7: "FC_ERR_CAPACITY", -8: "FC_ERR_INTERNAL",
}

# every function the header declares
EXPORTS = [
    "fc_plan_per_doc", "fc_plan_per_seq", "fc_plan_whole_lpt", "fc_plan_hybrid", "fc_plan_validate",
    "fc_plan_stats", "fc_view_create", "fc_view_get_info", "fc_view_export", "fc_view_bind",
    "fc_view_destroy", "fc_view_export_launch", "fc_view_export_split", "fc_workspace_size", "fc_kv_gather", "fc_attn_fwd",
    "fc_attn_fwd_partial", "fc_attn_fwd_partials", "fc_lse_merge", "fc_attn_bwd", "fc_bwd_preprocess",
    "fc_attn_bwd_pass", "fc_attn_bwd_dkdv", "fc_attn_bwd_dq", "fc_attn_bwd_noalloc", "fc_last_error",
]

# bytes of the static device scratch behind fc_attn_bwd_noalloc (flashcp.h)
NOALLOC_SCRATCH_BYTES = 64 * 1024 * 1024


class FlashCPError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"{ERRORS.get(code, code)}: {msg}")
        self.code = code


class Shard(C.Structure):
    _fields_ = [("doc", C.c_int32), ("rank", C.c_int32), ("offset", C.c_int32), ("len", C.c_int32)]


class TileCfg(C.Structure):
    _fields_ = [("bm_fwd", C.c_int32), ("bn_fwd", C.c_int32), ("bm_bwd", C.c_int32),
                ("bn_bwd", C.c_int32)]


class ViewInfo(C.Structure):
    _fields_ = [
        ("t_q", C.c_int32), ("t_recv", C.c_int32), ("n_seg", C.c_int32), ("n_pieces", C.c_int32),
        ("hq", C.c_int32), ("hkv", C.c_int32), ("d", C.c_int32),
        ("bm_fwd", C.c_int32), ("bn_fwd", C.c_int32), ("bm_bwd", C.c_int32), ("bn_bwd", C.c_int32),
        ("pad_", C.c_int32),
        ("n_fwd_local", C.c_int64), ("n_fwd_recv", C.c_int64), ("n_fwd_fused", C.c_int64),
        ("n_bwd", C.c_int64), ("pairs_loc", C.c_int64), ("pairs_recv", C.c_int64),
        ("meta_bytes", C.c_int64), ("n_bwd_launch", C.c_int64), ("n_bwd_reduce", C.c_int64),
        ("n_bwd_slots", C.c_int64), ("table_bytes", C.c_int64),
    ]

    def as_dict(self):
        return {k: getattr(self, k) for k, _ in self._fields_ if k != "pad_"}


_lib = _raw = None
P = C.c_void_p
I32P = C.POINTER(C.c_int32)


def _signatures():
    return {
        "fc_plan_per_doc": [I32P, C.c_int32, C.c_int32, C.POINTER(Shard), C.c_int64, C.POINTER(C.c_int64)],
        "fc_plan_per_seq": [I32P, C.c_int32, C.c_int32, C.POINTER(Shard), C.c_int64, C.POINTER(C.c_int64)],
        "fc_plan_whole_lpt": [I32P, C.c_int32, C.c_int32, C.POINTER(Shard), C.c_int64, C.POINTER(C.c_int64)],
        "fc_plan_hybrid": [I32P, C.c_int32, C.c_int32, C.c_double, C.POINTER(Shard), C.c_int64,
                           C.POINTER(C.c_int64), C.POINTER(C.c_uint8)],
        "fc_plan_validate": [I32P, C.c_int32, C.c_int32, C.POINTER(Shard), C.c_int64, C.c_int32],
        "fc_plan_stats": [I32P, C.c_int32, C.c_int32, C.POINTER(Shard), C.c_int64, C.c_int32, C.c_int32,
                          C.POINTER(C.c_int64), I32P, I32P, C.POINTER(C.c_int64), C.POINTER(C.c_int64),
                          C.POINTER(C.c_double)],
        "fc_view_create": [I32P, C.c_int32, C.POINTER(Shard), C.c_int64, C.c_int32, C.c_int32,
                           C.c_int32, C.c_int32, C.c_int32, C.POINTER(TileCfg), C.POINTER(P)],
        "fc_view_get_info": [P, C.POINTER(ViewInfo)],
        "fc_view_export": [P] + [I32P] * 11,
        "fc_view_bind": [P, P, C.c_size_t, P],
        "fc_view_export_launch": [P] + [I32P] * 6,
        "fc_view_export_split": [P] + [I32P] * 5,
        "fc_workspace_size": [P, C.c_int32, C.POINTER(C.c_size_t), C.POINTER(C.c_size_t),
                              C.POINTER(C.c_size_t)],
        "fc_kv_gather": [P, P, P, C.c_int64, P, P, P, P, P],
        "fc_attn_fwd": [P, P, P, P, P, P, C.c_float, C.c_int32, P, P, P, P, C.c_size_t, P],
        "fc_attn_fwd_partial": [P, C.c_int32, P, P, P, C.c_float, P, P, P],
        "fc_attn_fwd_partials": [P, P, P, P, P, P, C.c_float, P, P, P, P, P],
        "fc_lse_merge": [P, P, P, P, C.c_int32, C.c_int32, C.c_int32, P, P, P, P],
        "fc_attn_bwd": [P, P, P, P, P, P, P, P, P, P, C.c_float, C.c_int32, P, P, P, P, P, P,
                        C.c_size_t, P],
        "fc_bwd_preprocess": [P, P, P, P, P, P],
        "fc_attn_bwd_pass": [P, P, P, P, P, P, P, P, P, C.c_float, C.c_int32, P, P, P, P, P, P,
                             C.c_size_t, P],
        "fc_attn_bwd_dkdv": [P, P, P, P, P, P, P, P, P, C.c_float, P, P, P, P, P, C.c_size_t, P],
        "fc_attn_bwd_dq": [P, P, P, P, P, P, P, P, P, C.c_float, P, P],
        "fc_attn_bwd_noalloc": [P, P, P, P, P, P, P, P, P, P, C.c_float, C.c_int32, P, P, P, P,
                                P, P],
    }


def _open(raw):
    """The native library; its pointer arguments typed as declared, or (raw)
    plain addresses."""
    if not os.path.exists(_LIB_PATH):
        raise FileNotFoundError(f"{_LIB_PATH} is not built; run python -m paper_2606_08476_amd.build")
    L = C.CDLL(_LIB_PATH)
    for name, args in _signatures().items():
        f = getattr(L, name)
        f.argtypes = [P if raw and issubclass(a, C._Pointer) else a for a in args]
        f.restype = C.c_int
    L.fc_view_destroy.argtypes = [P]
    L.fc_view_destroy.restype = None
    L.fc_last_error.argtypes = []
    L.fc_last_error.restype = C.c_char_p
    return L


def lib():
    """The loaded native library (loaded once)."""
    global _lib
    if _lib is None:
        _lib = _open(False)
    return _lib


def _addr():
    """The same for calls made with addresses of numpy arrays whose types are
    set here (a typed pointer to one costs a microsecond or two)."""
    global _raw
    if _raw is None:
        _raw = _open(True)
    return _raw


def _check(rc: int):
    if rc != 0:
        raise FlashCPError(rc, lib().fc_last_error().decode())


def _i32(x):
    """x as a contiguous, aligned int32 array (keep it alive during the call) and
    its address."""
    a = np.ascontiguousarray(np.asarray(x, dtype=np.int32))
    if not a.flags.aligned:
        a = a.copy()
    return a, a.ctypes.data


def _cu(cu):
    a, p = _i32(cu)
    return a, p, int(a.size - 1)


def _shards(plan):
    """The plan as an int32 [n, 4] array (the layout of fc_shard), its address and
    n. (Addresses of numpy arrays throughout: an array type made per call, Shard *
    n, costs some 50 us.)"""
    a, p = _i32(np.asarray(plan, dtype=np.int32).reshape(-1, 4))
    return a, p, len(a)


def _plan_out(fn, *args):
    n = C.c_int64(0)
    cap = 1024
    while True:
        buf = np.empty((cap, 4), dtype=np.int32)
        rc = fn(*args, buf.ctypes.data, cap, C.byref(n))
        if rc == -7:
            cap = int(n.value)
            continue
        _check(rc)
        return buf[:n.value].copy()


# ------------------------------------------------------------------ planners

def fc_plan_per_doc(cu, cp: int) -> np.ndarray:
    a, p, n = _cu(cu)
    return _plan_out(_addr().fc_plan_per_doc, p, n, cp)


def fc_plan_per_seq(cu, cp: int) -> np.ndarray:
    a, p, n = _cu(cu)
    return _plan_out(_addr().fc_plan_per_seq, p, n, cp)


def fc_plan_whole_lpt(cu, cp: int) -> np.ndarray:
    a, p, n = _cu(cu)
    return _plan_out(_addr().fc_plan_whole_lpt, p, n, cp)


def fc_plan_hybrid(cu, cp: int, target_r: float = 1.05):
    a, p, n = _cu(cu)
    isp = np.zeros(n, dtype=np.uint8)
    cnt = C.c_int64(0)
    cap = 4 * n + 4 * cp + 16
    while True:
        buf = np.empty((cap, 4), dtype=np.int32)
        rc = _addr().fc_plan_hybrid(p, n, cp, float(target_r), buf.ctypes.data, cap, C.byref(cnt),
                                    isp.ctypes.data)
        if rc == -7:
            cap = int(cnt.value)
            continue
        _check(rc)
        return buf[:cnt.value].copy(), isp


def fc_plan_validate(cu, cp: int, plan, require_equal_tokens: bool = False) -> None:
    a, p, n = _cu(cu)
    s, sp, m = _shards(plan)
    _check(_addr().fc_plan_validate(p, n, cp, sp, m, int(bool(require_equal_tokens))))


def fc_plan_stats(cu, cp: int, plan, hkv: int, d: int) -> dict:
    a, p, n = _cu(cu)
    s, sp, m = _shards(plan)
    work = np.zeros(cp, dtype=np.int64)
    tok, rcv = np.zeros(cp, dtype=np.int32), np.zeros(cp, dtype=np.int32)
    eq4, eq5, imb = C.c_int64(0), C.c_int64(0), C.c_double(0)
    _check(_addr().fc_plan_stats(p, n, cp, sp, m, hkv, d, work.ctypes.data, tok.ctypes.data,
                                 rcv.ctypes.data, C.byref(eq4), C.byref(eq5), C.byref(imb)))
    return dict(work=work.tolist(), tokens=tok.tolist(), recv_tokens=rcv.tolist(), eq4=eq4.value,
                eq5=eq5.value, imbalance=imb.value)


# --------------------------------------------------------------------- views

class View:
    """An fc_view handle plus, once bound, the device buffer holding its
    tables. Destroyed with ``close()`` (or when garbage collected).
    ``tiles``: (bm_fwd, bn_fwd, bm_bwd, bn_bwd), 0 for a default; None for
    all defaults."""

    def __init__(self, cu, plan, cp: int, rank: int, hq: int, hkv: int, d: int, tiles=None):
        a, p, n = _cu(cu)
        s, sp, m = _shards(plan)
        h = P()
        t = C.byref(TileCfg(*[int(x) for x in tiles])) if tiles is not None else None
        _check(_addr().fc_view_create(p, n, sp, m, cp, rank, hq, hkv, d, t, C.byref(h)))
        self._h = h
        self.meta = None
        info = ViewInfo()
        _check(lib().fc_view_get_info(self._h, C.byref(info)))
        self._info = info
        # shapes every device call checks its tensors against
        tq, tr, hq, hkv, d = info.t_q, info.t_recv, info.hq, info.hkv, info.d
        self._q, self._kv, self._kvr, self._l = (tq, hq, d), (tq, hkv, d), (tr, hkv, d), (hq, tq)

    @property
    def info(self) -> dict:
        """The fields of fc_view_info."""
        d = self.__dict__.get("_info_dict")
        if d is None:
            d = self._info_dict = self._info.as_dict()
        return d

    @property
    def handle(self):
        if self._h is None:
            raise ValueError("view is closed")
        return self._h

    def export(self) -> dict:
        i = self.info
        sizes = dict(q_gpos=i["t_q"], recv_gpos=i["t_recv"], seg_doc=i["n_seg"],
                     q_cu_docseg=i["n_seg"] + 1, recv_cu=i["n_seg"] + 1, pieces=5 * i["n_pieces"],
                     lim=i["t_q"], fwd_local=8 * i["n_fwd_local"], fwd_recv=8 * i["n_fwd_recv"],
                     fwd_fused=8 * i["n_fwd_fused"], bwd=8 * i["n_bwd"])
        arrs = {k: np.zeros(max(1, v), dtype=np.int32) for k, v in sizes.items()}
        _check(lib().fc_view_export(self.handle, *[arrs[k].ctypes.data_as(I32P) for k in sizes]))
        out = {k: arrs[k][:sizes[k]] for k in sizes}
        out["pieces"] = out["pieces"].reshape(-1, 5)
        for k in ("fwd_local", "fwd_recv", "fwd_fused", "bwd"):
            out[k] = out[k].reshape(-1, 8)
        return out

    def export_launch(self) -> dict:
        """The launch tables exactly as uploaded (fc_view_export_launch)."""
        i = self.info
        nw = i["bn_bwd"] // 32
        sizes = dict(fwd_local=8 * i["n_fwd_local"], fwd_recv=8 * i["n_fwd_recv"],
                     fwd_fused=8 * i["n_fwd_fused"], bwd_launch=8 * i["n_bwd_launch"],
                     bwd_reduce=8 * i["n_bwd_reduce"], bwd_qfirst=nw * i["n_bwd_launch"])
        arrs = {k: np.zeros(max(1, v), dtype=np.int32) for k, v in sizes.items()}
        _check(lib().fc_view_export_launch(self.handle, *[arrs[k].ctypes.data_as(I32P) for k in sizes]))
        out = {k: arrs[k][:sizes[k]].reshape(-1, 8) for k in sizes if k != "bwd_qfirst"}
        out["bwd_qfirst"] = arrs["bwd_qfirst"][:sizes["bwd_qfirst"]].reshape(-1, nw)
        return out

    def export_split(self) -> dict:
        """The split key ranges (fc_view_export_split): ``fwd_chunk`` and the
        four tables."""
        n = np.zeros(5, dtype=np.int32)
        p = n.ctypes.data_as(I32P)
        _check(lib().fc_view_export_split(self.handle, p, None, None, None, None))
        out = {k: np.zeros((int(m), 8), dtype=np.int32)
               for k, m in zip(("dq_items", "dq_comb", "fwd_units", "fwd_comb"), n[1:])}
        _check(lib().fc_view_export_split(self.handle, p, *[a.ctypes.data_as(I32P)
                                                            for a in out.values()]))
        return dict(out, fwd_chunk=int(n[0]))

    def bind(self, device="cuda", buf=None, slots=True):
        """Upload the view's tables on the current stream into ``buf`` (a
        uint8 device tensor, allocated here if not given) and keep it.
        ``slots``: with the slots that the partial passes of a split view use
        (``meta_bytes``), as far as a given ``buf`` has room for them; without,
        the tables alone (``table_bytes``)."""
        need = self._info.table_bytes
        nbytes = self._info.meta_bytes if slots else need
        if buf is None:
            _load_torch()
            buf = torch.empty(nbytes + 256, dtype=torch.uint8, device=device)
        off = (-buf.data_ptr()) % 256
        if not buf.is_cuda or buf.numel() - off < need:
            raise ValueError("metadata buffer too small or not on the device")
        if buf.numel() - off < nbytes:
            nbytes = need
        self.meta = buf
        _check(lib().fc_view_bind(self.handle, buf.data_ptr() + off, nbytes, _stream()))
        return self

    def workspace_size(self, mode: int = FC_TWO_PASS):
        """(forward bytes, backward bytes, dK/dV-pass bytes)."""
        f, b, k = C.c_size_t(0), C.c_size_t(0), C.c_size_t(0)
        _check(lib().fc_workspace_size(self.handle, mode, C.byref(f), C.byref(b), C.byref(k)))
        return f.value, b.value, k.value

    def close(self):
        if getattr(self, "_h", None) is not None:
            lib().fc_view_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


# torch, loaded by the first call that needs it (the planners and views do not)
torch = _Tensor = _raw_stream = BF = F32 = None


def _load_torch():
    global torch, _Tensor, _raw_stream, BF, F32
    if torch is None:
        import torch as t
        _Tensor, BF, F32 = t.Tensor, t.bfloat16, t.float32
        # the current stream's handle without a Stream object, where torch has it
        raw, dev = getattr(t._C, "_cuda_getCurrentRawStream", None), getattr(t._C, "_cuda_getDevice", None)
        if raw is not None and dev is not None:
            _raw_stream = lambda: raw(dev())  # noqa: E731
        else:
            _raw_stream = lambda: t.cuda.current_stream().cuda_stream  # noqa: E731
        torch = t


def _stream():
    if torch is None:
        _load_torch()
    if not torch.cuda.is_initialized():
        torch.cuda.init()
    return _raw_stream()


def _ptr(t, shape, dtype, name):
    """Device address of tensor `t` after checking it; None for None."""
    if t is None:
        return None
    if (isinstance(t, _Tensor) and t.dtype is dtype and t.shape == shape and t.is_cuda
            and t.is_contiguous()):
        return t.data_ptr()
    if not isinstance(t, _Tensor) or not t.is_cuda:
        raise TypeError(f"{name} must be a device tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    raise ValueError(f"{name} must be contiguous")


def fc_kv_gather(view: View, k_packed, v_packed, k_loc, v_loc, k_recv, v_recv):
    if torch is None:
        _load_torch()
    KV, KR = view._kv, view._kvr
    T = k_packed.shape[0]
    packed = (T, KV[1], KV[2])
    _check(lib().fc_kv_gather(
        view.handle, _ptr(k_packed, packed, BF, "k_packed"), _ptr(v_packed, packed, BF, "v_packed"), T,
        _ptr(k_loc, KV, BF, "k_loc"), _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _stream()))


def fc_attn_fwd(view: View, q, k_loc, v_loc, k_recv, v_recv, scale, mode, o, o_f32, lse, ws):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    ws_ptr = ws.data_ptr() if ws is not None and ws.numel() else None
    ws_bytes = ws.numel() * ws.element_size() if ws is not None else 0
    _check(lib().fc_attn_fwd(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), float(scale), int(mode),
        _ptr(o, Q, BF, "o"), _ptr(o_f32, Q, F32, "o_f32"),
        _ptr(lse, L, F32, "lse"), ws_ptr, ws_bytes, _stream()))


def fc_attn_fwd_partial(view: View, src, q, k_src, v_src, scale, o_part, lse_part):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    K = KV if src == 0 else KR
    _check(lib().fc_attn_fwd_partial(
        view.handle, int(src), _ptr(q, Q, BF, "q"), _ptr(k_src, K, BF, "k_src"),
        _ptr(v_src, K, BF, "v_src"), float(scale), _ptr(o_part, Q, F32, "o_part"),
        _ptr(lse_part, L, F32, "lse_part"), _stream()))


def fc_attn_fwd_partials(view: View, q, k_loc, v_loc, k_recv, v_recv, scale, o_loc, lse_loc,
                         o_recv, lse_recv):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_fwd_partials(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), float(scale),
        _ptr(o_loc, Q, F32, "o_loc"), _ptr(lse_loc, L, F32, "lse_loc"),
        _ptr(o_recv, Q, F32, "o_recv"), _ptr(lse_recv, L, F32, "lse_recv"),
        _stream()))


def fc_lse_merge(o_a, lse_a, o_b, lse_b, o_bf16, o_f32, lse_out):
    if torch is None:
        _load_torch()
    t, h, d = o_a.shape
    _check(lib().fc_lse_merge(
        _ptr(o_a, (t, h, d), F32, "o_a"), _ptr(lse_a, (h, t), F32, "lse_a"),
        _ptr(o_b, (t, h, d), F32, "o_b"), _ptr(lse_b, (h, t), F32, "lse_b"), t, h, d,
        _ptr(o_bf16, (t, h, d), BF, "o_bf16"), _ptr(o_f32, (t, h, d), F32, "o_f32"),
        _ptr(lse_out, (h, t), F32, "lse_out"), _stream()))


def fc_attn_bwd(view: View, q, k_loc, v_loc, k_recv, v_recv, o, lse, dout, scale,
                dq, dk_loc, dv_loc, dk_recv, dv_recv, ws, deterministic: bool = True, o_f32=None):
    """o: the forward's bf16 output; o_f32 (optional): its fp32 output, from
    which delta is then computed (o may be None)."""
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_bwd(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _ptr(o, Q, BF, "o"),
        _ptr(o_f32, Q, F32, "o_f32"), _ptr(lse, L, F32, "lse"), _ptr(dout, Q, BF, "dout"), float(scale),
        int(bool(deterministic)),
        _ptr(dq, Q, F32, "dq"), _ptr(dk_loc, KV, F32, "dk_loc"),
        _ptr(dv_loc, KV, F32, "dv_loc"), _ptr(dk_recv, KR, F32, "dk_recv"),
        _ptr(dv_recv, KR, F32, "dv_recv"), ws.data_ptr(), ws.numel() * ws.element_size(),
        _stream()))


def fc_attn_bwd_noalloc(view: View, q, k_loc, v_loc, k_recv, v_recv, o, lse, dout, scale,
                        dq, dk_loc, dv_loc, dk_recv, dv_recv, deterministic: bool = True,
                        o_f32=None):
    """fc_attn_bwd with its workspace in the library's static device scratch
    (no device allocation)."""
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_bwd_noalloc(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _ptr(o, Q, BF, "o"),
        _ptr(o_f32, Q, F32, "o_f32"), _ptr(lse, L, F32, "lse"), _ptr(dout, Q, BF, "dout"), float(scale),
        int(bool(deterministic)),
        _ptr(dq, Q, F32, "dq"), _ptr(dk_loc, KV, F32, "dk_loc"),
        _ptr(dv_loc, KV, F32, "dv_loc"), _ptr(dk_recv, KR, F32, "dk_recv"),
        _ptr(dv_recv, KR, F32, "dv_recv"), _stream()))


def fc_bwd_preprocess(view: View, o, dout, delta, o_f32=None):
    """delta from the bf16 o, or from o_f32 when given (o may then be None)."""
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_bwd_preprocess(
        view.handle, _ptr(o, Q, BF, "o"),
        _ptr(o_f32, Q, F32, "o_f32"),
        _ptr(dout, Q, BF, "dout"),
        _ptr(delta, L, F32, "delta"), _stream()))


def _ws(ws):
    if ws is None or ws.numel() == 0:
        return None, 0
    return ws.data_ptr(), ws.numel() * ws.element_size()


def fc_attn_bwd_pass(view: View, q, k_loc, v_loc, k_recv, v_recv, lse, delta, dout, scale,
                     dq, dk_loc, dv_loc, dk_recv, dv_recv, ws=None, deterministic: bool = True):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_bwd_pass(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _ptr(lse, L, F32, "lse"),
        _ptr(delta, L, F32, "delta"), _ptr(dout, Q, BF, "dout"), float(scale),
        int(bool(deterministic)),
        _ptr(dq, Q, F32, "dq"), _ptr(dk_loc, KV, F32, "dk_loc"),
        _ptr(dv_loc, KV, F32, "dv_loc"), _ptr(dk_recv, KR, F32, "dk_recv"),
        _ptr(dv_recv, KR, F32, "dv_recv"), *_ws(ws), _stream()))


def fc_attn_bwd_dkdv(view: View, q, k_loc, v_loc, k_recv, v_recv, lse, delta, dout, scale,
                     dk_loc, dv_loc, dk_recv, dv_recv, ws=None):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_bwd_dkdv(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _ptr(lse, L, F32, "lse"),
        _ptr(delta, L, F32, "delta"), _ptr(dout, Q, BF, "dout"), float(scale),
        _ptr(dk_loc, KV, F32, "dk_loc"), _ptr(dv_loc, KV, F32, "dv_loc"),
        _ptr(dk_recv, KR, F32, "dk_recv"), _ptr(dv_recv, KR, F32, "dv_recv"),
        *_ws(ws), _stream()))


def fc_attn_bwd_dq(view: View, q, k_loc, v_loc, k_recv, v_recv, lse, delta, dout, scale, dq):
    if torch is None:
        _load_torch()
    Q, KV, KR, L = view._q, view._kv, view._kvr, view._l
    _check(lib().fc_attn_bwd_dq(
        view.handle, _ptr(q, Q, BF, "q"), _ptr(k_loc, KV, BF, "k_loc"),
        _ptr(v_loc, KV, BF, "v_loc"), _ptr(k_recv, KR, BF, "k_recv"),
        _ptr(v_recv, KR, BF, "v_recv"), _ptr(lse, L, F32, "lse"),
        _ptr(delta, L, F32, "delta"), _ptr(dout, Q, BF, "dout"), float(scale),
        _ptr(dq, Q, F32, "dq"), _stream()))
