"""ctypes marshalling for include/gcn.h.  No arithmetic happens here."""
from __future__ import annotations

import ctypes as C
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(HERE, "libgcn_hip.so")
_HEADER = os.path.join(os.path.dirname(HERE), "include", "gcn.h")

SYMMETRISE, ADD_SELF_LOOPS, NORM_SYM, BUILD_TRANSPOSE, NORM_ROW = 1, 2, 4, 8, 16
EPI_NONE, EPI_RELU, EPI_MASK = 0, 1, 2
ORDER_AUTO, ORDER_GEMM_FIRST, ORDER_SPMM_FIRST = 0, 1, 2
ACT_NONE, ACT_RELU = 0, 1
CFG_SPMM_ALGO, CFG_TIMING, CFG_SPMM_BLOCKS, CFG_SWEEP_HEAVY, CFG_SWEEP_WAVES, CFG_PATTERN_SPMM, CFG_HUB_MB, CFG_HUB_DMIN, CFG_HUB_BLOCK_COLS, CFG_SPLIT_LDS_KB, CFG_FUSED_LAST_LAYER = 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11

_lib = None


class GcnError(RuntimeError):
    def __init__(self, code: int, message: str):
        super().__init__(f"gcn error {code}: {message}")
        self.code = code


def library_path() -> str:
    return _LIB_PATH


def exported_symbols():
    """Names of the functions include/gcn.h declares."""
    with open(_HEADER) as fh:
        text = fh.read()
    return sorted(set(re.findall(r"\b(gcn_[a-z_0-9]+)\s*\(", text)))


def lib():
    """Load libgcn_hip.so (torch first, so both share one HIP runtime)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise RuntimeError(
                f"{_LIB_PATH} is missing: build it with `python -m paper_2005_03300_amd.build` "
                "(there is no CPU fallback)")
        import torch  # noqa: F401  -- loads the HIP runtime the library binds to
        L = C.CDLL(_LIB_PATH)
        L.gcn_last_error.restype = C.c_char_p
        L.gcn_version.restype = C.c_char_p
        L.gcn_epoch_workspace_bytes.restype = C.c_size_t
        L.gcn_build_count.restype = C.c_int64
        # Argument types of the compute calls: plain Python numbers then pass as they are.  Without them every argument
        # is wrapped in an object of its own, which made a product of a small graph wait for the host (8.7 us per call).
        p, i, i32, i64, f32, sz = C.c_void_p, C.c_int, C.c_int32, C.c_int64, C.c_float, C.c_size_t
        L.gcn_spmm.argtypes = [p, i, i32, p, i64, p, i64, i, p, i64, p]
        L.gcn_spmm_static.argtypes = L.gcn_spmm.argtypes
        L.gcn_spmm_pattern.argtypes = [p, i, i32, p, i64, p, i64, p, i, p, i64, p]
        L.gcn_scale_rows.argtypes = [i64, i32, p, i64, p, p, i64, p]
        L.gcn_gemm.argtypes = [i, i, i64, i64, i64, p, i64, p, i64, p, i64, p, i, p, i64, p]
        L.gcn_relu.argtypes = [i64, i32, p, i64, p, i64, p]
        L.gcn_relu_mask.argtypes = [i64, i32, p, i64, p, i64, p, i64, p]
        L.gcn_softmax_nll.argtypes = [i64, i32, p, i64, p, p, p, i64, p]
        L.gcn_softmax_nll_masked.argtypes = [i64, i32, p, i64, p, i64, p, p, i64, p]
        L.gcn_layer_forward.argtypes = [p, i32, i32, p, i64, p, p, p, p, p, i, i, p]
        L.gcn_layer_backward.argtypes = [p, i32, i32, p, i64, p, p, p, p, p, p, p, p, i, p]
        L.gcn_epoch.argtypes = [p, i32, p, p, p, p, p, f32, p, p, sz, i, p]
        L.gcn_epoch_masked.argtypes = [p, i32, p, p, p, i64, p, p, f32, p, p, sz, i, p]
        L.gcn_epoch_preaggregated.argtypes = L.gcn_epoch_masked.argtypes
        global _raw_stream, _device, _f32, _i32
        import torch
        _raw_stream, _device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice
        _f32, _i32 = torch.float32, torch.int32
        _lib = L
    return _lib


def _check(rc: int):
    if rc != 0:
        raise GcnError(rc, lib().gcn_last_error().decode())


def _stream():
    """The current stream's handle (0: the default stream)."""
    return C.c_void_p(_now())


def _now() -> int:
    return _raw_stream(_device())


def _ptr(t):
    return C.c_void_p(0 if t is None else t.data_ptr())


def _at(t) -> int:
    return 0 if t is None else t.data_ptr()


def _ld(t) -> int:
    rows, cols = t.shape
    s0, s1 = t.stride()
    assert cols == 1 or s1 == 1, "rows must be contiguous"
    return s0 if rows > 1 else max(s0, cols)


def _dev(t, dtype=None):
    assert t.is_cuda, "device tensor expected"
    assert dtype is None or t.dtype == dtype, (t.dtype, dtype)
    return t


class Csr:
    """Owner of a gcn_csr handle."""

    def __init__(self, handle: int):
        self._h = C.c_void_p(handle)
        n, nnz, md = C.c_int64(), C.c_int64(), C.c_int32()
        _check(lib().gcn_csr_info(self._h, C.byref(n), C.byref(nnz), C.byref(md)))
        self.n, self.nnz, self.max_degree = n.value, nnz.value, md.value
        nr, nc = C.c_int64(), C.c_int64()
        _check(lib().gcn_csr_shape(self._h, C.byref(nr), C.byref(nc)))
        self.n_rows, self.n_cols = nr.value, nc.value

    def arrays(self, transposed: bool = False):
        """Copies of (rowptr, colidx, val, deg) as torch tensors on the device."""
        import torch
        rowptr = torch.empty((self.n_cols if transposed else self.n_rows) + 1, dtype=torch.int64, device="cuda")
        colidx = torch.empty(self.nnz, dtype=torch.int32, device="cuda")
        val = torch.empty(self.nnz, dtype=torch.float32, device="cuda")
        deg = torch.empty(self.n, dtype=torch.int32, device="cuda")
        _check(lib().gcn_csr_export(self._h, int(transposed), _ptr(rowptr), _ptr(colidx), _ptr(val), _ptr(deg),
                                    _stream()))
        return rowptr, colidx, val, deg

    def views(self, transposed: bool = False):
        """(rowptr, colidx, val, deg) as torch tensors that ALIAS the library's own device arrays (no copy):
        read-only for the caller, valid until close()."""
        import torch
        rp, ci, va, dg = C.c_void_p(), C.c_void_p(), C.c_void_p(), C.c_void_p()
        _check(lib().gcn_csr_arrays(self._h, int(transposed), C.byref(rp), C.byref(ci), C.byref(va), C.byref(dg)))

        class _Borrowed:
            def __init__(self, ptr, count, typestr):
                self.__cuda_array_interface__ = {"shape": (count,), "typestr": typestr, "data": (ptr, False),
                                                 "version": 2, "strides": None}

        def wrap(p, count, typestr, dtype):
            if count == 0 or not p.value:
                return torch.empty(0, dtype=dtype, device="cuda")
            return torch.as_tensor(_Borrowed(p.value, count, typestr), device="cuda")
        rows = self.n_cols if transposed else self.n_rows
        return (wrap(rp, rows + 1, "<i8", torch.int64), wrap(ci, self.nnz, "<i4", torch.int32),
                wrap(va, self.nnz, "<f4", torch.float32), wrap(dg, self.n, "<i4", torch.int32))

    def close(self):
        if self._h is not None and self._h.value:
            lib().gcn_csr_destroy(self._h)
        self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def gcn_csr_create(n: int, src, dst, flags: int) -> Csr:
    import torch
    src, dst = _dev(src, torch.int32).contiguous(), _dev(dst, torch.int32).contiguous()
    assert src.shape == dst.shape and src.dim() == 1
    out = C.c_void_p()
    _check(lib().gcn_csr_create(C.byref(out), C.c_int64(n), C.c_int64(src.shape[0]), _ptr(src), _ptr(dst),
                                C.c_uint32(flags), _stream()))
    return Csr(out.value)


def gcn_csr_create_from_csr(n: int, rowptr, colidx, val, flags: int) -> Csr:
    import torch
    rowptr = _dev(rowptr, torch.int64).contiguous()
    colidx = _dev(colidx, torch.int32).contiguous()
    if val is not None:
        val = _dev(val, torch.float32).contiguous()
    out = C.c_void_p()
    _check(lib().gcn_csr_create_from_csr(C.byref(out), C.c_int64(n), _ptr(rowptr), _ptr(colidx), _ptr(val),
                                         C.c_uint32(flags), _stream()))
    return Csr(out.value)


def gcn_csr_create_from_csr_rect(n_rows: int, n_cols: int, rowptr, colidx, val, flags: int) -> Csr:
    import torch
    rowptr = _dev(rowptr, torch.int64).contiguous()
    colidx = _dev(colidx, torch.int32).contiguous()
    if val is not None:
        val = _dev(val, torch.float32).contiguous()
    out = C.c_void_p()
    _check(lib().gcn_csr_create_from_csr_rect(C.byref(out), C.c_int64(n_rows), C.c_int64(n_cols), _ptr(rowptr),
                                              _ptr(colidx), _ptr(val), C.c_uint32(flags), _stream()))
    return Csr(out.value)


def _product(a: Csr, trans: int, X, Z):
    """Checks the operands of a sparse product; returns its width and the leading dimensions."""
    assert X.is_cuda and Z.is_cuda, "device tensor expected"
    assert X.dtype is _f32 and Z.dtype is _f32, (X.dtype, Z.dtype)
    rows, f = X.shape
    assert tuple(Z.shape) == ((a.n_cols if trans else a.n_rows), f)
    assert rows == (a.n_rows if trans else a.n_cols)
    return f, _ld(X), _ld(Z)


def gcn_spmm(a: Csr, trans: int, X, Z, epilogue: int = EPI_NONE, Zprev=None):
    L = _lib or lib()
    f, ldx, ldz = _product(a, trans, X, Z)
    rc = L.gcn_spmm(a._h, trans, f, X.data_ptr(), ldx, Z.data_ptr(), ldz, epilogue, _at(Zprev),
                    0 if Zprev is None else _ld(Zprev), _raw_stream(_device()))
    if rc:
        _check(rc)
    return Z


def gcn_spmm_static(a: Csr, trans: int, X, Z, epilogue: int = EPI_NONE, Zprev=None):
    L = _lib or lib()
    f, ldx, ldz = _product(a, trans, X, Z)
    _check(L.gcn_spmm_static(a._h, trans, f, X.data_ptr(), ldx, Z.data_ptr(), ldz, epilogue, _at(Zprev),
                             0 if Zprev is None else _ld(Zprev), _now()))
    return Z


def gcn_spmm_pattern(a: Csr, trans: int, X, Z, row_scale=None, epilogue: int = EPI_NONE, Zprev=None):
    L = _lib or lib()
    f, ldx, ldz = _product(a, trans, X, Z)
    if row_scale is not None:
        _dev(row_scale, _f32)
        assert row_scale.numel() == Z.shape[0] and row_scale.is_contiguous()
    _check(L.gcn_spmm_pattern(a._h, trans, f, X.data_ptr(), ldx, Z.data_ptr(), ldz, _at(row_scale), epilogue, _at(Zprev),
                              0 if Zprev is None else _ld(Zprev), _now()))
    return Z


def gcn_scale_rows(X, scale, Y):
    L = _lib or lib()
    _dev(X, _f32), _dev(scale, _f32), _dev(Y, _f32)
    rows, cols = X.shape
    assert tuple(Y.shape) == (rows, cols) and scale.numel() == rows and scale.is_contiguous()
    _check(L.gcn_scale_rows(rows, cols, X.data_ptr(), _ld(X), scale.data_ptr(), Y.data_ptr(), _ld(Y), _now()))
    return Y


def gcn_csr_inv_sqrt_degrees(a: Csr, out):
    import torch
    _dev(out, torch.float32)
    assert out.numel() == a.n_rows and out.is_contiguous()
    _check(lib().gcn_csr_inv_sqrt_degrees(a._h, _ptr(out), _stream()))
    return out


def gcn_gemm(ta: int, tb: int, A, B, Cm, bias=None, epilogue: int = EPI_NONE, Zprev=None):
    L = _lib or lib()
    _dev(A, _f32), _dev(B, _f32), _dev(Cm, _f32)
    M, N = Cm.shape
    K = A.shape[0] if ta else A.shape[1]
    _check(L.gcn_gemm(int(ta), int(tb), M, N, K, A.data_ptr(), _ld(A), B.data_ptr(), _ld(B), Cm.data_ptr(), _ld(Cm), _at(bias),
                      int(epilogue), _at(Zprev), 0 if Zprev is None else _ld(Zprev), _now()))
    return Cm


def gcn_relu(Z, H):
    L = _lib or lib()
    _check(L.gcn_relu(Z.shape[0], Z.shape[1], Z.data_ptr(), _ld(Z), H.data_ptr(), _ld(H), _now()))
    return H


def gcn_relu_mask(G, Zprev, out):
    L = _lib or lib()
    _check(L.gcn_relu_mask(G.shape[0], G.shape[1], G.data_ptr(), _ld(G), Zprev.data_ptr(), _ld(Zprev), out.data_ptr(),
                           _ld(out), _now()))
    return out


def gcn_softmax_nll(Z, labels, loss, G=None):
    L = _lib or lib()
    _dev(Z, _f32), _dev(labels, _i32), _dev(loss, _f32)
    _check(L.gcn_softmax_nll(Z.shape[0], Z.shape[1], Z.data_ptr(), _ld(Z), labels.data_ptr(), loss.data_ptr(), _at(G),
                             0 if G is None else _ld(G), _now()))
    return loss


def gcn_softmax_nll_masked(Z, labels, n_labelled: int, loss, G=None):
    L = _lib or lib()
    _dev(Z, _f32), _dev(labels, _i32), _dev(loss, _f32)
    _check(L.gcn_softmax_nll_masked(Z.shape[0], Z.shape[1], Z.data_ptr(), _ld(Z), labels.data_ptr(), n_labelled,
                                    loss.data_ptr(), _at(G), 0 if G is None else _ld(G), _now()))
    return loss


def gcn_layer_forward(a: Csr, Hin, W, Z, Hout, T, order: int = ORDER_AUTO, act: int = ACT_RELU, bias=None):
    L = _lib or lib()
    f_in, f_out = W.shape
    assert W.is_contiguous() and Z.is_contiguous() and T.is_contiguous()
    assert Hout is None or Hout.is_contiguous()
    _check(L.gcn_layer_forward(a._h, f_in, f_out, _at(Hin), _ld(Hin), W.data_ptr(), _at(bias), Z.data_ptr(), _at(Hout),
                               T.data_ptr(), int(order), int(act), _now()))


def gcn_layer_backward(a: Csr, Hin, Zprev, W, G, T, S, Y, Gprev, order: int = ORDER_AUTO, dbias=None):
    L = _lib or lib()
    f_in, f_out = W.shape
    for t in (W, G, S, Y):
        assert t.is_contiguous()
    _check(L.gcn_layer_backward(a._h, f_in, f_out, _at(Hin), 0 if Hin is None else _ld(Hin), _at(Zprev), W.data_ptr(),
                                G.data_ptr(), _at(T), S.data_ptr(), Y.data_ptr(), _at(dbias), _at(Gprev), int(order), _now()))


def _dims_array(dims):
    return (C.c_int32 * len(dims))(*[int(d) for d in dims])


def gcn_epoch_workspace_bytes(n: int, dims, order: int = ORDER_AUTO) -> int:
    return int(lib().gcn_epoch_workspace_bytes(C.c_int64(n), C.c_int32(len(dims) - 1), _dims_array(dims), int(order)))


def _pointers(tensors):
    return (C.c_void_p * len(tensors))(*[t.data_ptr() for t in tensors])


def gcn_epoch(a: Csr, dims, H0, labels, W, Y, lr: float, loss, workspace, order: int = ORDER_AUTO):
    lib_ = _lib or lib()
    L = len(dims) - 1
    assert len(W) == L and len(Y) == L and H0.is_contiguous()
    _check(lib_.gcn_epoch(a._h, L, _dims_array(dims), _at(H0), _at(labels), _pointers(W), _pointers(Y), lr, _at(loss),
                          _at(workspace), workspace.numel() * workspace.element_size(), int(order), _now()))
    return loss


def gcn_epoch_masked(a: Csr, dims, H0, labels, n_labelled: int, W, Y, lr: float, loss, workspace,
                     order: int = ORDER_AUTO):
    lib_ = _lib or lib()
    L = len(dims) - 1
    assert len(W) == L and len(Y) == L and H0.is_contiguous()
    _check(lib_.gcn_epoch_masked(a._h, L, _dims_array(dims), _at(H0), _at(labels), n_labelled, _pointers(W), _pointers(Y), lr,
                                 _at(loss), _at(workspace), workspace.numel() * workspace.element_size(), int(order), _now()))
    return loss


def gcn_epoch_preaggregated(a: Csr, dims, P0, labels, n_labelled: int, W, Y, lr: float, loss, workspace,
                            order: int = ORDER_AUTO):
    lib_ = _lib or lib()
    L = len(dims) - 1
    assert len(W) == L and len(Y) == L and P0.is_contiguous() and tuple(P0.shape) == (a.n, dims[0])
    _check(lib_.gcn_epoch_preaggregated(a._h, L, _dims_array(dims), _at(P0), _at(labels), n_labelled, _pointers(W),
                                        _pointers(Y), lr, _at(loss), _at(workspace),
                                        workspace.numel() * workspace.element_size(), int(order), _now()))
    return loss


def gcn_epoch_view(n: int, dims, order: int, workspace, layer: int):
    """(Z^l, G^l) of the last gcn_epoch call as torch tensors aliasing the workspace."""
    import torch
    Zp, Gp = C.c_void_p(), C.c_void_p()
    _check(lib().gcn_epoch_view(C.c_int64(n), C.c_int32(len(dims) - 1), _dims_array(dims), int(order), _ptr(workspace),
                                C.c_int32(layer), C.byref(Zp), C.byref(Gp)))
    base = workspace.data_ptr()
    flat = workspace.view(torch.uint8).view(-1)
    f = int(dims[layer])

    def view(p):
        off = p.value - base
        return flat[off:off + n * f * 4].view(torch.float32).view(n, f)
    return view(Zp), view(Gp)


def gcn_config(key: int, value: int):
    _check(lib().gcn_config(int(key), int(value)))


def gcn_csr_config(a: Csr, key: int, value: int):
    _check(lib().gcn_csr_config(a._h, int(key), int(value)))


def gcn_spmm_prepare(a: Csr, trans: int, f: int):
    _check(lib().gcn_spmm_prepare(a._h, int(trans), C.c_int32(f), _stream()))


def gcn_spmm_describe(a: Csr, trans: int, f: int) -> str:
    buf = C.create_string_buffer(1024)
    _check(lib().gcn_spmm_describe(a._h, int(trans), C.c_int32(f), buf, C.c_size_t(1024), _stream()))
    return buf.value.decode()


def gcn_epoch_prepare(a: Csr, dims, order: int = ORDER_AUTO):
    _check(lib().gcn_epoch_prepare(a._h, C.c_int32(len(dims) - 1), _dims_array(dims), int(order), _stream()))


def gcn_scratch_release():
    _check(lib().gcn_scratch_release())


def gcn_build_count() -> int:
    return int(lib().gcn_build_count())


def gcn_csr_last_spmm_schedule(a: Csr) -> int:
    return int(lib().gcn_csr_last_spmm_schedule(a._h))


def gcn_timing_read():
    cnt, ms = C.c_int64(), C.c_double()
    _check(lib().gcn_timing_read(C.byref(cnt), C.byref(ms)))
    return cnt.value, ms.value


def gcn_timing_read_phases():
    """Returns {phase name: (spans, total ms)} and resets the record."""
    cnt = (C.c_int64 * 4)()
    ms = (C.c_double * 4)()
    _check(lib().gcn_timing_read_phases(cnt, ms))
    names = ("spmm_kernel", "spmm", "gemm", "other")
    return {k: (cnt[i], ms[i]) for i, k in enumerate(names)}


def gcn_radix_sort(keys, payload=None, end_bit=None, descending=False):
    """Stable radix sort of a 1-D tensor of 4- or 8-byte keys (their bit patterns as unsigned); payload: [n, w]
    int32 tensor with w in 1..3, or None.  Returns (sorted_keys, moved_payload or None)."""
    import torch
    keys = _dev(keys).contiguous()
    kb = keys.element_size()
    n = keys.numel()
    out = torch.empty_like(keys)
    pb, pout = 0, None
    if payload is not None:
        payload = _dev(payload, torch.int32).contiguous()
        assert payload.dim() == 2 and payload.shape[0] == n
        pb = 4 * payload.shape[1]
        pout = torch.empty_like(payload)
    _check(lib().gcn_radix_sort(C.c_int64(n), kb, _ptr(keys), _ptr(out), pb, _ptr(payload), _ptr(pout),
                                8 * kb if end_bit is None else int(end_bit), int(bool(descending)), _stream()))
    return out, pout


def gcn_exclusive_scan_i64(x, out=None):
    import torch
    x = _dev(x, torch.int64).contiguous()
    out = torch.empty_like(x) if out is None else _dev(out, torch.int64)
    _check(lib().gcn_exclusive_scan_i64(C.c_int64(x.numel()), _ptr(x), _ptr(out), _stream()))
    return out


def gcn_unique_u64(keys):
    """First key of every run of equal neighbours of an int64 tensor (bit patterns); returns the kept prefix."""
    import torch
    keys = _dev(keys, torch.int64).contiguous()
    out = torch.empty_like(keys)
    cnt = C.c_int64(0)
    _check(lib().gcn_unique_u64(C.c_int64(keys.numel()), _ptr(keys), _ptr(out), C.byref(cnt), _stream()))
    return out[:cnt.value]


def gcn_last_spmm_schedule() -> int:
    return int(lib().gcn_last_spmm_schedule())


SCHED_ROWWISE, SCHED_SPLIT, SCHED_SWEEP, SCHED_HUB, SCHED_BLOCKED = 1, 2, 3, 4, 5


def gcn_version() -> str:
    return lib().gcn_version().decode()
