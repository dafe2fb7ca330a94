"""ctypes binding of libbie.so (include/bie.h).

Argument marshalling only: every step of fill, excitation, products, solve
and far field runs in the library's HIP kernels.  torch supplies device
memory (tensors) and the current stream.  Importing this module loads the
library and raises if it has not been built (there is no fallback).
"""
from __future__ import annotations

import ctypes
import os
from dataclasses import dataclass

import numpy as np
import torch  # noqa: F401  (loads the HIP runtime the library shares)

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libbie.so")

BIE_OK, BIE_NOT_CONVERGED = 0, 1
BIE_EINVAL, BIE_EMESH, BIE_ENOMEM, BIE_EDEVICE, BIE_ENUMERIC = -1, -2, -3, -4, -5
BIE_C128, BIE_C64, BIE_SPLIT_BF16 = 0, 1, 2
BIE_APPLY_F64_BLOCK = 3
BIE_GMRES, BIE_CGNR, BIE_BGMRES = 0, 1, 2
BIE_SCC, BIE_RSCC, BIE_CCC = 0, 1, 2

_ERRNAMES = {BIE_EINVAL: "EINVAL", BIE_EMESH: "EMESH", BIE_ENOMEM: "ENOMEM",
             BIE_EDEVICE: "EDEVICE", BIE_ENUMERIC: "ENUMERIC"}


class BieError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"{_ERRNAMES.get(code, code)}: {msg}")
        self.code = code


class FillOpts(ctypes.Structure):
    _fields_ = [("storage", ctypes.c_int), ("near_factor", ctypes.c_double), ("keep_fp64", ctypes.c_int),
                ("star", ctypes.c_int)]


class SolveOpts(ctypes.Structure):
    _fields_ = [("method", ctypes.c_int), ("restart", ctypes.c_int), ("tol", ctypes.c_double),
                ("max_mvp", ctypes.c_int64), ("crit", ctypes.c_int), ("rscc_rows", ctypes.c_int64),
                ("rscc_seed", ctypes.c_uint64), ("use_x0", ctypes.c_int), ("precision", ctypes.c_int),
                ("inner_tol", ctypes.c_double), ("slots", ctypes.c_int64), ("inner_terms", ctypes.c_int),
                ("basis", ctypes.c_int), ("block", ctypes.c_int), ("calderon", ctypes.c_void_p)]


class CalderonInfo(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int64), ("Nb", ctypes.c_int64), ("nnz_bc", ctypes.c_int64),
                ("nnz_gram", ctypes.c_int64), ("cg_iters", ctypes.c_int64 * 2), ("cg_relres", ctypes.c_double * 2),
                ("setup_ms", ctypes.c_double)]


class WsOpts(ctypes.Structure):
    _fields_ = [("pod_rank", ctypes.c_int), ("hidden", ctypes.c_int), ("epochs", ctypes.c_int),
                ("batch", ctypes.c_int), ("lr_max", ctypes.c_double), ("lr_min", ctypes.c_double),
                ("seed", ctypes.c_uint64), ("oversample", ctypes.c_int), ("power_iters", ctypes.c_int),
                ("pol_model", ctypes.c_int)]


class FarOpts(ctypes.Structure):
    _fields_ = [("box", ctypes.c_double), ("s", ctypes.c_int), ("p", ctypes.c_int)]


class FastOpts(ctypes.Structure):
    _fields_ = [("box", ctypes.c_double), ("levels", ctypes.c_int), ("s", ctypes.c_int), ("p", ctypes.c_int),
                ("near_factor", ctypes.c_double)]


class FastInfo(ctypes.Structure):
    _fields_ = [("near_entries", ctypes.c_int64), ("leaf_cubes", ctypes.c_int64), ("levels", ctypes.c_int)]


class FarMLOpts(ctypes.Structure):
    _fields_ = [("box", ctypes.c_double), ("levels", ctypes.c_int), ("s", ctypes.c_int), ("p", ctypes.c_int)]


class FarInfo(ctypes.Structure):
    _fields_ = [("boxes", ctypes.c_int64), ("far_pairs", ctypes.c_int64), ("buffer_knots", ctypes.c_int64),
                ("splines", ctypes.c_int64), ("points_per_axis", ctypes.c_int64), ("protrusion", ctypes.c_double),
                ("origin", ctypes.c_double * 3)]


class SolveStat(ctypes.Structure):
    _fields_ = [("iters", ctypes.c_int64), ("mvps", ctypes.c_int64), ("relres_est", ctypes.c_double),
                ("relres_true", ctypes.c_double), ("converged", ctypes.c_int), ("checks", ctypes.c_int),
                ("x0_kept", ctypes.c_int)]

    def as_dict(self):
        return {f: getattr(self, f) for f, _ in self._fields_}


# (name, restype, argtypes) for every symbol declared in include/bie.h
_P = ctypes.c_void_p
_I64 = ctypes.c_int64
SYMBOLS = [
    ("bie_op_create", ctypes.c_int, [_P, _I64, _P, _I64, ctypes.c_double, _P, _P, ctypes.POINTER(_P)]),
    ("bie_op_destroy", None, [_P]),
    ("bie_release_memory", _I64, []),
    ("bie_op_create_fast", ctypes.c_int, [_P, _I64, _P, _I64, ctypes.c_double, _P, _P, ctypes.POINTER(_P)]),
    ("bie_op_fast_info", ctypes.c_int, [_P, _P]),
    ("bie_op_n", _I64, [_P]),
    ("bie_op_edges", ctypes.c_int, [_P, _P]),
    ("bie_op_near_pairs", _I64, [_P, _P, _I64]),
    ("bie_op_matrix", ctypes.c_int, [_P, _P, ctypes.c_int, _P]),
    ("bie_rhs_planewave", ctypes.c_int, [_P, _P, _P, _I64, _P, _P]),
    ("bie_apply", ctypes.c_int, [_P, _P, _P, _I64, ctypes.c_int, ctypes.c_int, _P]),
    ("bie_apply_noalloc", ctypes.c_int, [_P, _P, _P, _I64, ctypes.c_int, ctypes.c_int, _P]),
    ("bie_solve", ctypes.c_int, [_P, _P, _P, _I64, _P, _P, _P]),
    ("bie_farfield", ctypes.c_int, [_P, _P, _I64, _P, _I64, _P, _P]),
    ("bie_rcs", ctypes.c_int, [_P, _P, _I64, _P, _I64, _P, _P]),
    ("bie_batch_solve", ctypes.c_int, [_P, _I64, _P, _P, _P, _P, _P, _P]),
    ("bie_batch_solve_pc", ctypes.c_int, [_P, _P, _I64, _P, _P, _P, _P, _P, _P]),
    ("bie_batch_apply", ctypes.c_int, [_P, _I64, _P, _P, _P, ctypes.c_int, ctypes.c_int, ctypes.c_int, _P]),
    ("bie_batch_config", ctypes.c_int, [ctypes.c_int, ctypes.c_int, ctypes.c_int]),
    ("bie_batch_tuned", ctypes.c_int, [_P, _I64, _P]),
    ("bie_rscc_rows", ctypes.c_int, [_I64, _I64, ctypes.c_uint64, _P]),
    ("bie_far_create", ctypes.c_int, [_P, _P, _P, ctypes.POINTER(_P)]),
    ("bie_far_apply", ctypes.c_int, [_P, _P, _P, _I64, _P]),
    ("bie_far_get_info", ctypes.c_int, [_P, _P]),
    ("bie_far_boxes", ctypes.c_int, [_P, _P]),
    ("bie_far_destroy", None, [_P]),
    ("bie_farml_create", ctypes.c_int, [_P, _P, _P, ctypes.POINTER(_P)]),
    ("bie_farml_apply", ctypes.c_int, [_P, _P, _P, _I64, _P]),
    ("bie_farml_level_info", ctypes.c_int, [_P, ctypes.c_int, _P]),
    ("bie_farml_destroy", None, [_P]),
    ("bie_ws_train", ctypes.c_int, [_P, _P, _P, _P, _I64, _P, _P, ctypes.POINTER(_P)]),
    ("bie_ws_fit", ctypes.c_int, [_P, _P, _P, _P, _I64, ctypes.c_int, ctypes.c_int, ctypes.c_double,
                                  ctypes.c_double, ctypes.c_uint64, _P, _P]),
    ("bie_ws_predict", ctypes.c_int, [_P, _P, _P, _I64, _P, _P, _P, _P]),
    ("bie_ws_info", ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P]),
    ("bie_ws_basis", ctypes.c_int, [_P, _P, _P]),
    ("bie_ws_params", ctypes.c_int, [_P, _P, ctypes.c_int]),
    ("bie_ws_loss_grad", ctypes.c_int, [_P, _P, _P, _P, _I64, _P, _P]),
    ("bie_ws_forward", ctypes.c_int, [_P, _P, _I64, _P]),
    ("bie_ws_create", ctypes.c_int, [_P, ctypes.c_int, ctypes.c_int, ctypes.c_uint64, ctypes.c_int,
                                     ctypes.POINTER(_P)]),
    ("bie_ws_save", ctypes.c_int, [_P, ctypes.c_char_p]),
    ("bie_ws_load", ctypes.c_int, [_P, ctypes.c_char_p, ctypes.POINTER(_P)]),
    ("bie_ws_destroy", None, [_P]),
    ("bie_autotune", ctypes.c_int, [ctypes.c_int]),
    ("bie_autotune_report", _I64, [_P, _I64]),
    ("bie_prof_enable", ctypes.c_int, [ctypes.c_int]),
    ("bie_prof_read", ctypes.c_int, [ctypes.c_int, ctypes.POINTER(_I64), ctypes.POINTER(ctypes.c_double),
                                     ctypes.POINTER(_I64)]),
    ("bie_calderon_create", ctypes.c_int, [_P, _P, ctypes.POINTER(_P)]),
    ("bie_calderon_apply", ctypes.c_int, [_P, _P, _P, _I64, _P]),
    ("bie_calderon_get_info", ctypes.c_int, [_P, _P]),
    ("bie_calderon_destroy", None, [_P]),
    ("bie_last_error", ctypes.c_char_p, []),
]


def load(path: str = LIB_PATH) -> ctypes.CDLL:
    if not os.path.exists(path):
        raise ImportError(f"{path} not built: run `python -m paper_2606_13482_amd.build` "
                          "(or __graft_entry__.build())")
    lib = ctypes.CDLL(path)
    for name, res, args in SYMBOLS:
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    return lib


_lib = load()


def _check(rc: int, allow_nc: bool = False) -> int:
    if rc < 0 or (rc == BIE_NOT_CONVERGED and not allow_nc):
        raise BieError(rc, _lib.bie_last_error().decode())
    return rc


def _stream(stream=None):
    s = torch.cuda.current_stream() if stream is None else stream
    return ctypes.c_void_p(s.cuda_stream)


def _host(a, dtype):
    a = np.ascontiguousarray(a, dtype=dtype)
    return a, a.ctypes.data_as(ctypes.c_void_p)


def _dev(t: torch.Tensor, dtype, shape=None):
    if not (t.is_cuda and t.dtype == dtype and t.is_contiguous()):
        raise ValueError(f"need a contiguous {dtype} device tensor, got {t.dtype} on {t.device}")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"need shape {shape}, got {tuple(t.shape)}")
    return ctypes.c_void_p(t.data_ptr())


def release_memory() -> int:
    """Releases the device blocks that the library keeps of closed operators and
    preconditioners (at most 4 GiB a device); returns their bytes."""
    return int(_lib.bie_release_memory())


def _result(make):
    """make(): a device tensor for a result; tried again without the library's kept blocks."""
    try:
        return make()
    except torch.OutOfMemoryError:
        if not release_memory():
            raise
        return make()


def _empty(shape, dtype) -> torch.Tensor:
    return _result(lambda: torch.empty(shape, dtype=dtype, device="cuda"))


def _empty_like(x: torch.Tensor) -> torch.Tensor:
    return _result(lambda: torch.empty_like(x))


def rscc_rows(n: int, s: int, seed: int) -> np.ndarray:
    out = np.zeros(min(n, s), np.int64)
    _check(_lib.bie_rscc_rows(n, s, ctypes.c_uint64(seed), out.ctypes.data_as(ctypes.c_void_p)))
    return out


def prof_enable(on: bool = True):
    _check(_lib.bie_prof_enable(int(on)))


def prof_read(kernel: int = 0, columns: bool = False):
    """(launches, total_ms[, columns]) of a recorded kernel since the last read
    (0: packed symmetric product, 1: split-BF16 block product, 2: FP64 block
    product, 3: reduction of the packed product, 4: block GMRES basis dots, 5:
    block GMRES basis update); columns = summed right-hand sides of those launches
    (4: basis vector x column pairs; 5: basis vectors read)."""
    n = ctypes.c_int64(); ms = ctypes.c_double(); c = ctypes.c_int64()
    _check(_lib.bie_prof_read(int(kernel), ctypes.byref(n), ctypes.byref(ms), ctypes.byref(c)))
    return (n.value, ms.value, c.value) if columns else (n.value, ms.value)


def autotune(on: bool = True):
    """Autotuner on (default) or off (fixed launch shapes)."""
    _check(_lib.bie_autotune(int(on)))


def autotune_report() -> dict:
    """Launch shapes chosen so far: {key: [values]}."""
    n = int(_lib.bie_autotune_report(None, 0))
    buf = ctypes.create_string_buffer(n)
    _lib.bie_autotune_report(buf, n)
    out = {}
    for line in buf.value.decode().splitlines():
        parts = line.split()
        if parts:
            out[parts[0]] = [int(v) for v in parts[1:]]
    return out


@dataclass
class Solve:
    method: str = "gmres"
    restart: int = 30
    tol: float = 1e-6
    max_mvp: int = 10000
    crit: str = "scc"             # "scc", "rscc" or "ccc" (RSCC gates, SCC confirms)
    rscc_rows: int = 512
    rscc_seed: int = 1234
    precision: str = "plain"      # "plain" or "mixed" (FP32 inner GMRES + FP64 refinement)
    inner_tol: float = 0.0
    slots: int = 0                # mixed: right-hand sides in flight (continuous batch); 0 = all
    inner_terms: int = 0          # mixed, split-BF16: 3 or 2 terms of the inner block product; 0 = 3
    basis: str = "c64"            # mixed, split-BF16: inner Krylov basis "c64" or "f16" (FP16 pairs)
    block: int = 0                # method "bgmres": right-hand sides per block Krylov space (1..32); 0 = 32
    calderon: "Calderon | None" = None   # GMRES, precision "plain": right preconditioner built for the operator

    def c(self, use_x0: int) -> SolveOpts:
        return SolveOpts({"gmres": BIE_GMRES, "cgnr": BIE_CGNR, "bgmres": BIE_BGMRES}[self.method], self.restart, self.tol,
                         self.max_mvp, {"scc": BIE_SCC, "rscc": BIE_RSCC, "ccc": BIE_CCC}[self.crit], self.rscc_rows,
                         self.rscc_seed, int(use_x0), {"plain": 0, "mixed": 1}[self.precision],
                         self.inner_tol, self.slots, self.inner_terms, {"c64": 0, "f16": 1}[self.basis],
                         self.block, None if self.calderon is None else self.calderon._h)


class Operator:
    """Dense EFIE operator T of a closed PEC surface at wavenumber k (Sec. II)."""

    def __init__(self, V, T, k: float, storage: str = "c128", near_factor: float = 2.0,
                 keep_fp64: bool = False, star: bool = False, stream=None):
        """star: store the star-split form T_A' = jk T_A and V' = V/(jk) (Sec. VI-A);
        products are T_A' x + Sigma V' Sigma^T x."""
        V, pv = _host(V, np.float64)
        T, pt = _host(T, np.int32)
        opts = FillOpts({"c128": BIE_C128, "c64": BIE_C64, "split_bf16": BIE_SPLIT_BF16}[storage], near_factor,
                        int(keep_fp64), int(star))
        h = ctypes.c_void_p()
        _check(_lib.bie_op_create(pv, V.shape[0], pt, T.shape[0], float(k), ctypes.byref(opts),
                                  _stream(stream), ctypes.byref(h)))
        self._h = h
        self.k = float(k)
        self.storage = storage
        self.star = bool(star)
        self.N = int(_lib.bie_op_n(h))

    def close(self):
        if getattr(self, "_h", None):
            _lib.bie_op_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def edges(self) -> np.ndarray:
        out = np.zeros((self.N, 4), np.int32)
        _check(_lib.bie_op_edges(self._h, out.ctypes.data_as(ctypes.c_void_p)))
        return out

    def near_pairs(self) -> np.ndarray:
        n = int(_lib.bie_op_near_pairs(self._h, None, 0))
        out = np.zeros((n, 2), np.int32)
        _lib.bie_op_near_pairs(self._h, out.ctypes.data_as(ctypes.c_void_p), n)
        return out

    def matrix(self, dtype=torch.complex128, stream=None) -> torch.Tensor:
        out = _empty((self.N, self.N), dtype)
        code = BIE_C128 if dtype == torch.complex128 else BIE_C64
        _check(_lib.bie_op_matrix(self._h, _dev(out, dtype), code, _stream(stream)))
        return out

    def rhs(self, dirs, pols, stream=None) -> torch.Tensor:
        d, pd = _host(np.atleast_2d(dirs), np.float64)
        p, pp = _host(np.atleast_2d(pols), np.float64)
        R = d.shape[0]
        B = _empty((R, self.N), torch.complex128)
        _check(_lib.bie_rhs_planewave(self._h, pd, pp, R, _dev(B, torch.complex128), _stream(stream)))
        return B

    def apply(self, X: torch.Tensor, conj: bool = False, out: torch.Tensor | None = None, stream=None,
              block: bool | str = False):
        """Y = T X (or T^H X).  block=True or "bf16": complex128 vectors through the
        split-BF16 block product on the matrix cores (storage "split_bf16");
        block="fp64": the FP64 block product on the matrix cores."""
        X2 = X.reshape(-1, self.N)
        Y = _empty_like(X2) if out is None else out
        if block == "fp64":
            code = BIE_APPLY_F64_BLOCK
        elif block:
            code = BIE_SPLIT_BF16
        else:
            code = BIE_C128 if X2.dtype == torch.complex128 else BIE_C64
        _check(_lib.bie_apply(self._h, _dev(X2, X2.dtype), _dev(Y, X2.dtype, X2.shape), X2.shape[0], code,
                              int(conj), _stream(stream)))
        return Y.reshape(X.shape)

    def solve(self, B: torch.Tensor, opts: Solve | None = None, x0: torch.Tensor | None = None,
              stream=None, out: torch.Tensor | None = None, x0_fallback: bool = False):
        """Solve T X = B; x0: initial guesses (x0_fallback: a guess no better than
        zero, ||b - T x0|| >= ||b||, is replaced by zero inside the solve)."""
        opts = opts or Solve()
        B2 = B.reshape(-1, self.N)
        R = B2.shape[0]
        if out is not None:
            X = out
        elif x0 is not None:
            X = x0.reshape(-1, self.N).clone()
        else:
            X = _empty_like(B2)
        if x0 is not None and out is not None:
            X.copy_(x0.reshape(-1, self.N))
        st = (SolveStat * R)()
        co = opts.c(0 if x0 is None else (2 if x0_fallback else 1))
        rc = _lib.bie_solve(self._h, _dev(B2, torch.complex128), _dev(X, torch.complex128, B2.shape), R,
                            ctypes.byref(co), st, _stream(stream))
        _check(rc, allow_nc=True)
        return X.reshape(B.shape), [s.as_dict() for s in st]

    def farfield(self, X: torch.Tensor, obs, stream=None) -> torch.Tensor:
        X2 = X.reshape(-1, self.N)
        o, po = _host(np.atleast_2d(obs), np.float64)
        F = _empty((X2.shape[0], o.shape[0], 3), torch.complex128)
        _check(_lib.bie_farfield(self._h, _dev(X2, torch.complex128), X2.shape[0], po, o.shape[0],
                                 _dev(F, torch.complex128), _stream(stream)))
        return F

    def rcs(self, X: torch.Tensor, obs, stream=None) -> torch.Tensor:
        """Bistatic RCS (m^2) for unit-amplitude incidence (bie_rcs): R x M, device."""
        X2 = X.reshape(-1, self.N)
        o, po = _host(np.atleast_2d(obs), np.float64)
        S = _empty((X2.shape[0], o.shape[0]), torch.float64)
        _check(_lib.bie_rcs(self._h, _dev(X2, torch.complex128), X2.shape[0], po, o.shape[0],
                            _dev(S, torch.float64), _stream(stream)))
        return S


class Calderon:
    """Multiplicative Calderon preconditioner M = -G^{-1} T_BC G^{-T} of an
    operator (bie_calderon_create): pass it as Solve(calderon=...) to run GMRES
    on T M u = b, x = M u."""

    def __init__(self, op: Operator, stream=None):
        h = ctypes.c_void_p()
        _check(_lib.bie_calderon_create(op._h, _stream(stream), ctypes.byref(h)))
        self._h = h
        self.op = op            # the operator must outlive the preconditioner
        self.N = op.N

    def apply(self, X: torch.Tensor, out: torch.Tensor | None = None, stream=None) -> torch.Tensor:
        """Y = M X for complex128 vectors (rows of X)."""
        X2 = X.reshape(-1, self.N)
        Y = _empty_like(X2) if out is None else out
        _check(_lib.bie_calderon_apply(self._h, _dev(X2, torch.complex128), _dev(Y, torch.complex128, X2.shape),
                                       X2.shape[0], _stream(stream)))
        return Y.reshape(X.shape)

    def info(self) -> dict:
        i = CalderonInfo()
        _check(_lib.bie_calderon_get_info(self._h, ctypes.byref(i)))
        return dict(N=i.N, Nb=i.Nb, nnz_bc=i.nnz_bc, nnz_gram=i.nnz_gram, cg_iters=list(i.cg_iters),
                    cg_relres=list(i.cg_relres), setup_ms=i.setup_ms)

    def close(self):
        if getattr(self, "_h", None):
            _lib.bie_calderon_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class FastOperator(Operator):
    """The paper's fast operator (bie_op_create_fast): near entries between the
    RWG functions of near leaf cubes, stored sparse, plus the multilevel B-spline
    far field; no dense matrix.  apply() and solve() (GMRES, plain precision,
    SCC) as for Operator."""

    def __init__(self, V, T, k: float, box: float, levels: int, s: int, p: int = 3, near_factor: float = 2.0,
                 stream=None):
        V, pv = _host(V, np.float64)
        T, pt = _host(T, np.int32)
        o = FastOpts(float(box), int(levels), int(s), int(p), float(near_factor))
        h = ctypes.c_void_p()
        _check(_lib.bie_op_create_fast(pv, V.shape[0], pt, T.shape[0], float(k), ctypes.byref(o), _stream(stream),
                                       ctypes.byref(h)))
        self._h = h
        self.k = float(k)
        self.storage = "fast"
        self.star = False
        self.N = int(_lib.bie_op_n(h))

    def fast_info(self) -> dict:
        i = FastInfo()
        _check(_lib.bie_op_fast_info(self._h, ctypes.byref(i)))
        return dict(near_entries=i.near_entries, leaf_cubes=i.leaf_cubes, levels=i.levels)


class FarFieldML:
    """Multilevel far field of an operator (bie_farml_create): knot-insertion
    transfers between the octree levels, FFT translations; apply() gives Z~_far X
    for the pairs of far leaf cubes."""

    def __init__(self, op: Operator, box: float, levels: int, s: int, p: int = 3, stream=None):
        h = ctypes.c_void_p()
        o = FarMLOpts(float(box), int(levels), int(s), int(p))
        _check(_lib.bie_farml_create(op._h, ctypes.byref(o), _stream(stream), ctypes.byref(h)))
        self._h = h
        self.op = op
        self.N = op.N
        self.levels = int(levels)

    def apply(self, X: torch.Tensor, out: torch.Tensor | None = None, stream=None) -> torch.Tensor:
        X2 = X.reshape(-1, self.N)
        Y = _empty_like(X2) if out is None else out
        _check(_lib.bie_farml_apply(self._h, _dev(X2, torch.complex128), _dev(Y, torch.complex128, X2.shape),
                                    X2.shape[0], _stream(stream)))
        return Y.reshape(X.shape)

    def level_info(self, level: int) -> dict:
        i = FarInfo()
        _check(_lib.bie_farml_level_info(self._h, int(level), ctypes.byref(i)))
        return dict(boxes=i.boxes, far_pairs=i.far_pairs, buffer_knots=i.buffer_knots, splines=i.splines,
                    points_per_axis=i.points_per_axis, protrusion=i.protrusion, origin=list(i.origin))

    def close(self):
        if getattr(self, "_h", None):
            _lib.bie_farml_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class FarField:
    """Single-level far field of an operator by B-spline interpolation of g
    (bie_far_create): apply() gives Z~_far X for the pairs of far cubes."""

    def __init__(self, op: Operator, box: float, s: int, p: int = 3, stream=None):
        h = ctypes.c_void_p()
        o = FarOpts(float(box), int(s), int(p))
        _check(_lib.bie_far_create(op._h, ctypes.byref(o), _stream(stream), ctypes.byref(h)))
        self._h = h
        self.op = op
        self.N = op.N

    def apply(self, X: torch.Tensor, out: torch.Tensor | None = None, stream=None) -> torch.Tensor:
        X2 = X.reshape(-1, self.N)
        Y = _empty_like(X2) if out is None else out
        _check(_lib.bie_far_apply(self._h, _dev(X2, torch.complex128), _dev(Y, torch.complex128, X2.shape),
                                  X2.shape[0], _stream(stream)))
        return Y.reshape(X.shape)

    def info(self) -> dict:
        i = FarInfo()
        _check(_lib.bie_far_get_info(self._h, ctypes.byref(i)))
        return dict(boxes=i.boxes, far_pairs=i.far_pairs, buffer_knots=i.buffer_knots, splines=i.splines,
                    points_per_axis=i.points_per_axis, protrusion=i.protrusion, origin=list(i.origin))

    def boxes(self) -> np.ndarray:
        out = np.zeros((self.N, 3), np.int32)
        _check(_lib.bie_far_boxes(self._h, out.ctypes.data_as(ctypes.c_void_p)))
        return out

    def close(self):
        if getattr(self, "_h", None):
            _lib.bie_far_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def batch_solve(ops, Bs, opts: Solve | None = None, x0s=None, x0_fallback: bool = False, stream=None,
                pcs=None):
    """Solve T_p X_p = B_p for several operators at once (bie_batch_solve):
    grouped products, one captured graph per restart cycle.  pcs: one Calderon
    preconditioner per operator (bie_batch_solve_pc).  Returns the list of
    solutions and the list of per-operator statistics lists."""
    opts = opts or Solve()
    if opts.calderon is not None:
        raise ValueError("batched solves take their preconditioners per operator (pcs=...)")
    P = len(ops)
    Bs = [b.reshape(-1, op.N) for b, op in zip(Bs, ops)]
    R = np.array([b.shape[0] for b in Bs], np.int64)
    if x0s is not None:
        Xs = [x.reshape(-1, op.N).clone() for x, op in zip(x0s, ops)]
    else:
        Xs = [_empty_like(b) for b in Bs]
    oph = (ctypes.c_void_p * P)(*[op._h.value for op in ops])
    bp = (ctypes.c_void_p * P)(*[_dev(b, torch.complex128).value for b in Bs])
    xp = (ctypes.c_void_p * P)(*[_dev(x, torch.complex128, b.shape).value for x, b in zip(Xs, Bs)])
    st = (SolveStat * int(max(1, R.sum())))()
    use = 0 if x0s is None else (2 if x0_fallback else 1)
    co = opts.c(use)
    if pcs is None:
        rc = _lib.bie_batch_solve(oph, P, bp, xp, R.ctypes.data_as(ctypes.c_void_p), ctypes.byref(co), st,
                                  _stream(stream))
    else:
        if len(pcs) != P:
            raise ValueError("one preconditioner per operator")
        pch = (ctypes.c_void_p * P)(*[pc._h.value for pc in pcs])
        rc = _lib.bie_batch_solve_pc(oph, pch, P, bp, xp, R.ctypes.data_as(ctypes.c_void_p), ctypes.byref(co), st,
                                     _stream(stream))
    _check(rc, allow_nc=True)
    out, k = [], 0
    for r in R:
        out.append([st[k + i].as_dict() for i in range(int(r))])
        k += int(r)
    return Xs, out


_BATCH_MAT = {"fp64": 0, "fp32": 1, "fp32_mfma": 2, "fp64_mfma": 3}


def batch_apply(ops, Xs, mat: str = "fp64", unit_tiles: int = 0, cols_per_item: int = 0, stream=None):
    """Y_p = T_p X_p for several operators in one grouped launch
    (bie_batch_apply).  mat: "fp64" (FP64 tiles), "fp32" (FP32 tiles, vector
    units), "fp32_mfma" (FP32 tiles on the matrix cores) or "fp64_mfma" (FP64
    tiles on the FP64 matrix cores).  Returns the list of
    products (R_p x N_p complex128 each)."""
    if mat not in _BATCH_MAT:
        raise ValueError(f"mat must be one of {sorted(_BATCH_MAT)}")
    P = len(ops)
    Xs = [x.reshape(-1, op.N) for x, op in zip(Xs, ops)]
    R = np.array([x.shape[0] for x in Xs], np.int64)
    Ys = [_empty_like(x) for x in Xs]
    oph = (ctypes.c_void_p * P)(*[op._h.value for op in ops])
    xp = (ctypes.c_void_p * P)(*[_dev(x, torch.complex128).value for x in Xs])
    yp = (ctypes.c_void_p * P)(*[_dev(y, torch.complex128, x.shape).value for y, x in zip(Ys, Xs)])
    _check(_lib.bie_batch_apply(oph, P, xp, yp, R.ctypes.data_as(ctypes.c_void_p), _BATCH_MAT[mat], int(unit_tiles),
                                int(cols_per_item), _stream(stream)))
    return Ys


def batch_config(unit_tiles: int = 0, graph: bool = True, matrix_cores: bool = True):
    """Tiles per unit of the grouped product (0: autotune; -1: each operator's own
    single-product units, bitwise equal to single solves), graph replay, and the
    FP32 matrix cores for the grouped products of precision-1 batches."""
    _check(_lib.bie_batch_config(int(unit_tiles), int(graph), int(matrix_cores)))


def batch_tuned(ops, R) -> int:
    oph = (ctypes.c_void_p * len(ops))(*[op._h.value for op in ops])
    Rv = np.ascontiguousarray(R, np.int64)
    return int(_lib.bie_batch_tuned(oph, len(ops), Rv.ctypes.data_as(ctypes.c_void_p)))


def features(dirs, pol_flags):
    """Network inputs (d_x, d_y, d_z, s): propagation direction and +1 (theta-hat) / -1 (phi-hat)."""
    d = np.atleast_2d(np.asarray(dirs, np.float64))
    f = np.asarray(pol_flags, np.float64).reshape(-1, 1)
    return np.ascontiguousarray(np.concatenate([d, f], axis=1))


class WarmStart:
    """Learned warm start: POD basis + MLP (bie_ws_* in include/bie.h)."""

    def __init__(self, op: Operator, handle):
        self.op = op
        self._h = handle
        K = ctypes.c_int64(); H = ctypes.c_int64(); n = ctypes.c_int64()
        sc = ctypes.c_double(); loss = ctypes.c_double()
        _check(_lib.bie_ws_info(self._h, ctypes.byref(K), ctypes.byref(H), ctypes.byref(n), ctypes.byref(sc),
                                ctypes.byref(loss), None))
        self.K, self.H, self.nparams = K.value, H.value, n.value
        self.scale, self.final_loss = sc.value, loss.value

    @classmethod
    def train(cls, op: Operator, feats, X: torch.Tensor, pod_rank=256, hidden=512, epochs=3000, batch=256,
              lr_max=1e-3, lr_min=1e-5, seed=555, oversample=32, power_iters=2, pols=None, pol_model=0,
              stream=None):
        f, pf = _host(feats, np.float64)
        pp = None
        if pols is not None:
            e, pp = _host(pols, np.float64)
        X2 = X.reshape(-1, op.N)
        o = WsOpts(pod_rank, hidden, epochs, batch, lr_max, lr_min, seed, oversample, power_iters, pol_model)
        h = ctypes.c_void_p()
        _check(_lib.bie_ws_train(op._h, pf, pp, _dev(X2, torch.complex128), X2.shape[0], ctypes.byref(o),
                                 _stream(stream), ctypes.byref(h)))
        ws = cls(op, h)
        ws.pol_model = pol_model
        return ws

    @classmethod
    def create(cls, op: Operator, pod_rank=256, hidden=512, seed=555, pol_model=0):
        h = ctypes.c_void_p()
        _check(_lib.bie_ws_create(op._h, pod_rank, hidden, ctypes.c_uint64(seed), pol_model, ctypes.byref(h)))
        return cls(op, h)

    @classmethod
    def load(cls, op: Operator, path: str):
        h = ctypes.c_void_p()
        _check(_lib.bie_ws_load(op._h, path.encode(), ctypes.byref(h)))
        return cls(op, h)

    def save(self, path: str):
        _check(_lib.bie_ws_save(self._h, path.encode()))

    def close(self):
        if getattr(self, "_h", None):
            _lib.bie_ws_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def sigma(self) -> np.ndarray:
        out = np.zeros(self.K)
        _check(_lib.bie_ws_info(self._h, None, None, None, None, None, out.ctypes.data_as(ctypes.c_void_p)))
        return out

    def basis(self, stream=None) -> torch.Tensor:
        U = _empty((self.K, self.op.N), torch.complex128)
        _check(_lib.bie_ws_basis(self._h, _dev(U, torch.complex128), _stream(stream)))
        return U

    def params(self) -> np.ndarray:
        p = np.zeros(self.nparams, np.float32)
        _check(_lib.bie_ws_params(self._h, p.ctypes.data_as(ctypes.c_void_p), 0))
        return p

    def set_params(self, p):
        p = np.ascontiguousarray(p, np.float32)
        _check(_lib.bie_ws_params(self._h, p.ctypes.data_as(ctypes.c_void_p), 1))

    def loss_grad(self, feats, targets, pols=None):
        f, pf = _host(feats, np.float64)
        t, pt = _host(targets, np.float32)
        pp = None
        if pols is not None:
            e, pp = _host(pols, np.float64)
        g = np.zeros(self.nparams, np.float32)
        loss = ctypes.c_double()
        _check(_lib.bie_ws_loss_grad(self._h, pf, pp, pt, f.shape[0], ctypes.byref(loss),
                                     g.ctypes.data_as(ctypes.c_void_p)))
        return loss.value, g

    @property
    def outputs(self) -> int:
        """Network outputs: 2K, or 6K for the linear-in-polarisation model."""
        H = self.H
        return (self.nparams - 6 * H - H * H) // (H + 1)

    def fit(self, feats, targets, epochs: int, batch: int, lr_max: float = 1e-3, lr_min: float = 1e-5,
            seed: int = 555, pols=None, stream=None) -> float:
        """Train on given inputs and targets (S x 2K) with the library's kernels
        (bie_ws_fit); returns the mean squared error of the last epoch."""
        f, pf = _host(feats, np.float64)
        t, pt = _host(targets, np.float32)
        pp = None
        if pols is not None:
            e, pp = _host(pols, np.float64)
        loss = ctypes.c_double()
        _check(_lib.bie_ws_fit(self._h, pf, pp, pt, f.shape[0], int(epochs), int(batch), float(lr_max),
                               float(lr_min), ctypes.c_uint64(seed), ctypes.byref(loss), _stream(stream)))
        return loss.value

    def forward(self, feats) -> np.ndarray:
        f, pf = _host(feats, np.float64)
        out = np.zeros((f.shape[0], self.outputs), np.float32)
        _check(_lib.bie_ws_forward(self._h, pf, f.shape[0], out.ctypes.data_as(ctypes.c_void_p)))
        return out

    def predict(self, feats, B: torch.Tensor | None = None, pols=None, stream=None):
        """x0 (R x N complex128) and which predictions were kept (fallback to 0 when
        ||b - T x0|| >= ||b||; all kept when B is None)."""
        f, pf = _host(feats, np.float64)
        pp = None
        if pols is not None:
            e, pp = _host(pols, np.float64)
        R = f.shape[0]
        X0 = _empty((R, self.op.N), torch.complex128)
        used = np.zeros(R, np.int32)
        pb = None if B is None else _dev(B.reshape(R, self.op.N), torch.complex128)
        _check(_lib.bie_ws_predict(self._h, pf, pp, R, pb, _dev(X0, torch.complex128),
                                   used.ctypes.data_as(ctypes.c_void_p), _stream(stream)))
        return X0, used.astype(bool)
