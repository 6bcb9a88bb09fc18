"""ctypes binding of the C ABI declared in include/cheb.h (argument marshalling only).

The shared library ``libchebfft.so`` is built in-tree by
``paper_2606_21410_amd.csrc.build``; importing the binding fails loudly when it
is missing -- there is no fallback implementation.
"""
from __future__ import annotations

import ctypes
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libchebfft.so")

CHEB_OK = 0
CHEB_NOT_CONVERGED = 1
CHEB_STAGNATED = 2
CHEB_ERR_INVALID_ARG = -1
CHEB_ERR_SINGULAR_BC = -2
CHEB_ERR_BAD_INPUT = -3
CHEB_ERR_DEVICE = -4
CHEB_ERR_WORKSPACE = -5
CHEB_ERR_UNSUPPORTED = -6

CHEB_F64, CHEB_F32, CHEB_MIXED = 0, 1, 2
CHEB_DIRICHLET, CHEB_NEUMANN = 0, 1
CHEB_APPLY_FULL, CHEB_APPLY_REDUCED, CHEB_APPLY_TRANSPOSE = 0, 1, 2
CHEB_ROUTE_AUTO, CHEB_ROUTE_FFT, CHEB_ROUTE_MATRIX = 0, 1, 2


class cheb_grid(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int32 * 3), ("lo", ctypes.c_double * 3),
                ("hi", ctypes.c_double * 3), ("bc", ctypes.c_int32 * 6),
                ("robin", ctypes.c_double * 6)]


class cheb_solve_opts(ctypes.Structure):
    _fields_ = [("rtol", ctypes.c_double), ("atol", ctypes.c_double),
                ("maxiter", ctypes.c_int32), ("inner_m", ctypes.c_int32),
                ("outer_k", ctypes.c_int32), ("ir_inner_rtol", ctypes.c_double),
                ("ir_max_outer", ctypes.c_int32), ("flags", ctypes.c_int32),
                ("history", ctypes.POINTER(ctypes.c_double)), ("history_len", ctypes.c_int32),
                ("reserved", ctypes.c_int32 * 3)]


class cheb_solve_info(ctypes.Structure):
    _fields_ = [("status", ctypes.c_int32), ("matvecs", ctypes.c_int32),
                ("matvecs_f32", ctypes.c_int32), ("restarts", ctypes.c_int32),
                ("ir_steps", ctypes.c_int32), ("history_used", ctypes.c_int32),
                ("relres_final", ctypes.c_double), ("seconds", ctypes.c_double)]

    def as_dict(self):
        return {k: getattr(self, k) for k, _ in self._fields_}


_vp = ctypes.c_void_p
_SIGS = {
    "cheb_plan_create": (ctypes.c_int, [ctypes.POINTER(cheb_grid), ctypes.c_int32, _vp, ctypes.POINTER(_vp)]),
    "cheb_plan_workspace_bytes": (ctypes.c_int, [_vp, ctypes.POINTER(cheb_solve_opts),
                                                 ctypes.POINTER(ctypes.c_size_t)]),
    "cheb_plan_set_workspace": (ctypes.c_int, [_vp, _vp, ctypes.c_size_t]),
    "cheb_plan_set_stream": (ctypes.c_int, [_vp, _vp]),
    "cheb_plan_set_route": (ctypes.c_int, [_vp, ctypes.c_int32]),
    "cheb_plan_set_robin_nodes": (ctypes.c_int, [_vp, _vp]),
    "cheb_plan_set_tile_shape": (ctypes.c_int, [_vp, ctypes.c_int32, ctypes.c_int32]),
    "cheb_plan_autotune": (ctypes.c_int, [_vp, ctypes.c_int32, _vp, _vp, _vp, ctypes.POINTER(ctypes.c_double),
                                          ctypes.c_int32]),
    "cheb_plan_destroy": (ctypes.c_int, [_vp]),
    "cheb_apply": (ctypes.c_int, [_vp, _vp, _vp, _vp, ctypes.c_uint32]),
    "cheb_apply_scratch": (ctypes.c_int, [_vp, _vp, _vp, _vp, ctypes.c_uint32, _vp]),
    "cheb_solve": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, ctypes.POINTER(cheb_solve_opts),
                                  ctypes.POINTER(cheb_solve_info)]),
    "cheb_prolong": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, ctypes.POINTER(ctypes.c_double)]),
    "cheb_prolong_noalloc": (ctypes.c_int, [_vp, _vp, _vp, _vp]),
    "cheb_refine": (ctypes.c_int, [ctypes.POINTER(_vp), ctypes.c_int32, ctypes.POINTER(_vp), ctypes.POINTER(_vp),
                                   ctypes.POINTER(_vp), ctypes.POINTER(_vp), _vp, ctypes.POINTER(cheb_solve_opts),
                                   ctypes.c_double, ctypes.POINTER(ctypes.c_double),
                                   ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(cheb_solve_info)]),
    "cheb_adjoint": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, _vp, ctypes.POINTER(cheb_solve_opts),
                                    ctypes.POINTER(cheb_solve_info)]),
    "cheb_picard": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_double, ctypes.c_int32,
                                   ctypes.POINTER(cheb_solve_opts), ctypes.POINTER(cheb_solve_info),
                                   ctypes.POINTER(ctypes.c_int32)]),
    "cheb_newton_work_bytes": (ctypes.c_int, [_vp, ctypes.POINTER(ctypes.c_size_t)]),
    "cheb_newton_residual": (ctypes.c_int, [_vp, _vp, ctypes.c_double, _vp, _vp, _vp, _vp]),
    "cheb_newton_jacobian": (ctypes.c_int, [_vp, _vp, ctypes.c_double, _vp, _vp, _vp, _vp]),
    "cheb_newton": (ctypes.c_int, [_vp, _vp, ctypes.c_double, _vp, _vp, _vp, _vp, ctypes.c_double,
                                   ctypes.c_int32, ctypes.POINTER(cheb_solve_opts),
                                   ctypes.POINTER(cheb_solve_info), ctypes.POINTER(ctypes.c_int32),
                                   ctypes.POINTER(ctypes.c_int32)]),
    "cheb_derivative": (ctypes.c_int, [_vp, _vp, _vp, ctypes.c_int32]),
    "cheb_flux_average": (ctypes.c_int, [_vp, _vp, _vp, ctypes.POINTER(ctypes.c_double)]),
    "cheb_precond_apply": (ctypes.c_int, [_vp, ctypes.c_int32, ctypes.c_double, _vp, _vp, ctypes.c_uint32]),
    "cheb_apparent_conductivity": (ctypes.c_int, [_vp, _vp, _vp, ctypes.c_int32, ctypes.c_double,
                                                  ctypes.POINTER(ctypes.c_double)]),
    "cheb_debug_copy": (ctypes.c_int, [_vp, _vp, ctypes.c_size_t, _vp]),
    "cheb_debug_gemm": (ctypes.c_int, [ctypes.c_int32, _vp, _vp, _vp, ctypes.c_int32, ctypes.c_int32,
                                       ctypes.c_int32, _vp]),
    "cheb_batch_create": (ctypes.c_int, [ctypes.POINTER(cheb_grid), ctypes.c_int32, ctypes.c_int32, _vp,
                                         ctypes.POINTER(_vp)]),
    "cheb_batch_workspace_bytes": (ctypes.c_int, [_vp, ctypes.POINTER(cheb_solve_opts),
                                                  ctypes.POINTER(ctypes.c_size_t)]),
    "cheb_batch_set_workspace": (ctypes.c_int, [_vp, _vp, ctypes.c_size_t]),
    "cheb_batch_set_stream": (ctypes.c_int, [_vp, _vp]),
    "cheb_batch_solve": (ctypes.c_int, [_vp, ctypes.POINTER(_vp), ctypes.POINTER(_vp), ctypes.POINTER(_vp),
                                        ctypes.POINTER(_vp), ctypes.POINTER(cheb_solve_opts),
                                        ctypes.POINTER(cheb_solve_info)]),
    "cheb_batch_tile_shapes": (ctypes.c_int, [_vp, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32), ctypes.c_int32]),
    "cheb_batch_destroy": (ctypes.c_int, [_vp]),
    "cheb_status_string": (ctypes.c_char_p, [ctypes.c_int]),
    "cheb_last_error": (ctypes.c_char_p, []),
}

_lib = None


def load() -> ctypes.CDLL:
    """Load libchebfft.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} not found: build it with `python -m paper_2606_21410_amd.csrc.build`")
    lib = ctypes.CDLL(LIB_PATH)
    for name, (res, args) in _SIGS.items():
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    _lib = lib
    return lib


class ChebError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"[{code}] {msg}")
        self.code = code


def check(rc: int) -> int:
    """Raise ChebError for hard errors (negative codes); return soft statuses."""
    if rc < 0:
        lib = load()
        raise ChebError(rc, f"{lib.cheb_status_string(rc).decode()}: {lib.cheb_last_error().decode()}")
    return rc


def declared_functions(header_path: str | None = None) -> list[str]:
    """Names of the functions a header under include/ declares (default cheb.h)."""
    import re
    if header_path is None:
        header_path = os.path.join(os.path.dirname(_HERE), "include", "cheb.h")
    text = open(header_path).read()
    return sorted(set(re.findall(r"^\s*(?:int|const char\*)\s+(cheb_\w+)\s*\(", text, re.M)))
