"""Which kernel a matmul runs, asked of the library on the host: tests name the kernel that
they are about, so that a retuned dispatch rule cannot move them to another one unnoticed."""
import ctypes
from typing import NamedTuple

from oracle import ssq_oracle as O
from paper_2607_08779_amd import ssq

KERNELS = ("gemv", "exact", "rounded", "stat", "split", "tile", "gemm", "q8_gemv", "q8_tile")


class Route(NamedTuple):
    kernel: str
    tokens: int      # of a workgroup
    rows: int        # weight rows of a workgroup ("stat": row tiles of a run)
    slices: int      # of K


def route(M, N, K, group, q, mode, workspace=False, q8=False, aligned=True):
    """`workspace`: with one of ssq_matmul_workspace_size() bytes."""
    fn = ssq.lib().ssq_internal_route
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 4 + [ctypes.c_size_t, ctypes.c_int, ctypes.c_int * 4]
    out = (ctypes.c_int * 4)()
    kind = {O.ASYM: 1, O.ASYM_MIN: 2}.get(mode, 0)
    room = ssq.ssq_matmul_workspace_size(M, N, K, group, q) if workspace else 0
    st = fn(M, N, K, group, q, kind, int(aligned), room, int(q8), out)
    assert st == 0, ssq.ssq_strerror(st)
    return Route(KERNELS[out[0]], *list(out)[1:])
