"""The library's choice of kernel for a product, asked from the built library on the host (no GPU): the functions of
paper_2407_00952_amd/csrc that its own launches ask."""
import ctypes
from ctypes import c_bool, c_int, c_size_t

from paper_2407_00952_amd import binding as B

STORE, RESID, GELU, DGELU, STORE_DELTA = range(5)        # epilogues (csrc/common.h)


class TilePlan(ctypes.Structure):
    _fields_ = [("tm", c_int), ("tn", c_int), ("splits", c_int)]


class SplitPlan(ctypes.Structure):
    _fields_ = [("shared", c_bool), ("most_rows", c_int), ("bytes", c_size_t)]


def _fn(name, res, *args):
    f = getattr(B.lib(), name)
    f.restype, f.argtypes = res, args
    return f


def tile(M, N, K, epi=STORE, nz=0, can_split=False, nseg=1, whole=True):
    """(rows, columns, blocks that share a tile's contraction) of a bf16 product with nseg segments of N / nseg columns"""
    p = _fn("plan_gemm_tile", TilePlan, *[c_int] * 6, c_bool, c_bool)(M, N // nseg, nseg, K, epi, nz, can_split, whole)
    return p.tm, p.tn, p.splits


def split(M, N, K, nz=16):
    p = _fn("plan_gemm_split", SplitPlan, c_int, c_int, c_int, c_int)(M, N, K, nz)
    return p.shared, p.most_rows, p.bytes


def layer(T, n_in, n_out):
    """the plans of a bf16 LoRA layer's two products: forward, input gradient"""
    return [tile(T, n, k, nz=16, can_split=split(T, n, k)[0]) for n, k in ((n_out, n_in), (n_in, n_out))]
