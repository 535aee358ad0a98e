"""The library's choice of kernel for a product, asked from the built library on the host (no GPU): the functions of
paper_2407_00952_amd/csrc that its own launches ask."""
import ctypes
from ctypes import c_bool, c_int, c_size_t

from paper_2407_00952_amd import binding as B

STORE, RESID, GELU, DGELU, STORE_DELTA = range(5)        # epilogues (csrc/common.h)


class TilePlan(ctypes.Structure):
    _fields_ = [("tm", c_int), ("tn", c_int), ("splits", c_int), ("pair", c_int)]

    def form(self):
        return (self.tm, self.tn) + (("pair",) if self.pair else ())


class SplitPlan(ctypes.Structure):
    _fields_ = [("shared", c_bool), ("most_rows", c_int), ("bytes", c_size_t)]


def _fn(name, res, *args):
    f = getattr(B.lib(), name)
    f.restype, f.argtypes = res, args
    return f


def tile(M, N, K, epi=STORE, nz=0, can_split=False, nseg=1, whole=True):
    """((rows, columns[, "pair"]), blocks that share a tile's contraction) of a bf16 product with nseg segments of N / nseg columns"""
    p = _fn("plan_gemm_tile", TilePlan, *[c_int] * 6, c_bool, c_bool)(M, N // nseg, nseg, K, epi, nz, can_split, whole)
    return p.form(), p.splits


def split(M, N, K, nz=16):
    p = _fn("plan_gemm_split", SplitPlan, c_int, c_int, c_int, c_int)(M, N, K, nz)
    return p.shared, p.most_rows, p.bytes


def layer(T, n_in, n_out):
    """the plans of a bf16 LoRA layer's two products: forward, input gradient"""
    return [tile(T, n, k, nz=16, can_split=split(T, n, k)[0]) for n, k in ((n_out, n_in), (n_in, n_out))]


class F32Plan(ctypes.Structure):
    _fields_ = [("tm", c_int), ("tn", c_int), ("stages", c_int)]


def mx(M, N, K, nseg=1, epi=STORE, low_rank=False):
    """(rows, columns) of a product with fp8 weights"""
    p = _fn("plan_gemm_mx", TilePlan, *[c_int] * 5, c_bool)(M, N // nseg, nseg, K, epi, low_rank)
    return p.tm, p.tn


def mx_layer(T, n_in, n_out):
    return [mx(T, n_out, n_in, low_rank=True), mx(T, n_in, n_out, low_rank=True)]


def f32_layer(T, n_in, n_out):
    """(rows, columns, pairs of waves or ring stages of the kernel on bf16 pieces, or 0) of an fp32 layer's two products, on aligned
    operands"""
    f = _fn("plan_f32", F32Plan, c_int, c_int, c_int, c_bool)
    plan = [f(T, n_out, n_in, n_in % 4 == 0), f(T, n_in, n_out, n_in % 4 == 0 and n_out % 4 == 0)]
    return [(p.tm, p.tn, p.stages) for p in plan]


def stack(T, d, f, proj, seq_len, fp8=False):
    """{(epilogue, rank-space columns, rows, columns)} of the eight products of a block"""
    on = {p: p in proj for p in "q k v o fc pr".split()}
    qkv = sum(on[p] for p in "qkv")
    ad = lambda p: 16 if on[p] else 0
    delta = STORE_DELTA if seq_len <= 512 and not on["o"] else STORE
    prods = [(STORE, 16 if qkv else 0, 3 * d, d, 3), (RESID, ad("o"), d, d, 1), (GELU, ad("fc"), f, d, 1),
             (RESID, ad("pr"), d, f, 1), (DGELU, ad("pr"), f, d, 1), (STORE, ad("fc"), d, f, 1),
             (delta, ad("o"), d, d, 1), (STORE, 16 * qkv, d, 3 * d, 1)]
    return {(epi, nz) + (mx(T, N, K, nseg, epi, nz > 0) if fp8 else tile(T, N, K, epi, nz, nseg=nseg)[0])
            for epi, nz, N, K, nseg in prods}


def one_pass(T, jobs, r, width):
    """whether rank-space gradients of `jobs` adapters and their dB come from one pass over a gradient of that width"""
    return _fn("rank_grad_fills", c_bool, c_int, c_int, c_int, c_int)(T, jobs, r, width)


def counted(M, N, K):
    """(rows, columns) of a plain store over counted rows on a kernel that computes all M, None for the one that counts"""
    p = _fn("plan_gemm_counted", TilePlan, c_int, c_int, c_int)(M, N, K)
    return p.form() if p.tm else None
