"""GPU parity of the single LoRA-adapted linear layer (SplitLoRA Sec. II-C) through the C ABI."""
import numpy as np
import pytest

from oracle import slora_oracle as so
from paper_2407_00952_amd import binding as B
from paper_2407_00952_amd import synth
from gpu_util import BF16_TOL, F32_TOL, norm_err, one_by_one, relerr, say

pytestmark = pytest.mark.gpu


def _run_f32(c):
    import torch
    T, n_in = c["x"].shape
    n_out, r = c["W"].shape[0], c["r"]
    dev = {k: torch.from_numpy(np.ascontiguousarray(c[k], dtype=np.float32)).cuda()
           for k in ("x", "W", "A", "B", "dy")}
    bias = None if c["b"] is None else torch.from_numpy(c["b"]).cuda()
    nws = B.slora_lora_linear_ws_bytes(B.DTYPE_F32, T, n_in, n_out, r)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    y = torch.empty((T, n_out), dtype=torch.float32, device="cuda")
    dx = torch.empty((T, n_in), dtype=torch.float32, device="cuda")
    dA = torch.empty((r, n_in), dtype=torch.float32, device="cuda")
    dB = torch.empty((n_out, r), dtype=torch.float32, device="cuda")
    B.slora_lora_linear_fwd(B.DTYPE_F32, T, n_in, n_out, r, c["alpha"], dev["x"], dev["W"], bias, dev["A"],
                            dev["B"], y, ws, nws)
    B.slora_lora_linear_bwd(B.DTYPE_F32, T, n_in, n_out, r, c["alpha"], dev["x"], dev["dy"], dev["W"], dev["A"],
                            dev["B"], dx, dA, dB, ws, nws)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (y, dx, dA, dB)]


def _run_bf16(c):
    import torch
    T, n_in = c["x"].shape
    n_out, r = c["W"].shape[0], c["r"]
    x, W, dy = (B.to_device_bf16(c[k]) for k in ("x", "W", "dy"))
    bias = None if c["b"] is None else B.to_device_bf16(c["b"])
    A = torch.from_numpy(c["A"]).cuda()
    Bm = torch.from_numpy(c["B"]).cuda()
    nws = B.slora_lora_linear_ws_bytes(B.DTYPE_BF16, T, n_in, n_out, r)
    assert nws > 0
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    y = torch.empty((T, n_out), dtype=torch.bfloat16, device="cuda")
    dx = torch.empty((T, n_in), dtype=torch.bfloat16, device="cuda")
    dA = torch.empty((r, n_in), dtype=torch.float32, device="cuda")
    dB = torch.empty((n_out, r), dtype=torch.float32, device="cuda")
    B.slora_lora_linear_fwd(B.DTYPE_BF16, T, n_in, n_out, r, c["alpha"], x, W, bias, A, Bm, y, ws, nws)
    torch.cuda.synchronize()
    B.slora_lora_linear_bwd(B.DTYPE_BF16, T, n_in, n_out, r, c["alpha"], x, dy, W, A, Bm, dx, dA, dB, ws, nws)
    torch.cuda.synchronize()
    return [B.from_device_bf16(y), B.from_device_bf16(dx), dA.cpu().numpy(), dB.cpu().numpy()]


def _oracle(c):
    s = c["alpha"] / c["r"]
    y, _ = so.lora_linear_fwd(c["x"], c["W"], c["b"], c["A"], c["B"], s)
    dx, dA, dB = so.lora_linear_bwd(c["x"], c["dy"], c["W"], c["A"], c["B"], s)
    return [y, dx, dA, dB]


def test_workload1_fp32():
    """x [1024,768], W [768,768], r = 4, alpha = 32: y, dx, dA, dB within 1e-4 of the fp64 oracle."""
    c = synth.make_single_layer()
    say("fp32 single layer 1024x768x768 r=4")
    got, ref = _run_f32(c), _oracle(c)
    for name, g, r in zip(("y", "dx", "dA", "dB"), got, ref):
        e = relerr(g, r)
        say("   %s rel err %.2e" % (name, e))
        assert e <= F32_TOL, (name, e)


@pytest.mark.parametrize("T,n_in,n_out,r,bias", [(100, 72, 40, 1, True), (257, 64, 200, 16, False)])
def test_fp32_ragged_shapes(T, n_in, n_out, r, bias):
    c = synth.make_single_layer(T, n_in, n_out, r, seed=7 + T, bias=bias)
    say("fp32 single layer", T, n_in, n_out, r)
    for name, g, ref in zip(("y", "dx", "dA", "dB"), _run_f32(c), _oracle(c)):
        assert relerr(g, ref) <= F32_TOL, name


# Where the fp32 products change kernel, and ragged edges on both sides of each line: tiles on bf16 pieces where rows are whole float4s
# and the contraction whole 64s (or 16 x 16 outputs per block, where a cost in us says so), otherwise 16 x 16 outputs per block up to
# 95 tiles of 64 x 64, 64 x 64 tiles up to 511 tiles of 128 x 128, and those.
# Sums of up to 16 400 fp32 products in whatever order: 1e-4 is the bar of the fp32 path.
@pytest.mark.parametrize("T,n_in,n_out,r,bias", [
    (1, 768, 768, 4, True),
    (17, 1280, 1288, 5, False),
    (500, 768, 704, 2, False),       # 32 x 64 tiles, ragged rows
    (333, 259, 130, 3, True),        # odd rows, 16 x 16 outputs per block
    (700, 331, 1027, 9, True),       # odd rows, 64 x 64 tiles forward, 16 x 16 back
    (8200, 64, 1030, 16, True),      # 128 x 128 tiles on a ring forward, odd columns; 64 x 64 tiles back
    (16400, 512, 36, 4, False),      # 64 x 64 tiles, two to a CU, forward; 516 tiles of 128 x 128 in the input gradient
])
def test_fp32_dispatch_edges(T, n_in, n_out, r, bias):
    c = synth.make_single_layer(T, n_in, n_out, r, seed=17 + T, bias=bias)
    say("fp32 single layer", T, n_in, n_out, r)
    for name, g, ref in zip(("y", "dx", "dA", "dB"), _run_f32(c), _oracle(c)):
        assert relerr(g, ref) <= F32_TOL, name


# The forms of the kernel on bf16 pieces (contraction a multiple of 64), forward (W as [n, k]) and input gradient (W as [k, n]), with
# ragged rows and columns; 64 is one stage of the contraction.  (The other product of each layer has a contraction that is no
# multiple of 64.)  T, n_in, n_out: which product, and its tile and the last argument of its kernel (tests/test_plans.py).
FP32_TILE_FORMS = {
    (601, 768, 700): ("forward", (32, 64, 4)), (601, 700, 768): ("input gradient", (32, 64, 4)),
    (601, 768, 836): ("forward", (64, 48, 4)), (601, 836, 768): ("input gradient", (64, 48, 4)),
    (1001, 768, 764): ("forward", (64, 48, 4)), (1001, 764, 768): ("input gradient", (64, 48, 4)),
    (1001, 1024, 1020): ("forward", (64, 64, 4)), (1001, 1020, 1024): ("input gradient", (64, 64, 4)),
    (2101, 192, 764): ("forward", (64, 64, 2)), (2101, 764, 192): ("input gradient", (64, 64, 2)),       # two to a CU
    (3900, 320, 1020): ("forward", (128, 128, 2)), (3900, 1020, 320): ("input gradient", (128, 128, 2)),
    (3900, 64, 1028): ("forward", (64, 64, 2)),      # one stage of the contraction
}


@pytest.mark.parametrize("T,n_in,n_out", list(FP32_TILE_FORMS))
def test_fp32_tile_forms(T, n_in, n_out):
    test_fp32_dispatch_edges(T, n_in, n_out, 5, True)


# The adapter gradients of up to 4 columns take a half-wave's rows 16, 4 and 1 at a time (32 half-waves): none, one and several of
# each, half-waves with and without the last row.
@pytest.mark.parametrize("T", [1, 31, 32, 97, 128, 129, 480, 481, 512, 513, 1000, 1024, 1185])
def test_fp32_adapter_gradient_rows(T):
    test_fp32_dispatch_edges(T, 72, 40, 3, False)


# The low-rank term may not cost the fp32 product precision: error (2-norm, against fp64) of y no larger than that of the sums
# taken one after the other, the frozen product and the low-rank one each on its own (the 5 % cover the sample: some 1e5
# independent roundings).  Short contractions, where 16 more roundings at the size of the result show most.
# A low-rank term that is small beside the frozen product, and one that is larger.
# T, n_in, n_out: tile and the last argument of its kernel.
FP32_PRECISION = {(20, 16, 768): (16, 16, 0), (700, 32, 704): (64, 64, 0), (8200, 16, 1030): (128, 128, 0), (700, 64, 704): (32, 64, 4)}


@pytest.mark.parametrize("boost", [1, 30])
@pytest.mark.parametrize("T,n_in,n_out", list(FP32_PRECISION))
def test_fp32_low_rank_term_costs_no_precision(T, n_in, n_out, boost):
    c = synth.make_single_layer(T, n_in, n_out, 16, seed=23 + T, bias=True)
    c["B"] = c["B"] * np.float32(boost)
    rows = slice(0, min(T, 256))
    f32, f64 = np.float32, np.float64
    s = c["alpha"] / c["r"]
    x = c["x"][rows]
    plain = one_by_one(x, c["W"]) + c["b"]
    plain = plain + f32(s) * one_by_one(one_by_one(x, c["A"]), c["B"])
    got = _run_f32(c)[0][rows]
    x, W, A, Bm = (v.astype(f64) for v in (x, c["W"], c["A"], c["B"]))
    ref = x @ W.T + c["b"].astype(f64) + s * (x @ A.T) @ Bm.T
    e_got, e_plain = norm_err(got, ref), norm_err(plain, ref)
    say("fp32 layer", T, n_in, n_out, boost, "error %.3e, one by one %.3e, ratio %.3f" % (e_got, e_plain, e_got / e_plain))
    assert e_got <= 1.05 * e_plain


FP32_INFINITY = {(20, 64, 96): ((16, 16, 0),) * 2, (700, 768, 704): ((32, 64, 4), (64, 48, 4)),
                 (700, 780, 716): ((64, 64, 0),) * 2, (8200, 100, 1028): ((128, 128, 0), (64, 64, 0)),
                 (3900, 320, 1020): ((128, 128, 2), (64, 64, 0)), (3900, 1020, 320): ((64, 64, 0), (128, 128, 2))}


@pytest.mark.parametrize("T,n_in,n_out", list(FP32_INFINITY))
def test_fp32_infinity_stays_an_infinity(T, n_in, n_out):
    # rank 3 is kept as 4 columns: the empty one must not turn inf * 0 into a NaN of the result
    c = synth.make_single_layer(T, n_in, n_out, 3, seed=5, bias=False)
    for k in ("W", "A", "B"):
        c[k] = np.abs(c[k]) + np.float32(1e-3)
    c["x"][7, 5] = c["dy"][9, 11] = np.inf
    say("fp32 layer with an infinity", T, n_in, n_out)
    y, dx = _run_f32(c)[:2]
    assert np.all(y[7] == np.inf) and np.all(dx[9] == np.inf)
    assert np.isfinite(np.delete(y, 7, 0)).all() and np.isfinite(np.delete(dx, 9, 0)).all()


# A sum that is formed again because an operand is infinite, or has no bf16 neighbour but infinity (3.39e38 and above), leaves the
# sums beside it alone: the same bits as without that operand, in every form of the kernel on bf16 pieces and both directions.
@pytest.mark.parametrize("value", [np.inf, 3.4e38])
@pytest.mark.parametrize("T,n_in,n_out", list(FP32_TILE_FORMS))
def test_fp32_sums_do_not_depend_on_their_neighbours(T, n_in, n_out, value):
    c = synth.make_single_layer(T, n_in, n_out, 5, seed=19 + T, bias=True)
    for k in ("W", "A", "B"):
        c[k] = c[k] * np.float32(1e-3)
    y, dx = _run_f32(c)[:2]
    say("fp32 layer with one", value, T, n_in, n_out)
    rows = dict(c, x=c["x"].copy(), dy=c["dy"].copy())   # an element of a row each
    rows["x"][7, 5] = rows["dy"][9, 11] = value
    y1, dx1 = _run_f32(rows)[:2]
    assert not np.array_equal(y1[7], y[7]) and not np.array_equal(dx1[9], dx[9])
    assert np.array_equal(np.delete(y1, 7, 0), np.delete(y, 7, 0)) and np.array_equal(np.delete(dx1, 9, 0), np.delete(dx, 9, 0))
    cols = dict(c, W=c["W"].copy())                      # of a column of either product
    cols["W"][13, 6] = value
    y2, dx2 = _run_f32(cols)[:2]
    assert not np.array_equal(y2[:, 13], y[:, 13]) and not np.array_equal(dx2[:, 6], dx[:, 6])
    assert np.array_equal(np.delete(y2, 13, 1), np.delete(y, 13, 1)) and np.array_equal(np.delete(dx2, 6, 1), np.delete(dx, 6, 1))


# Operands times powers of two are sums times powers of two, bit by bit, while nothing rounds at the edge of the range: x and dy at
# 2^-118, where a bf16 piece of 16 bits less would be no normal number, against W at 2^60; W at 2^-118 against x and dy at 2^60; and
# subnormal ones at 2^-140.
@pytest.mark.parametrize("tiny", ["x", "W", "subnormal x", "subnormal W"])
@pytest.mark.parametrize("T,n_in,n_out", list(FP32_TILE_FORMS))
def test_fp32_tiny_operands_keep_their_bits(T, n_in, n_out, tiny):
    c = synth.make_single_layer(T, n_in, n_out, 5, seed=29 + T, bias=False)
    down = -140 if "subnormal" in tiny else -118
    ex = {k: down if tiny.endswith("x") == (k != "W") else 60 - down - 118 for k in ("x", "dy", "W")}
    for k in ("x", "dy") if tiny.endswith("x") else ("W",):         # whole multiples of 2^-149 there
        c[k] = np.ldexp(np.round(np.ldexp(c[k].astype(np.float64), 149 + down + (k == "W") * 5)), -149 - down).astype(np.float32)
    z = 40 if ex["x"] < 0 else -60                       # (the rank-space activations between 2^-100 and 2^22)
    ex["A"], ex["B"] = z, ex["W"] - z                    # (both terms of a result in one scale)
    t = dict(c)
    for k, e in ex.items():
        t[k] = np.ldexp(c[k], e).astype(np.float32)
        assert np.array_equal(np.ldexp(t[k].astype(np.float64), -e), c[k]), k
    say("fp32 layer, tiny", tiny, T, n_in, n_out, ex)
    (y, dx), (ty, tdx) = _run_f32(c)[:2], _run_f32(t)[:2]
    for name, got, want, e in (("y", ty, y, ex["x"] + ex["W"]), ("dx", tdx, dx, ex["dy"] + ex["W"])):
        want = np.ldexp(want, e).astype(np.float32)
        assert np.array_equal(got, want), (name, relerr(got, want))


# The products on three bf16 pieces an operand: fewer k-steps than waves, ragged tiles, an adapter that is not 16-byte aligned
# (projection in a launch of its own), backward projections in the product's launch (rank up to 8) and not (16); and numbers
# that bf16 rounds to an infinity, whose sums are formed again.  T, n_in, n_out, r, floats the adapter is off by: forms of
# the two products (tests/test_plans.py).
FP32_SPLIT = {
    (300, 64, 2052, 4, 0): ((64, 48, 4), (16, 16, 0)),
    (97, 1024, 1536, 16, 1): ((32, 64, 4), (32, 64, 4)),
    (300, 576, 1152, 8, 0): ((32, 64, 4), (32, 64, 4)),
    (300, 1152, 576, 16, 0): ((32, 64, 4), (32, 64, 4)),
    (2050, 192, 772, 5, 0): ((64, 64, 2), (64, 64, 0)),
    (2100, 384, 1984, 3, 0): ((64, 64, 2), (64, 64, 4)),
    (4100, 256, 1988, 2, 0): ((128, 128, 2), (64, 64, 0)),
    (4100, 1988, 256, 6, 0): ((64, 64, 0), (128, 128, 2)),
}


@pytest.mark.parametrize("huge", [False, True])
@pytest.mark.parametrize("T,n_in,n_out,r,off", list(FP32_SPLIT))
def test_fp32_split_products(T, n_in, n_out, r, off, huge):
    import torch
    c = synth.make_single_layer(T, n_in, n_out, r, seed=31 + T, bias=True)
    if huge:                                             # (3.39e38 and above have no bf16 neighbour but infinity)
        for k in ("W", "A", "B"):
            c[k] = c[k] * np.float32(1e-3)
        c["x"][T // 2, 3] = c["dy"][T // 3, 5] = np.float32(3.4e38)
    flat = torch.empty(r * n_in + off, dtype=torch.float32, device="cuda")
    A = flat[off:].view(r, n_in)
    A.copy_(torch.from_numpy(c["A"]))
    x, W, dy, bias, Bm = (torch.from_numpy(c[k]).cuda() for k in ("x", "W", "dy", "b", "B"))
    nws = B.slora_lora_linear_ws_bytes(B.DTYPE_F32, T, n_in, n_out, r)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    y, dx, dA, dB = (torch.empty(s, dtype=torch.float32, device="cuda") for s in ((T, n_out), (T, n_in), (r, n_in), (n_out, r)))
    say("fp32 split", T, n_in, n_out, r, off, huge)
    B.slora_lora_linear_fwd(B.DTYPE_F32, T, n_in, n_out, r, c["alpha"], x, W, bias, A, Bm, y, ws, nws)
    B.slora_lora_linear_bwd(B.DTYPE_F32, T, n_in, n_out, r, c["alpha"], x, dy, W, A, Bm, dx, dA, dB, ws, nws)
    torch.cuda.synchronize()
    # element by element: no more roundings of half an ulp (of the sum of magnitudes) than 6 sums for 32 products, each
    # with up to 3 more inside the instruction, and 32 for the pieces left out, the low-rank term, the bias and the waves
    a = {k: np.abs(c[k].astype(np.float64)) for k in ("x", "dy", "W", "A", "B")}
    s = c["alpha"] / c["r"]
    size = [a["x"] @ a["W"].T + np.abs(c["b"]) + s * (a["x"] @ a["A"].T) @ a["B"].T, a["dy"] @ a["W"] + s * (a["dy"] @ a["B"]) @ a["A"],
            s * (a["dy"] @ a["B"]).T @ a["x"], s * a["dy"].T @ (a["x"] @ a["A"].T)]
    sums = [24 * n_in / 32, 24 * n_out / 32, 24 * n_out / 32 + T, 24 * n_in / 32 + T]
    for name, got, ref, m, n in zip(("y", "dx", "dA", "dB"), (y, dx, dA, dB), _oracle(c), size, sums):
        got = got.cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all(), name
        assert (np.abs(got - ref) <= (n + 32) * 2.0 ** -24 * m).all(), (name, np.max(np.abs(got - ref) / m) * 2 ** 24)
    if huge:
        return
    # and no further from the sums in 64 bits than a fused multiply-add for each product in turn (5 % for the sample, 1e5 roundings
    # or so): 1.4e-7 at a contraction of 64, 7e-7 at 1536, where one of the six products left out is 2.4e-6 (test_oracle_linear.py)
    f32 = np.float32
    p, z = one_by_one(c["dy"], c["B"].T), one_by_one(c["x"], c["A"])
    rows = slice(0, 64)
    plain = [one_by_one(c["x"][rows], c["W"]) + c["b"] + f32(s) * one_by_one(z[rows], c["B"]),
             one_by_one(c["dy"][rows], c["W"].T) + f32(s) * one_by_one(p[rows], c["A"].T),
             f32(s) * one_by_one(p.T, c["x"].T), f32(s) * one_by_one(c["dy"].T, z.T)]
    for name, got, ref, one in zip(("y", "dx", "dA", "dB"), (y, dx, dA, dB), _oracle(c), plain):
        n = one.shape[0]
        e_got, e_plain = norm_err(got[:n].cpu().numpy(), ref[:n]), norm_err(one, ref[:n])
        say("   %s error %.2e, one by one %.2e" % (name, e_got, e_plain))
        assert e_got <= 1.05 * e_plain, (name, e_got, e_plain)


def test_fp32_zero_B_is_bitwise_base():
    import torch
    c = synth.make_single_layer(300, 128, 192, 4, seed=11)
    c0 = dict(c); c0["B"] = np.zeros_like(c["B"])
    y_lora = _run_f32(c0)[0]
    # base layer: W only, expressed through the same call with A = 0 as well
    c1 = dict(c0); c1["A"] = np.zeros_like(c["A"])
    y_base = _run_f32(c1)[0]
    assert np.array_equal(y_lora, y_base)
    assert relerr(y_base, c["x"].astype(np.float64) @ c["W"].astype(np.float64).T) <= F32_TOL


@pytest.mark.parametrize("T,n_in,n_out,r,bias", [
    (1024, 768, 768, 4, False),      # workload 1 shapes, bf16 path
    (700, 320, 448, 3, True),        # ragged row tile, column tile and rank
    (256, 64, 64, 16, True),         # one tile, full rank
    (1300, 1024, 3072, 8, True),     # several column tiles
    (64, 128, 128, 1, False),
    (512, 768, 768, 2, True),        # the remaining ranks of the paper's sweep r in {1, 2, 4, 8} (Sec. IV)
    (512, 768, 2304, 8, False),
    # 133 chunks of 128 tokens, the last one ragged: nine for each wavefront of the adapter-gradient reduction (the body with
    # eight loads in flight, and its tail), seven for the 15th, none for the last
    (16960, 256, 64, 4, True),
    (16960, 64, 256, 16, False),
    # both sides of tokens x the wider side = 2^24, where chunks of 128 tokens become chunks of 512 (for both gradients): 128 short
    # chunks, the last one ragged; 33 long ones, the last of 16 tokens, three for each of 11 wavefronts (tail only)
    (16383, 1024, 64, 4, False),
    (16400, 1024, 64, 4, True),
    (16400, 64, 1024, 16, False),
    (700, 19840, 640, 4, False),     # scratch with 512-token partial sums only, the last one ragged
])
def test_bf16_layer(T, n_in, n_out, r, bias):
    c = synth.make_single_layer(T, n_in, n_out, r, seed=100 + T + r, quant=True, bias=bias)
    c["B"] = synth.round_bf16(c["B"] * 10)       # make the low-rank term visible next to x W^T
    say("bf16 single layer", T, n_in, n_out, r)
    got, ref = _run_bf16(c), _oracle(c)
    for name, g, rf in zip(("y", "dx", "dA", "dB"), got, ref):
        e = relerr(g, rf)
        say("   %s rel err %.2e" % (name, e))
        assert e <= BF16_TOL, (name, e)


# chunks of 128 tokens: 31 (4 waves of the reduction share them), 32 and 33 (16 waves; the last of 11 with 33), 49, 160
@pytest.mark.parametrize("T", [3968, 3969, 4096, 4097, 6145, 20480])
def test_bf16_adapter_gradient_chunks(T):
    c = synth.make_single_layer(T, 64, 128, 3, seed=53, quant=True)
    c["B"] = synth.round_bf16(c["B"] * 10)
    _, _, dA, dB = _run_bf16(c)
    _, _, rdA, rdB = _oracle(c)
    say("bf16 gradient chunks", T, relerr(dA, rdA), relerr(dB, rdB))
    # (each chunk is one of up to 160 equal parts of the sum: one left out or read twice is an error of 1/sqrt(160) = 8e-2 or more)
    assert relerr(dA, rdA) <= BF16_TOL and relerr(dB, rdB) <= BF16_TOL


def test_bf16_zero_B_is_bitwise_base():
    c = synth.make_single_layer(512, 256, 320, 4, seed=21, quant=True, bias=True)
    c0 = dict(c); c0["B"] = np.zeros_like(c["B"])
    c1 = dict(c0); c1["A"] = np.zeros_like(c["A"])
    y_lora, dx_lora = _run_bf16(c0)[:2]
    y_base, dx_base = _run_bf16(c1)[:2]
    assert np.array_equal(y_lora, y_base) and np.array_equal(dx_lora, dx_base)


# The frozen product on its own (Sec. II-C without the adapter), the stack's products that have no rank-space branch with the
# plain-store epilogue.  One k-slab, an odd number of slabs, ragged row and column tiles, a single row, with and without bias.
@pytest.mark.parametrize("T,n_in,n_out,bias", [
    (700, 320, 448, True),
    (1, 64, 8, True),
    (257, 64, 264, False),
    (300, 704, 320, True),
    (1300, 1024, 3072, False),
    (4096, 4096, 1024, True),
])
def test_frozen_linear_bf16(T, n_in, n_out, bias):
    import torch
    c = synth.make_single_layer(T, n_in, n_out, 1, seed=300 + T + n_in, quant=True, bias=bias)
    x, W = B.to_device_bf16(c["x"]), B.to_device_bf16(c["W"])
    b = None if c["b"] is None else B.to_device_bf16(c["b"])
    y = torch.empty((T, n_out), dtype=torch.bfloat16, device="cuda")
    B.slora_frozen_linear_bf16(T, n_in, n_out, x, W, b, y)
    torch.cuda.synchronize()
    ref, _ = so.lora_linear_fwd(c["x"], c["W"], c["b"], np.zeros_like(c["A"]), np.zeros_like(c["B"]), 1.0)
    e = relerr(B.from_device_bf16(y), ref)
    say("frozen linear", T, n_in, n_out, "rel err %.2e" % e)
    # fp32 accumulation and one rounding to bf16: half a bf16 ulp of the largest output
    assert e <= 2.0 ** -8


# Products with ragged rows and columns and one or an odd number of slabs.
@pytest.mark.parametrize("T,n_in,n_out,bias", [
    (1, 1152, 64, True),             # one row
    (130, 2432, 72, False),          # columns past a tile
    (300, 1216, 776, True),
    (1020, 64, 2040, True),          # one slab
    (1030, 192, 2040, False),        # three
    (2050, 320, 2056, True),         # five
])
def test_frozen_linear_dispatch_edges(T, n_in, n_out, bias):
    import torch
    c = synth.make_single_layer(T, n_in, n_out, 1, seed=400 + T + n_in, quant=True, bias=bias)
    x, W = B.to_device_bf16(c["x"]), B.to_device_bf16(c["W"])
    b = None if c["b"] is None else B.to_device_bf16(c["b"])
    y = torch.full((T, n_out), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.slora_frozen_linear_bf16(T, n_in, n_out, x, W, b, y)
    torch.cuda.synchronize()
    ref, _ = so.lora_linear_fwd(c["x"], c["W"], c["b"], np.zeros_like(c["A"]), np.zeros_like(c["B"]), 1.0)
    e = relerr(B.from_device_bf16(y), ref)
    say("frozen linear", T, n_in, n_out, "rel err %.2e" % e)
    assert e <= 2.0 ** -8                # as above: one rounding to bf16


# The tile forms of the bf16 products, each with ragged rows and columns and an odd number of slabs (forms with two slabs to
# a barrier end on a single one).  T, n_in, n_out: tile (tests/test_plans.py).
FROZEN_FORMS = {
    (70, 704, 776): (32, 32),
    (33, 192, 104): (32, 64),
    (200, 448, 4088): (64, 64),
    (450, 192, 3080): (64, 128),
    (1090, 320, 2056): (128, 128),
    (1500, 1088, 3080): (192, 128),
    (2000, 1088, 3080): (256, 128),
    (2100, 192, 3080): (128, 128, "pair"),
    (1818, 832, 4104): (128, 256),
    (3700, 192, 4104): (256, 256),
    (10803, 64, 4040): (128, 128, "pair"),       # one slab
}


@pytest.mark.parametrize("T,n_in,n_out", list(FROZEN_FORMS))
def test_frozen_linear_tile_forms(T, n_in, n_out):
    test_frozen_linear_dispatch_edges(T, n_in, n_out, True)


# A row's bits are the same on whichever form its call ran.
@pytest.mark.parametrize("T,n_in,n_out", [(10803, 64, 4040), (2100, 192, 3080), (2900, 640, 2568)])      # pair forms
def test_frozen_linear_rows_are_the_same_on_every_form(T, n_in, n_out):
    import torch
    c = synth.make_single_layer(T, n_in, n_out, 1, seed=450 + T, quant=True, bias=True)
    x, W, b = (B.to_device_bf16(c[k]) for k in ("x", "W", "b"))
    y = torch.empty((T, n_out), dtype=torch.bfloat16, device="cuda")
    B.slora_frozen_linear_bf16(T, n_in, n_out, x, W, b, y)
    for rows in (1, 33, 200, 450, 1090, 1500, 2000):
        part = torch.empty((rows, n_out), dtype=torch.bfloat16, device="cuda")
        B.slora_frozen_linear_bf16(rows, n_in, n_out, x, W, b, part)
        torch.cuda.synchronize()
        assert torch.equal(part, y[:rows]), rows


# The same with the rank-space branch (contraction n_in forward, n_out in the input gradient).  T, n_in, n_out: tile forward
# (and in the input gradient: whichever).
LAYER_FORMS = {
    (70, 704, 768): (32, 32),
    (130, 704, 2048): (32, 64),
    (200, 448, 4096): (64, 64),
    (450, 192, 3072): (64, 128),
    (1090, 320, 2048): (128, 128),
    (1400, 704, 3072): (192, 128),
    (2000, 1088, 3072): (256, 128),
    (2700, 192, 3072): (256, 256),
}


@pytest.mark.parametrize("T,n_in,n_out", list(LAYER_FORMS))
def test_bf16_layer_tile_forms(T, n_in, n_out):
    test_bf16_layer_dispatch_edges(T, n_in, n_out, (T // 10) % 16 + 1)


# Contractions long enough to be shared over blocks: T, n_in, n_out: blocks to a tile forward, in the input gradient.
SHARED = {
    (3, 5120, 128): (4, 1),          # two tiles of 64 x 64
    (130, 128, 5120): (1, 4),        # six
    (160, 4096, 1024): (3, 1),       # 48
    (160, 1024, 4096): (1, 3),
    (300, 3584, 832): (2, 1),        # 65
    (1024, 5120, 512): (2, 1),       # 128
    (2048, 256, 5120): (1, 2),
    (33, 4160, 2048): (4, 1),        # 65 slabs: shares of 16 and 17
}


@pytest.mark.parametrize("T,n_in,n_out", list(SHARED))
def test_bf16_layer_long_contractions_are_shared(T, n_in, n_out):
    r = T % 16 + 1
    test_bf16_layer_dispatch_edges(T, n_in, n_out, r)
    test_bf16_layer_shared_contraction_repeats_itself(T, n_in, n_out, r)


@pytest.mark.parametrize("T,n_in,n_out,r", [
    (3, 2432, 128, 16),              # one row of tiles, an odd number of slabs
    (130, 128, 2432, 3),             # the same in the input gradient
    (1100, 192, 1984, 5),            # odd number of slabs
    (260, 1216, 832, 2),
    (2100, 2048, 320, 8),
    (2048, 2048, 256, 4),
])
def test_bf16_layer_dispatch_edges(T, n_in, n_out, r):
    c = synth.make_single_layer(T, n_in, n_out, r, seed=500 + T + r, quant=True, bias=True)
    c["B"] = synth.round_bf16(c["B"] * 10)
    say("bf16 single layer", T, n_in, n_out, r)
    for name, g, rf in zip(("y", "dx", "dA", "dB"), _run_bf16(c), _oracle(c)):
        e = relerr(g, rf)
        say("   %s rel err %.2e" % (name, e))
        assert e <= BF16_TOL, (name, e)


# Products that share their contraction over blocks: the blocks of a tile finish in any order, and their sums are added in
# share order all the same; the counters are left as the next call expects them; nothing behind the workspace is written.
# (38 slabs here, which no launch shares: the same must hold.  SHARED has those that do.)
@pytest.mark.parametrize("T,n_in,n_out,r", [
    (3, 2432, 128, 16),
    (130, 128, 2432, 3),
])
def test_bf16_layer_shared_contraction_repeats_itself(T, n_in, n_out, r):
    import torch
    c = synth.make_single_layer(T, n_in, n_out, r, seed=600 + T + r, quant=True, bias=False)
    x, W, dy = (B.to_device_bf16(c[k]) for k in ("x", "W", "dy"))
    A, Bm = torch.from_numpy(c["A"]).cuda(), torch.from_numpy(c["B"]).cuda()
    nws = B.slora_lora_linear_ws_bytes(B.DTYPE_BF16, T, n_in, n_out, r)
    ws = torch.full((nws + 4096,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN in either type
    first = None
    for k in range(4):
        out = [torch.full(sh, float("nan"), dtype=dt, device="cuda") for sh, dt in
               (((T, n_out), torch.bfloat16), ((T, n_in), torch.bfloat16), ((r, n_in), torch.float32), ((n_out, r), torch.float32))]
        if k == 2:
            ws[:nws].fill_(0xFF)
        B.slora_lora_linear_fwd(B.DTYPE_BF16, T, n_in, n_out, r, c["alpha"], x, W, None, A, Bm, out[0], ws, nws)
        B.slora_lora_linear_bwd(B.DTYPE_BF16, T, n_in, n_out, r, c["alpha"], x, dy, W, A, Bm, *out[1:], ws, nws)
        torch.cuda.synchronize()
        assert all(bool(torch.isfinite(t).all()) for t in out)
        first = first or out
        assert all(torch.equal(a, b) for a, b in zip(out, first)), k
    assert bool((ws[nws:] == 0xFF).all())
