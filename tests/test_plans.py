"""The cases of the GPU tests reach the kernels that they are there for: the library's own choice for each, asked on the host.  A
change of a cost table that moves a case to another kernel fails here."""
import plans
import test_gpu_linear as linear
import test_gpu_loss_head as head
import test_gpu_mx as mx
import test_gpu_stack as stack
import test_zz_no_alloc as no_alloc
from paper_2407_00952_amd import synth

BF16_FORMS = {(32, 32), (32, 64), (64, 64), (64, 128), (128, 128), (192, 128), (256, 128), (128, 256), (256, 256)}
FP8_FORMS = {(32, 64), (64, 64), (64, 128), (128, 128), (192, 128), (256, 128), (256, 256)}


def test_fp32_tile_forms():
    for case, (which, want) in linear.FP32_TILE_FORMS.items():
        fwd, bwd = plans.f32_layer(*case)
        assert (fwd if which == "forward" else bwd) == want, case
    for which in ("forward", "input gradient"):
        assert {f for w, f in linear.FP32_TILE_FORMS.values() if w == which} == {
            (32, 64, 4), (64, 48, 4), (64, 64, 4), (64, 64, 2), (128, 128, 2)}
    for case, want in linear.FP32_PRECISION.items():
        assert plans.f32_layer(*case)[0] == want, case
    for case, want in linear.FP32_INFINITY.items():
        assert tuple(plans.f32_layer(*case)) == want, case


def test_fp32_split_forms():
    for (T, n_in, n_out, _, _), want in linear.FP32_SPLIT.items():
        assert tuple(plans.f32_layer(T, n_in, n_out)) == want, (T, n_in, n_out)


def test_bf16_forms():
    for (T, n_in, n_out), want in linear.FROZEN_FORMS.items():
        assert plans.tile(T, n_out, n_in) == (want, 1), (T, n_in, n_out)
    assert set(linear.FROZEN_FORMS.values()) == BF16_FORMS | {(128, 128, "pair")}
    for case, want in linear.LAYER_FORMS.items():
        assert plans.layer(*case)[0] == (want, 1), case
    assert set(linear.LAYER_FORMS.values()) == BF16_FORMS - {(128, 256)}


def test_pair_forms():
    """up to the rows of which the pair form takes all at once, other forms take fewer"""
    for T, n_in, n_out in ((10803, 64, 4040), (2100, 192, 3080), (2900, 640, 2568)):
        assert plans.tile(T, n_out, n_in)[0] == (128, 128, "pair"), (T, n_in, n_out)
        assert len({plans.tile(rows, n_out, n_in)[0] for rows in (1, 33, 200, 450, 1090, 1500, 2000)} - {(128, 128, "pair")}) >= 3
    assert plans.tile(10803, 4040, 64, epi=plans.RESID)[0] != (128, 128, "pair") != plans.tile(10803, 4040, 64, nz=16)[0]
    assert plans.tile(13197, 2520, 768)[0] != (128, 128, "pair")             # 12 slabs


def test_shared_contractions():
    for case, want in linear.SHARED.items():
        assert tuple(p[1] for p in plans.layer(*case)) == want, case
    for case, want in no_alloc.SHARED.items():
        assert plans.layer(*case)[1][1] == want, case
    assert {w[0] for w in linear.SHARED.values()} == {w[1] for w in linear.SHARED.values()} == {1, 2, 3, 4}


def test_fp8_forms():
    for (T, K, N), want in mx.FP8_FORMS.items():
        assert plans.mx(T, N, K) == want, (T, K, N)
    assert set(mx.FP8_FORMS.values()) == FP8_FORMS
    for case, want in mx.FP8_LAYER_FORMS.items():
        assert tuple(plans.mx_layer(*case)) == want, case


def test_stacks_reach_every_form_and_epilogue():
    """every (epilogue, rank-space columns, form) that any batch of up to 200 sequences of the test's stack would run on is run on
    by its batches; and what that leaves out of the forms altogether"""
    d, f, S = (stack.FORM_STACK[k] for k in ("d_model", "d_ff", "seq_len"))
    for (dtype, proj), sizes in stack.FORM_BATCHES.items():
        reached, possible = ([plans.stack(n * S, d, f, proj, S, dtype == "mxfp8") for n in ns] for ns in (sizes, range(1, 201)))
        assert set().union(*reached) == set().union(*possible), (dtype, proj)
        forms = {p[2:] for p in set().union(*reached)}
        if dtype == "mxfp8":
            assert forms == FP8_FORMS
        else:                                            # 128 x 256 has no rank-space branch
            assert forms == BF16_FORMS - ({(128, 256)} if proj == synth.PROJ_NAMES else set())


def test_batches_of_the_wider_stack():
    forms = lambda n, S, proj: {p[2:] for p in plans.stack(n * S, 768, 3072, proj, S)}
    for proj in ((), synth.PROJ_NAMES):
        assert {(32, 64), (64, 128)} <= forms(1, 512, proj) <= {(32, 64), (64, 64), (64, 128)}
        assert forms(3, 512, proj) == {(64, 128), (128, 128), (192, 128)}
        assert forms(11, 512, proj) == {(192, 128), (256, 256)}
    for proj in (("q", "v"), synth.PROJ_NAMES):
        assert forms(1, 128, proj) == {(32, 32), (32, 64)} and forms(33, 128, proj) == {(128, 128), (256, 256)}
        assert set().union(*(forms(n, 128, proj) for n in (1, 2, 4, 8, 16, 24, 33))) == BF16_FORMS - {(128, 256)}


def test_stacks_of_the_rank_gradient_pass():
    """input gradients of the adapted projections on 256 x 256 tiles, where the rank-space tail is, behind a pass; of a client's tokens
    on other tiles, without one"""
    for name, (d, f, r, proj, batch) in stack.AHEAD.items():
        n = sum(p in proj for p in "qkv")
        prods = {"pr": (f, d, plans.DGELU, 16, 1), "fc": (d, f, plans.STORE, 16, 1), "o": (d, d, plans.STORE, 16, 1)}
        prods = [v for k, v in prods.items() if k in proj] + ([(d, 3 * d, plans.STORE, 16 * n, n)] if n else [])
        for N, K, epi, nz, jobs in prods:
            few = name == "rank 16" and jobs == 1        # (113 blocks: only q, k and v together are enough)
            assert plans.one_pass(320 * batch, jobs, r, K) != few and not plans.one_pass(64 * batch, jobs, r, K), (name, N, K)
            assert plans.tile(320 * batch, N, K, epi, nz)[0] == (256, 256) != plans.tile(64 * batch, N, K, epi, nz)[0], (name, N, K)
    for (T, r, width), want in mx.ONE_PASS.items():
        assert plans.one_pass(T, 1, r, width) == want, (T, r, width)


def test_logits_of_a_loss_head():
    """all rows are computed where 512 tiles of 128 x 128 or fewer hold them, and up to 128 rows; elsewhere they are counted"""
    for (T, d, V), want in head.LOGIT_FORMS.items():
        assert plans.counted(T, -(-V // 64) * 64, d) == want, (T, d, V)
    for d in (64, 768, 1280, 2048):
        for T in (1, 64, 128, 129, 256, 300, 600, 1000, 1500, 4096, 16384):
            for Vp in (64, 1024, 1344, 4288, 8000, 12032, 20032, 31168, 50304, 65536):
                few = T <= 128 or -(-T // 128) * -(-Vp // 128) <= 512
                plan = plans.counted(T, Vp, d)
                assert (plan is not None) == few and (not few or plan == plans.tile(T, Vp, d, whole=T <= 128)[0]), (T, Vp, d)


def test_short_contractions():
    """one to six slabs over many rows: a small tile's price is not the line through the long contractions alone"""
    for T, K, N in ((10803, 128, 4224), (20820, 128, 1024), (13197, 256, 4320), (20820, 256, 2048), (8192, 384, 4320), (8192, 512, 4696),
                    (8192, 1024, 3072), (20820, 1024, 1024)):           # (and eight, without a low-rank branch)
        assert plans.mx(T, N, K) == (256, 256), (T, K, N)
    for T, K, N in ((20820, 64, 3072), (13197, 64, 4320), (20820, 128, 3072), (13197, 192, 4320), (20820, 192, 4696)):
        assert plans.tile(T, N, K)[0] in ((256, 256), (128, 256), (128, 128, "pair")), (T, K, N)
