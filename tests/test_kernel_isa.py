"""Build-time checks of the compiled GEMM kernels (gfx950 assembly as hipcc emits it for the library's own
sources with the library's own flags; nothing runs on a GPU).

The 4-wave GEMM kernel writes its MFMAs as inline assembly, so the compiler no longer sees their data
hazards, and the GEMM sources write the M0 register behind the compiler's back for their asynchronous
global -> LDS copies.  What the source guarantees by construction is checked here in the instruction stream
of every instantiation, so that a compiler upgrade or a changed flag that breaks an assumption fails the
test suite instead of corrupting results:

  1. every MFMA of gemm_kernel4 accumulates in place in the accumulation registers (destination = addend,
     the form whose back-to-back dependency the hardware interlocks) and no two MFMAs use overlapping but
     different accumulator ranges;
  2. the same accumulator is not touched again by anything but its own MFMA inside the main loop (no copies
     in and out of the accumulation registers around the MFMAs);
  3. on every control-flow path from the last MFMA, at least 19 wait states (the requirement for the
     longest, 16-pass, matrix instruction; the 16x16x32 bf16 one needs fewer) pass before the first
     instruction other than an MFMA that reads or writes an accumulation register;
  4. M0 is written only by the copy sequence (s_mov_b32 m0 / s_nop 0 / global_load_lds_*) and read by
     nothing else, in every source whose kernels issue it;
  5. no vector memory instruction reads a scalar register that a vector instruction (v_readlane,
     v_readfirstlane, a compare, a carry) wrote fewer than 5 wait states earlier, vcc included.  The
     compiler keeps that distance for its own instructions but does not look into inline assembly, and the
     copies take their base address in scalar registers: a spilled scalar restored right in front of one
     would make it read a stale address.
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2407_00952_amd import build as libbuild

CSRC = libbuild.CSRC
MIN_WAIT_STATES = 19


def _assembly(src):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        cmd = ["hipcc", *[f for f in libbuild.FLAGS if f != "-fPIC"], "--cuda-device-only", "-S",
               os.path.join(CSRC, src), "-o", out]
        p = subprocess.run(cmd, capture_output=True, text=True)
        assert p.returncode == 0, p.stderr[-2000:]
        return open(out).read()


def _functions(text):
    """{mangled name: [instruction lines]} for every kernel in an assembly file (labels kept, comments dropped)."""
    funcs, name, body = {}, None, []
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
            continue
        if name is None:
            continue
        if line.startswith(".Lfunc_end"):
            funcs[name] = body
            name = None
            continue
        code = line.split(";")[0].rstrip()
        if not code.strip() or code.strip().startswith((".", "//")) and not re.match(r"^\.L\w+:", code.strip()):
            continue
        body.append(code.strip())
    return funcs


def _is_label(ins):
    return ins.endswith(":")


def _wait_states(ins):
    if _is_label(ins):
        return 0
    m = re.match(r"s_nop\s+(\d+)", ins)
    return int(m.group(1)) + 1 if m else 1


_AGPR = re.compile(r"\ba(\d+)\b|\ba\[(\d+):(\d+)\]")


def _agprs(ins):
    regs = set()
    for m in _AGPR.finditer(ins):
        if m.group(1) is not None:
            regs.add(int(m.group(1)))
        else:
            regs.update(range(int(m.group(2)), int(m.group(3)) + 1))
    return regs


@pytest.fixture(scope="module")
def gemm_asm():
    return _assembly("gemm.hip")


@pytest.fixture(scope="module")
def tile_asm():
    text = _assembly("gemm_tile.hip")
    assert sum("gemm_tile_kernel" in n for n in _functions(text)) == 33     # 11 epilogues and ranks x three tile forms
    assert sum("gemm_tile128_kernel" in n for n in _functions(text)) == 1   # plain store
    return text


def test_four_wave_gemm_mfma_hazards(gemm_asm):
    funcs = {n: b for n, b in _functions(gemm_asm).items() if "gemm_kernel4" in n}
    assert len(funcs) == 10, sorted(funcs)         # five epilogues x two tile heights
    _check_mfma_hazards(funcs)


def test_counted_gemm_mfma_hazards(gemm_asm):
    funcs = {n: b for n, b in _functions(gemm_asm).items() if "gemm_counted4" in n}
    assert len(funcs) == 3, sorted(funcs)          # plain store, and shared contraction x two tile heights
    _check_mfma_hazards(funcs)


def test_tail_gemm_mfma_hazards(gemm_asm):
    """the main loop of gemm_kernel4 and the rank-space tail behind it: MFMAs in place, nothing else on an accumulator inside
    either, and wait states behind the last of each before anything else reads one"""
    funcs = {n: b for n, b in _functions(gemm_asm).items() if "gemm_tail4" in n}
    assert len(funcs) == 2, sorted(funcs)          # plain store, saved GELU'
    for name, body in funcs.items():
        mf = [i for i, ins in enumerate(body) if ins.startswith("v_mfma")]
        assert len(mf) == 3 * 64, (name, len(mf))  # two k-steps of a slab, one of the tail
        for first, last in ((mf[0], mf[127]), (mf[128], mf[191])):
            acc = set()
            for ins in body[first:last + 1]:
                if ins.startswith("v_mfma"):
                    m = re.match(r"v_mfma_f32_16x16x32_bf16 a\[(\d+):(\d+)\], v\[\d+:\d+\], v\[\d+:\d+\], a\[(\d+):(\d+)\]$", ins)
                    assert m and m.group(1, 2) == m.group(3, 4) and int(m.group(1)) % 4 == 0, (name, ins)
                    acc.add(m.group(1))
                else:
                    assert not _agprs(ins), (name, ins)
            assert len(acc) == 64, name
            worst, where = _min_wait_states_to_acc_access(body, last)
            assert worst >= MIN_WAIT_STATES, (name, worst, where)
            # what the kernel spills (it has all 512 registers) stays out of both loops
            assert not any("scratch_" in ins for ins in body[first:last]), name
        # the tail's operands are zeroed by vector instructions; the main loop's come from LDS alone
        assert not _operands_too_close(body, "v_"), (name, _operands_too_close(body, "v_")[:2])


def _check_mfma_hazards(funcs):
    for name, body in funcs.items():
        ni = int(re.search(r"gemm_(?:kernel|counted)4ILi\d+ELi(\d+)E", name).group(1))      # 16-row MFMA tiles per wave along M
        assert ni in (4, 8), name
        mf = [(i, ins) for i, ins in enumerate(body) if ins.startswith("v_mfma")]
        # the unrolled loop body: 2 k-steps x (ni x 8) MFMAs
        assert len(mf) == 2 * 8 * ni, (name, len(mf))
        ranges = []
        for _, ins in mf:
            m = re.match(r"v_mfma_f32_16x16x32_bf16 a\[(\d+):(\d+)\], v\[\d+:\d+\], v\[\d+:\d+\], a\[(\d+):(\d+)\]$", ins)
            assert m, (name, ins)
            d0, d1, c0, c1 = map(int, m.groups())
            assert (d0, d1) == (c0, c1) and d1 - d0 == 3 and d0 % 4 == 0, (name, ins)      # (1) in place, aligned
            ranges.append(d0)
        # ni x 8 distinct accumulators per k-step, the same ones in both: a register is written again that many
        # MFMAs later at the earliest and ranges never overlap partially
        half = 8 * ni
        assert sorted(ranges[:half]) == sorted(ranges[half:]) and len(set(ranges[:half])) == half, name
        first, last = mf[0][0], mf[-1][0]
        # (2) nothing else touches an accumulation register between the first and the last MFMA
        for ins in body[first:last + 1]:
            if not ins.startswith("v_mfma"):
                assert not _agprs(ins), (name, ins)
        # (3) every path from the last MFMA to an access of an accumulation register that is not an MFMA
        worst, where = _min_wait_states_to_acc_access(body, last)
        assert worst >= MIN_WAIT_STATES, (name, worst, where)


def _min_wait_states_to_acc_access(body, start):
    """Follow every control-flow path from the instruction after body[start]; a path ends at the next MFMA
    (inside the loop nothing else touches the accumulators, check 2), at s_endpgm, or once it has collected
    the required wait states.  Returns the fewest wait states in front of any other instruction that reads
    or writes an accumulation register, and that instruction."""
    labels = {ins[:-1]: i for i, ins in enumerate(body) if _is_label(ins)}
    best = {}
    worst, where = 10 ** 9, None
    todo = [(start + 1, 0)]
    while todo:
        i, ws = todo.pop()
        while i < len(body):
            if ws >= MIN_WAIT_STATES or best.get(i, 10 ** 9) <= ws:
                break
            best[i] = ws
            ins = body[i]
            if ins.startswith("v_mfma") or ins.startswith("s_endpgm"):
                break
            if _agprs(ins):
                if ws < worst:
                    worst, where = ws, ins
                break
            m = re.match(r"s_(c?)branch\w*\s+(\S+)", ins)
            ws += _wait_states(ins)
            if m:
                assert m.group(2) in labels, ins
                todo.append((labels[m.group(2)], ws))
                if not m.group(1):                  # unconditional: no fall-through
                    break
            i += 1
    return (worst if where is not None else MIN_WAIT_STATES), where


def _check_m0(text, what):
    for name, body in _functions(text).items():
        code = [ins for ins in body if not _is_label(ins)]
        for i, ins in enumerate(code):
            if not re.search(r"\bm0\b", ins):
                continue
            if re.match(r"s_mov_b32 m0, (?:s\d+|vcc_lo|vcc_hi)$", ins):        # (a scalar may live in a half of vcc)
                assert code[i + 1] == "s_nop 0" and code[i + 2].startswith("global_load_lds_dword"), \
                    (what, name, code[i:i + 3])
            else:
                raise AssertionError("%s: %s: M0 used outside the copy sequence: %s" % (what, name, ins))
        # the copies read M0 implicitly: each one must be preceded by the write that belongs to it
        for i, ins in enumerate(code):
            if ins.startswith("global_load_lds_dword"):
                assert i >= 2 and code[i - 1] == "s_nop 0" and code[i - 2].startswith("s_mov_b32 m0,"), \
                    (what, name, code[max(i - 2, 0):i + 1])


def test_m0_is_only_used_by_the_async_copies(gemm_asm, tile_asm):
    _check_m0(gemm_asm, "gemm.hip")
    _check_m0(tile_asm, "gemm_tile.hip")
    _check_m0(_assembly("mx.hip"), "mx.hip")


_SREG = re.compile(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]|\b(vcc(?:_lo|_hi)?)\b")
_VCC = {"vcc": {"vcc_lo", "vcc_hi"}, "vcc_lo": {"vcc_lo"}, "vcc_hi": {"vcc_hi"}}
_VMEM = ("global_load", "global_store", "global_atomic", "buffer_load", "buffer_store", "scratch_load", "scratch_store")


def _sregs(text):
    regs = set()
    for m in _SREG.finditer(text):
        if m.group(1) is not None:
            regs.add(int(m.group(1)))
        elif m.group(4) is not None:
            regs |= _VCC[m.group(4)]
        else:
            regs.update(range(int(m.group(2)), int(m.group(3)) + 1))
    return regs


def _valu_scalar_dest(ins):
    """Scalar registers written by a vector instruction (empty for everything else): the first operand of lane reads and
    compares, the second of what leaves a carry or a scale flag."""
    op, _, args = ins.partition(" ")
    args = args.split(",")
    if op.startswith(("v_readlane_b32", "v_readfirstlane_b32", "v_cmp")):
        return _sregs(args[0])
    if re.match(r"v_(?:\w+_co_|div_scale_|mad_[ui]64_[ui]32)", op):
        return _sregs(args[1])
    return set()


def _salu_dest(ins):
    """Scalar registers written by a scalar arithmetic instruction: what a vector instruction before it left there (the carry
    of a multiply-add that nobody asked for) is not what is read behind it."""
    m = re.match(r"s_(?:mov|add|addc|sub|subb|mul|and|or|lshl|lshr|ashr|cselect)\w*\s+([^,]+),", ins)
    return _sregs(m.group(1)) if m else set()


def _check_valu_sgpr_to_vmem(text, what):
    for name, body in _functions(text).items():
        code = [ins for ins in body if not _is_label(ins)]
        for i, ins in enumerate(code):
            if not ins.startswith(_VMEM):
                continue
            used = _sregs(ins)
            if not used:
                continue
            ws, j = 0, i - 1
            while j >= 0 and ws < 5:
                hit = _valu_scalar_dest(code[j]) & used
                assert not hit, (what, name, code[j], ins, "only %d wait states between" % ws)
                used -= _salu_dest(code[j])
                ws += _wait_states(code[j])
                j -= 1


def test_wide_tile_gemm_copies_and_scalars():
    text = _assembly("gemm_wide.hip")
    assert sum("gemm_wide_kernel" in n for n in _functions(text)) == 31     # 11 epilogues and ranks x three tile heights, less two
    _check_m0(text, "gemm_wide.hip")
    _check_valu_sgpr_to_vmem(text, "gemm_wide.hip")
    text = _assembly("gemm_mx.hip")
    assert sum("gemm_mx_tile_kernel" in n for n in _functions(text)) == 30      # five epilogues x six tile forms
    _check_m0(text, "gemm_mx.hip")
    _check_valu_sgpr_to_vmem(text, "gemm_mx.hip")


def test_fp32_tile_copies_and_scalars():
    text = _assembly("f32_linear.hip")
    assert sum("f32_tile_kernel" in n for n in _functions(text)) == 10      # five tile forms x two orientations of W
    _check_m0(text, "f32_linear.hip")
    _check_valu_sgpr_to_vmem(text, "f32_linear.hip")


_VGPR = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")


def _vgprs(text):
    regs = set()
    for m in _VGPR.finditer(text):
        regs.update([int(m.group(1))] if m.group(1) is not None else range(int(m.group(2)), int(m.group(3)) + 1))
    return regs


def _operands_too_close(body, writer):
    """(vector instruction, MFMA) pairs of which the second reads as an operand what the first, one that starts with `writer`,
    wrote fewer than 2 wait states earlier"""
    code = [ins for ins in body if not _is_label(ins)]
    found = []
    for i, ins in enumerate(code):
        if not ins.startswith("v_mfma"):
            continue
        used, ws, j = _vgprs(ins.split(",", 1)[1]), 0, i - 1
        while j >= 0 and ws < 2:
            if code[j].startswith(writer) and not code[j].startswith("v_mfma") and _vgprs(code[j].split(",")[0]) & used:
                found.append((code[j], ins))
            ws += _wait_states(code[j])
            j -= 1
    return found


def test_fp32_pieces_are_settled_before_the_products():
    """the conversions are inline assembly, whose results the compiler keeps no distance to"""
    funcs = {n: b for n, b in _functions(_assembly("f32_linear.hip")).items() if "f32_tile_kernel" in n}
    assert all(sum(x.startswith("v_cvt_pk_bf16_f32") for x in b) >= 60 for b in funcs.values())
    for name, body in funcs.items():
        assert not _operands_too_close(body, "v_cvt_pk_bf16_f32"), (name, _operands_too_close(body, "v_cvt_pk_bf16_f32")[:2])
    bad = ["v_cvt_pk_bf16_f32 v5, v1, v2", "s_mov_b32 s1, s2", "v_mfma_f32_16x16x32_bf16 v[8:11], v[4:7], v[0:3], v[8:11]"]
    for writer in ("v_cvt_pk_bf16_f32", "v_"):
        assert _operands_too_close(bad, writer) and not _operands_too_close(bad[:1] + ["s_nop 1"] + bad[2:], writer)
    assert _operands_too_close(["v_mov_b64_e32 v[6:7], v[0:1]"] + bad[1:], "v_")


def _loops(body):
    """[instructions] of every loop without a label inside (a label, its body, a branch back to it)"""
    loops = []
    for i, ins in enumerate(body):
        m = re.match(r"s_c?branch\w*\s+(\S+)", ins)
        if m and m.group(1) + ":" in body[:i]:
            inner = body[body.index(m.group(1) + ":") + 1:i]
            if not any(_is_label(x) for x in inner):
                loops.append(inner)
    return loops


def test_fp32_adapter_gradient_rows_are_in_flight_together():
    """the loops over a half-wave's rows (two loads each at up to 4 columns): 16 of them, then 4, then single ones, so that
    behind the last 16 there are three groups of 4 and three single rows at most"""
    body = next(b for n, b in _functions(_assembly("f32_linear.hip")).items() if "f32_grad_kernelILi4E" in n)
    loads = [[i for i, x in enumerate(lp) if x.startswith("global_load")] for lp in _loops(body)]
    loops = [(lp, ld) for lp, ld in zip(_loops(body), loads) if ld]
    assert [len(ld) for _, ld in loops] == [32, 8, 2]
    for (lp, ld), first in zip(loops[:2], (16, 8)):      # loads in front of the first wait for one
        assert sum(i < next(j for j, x in enumerate(lp) if "vmcnt" in x) for i in ld) >= first


def test_rank_gradient_pass_copies_and_stores():
    """copies and scalars as elsewhere; and each unit of 64 tokens stores codes and scales as often as its wait allows for: 4
    of either where all rows are tokens (and one in the loop for the last block)"""
    text = _assembly("rank_grad.hip")
    _check_m0(text, "rank_grad.hip")
    _check_valu_sgpr_to_vmem(text, "rank_grad.hip")
    for ht in (1, 2):
        body = next(b for n, b in _functions(text).items() if "rank_grad_kernelILi%dELb1E" % ht in n)
        assert sum(x.startswith("global_store_dwordx2") for x in body) == 2 * ht * 5
        assert sum(x.startswith("global_store_byte") for x in body) == 2 * ht * 5


def test_attention_copies_and_scalars():
    text = _assembly("attention.hip")
    funcs = _functions(text)
    assert sum("attn_" in n for n in funcs) == 4
    _check_m0(text, "attention.hip")
    _check_valu_sgpr_to_vmem(text, "attention.hip")
    # the copies of the next tile run beside the products of this one: no wait for memory between a tile's first MFMA
    # and its last in the backward of long sequences
    for name, body in funcs.items():
        if "attn_bwd_dq" in name or "attn_bwd_dkv" in name:
            mf = [i for i, ins in enumerate(body) if ins.startswith("v_mfma")]
            assert not any("vmcnt" in ins for ins in body[mf[0]:mf[-1] + 1]), name


def test_vector_written_scalars_are_settled_before_vector_memory_reads_them(gemm_asm, tile_asm):
    _check_valu_sgpr_to_vmem(gemm_asm, "gemm.hip")
    _check_valu_sgpr_to_vmem(tile_asm, "gemm_tile.hip")
    _check_valu_sgpr_to_vmem(_assembly("mx.hip"), "mx.hip")
    _check_valu_sgpr_to_vmem(_assembly("attention.hip"), "attention.hip")


def test_the_scalar_hazard_check_sees_a_planted_hazard():
    bad = ("_Z3foov:\n\tv_readlane_b32 s0, v255, 16\n\tv_readlane_b32 s1, v255, 17\n\tv_readlane_b32 s51, v255, 19\n"
           "\tglobal_load_dwordx4 v[178:181], v221, s[0:1]\n\ts_endpgm\n.Lfunc_end0:\n")
    with pytest.raises(AssertionError):
        _check_valu_sgpr_to_vmem(bad, "planted")
    _check_valu_sgpr_to_vmem(bad.replace("\tglobal_load", "\ts_nop 4\n\tglobal_load"), "planted, with wait states")


# the same for a base in vcc, as a whole or by halves, written by each kind of vector instruction that can
@pytest.mark.parametrize("write", ["v_cmp_gt_i32_e32 vcc, s3, v1", "v_cmp_lt_u32_e64 vcc, v1, v2", "v_readlane_b32 vcc_lo, v255, 16",
                                   "v_readfirstlane_b32 vcc_hi, v3", "v_add_co_u32_e32 v0, vcc, v1, v2",
                                   "v_addc_co_u32_e64 v0, vcc, v1, v2, s[4:5]", "v_div_scale_f32 v0, vcc, v1, v2, v1",
                                   "v_mad_u64_u32 v[0:1], vcc, v2, v3, v[4:5]"])
def test_the_scalar_hazard_check_knows_vcc(write):
    bad = "_Z3foov:\n\t%s\n\tglobal_load_lds_dwordx4 v221, vcc\n\ts_endpgm\n.Lfunc_end0:\n" % write
    with pytest.raises(AssertionError):
        _check_valu_sgpr_to_vmem(bad, "planted")
    _check_valu_sgpr_to_vmem(bad.replace("\tglobal_load", "\ts_nop 4\n\tglobal_load"), "planted, with wait states")
    _check_valu_sgpr_to_vmem(bad.replace("v221, vcc", "v221, s[6:7]"), "another base")
    half = bad.replace("\tglobal_load", "\ts_add_u32 vcc_lo, s4, 64\n\tglobal_load")
    if not write.startswith("v_readlane"):               # (that one writes the low half only)
        with pytest.raises(AssertionError):
            _check_valu_sgpr_to_vmem(half, "planted, half of it written again")
    _check_valu_sgpr_to_vmem(half.replace("\tglobal_load", "\ts_addc_u32 vcc_hi, s5, 0\n\tglobal_load"), "written again")
