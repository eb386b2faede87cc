"""Wait states in the built gfx950 code of the kernels (no GPU needed). The
compiler keeps them between the instructions that it schedules, but it cannot see
into inline assembly. Checked in program order over every kernel:
  - a scalar or condition register that a vector instruction wrote is read by a
    vector instruction two wait states later at the earliest, and as the lane
    number of a lane read or write four;
  - a vector register is read by a lane read one wait state after a vector
    instruction wrote it, and as the shifted operand of a lane move (DPP) two.
And no reversed instruction (v_subrev and the like) takes a shifted operand: here
d = v_subrev_u32_dpp(s0, s1) gave shifted(s1) - s0, not s1 - shifted(s0)."""
import re

import pytest

from tests.test_kernel_asm import device_asm, kernel_meta  # noqa: F401

pytestmark = pytest.mark.slow

REGISTER = re.compile(r"\b(vcc(?:_lo|_hi)?|[sv]\d+|[sv]\[\d+:\d+\]|m0)\b")


def registers(operand):
    out = set()
    for r in REGISTER.findall(operand):
        if r == "vcc":
            out |= {"vcc_lo", "vcc_hi"}
        elif "[" in r:
            first, last = map(int, re.findall(r"\d+", r))
            out |= {f"{r[0]}{k}" for k in range(first, last + 1)}
        else:
            out.add(r)
    return out


def is_scalar(r):
    return r[0] != "v" or r.startswith("vcc")


def missing_waits(asm):
    """(kernel, writer, reader) of each pair of instructions too close together."""
    bad, kernel, written = [], "", []  # written: [wait states since, registers, instruction]
    for line in asm.splitlines():
        label = re.match(r"([A-Za-z_]\w*):", line)
        text = line.split(";")[0].strip()
        if label:
            kernel, written = label.group(1), []
            continue
        if not text or text[0] == "." or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        ops = [registers(x) for x in re.split(r",(?![^\[]*\])", rest)]
        if op.startswith("v_"):
            outs = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[iu]64", op) else 1
            lane_op = op.startswith(("v_readlane", "v_writelane"))
            for age, regs, by in written:
                reads = [r for r in ops[outs:] if r]
                close = [r for at, r in enumerate(reads) for x in r & regs
                         if (is_scalar(x) and age < (4 if lane_op and at == 1 else 2)) or
                         (not is_scalar(x) and age < 1 and op.startswith(("v_readlane", "v_readfirstlane")) and at == 0) or
                         (not is_scalar(x) and age < 2 and "_dpp" in op and at == 0)]
                if close:
                    bad.append((kernel, by, text))
        states = int(rest, 0) + 1 if op == "s_nop" else 1
        written = [(age + states, regs, by) for age, regs, by in written if age + states < 4]
        if op.startswith("v_"):
            written.append((0, set().union(*ops[:outs]), text))
    return bad


def test_planted_missing_waits_are_seen():
    near = "k:\n\tv_cmp_eq_u64_e32 vcc, 0, v[2:3]\n{}\tv_addc_co_u32_e32 v4, vcc, v4, v4, vcc\n"
    lane = "k:\n\tv_add_u32_e32 v1, v2, v3\n{}\tv_readlane_b32 s4, v1, s5\n"
    move = "k:\n\tv_add_u32_e32 v1, v2, v3\n{}\tv_mov_b32_dpp v4, v1 row_shr:1 row_mask:0xf bank_mask:0xf\n"
    for text, needed in ((near, 2), (lane, 1), (move, 2)):
        assert len(missing_waits(text.format(""))) == 1
        assert len(missing_waits(text.format("\ts_mov_b32 s9, 0\n" * (needed - 1)))) == 1
        assert not missing_waits(text.format(f"\ts_nop {needed - 1}\n"))
        assert not missing_waits(text.format("\ts_mov_b32 s9, 0\n" * needed))


def test_no_missing_waits(device_asm):  # noqa: F811
    bad = missing_waits(device_asm)
    assert not bad, (len(bad), bad[:3])


def test_no_reversed_lane_moves(device_asm):  # noqa: F811
    # what the compiler makes of x - lane_below(y), unless here() keeps it apart
    found = re.findall(r"\bv_\w*rev\w*_dpp\b[^\n]*", device_asm)
    assert not found, found[:3]


def test_lone_wavefronts_take_a_simd(device_asm):  # noqa: F811
    # instances that rely on no two wavefronts fitting a SIMD's 512 registers, and
    # the ones of which two have to
    meta = kernel_meta(device_asm)
    regs = {k: int(re.search(r"\.vgpr_count:\s+(\d+)", v).group(1)) for k, v in meta.items() if "k_windows_lane" in k}
    alone = {k: v for k, v in regs.items() if "ELb1EEEv" in k}
    assert len(alone) == 3 and all(v > 256 for v in alone.values()), regs
    assert len(regs) == 5 and all(v <= 256 for k, v in regs.items() if k not in alone), regs
