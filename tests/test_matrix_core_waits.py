"""Wait states around the dK/dV kernel's matrix instructions (no GPU needed).

The kernel issues its MFMAs from inline asm, where the compiler does not insert
the waits the hardware asks for: a result is not to be touched by a VALU or
memory instruction before the matrix core has written it, an operand written by
a VALU instruction is readable two instructions later, and the starting value of
a product (its third operand) is not to be overwritten while the matrix core
still reads it.  This reads the assembly that the build's own flags produce and
counts the distances, the loop's back edge included."""

import os
import re
import subprocess

import pytest

from paper_2607_20940_amd import build

MFMAS, CYCLES = 2, 19  # MFMAs or wait states behind a result
OPERAND = 2            # wait states before an operand
SOURCE = 16            # wait states, or an MFMA, before a starting value is overwritten


def _registers(text):
    out = set()
    for m in re.finditer(r"\b([va])(\d+)\b|\b([va])\[(\d+):(\d+)\]", text):
        out |= {(m[1], int(m[2]))} if m[1] else {(m[3], k) for k in range(int(m[4]), int(m[5]) + 1)}
    return out


def _instructions(lines):
    """[(opcode, operands)], the longest loop's body a second time after it."""
    ins, labels, loop = [], {}, (0, 0)
    for line in lines:
        line = line.split(";")[0]
        m = re.match(r"^(\.L\w+):", line)
        if m:
            labels[m[1]] = len(ins)
        m = re.match(r"^\s+([a-z]\w+)\s*(.*)$", line)
        if not m:
            continue
        ins.append((m[1], [x.strip() for x in re.split(r",(?![^\[]*\])", m[2])] if m[2] else []))
        if m[1].startswith("s_cbranch") and m[2].strip() in labels:
            b = labels[m[2].strip()]
            if sum("mfma" in op for op, _ in ins[b:]) > sum("mfma" in op for op, _ in ins[slice(*loop)]):
                loop = (b, len(ins))
    return ins[: loop[1]] + ins[loop[0]:] if loop[1] else ins


def _violations(ins):
    bad, n_mfma, pos, result, written, source = [], 0, 0, {}, {}, {}
    for op, args in ins:
        if "mfma" in op:
            n_mfma += 1
            for r in set().union(*(_registers(a) for a in args[1:4])):
                if r in written and pos - written[r] < OPERAND:
                    bad.append(("operand", op, args, r))
            for r in _registers(args[0]):
                result[r] = (n_mfma, pos)
            for r in _registers(args[3]) - _registers(args[0]):
                source[r] = (n_mfma, pos)
        elif op.startswith(("v_", "ds_", "buffer_", "global_", "scratch_", "flat_")):
            for r in set().union(set(), *(_registers(a) for a in args)):
                if r in result and n_mfma - result[r][0] < MFMAS and pos - result[r][1] < CYCLES:
                    bad.append(("result", op, args, r))
            if op.startswith("v_") and args and not op.startswith("v_cmp"):
                for r in _registers(args[0]):
                    if r in source and n_mfma == source[r][0] and pos - source[r][1] < SOURCE:
                        bad.append(("source", op, args, r))
                    written[r] = pos + 1
                    result.pop(r, None)
        pos += int(args[0], 0) + 1 if op == "s_nop" else 1
    return bad


@pytest.fixture(scope="module")
def kernels():
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    src = os.path.join(build.CSRC, "attention_bwd.hip")
    r = subprocess.run([hipcc, "-x", "hip", *build.COMMON, *build.HIP_FLAGS, "--cuda-device-only", "-S", src, "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out, name = {}, None
    for line in r.stdout.splitlines():
        m = re.match(r"^(_Z\w*dkdv_kernel\w*):", line)
        if m:
            name = m[1]
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            out[name].append(line)
    return out


def test_waits_of_the_dkdv_kernel(kernels):
    assert len(kernels) >= 4
    for name, lines in kernels.items():
        ins = _instructions(lines)
        assert sum("mfma" in op for op, _ in ins) > 100, name
        assert not _violations(ins), name


def test_the_check_finds_missing_waits():
    mfma = "\tv_mfma_f32_32x32x16_bf16 {0}, v[80:83], v[84:87], {0}"
    a, b, c = (mfma.format(r) for r in ("v[0:15]", "v[16:31]", "a[0:15]"))
    read, store = "\tv_mul_f32_e32 v40, s3, v5", "\tds_write_b32 v41, v17"
    first = "\\tv_mfma_f32_32x32x16_bf16 v[0:15], v[80:83], v[84:87], v[48:63]"
    ok = [[first, b, "\\tv_mov_b32_e32 v60, v2"], [a, b, c, read], [a, "\ts_nop 15", "\ts_nop 2", read], [b, a, c, store],
          ["\tv_mov_b32_e32 v80, v2", "\ts_nop 1", a]]
    missing = [[a, b, read], [a, read], [b, a, store], [a, "\ts_nop 15", read], [c, "\tv_accvgpr_read_b32 v40, a3"],
               ["\tv_mov_b32_e32 v80, v2", a], ["\tv_mov_b32_e32 v80, v2", "\ts_nop 0", a],
               [".LBB0_1:", read, a, b, "\ts_cbranch_scc1 .LBB0_1"]]  # around the back edge
    assert all(not _violations(_instructions(t)) for t in ok)
    assert all(_violations(_instructions(t)) for t in missing)
