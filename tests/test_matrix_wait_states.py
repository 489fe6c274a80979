"""The compiled kernels keep the distance the hardware wants between a matrix instruction and the use of its result.

The result registers of a matrix instruction are written some cycles after it issues, and nothing in the hardware holds back
another instruction that reads (or writes) them earlier: the compiler has to place enough instructions or s_nop in between.  It
counts along the paths of the control flow and can miss a short one: where a result is used behind a branch and at the
point where the branch joins again, it has taken the longer way round for both.  The kernel then reads old register
contents now and then.  So the assembly of every kernel is followed here along every path.

Wait states (one per instruction, k + 1 for s_nop k) between a matrix instruction and the first other instruction that
touches its result, by the number of passes the instruction takes; those a straight piece of code gets from the compiler."""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess

import pytest

# (vector instruction or matrix operand A / B, memory instruction)
NEED = {"v_mfma_f32_4x4x1_16b_f32": (4, 4), "v_mfma_f32_16x16x4_f32": (10, 10), "v_mfma_f32_32x32x2_f32": (18, 18),
        "v_mfma_f64_16x16x4_f64": (19, 18)}
REGISTER = re.compile(r"\b([va])(\d+)\b|\b([va])\[(\d+):(\d+)\]")


def _registers(text):
    out = set()
    for m in REGISTER.finditer(text):
        if m.group(1):
            out.add((m.group(1), int(m.group(2))))
        else:
            out |= {(m.group(3), i) for i in range(int(m.group(4)), int(m.group(5)) + 1)}
    return out


def _operands(rest):
    return [o.strip() for o in re.split(r",(?![^\[]*\])", rest)]


def _kernels(lines):
    """(name, [(operation, operands)], {label: index}) of every function in the assembly"""
    name, code, labels = None, [], {}
    for line in lines:
        line = line.split(";")[0].rstrip()
        m = re.match(r"(\.?\w+):", line)
        if m and not m.group(1).startswith("."):
            name, code, labels = m.group(1), [], {}
        elif m and m.group(1).startswith(".Lfunc_end"):
            if name and code:
                yield name, code, labels
            name = None
        elif m:
            labels[m.group(1)] = len(code)
        elif name and line.startswith("\t") and not line.strip().startswith("."):
            op, _, rest = line.strip().partition(" ")
            code.append((op, rest.strip()))


def _too_early(code, labels):
    """(matrix instruction, instruction that touches its result, wait states in between) of every pair that is too close"""
    info = []
    for op, rest in code:
        if op.startswith("v_mfma"):
            o = _operands(rest)
            info.append(("matrix", _registers(o[0]), _registers(o[1]) | _registers(o[2])))
        elif op.startswith("v_"):
            info.append(("vector", _registers(rest), set()))
        elif op.startswith(("ds_", "global_", "scratch_", "buffer_", "flat_")):
            info.append(("memory", _registers(rest), set()))
        else:
            info.append(("scalar", set(), set()))
    found = set()
    for i, (op, _) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        assert op in NEED, f"{op}: add the distance it needs"
        need = NEED[op]
        paths, seen = [(i + 1, 0, frozenset(info[i][1]))], {}
        while paths:
            pc, waited, regs = paths.pop()
            while pc < len(code) and waited < max(need) and regs and seen.get((pc, regs), 1 << 30) > waited:
                seen[pc, regs] = waited
                o, rest = code[pc]
                kind, touched, ab = info[pc]
                if kind == "matrix":
                    if ab & regs and waited < need[0]:
                        found.add((op, o, waited))
                    regs = regs - touched                   # (as operand C it may follow at once; its result counts on its own)
                elif kind != "scalar" and touched & regs:
                    if waited < need[kind == "memory"]:
                        found.add((op, o, waited))
                    regs = regs - touched
                waited += int(rest, 0) + 1 if o == "s_nop" else 1
                if o.startswith("s_cbranch"):
                    paths.append((labels[rest], waited, regs))
                if o == "s_endpgm":
                    break
                pc = labels[rest] if o == "s_branch" else pc + 1
    return found


def test_the_check_follows_the_shorter_path():
    """A result used four wait states later at the join of a branch around a use that waits long enough."""
    text = ["k:", "\tv_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[0:3]", "\ts_cbranch_vccnz .LBB0_2", "\ts_xor_b64 s[0:1], s[2:3], -1",
            "\ts_andn2_b64 vcc, exec, s[0:1]", "\ts_cbranch_vccnz .LBB0_1", "\ts_nop 4", "\tv_add_f32_e32 v3, v7, v3", ".LBB0_1:",
            "\tv_mov_b64_e32 v[4:5], v[2:3]", ".LBB0_2:", "\ts_endpgm", ".Lfunc_end0:"]
    (_, code, labels), = _kernels(text)
    assert _too_early(code, labels) == {("v_mfma_f32_16x16x4_f32", "v_mov_b64_e32", 4),
                                        ("v_mfma_f32_16x16x4_f32", "v_add_f32_e32", 9)}
    (_, code, labels), = _kernels(text[:6] + ["\ts_nop 5"] + text[7:8] + ["\ts_nop 0", ".LBB0_3:", "\ts_endpgm", ".LBB0_1:", "\ts_branch .LBB0_3",
                                                                          ".LBB0_2:", "\ts_endpgm", ".Lfunc_end0:"])
    assert _too_early(code, labels) == set()


@pytest.mark.slow
@pytest.mark.timeout(600)
def test_results_of_matrix_instructions_are_waited_for(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    from paper_2202_13638_amd import build

    def assembly(src):
        out = str(tmp_path / (src + ".s"))
        r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        with open(out) as f:
            return f.readlines()

    with cf.ThreadPoolExecutor(max_workers=6) as ex:
        texts = list(ex.map(assembly, build.SOURCES))
    matrix, bad = 0, {}
    for lines in texts:
        for name, code, labels in _kernels(lines):
            matrix += sum(op.startswith("v_mfma") for op, _ in code)
            found = _too_early(code, labels)
            if found:
                bad[name] = sorted(found)
    assert matrix > 1000
    assert not bad, bad
