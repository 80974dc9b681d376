"""Matrix and dot-product instructions that the kernels write as statements of their own are unknown to the compiler as such: it puts no wait
between them and what writes their operands or reads their results.  Checked in the assembly of the present sources:
  - no vector instruction writes an operand of such an instruction within the two wait states before it;
  - nothing but another matrix instruction touches the result of v_mfma_f32_16x16x32_* for 11 wait states (its 8 passes and 3);
  - nothing but the next v_dot2_f32_f16 on the same sum touches the result of one for 3.
An instruction counts as one wait state, an s_nop as many as it says; both ways of a branch are followed."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2210_17323_amd import build

SOURCES = {"gemm_split.hip": 1, "hessian.hip": 1, "consume.hip": 1}        # and at least how many such instructions each has
OPERAND = re.compile(r"([va])(?:\[(\d+):(\d+)\]|(\d+))$")


def _registers(operand):
    m = OPERAND.match(operand)
    if not m:
        return frozenset()
    first, last = (int(m[2]), int(m[3])) if m[2] else (int(m[4]), int(m[4]))
    return frozenset((m[1], i) for i in range(first, last + 1))


class Function:
    """Instructions as (line, name, registers of each operand, written by hand, wait states), and which may follow and precede each."""

    def __init__(self):
        self.code, self.labels, self.targets = [], {}, {}

    def link(self):
        self.after, self.before = [[] for _ in self.code], [[] for _ in self.code]
        for k, (_, name, _, _, _) in enumerate(self.code):
            follow = [] if name in ("s_branch", "s_endpgm", "s_setpc_b64") else [k + 1]
            if k in self.targets:
                follow.append(self.labels[self.targets[k]])
            for f in follow:
                if f < len(self.code):
                    self.after[k].append(f)
                    self.before[f].append(k)


def instructions(text):
    functions, by_hand = [], False
    for number, line in enumerate(text.splitlines(), 1):
        if "#ASMSTART" in line or "#ASMEND" in line:
            by_hand = "#ASMSTART" in line
            continue
        code = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", code):
            functions.append(Function())
        if not functions or not code:
            continue
        f = functions[-1]
        if code.endswith(":"):
            f.labels[code[:-1]] = len(f.code)
        elif not code.startswith("."):
            name, _, rest = code.partition(" ")
            if name == "s_branch" or name.startswith("s_cbranch"):
                f.targets[len(f.code)] = rest.strip()
            ops = [_registers(o.strip().split(" ")[0]) for o in rest.split(",")] if rest else []
            f.code.append((number, name, ops, by_hand, int(rest, 0) + 1 if name == "s_nop" else 1))
    for f in functions:
        f.link()
    return functions


def _within(ways, code, k, states):
    """(wait states in between, instruction) of everything less than `states` away from instruction k, each at its nearest."""
    nearest, todo = {}, [(0, n) for n in ways[k]]
    while todo:
        passed, n = todo.pop()
        if passed >= states or nearest.get(n, states) <= passed:
            continue
        nearest[n] = passed
        todo += [(passed + code[n][4], m) for m in ways[n]]
    return sorted((passed, code[n]) for n, passed in nearest.items())


def violations(function):
    found, checked, code = [], 0, function.code
    for k, (line, name, ops, by_hand, _) in enumerate(code):
        matrix, dot = name.startswith("v_mfma_f32_16x16x32"), name.startswith("v_dot2_f32_f16")
        if not by_hand or not (matrix or dot):
            continue
        checked += 1
        if matrix:
            sources = frozenset().union(*ops[1:4])
            for passed, (at, other, theirs, _, _) in _within(function.before, code, k, 2):
                if other.startswith("v_") and not other.startswith(("v_mfma", "v_cmp")) and theirs and theirs[0] & sources:
                    found.append(f"line {line}: {name} reads what line {at} ({other}) wrote {passed} wait states before")
        for passed, (at, other, theirs, _, _) in _within(function.after, code, k, 11 if matrix else 3):
            if matrix:
                touched = not other.startswith("v_mfma") and any(o & ops[0] for o in theirs)
            else:                                           # the same sum's next product takes it as its addend
                touched = any(o & ops[0] for o in (theirs[1:3] if other.startswith("v_dot2_f32_f16") and theirs[0] == ops[0] else theirs))
            if touched:
                found.append(f"line {at}: {other} touches the result of line {line} ({name}) after {passed} wait states")
    return found, checked


def test_the_check_finds_what_it_is_for():
    lead = "_Zf:\n;;#ASMSTART\n"
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n;;#ASMEND\n"
    ok = lead + mfma + "s_nop 15\nv_accvgpr_read_b32 v9, a0\n"
    assert violations(instructions(ok)[0]) == ([], 1)
    early = lead + mfma + "s_nop 9\nv_accvgpr_read_b32 v9, a0\n"
    assert len(violations(instructions(early)[0])[0]) == 1
    fed = "_Zf:\nv_add_u32 v5, v9, v9\ns_nop 0\n" + lead[5:] + mfma
    assert len(violations(instructions(fed)[0])[0]) == 1
    assert violations(instructions(fed.replace("s_nop 0", "s_nop 1"))[0])[0] == []
    dot = "v_dot2_f32_f16 v0, v1, v2, v0\n"
    away = lead + mfma + "s_branch .L1\n.L0:\nv_accvgpr_write_b32 a0, 0\n.L1:\ns_nop 15\nv_accvgpr_read_b32 v9, a0\n"
    assert violations(instructions(away)[0])[0] == []
    assert len(violations(instructions(away.replace("s_branch .L1", "s_cbranch_vccz .L1"))[0])[0]) == 1
    assert violations(instructions(lead + dot + dot + ";;#ASMEND\ns_nop 2\nv_add_f32 v3, v0, v0\n")[0]) == ([], 2)
    assert len(violations(instructions(lead + dot + ";;#ASMEND\ns_nop 1\nv_add_f32 v3, v0, v0\n")[0])[0]) == 1


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    folder = tmp_path_factory.mktemp("asm")

    def compiled(source):
        out = folder / (source + ".s")
        subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
        return out.read_text()

    with concurrent.futures.ThreadPoolExecutor(len(SOURCES)) as pool:
        return dict(zip(SOURCES, pool.map(compiled, SOURCES)))


@pytest.mark.parametrize("source", SOURCES)
def test_hand_written_instructions_have_their_waits(assembly, source):
    found, checked = [], 0
    for function in instructions(assembly[source]):
        f, c = violations(function)
        found += f
        checked += c
    print(f"{source}: {checked} instructions")
    assert checked >= SOURCES[source]
    assert not found, "\n".join(found[:20])
