"""Every path of the built kernels keeps the wait states between a matrix
instruction and the first other instruction that touches its result.

The hardware does not interlock a vector instruction with the matrix
instruction that produces its operand: the compiler counts the instructions in
between and fills up with s_nop.  ROCm 7.2's compiler counts them along the
longer path only where a branch lies between the two, so kernels with such a
branch spell the wait out (mfma_settled); this test walks the disassembly of
the library, every branch both ways, and fails on a path that is short.
"""
import os
import re
import shutil
import subprocess
from collections import defaultdict

import pytest

from paper_2606_00422_amd import upr

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# Wait states by instruction: passes of four cycles, plus four for the
# reduced-precision instructions (plus two for fp32's), the distances that the
# compiler itself keeps in straight-line code on gfx950.
NEED = {
    "v_mfma_f32_16x16x32_bf16": 8,
    "v_mfma_f32_32x32x16_f16": 12,
    "v_mfma_scale_f32_32x32x64_f8f6f4": 20,
    "v_mfma_f32_16x16x4_f32": 10,
}

_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
_FUNC = re.compile(r"^([0-9a-f]+) <(.+)>:$")
_INS = re.compile(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+):")
_TARGET = re.compile(r"\+0x([0-9a-f]+)>\s*$")


def _regs(operands):
    got = set()
    for kind, lo, hi, one in _REG.findall(operands):
        a, b = (int(lo), int(hi)) if lo else (int(one), int(one))
        got.update((kind, r) for r in range(a, b + 1))
    return got


def parse(text):
    """{kernel: [(mnemonic, operands, address, branch target or None)]}"""
    kernels, cur, base = {}, None, 0
    for line in text.splitlines():
        m = _FUNC.match(line)
        if m:
            base, cur = int(m.group(1), 16), kernels.setdefault(m.group(2), [])
            continue
        m = _INS.match(line)
        if m and cur is not None:
            name, ops, at = m.group(1), m.group(2).strip(), int(m.group(3), 16)
            target = None
            if name.startswith(("s_branch", "s_cbranch")):
                t = _TARGET.search(line)
                target = base + (int(t.group(1), 16) if t else 0)
            cur.append((name, ops, at, target))
    return kernels


def short_paths(code):
    """Paths of one kernel on which a result is touched too early:
    [(address of the matrix instruction, address of the other, distance)]."""
    at = {ins[2]: i for i, ins in enumerate(code)}
    bad = []
    for i, (name, ops, addr, _) in enumerate(code):
        if not name.startswith(("v_mfma", "v_smfma")):
            continue
        need = NEED[name]                       # a new instruction needs a line above
        dst = _regs(ops.split(",")[0])
        best = {}
        todo = [(i + 1, 0)]
        while todo:
            j, waited = todo.pop()
            if waited >= need or j >= len(code) or best.get(j, need) <= waited:
                continue
            best[j] = waited
            n, o, a, target = code[j]
            if n.startswith(("v_mfma", "v_smfma")):
                # the accumulator goes from one to the next by rules of its
                # own; what it overwrites is its own result to wait for
                if dst & _regs(o.split(",")[0]):
                    continue
            elif not n.startswith("s_") and dst & _regs(o):
                bad.append((addr, a, waited))
                continue
            if n == "s_endpgm":
                continue
            step = int(o) + 1 if n == "s_nop" else 1
            if target is not None:
                todo.append((at[target], waited + step))
                if n == "s_branch":
                    continue
            todo.append((j + 1, waited + step))
    return bad


def test_a_short_path_is_found():
    """The walker itself: a result read eight states late straight on, and two
    states late where the branch is taken."""
    def kernel(nop, jump):
        lines = ["0000000000000100 <k>:"]
        code = ["v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]", jump, f"s_nop {nop}",
                "v_add_f32_e32 v4, v5, v6", "v_add_f32_e32 v7, v0, v6", "s_endpgm"]
        for i, c in enumerate(code):        # a branch goes to the v_add of v4, past the s_nop
            lines.append(f"\t{c}// {0x100 + 4 * i:012X}: 00000000" + (" <k+0xc>" if "cbranch" in c else ""))
        return parse("\n".join(lines))["k"]
    assert short_paths(kernel(5, "s_mov_b32 s0, s1")) == []
    assert [d for _, _, d in short_paths(kernel(4, "s_mov_b32 s0, s1"))] == [7]
    assert [d for _, _, d in short_paths(kernel(5, "s_cbranch_scc1 2"))] == [2]


def test_no_kernel_reads_a_matrix_result_early(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(upr.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(f for f in os.listdir(tmp_path) if "gfx950" in f)
    assert objects
    bad = defaultdict(list)
    for f in objects:
        dis = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name, code in parse(dis).items():
            for at, to, waited in short_paths(code):
                bad[name].append(f"{at:x} -> {to:x}: {waited} wait states")
        assert dis.count("\tv_mfma") == sum(ins[0].startswith("v_mfma") for code in parse(dis).values() for ins in code)
    assert not bad, "\n".join(f"{k}: {'; '.join(v[:4])}" for k, v in bad.items())
