"""Waits between the FP64 matrix instructions and the first use of their
results, in the machine code of the built library (CPU only).

A v_mfma_f64_16x16x4 takes 16 passes; an instruction that is not itself a
matrix instruction accumulating into the same registers may touch its result 19
wait states after the issue (an s_nop k counts k + 1, every other instruction
one).  The hardware does not check this.  Compiled code has waited too little
where a loop's branch lay between the two, so every path is followed here."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1304_2062_amd", "libse2n.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT = 19

INSN = re.compile(r"^\s+(\S+)(?:\s+(.*?))?\s*// ([0-9A-F]+): .*?(?:<.*\+0x([0-9a-f]+)>)?$")
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(text):
    out = set()
    for bank, lo, hi, one in REG.findall(text):
        out.update((bank, r) for r in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def functions(disassembly):
    """name -> [(address, mnemonic, operands, branch target)]"""
    res, cur, base = {}, None, 0
    for line in disassembly.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
        if m:
            base = int(m.group(1), 16)
            cur = res.setdefault(m.group(2), [])
            continue
        m = INSN.match(line)
        if m and cur is not None:
            op, args, addr, off = m.groups()
            cur.append((int(addr, 16), op, args or "", base + int(off, 16) if off else None))
            if op in ("s_branch",) or op.startswith("s_cbranch"):
                # a target at the function's first instruction carries no offset
                cur[-1] = (*cur[-1][:3], cur[-1][3] if cur[-1][3] is not None else base)
    return res


def too_early(code):
    """[(instruction, wait states since the matrix instruction)] of uses before WAIT."""
    at = {a: i for i, (a, *_) in enumerate(code)}
    found = []
    for i, (_, op, args, _) in enumerate(code):
        if not op.startswith("v_mfma_f64_16x16x4"):
            continue
        dst = _regs(args.split(", ")[0])
        best, todo = {}, [(i + 1, 0)]
        while todo:
            k, waited = todo.pop()
            if k >= len(code) or waited >= WAIT or best.get(k, WAIT) <= waited:
                continue
            best[k] = waited
            _, o, a, target = code[k]
            if o.startswith("v_mfma"):
                d, srca, srcb, srcc = a.split(", ")[:4]
                if (_regs(srca) | _regs(srcb)) & dst:
                    found.append((o + " " + a, waited))
                if _regs(d) & dst:
                    continue  # the next product into the same registers is looked at by itself
            elif _regs(a) & dst:
                found.append((o + " " + a, waited))
            if o == "s_endpgm":
                continue
            states = int(a, 0) + 1 if o == "s_nop" else 1
            if target is not None:
                todo.append((at[target], waited + states))
            if o != "s_branch":
                todo.append((k + 1, waited + states))
    return found


def _build_kernels(tmp):
    shutil.copy(LIB, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    codes = {}
    for f in sorted(glob.glob(os.path.join(tmp, "lib.so.*gfx950*"))):
        with open(f, "rb") as fh:
            if b"k_precompute_mfma" not in fh.read():
                continue
        text = subprocess.run([OBJDUMP, "-d", f], check=True, capture_output=True, text=True).stdout
        codes.update({n: c for n, c in functions(text).items() if "k_precompute_mfma" in n})
    return codes


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not available")
def test_results_of_the_propagator_build_are_read_in_time(tmp_path):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built (run python -m paper_1304_2062_amd.build)")
    codes = _build_kernels(str(tmp_path))
    assert len(codes) == 4  # two types, one or four tiles per block
    for name, code in codes.items():
        assert sum(op.startswith("v_mfma_f64") for _, op, _, _ in code) >= 4, name
        assert any(t is not None for *_, t in code), name
        assert too_early(code) == [], name


LOOP = """
0000000000000100 <k>:
\tv_mov_b32_e32 v0, 0                                        // 000000000100: 00000000
\tv_accvgpr_read_b32 v17, a7                                 // 000000000104: 00000000
\ts_nop 11                                                   // 000000000108: 00000000
\tv_accvgpr_read_b32 v10, a0                                 // 00000000010C: 00000000
\tv_mfma_f64_16x16x4_f64 a[0:7], v[10:11], v[10:11], 0       // 000000000110: 00000000 00000000
\tv_mfma_f64_16x16x4_f64 a[0:7], v[12:13], v[12:13], a[0:7]  // 000000000118: 00000000 00000000
\ts_cbranch_scc1 65529                                       // 000000000120: 00000000 <k+0x4>
\ts_nop 15                                                   // 000000000124: 00000000
\ts_nop 1                                                    // 000000000128: 00000000
\tv_mfma_f64_16x16x4_f64 a[8:15], a[0:1], v[2:3], 0          // 00000000012C: 00000000 00000000
\ts_endpgm                                                   // 000000000134: 00000000
"""


def test_the_check_sees_a_read_across_a_loop_branch():
    """On the way back the last register is read one state after the product; the
    way on waits 19 states."""
    found = too_early(functions(LOOP)["k"])
    assert found == [("v_accvgpr_read_b32 v17, a7", 1), ("v_accvgpr_read_b32 v10, a0", 14)]
