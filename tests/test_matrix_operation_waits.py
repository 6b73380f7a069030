"""Wait states behind matrix operations in the compiled kernels.

The hardware does not hold an instruction back that reads or overwrites the result of a matrix operation too early; the
compiler counts wait states and inserts s_nop.  This follows every path from every matrix operation of the built library and
looks for an instruction that touches the result before they are over (the same accumulator as the C operand of the next
matrix operation is forwarded and needs none of them)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2007_06000_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# wait states before any other instruction may touch the result: 4-cycle passes (8, 4, 16, 8) plus 4 for bf16, plus 2 for fp32
NEED = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x2_f32": 18, "v_mfma_f32_16x16x4_f32": 10}
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, i) for i in range(int(lo or one), int(hi or one) + 1))
    return out


def functions(listing):
    """[(name, [(operation, arguments, address, branch target or None)])] of a disassembly."""
    out, base, ins = [], 0, None
    for ln in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", ln)
        if m:
            base, ins = int(m[1], 16), []
            out.append((m[2], ins))
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^+>]+(?:\+0x([0-9a-f]+))?>)?", ln)
        if m and ins is not None:
            branch = m[1].startswith(("s_branch", "s_cbranch"))
            ins.append((m[1], m[2], int(m[3], 16), base + int(m[4] or "0", 16) if branch else None))
    return out


def early_uses(ins):
    at = {a: i for i, (_, _, a, _) in enumerate(ins)}

    def following(i):
        op, _, _, target = ins[i]
        if op == "s_endpgm":
            return []
        to = [at[target]] if target is not None else []
        return to if op == "s_branch" else to + ([i + 1] if i + 1 < len(ins) else [])
    used = [registers(args) for _, args, _, _ in ins]
    bad, count = [], 0
    for i, (op, args, _, _) in enumerate(ins):
        if not op.startswith("v_mfma"):
            continue
        count += 1
        need, result = NEED[op], registers(args.split(",")[0])
        best, todo = {}, [(j, 0) for j in following(i)]
        while todo:
            j, waited = todo.pop()
            if waited >= need or best.get(j, need) <= waited:
                continue
            best[j] = waited
            o, a, _, _ = ins[j]
            if o.startswith("v_mfma"):
                _, x, y, _ = [registers(part) for part in a.split(", ")[:4]]
                touched = x | y
            else:
                touched = used[j] if o.startswith(("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")) else set()
            if touched & result:
                bad.append((op, args, o, a, waited))
            todo += [(k, waited + (int(a) + 1 if o == "s_nop" else 1)) for k in following(j)]
    return bad, count


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_results_of_matrix_operations_are_not_touched_early(tmp_path):
    lib = shutil.copy(B.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    seen = 0
    for part in sorted(tmp_path.glob("*gfx950")):
        listing = subprocess.run([OBJDUMP, "-d", str(part)], check=True, capture_output=True, text=True).stdout
        for name, ins in functions(listing):
            bad, count = early_uses(ins)
            seen += count
            assert not bad, (name, bad[:4])
    assert seen > 10000


def test_the_search_finds_a_use_on_the_short_way_round_a_branch():
    text = """0000000000000100 <f>:
	v_mfma_f32_32x32x16_bf16 v[16:31], v[0:3], v[4:7], v[16:31]// 000000000100: 00000000
	s_cbranch_scc1 9                                           // 000000000108: BF850009 <f+0x30>
	s_nop 15                                                   // 00000000010C: BF80000F
	v_mov_b32_e32 v40, v16                                     // 000000000130: 7E500310
	s_endpgm                                                   // 000000000134: BF810000
"""
    (_, ins), = functions(text)
    bad, count = early_uses(ins)
    assert count == 1 and len(bad) == 1 and bad[0][2] == "v_mov_b32_e32" and bad[0][4] == 1
    assert early_uses([i for i in ins if not i[0].startswith("s_cbranch")]) == ([], 1)
