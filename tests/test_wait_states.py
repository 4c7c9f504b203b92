"""Wait states in the built library (no GPU needed): results of one instruction that another may read only some cycles later.
The compiler puts them in for the instructions it knows and for none in inline assembly, so every kernel is read back:
whatever stands between a write and such a read, in program order, has to last long enough."""
import os
import re
import subprocess

import pytest

from paper_2501_15021_amd import binding as akvq
from test_kernel_resources import _code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\s+(\w+)\s*(.*?)\s*(?://.*)?$")
REG = re.compile(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)")
TRANS = ("v_exp", "v_rcp", "v_log", "v_rsq", "v_sqrt", "v_sin", "v_cos")
# wait states from a write of a vector register to a read of it
VALU_TO_SWAP, VALU_TO_DPP, TRANS_TO_VALU, PRODUCT_TO_VALU = 2, 2, 1, 8  # (products: 16 x 16 x 32, four passes)


def _regs(operand):
    out = set()
    for lo, hi, one in REG.findall(operand):
        out.update(range(int(lo), int(hi) + 1) if lo else (int(one),))
    return out


def violations(text):
    """(kernel, what, instruction) of every read that comes too early; also how many reads of each kind were looked at."""
    bad, seen, kernel, clock, last = [], {}, None, 0, {}
    for line in text.splitlines():
        if line.endswith(">:"):
            kernel, clock, last = line, 0, {}
            continue
        m = LINE.match(line)
        if not m or kernel is None:
            continue
        op, operands = m.groups()
        if op == "s_nop":
            clock += int(operands, 0) + 1
            continue
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            clock, last = 0, {}
            continue
        vector, swap, product = op.startswith("v_"), "permlane" in op, op.startswith("v_mfma")
        parts = operands.split(",")
        dst = _regs(parts[0]) if vector else set()
        accumulates = swap or op.startswith(("v_fmac", "v_dot")) or "_dpp" in op
        src = _regs(",".join(parts[1:])) | (dst if accumulates else set())
        if swap:
            dst |= src
        if vector:
            for r in src:
                at, kind = last.get(r, (None, None))
                need = []
                if kind in ("valu", "trans") and swap:
                    need.append(("swap", VALU_TO_SWAP))
                if kind in ("valu", "trans") and "_dpp" in op and r in _regs(parts[1]):
                    need.append(("dpp", VALU_TO_DPP))
                if kind == "trans" and not op.startswith(TRANS) and not product:
                    need.append(("trans", TRANS_TO_VALU))
                if kind == "product" and not product:
                    need.append(("product", PRODUCT_TO_VALU))
                for what, n in need:
                    seen[what] = seen.get(what, 0) + 1
                    if clock - at < n:
                        bad.append((kernel, what, line.strip()))
            clock += 1
            kind = "product" if product else "trans" if op.startswith(TRANS) else "valu"
            for r in dst:
                last[r] = (clock, kind)
        else:
            clock += 1
            if "load" in op or op.startswith("ds_read"):
                for r in _regs(parts[0]):
                    last.pop(r, None)
    return bad, seen


def test_the_scan_itself():
    def count(body):
        return len(violations("<k>:\n" + "".join(f"\t{x}\n" for x in body))[0])

    top, swap = "v_max3_f32 v68, v1, v2, v68", "v_permlane32_swap_b32_e32 v66, v68"
    assert count([top, swap]) == 1 and count([top, "s_nop 0", swap]) == 1 and count([top, "s_nop 1", swap]) == 0
    assert count([top, "v_mov_b32_e32 v3, v4", "s_waitcnt lgkmcnt(0)", swap]) == 0
    product, read = "v_mfma_f32_16x16x32_bf16 v[6:9], v[1:4], v[10:13], v[6:9]", "v_max3_f32 v20, v5, v6, v21"
    assert count([product, "s_nop 6", read]) == 1 and count([product, "s_nop 7", read]) == 0
    assert count([product, "v_mfma_f32_16x16x32_bf16 v[14:17], v[1:4], v[10:13], v[6:9]"]) == 0
    assert count(["v_exp_f32_e32 v1, v2", "v_add_f32_e32 v3, v1, v2"]) == 1
    assert count(["v_add_f32_e32 v1, v2, v2", "v_fmac_f32_dpp v3, v1, v4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"]) == 1


def test_every_read_comes_late_enough(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    with open(akvq.LIB_PATH, "rb") as f:
        blob = f.read()
    seen = {}
    for i, image in enumerate(_code_objects(blob)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(image)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout
        bad, looked_at = violations(text)
        assert not bad, bad[:20]
        for what, n in looked_at.items():
            seen[what] = seen.get(what, 0) + n
    assert all(seen.get(what, 0) > 20 for what in ("swap", "dpp", "trans", "product")), seen
