"""Weights of the pivot score in the built library (no GPU needed): every scoring kernel divides by a row's sum, correctly rounded,
so that the kernel a prompt's size chooses does not change how a weight is rounded."""
import os
import re
import subprocess

import pytest

from paper_2501_15021_amd import binding as akvq
from test_kernel_resources import _code_objects
from test_wait_states import OBJDUMP


def reciprocals(text):
    """kernel -> (reciprocal approximations, divisions), of the kernels that turn exponentials into masses"""
    found, name = {}, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if head:
            name = head.group(1) if re.search(r"psa_(once|small|mass|mass_gqa)_kernel", head.group(1)) else None
        elif name:
            approximate, divided = found.get(name, (0, 0))
            found[name] = (approximate + ("v_rcp_f32" in line), divided + ("v_div_fixup_f32" in line))
    return found


def test_every_weight_is_a_division(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    with open(akvq.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {}
    for i, image in enumerate(_code_objects(blob)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(image)
        found.update(reciprocals(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout))
    for kind in ("once", "small", "mass", "mass_gqa"):
        assert any(f"psa_{kind}_kernel" in name for name in found), kind
    # (a division starts from an approximate reciprocal of its own)
    assert {name: n for name, n in found.items() if n[1] == 0 or n[0] != n[1]} == {}
