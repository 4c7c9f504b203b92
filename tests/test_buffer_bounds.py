"""Accesses through buffer descriptors in the built library (no GPU needed).  What lies past the end is left out by the
comparison of the lane's offset with the descriptor's size; a scalar offset beside it is not sure to be part of that
comparison, so an access that may pass the end has none."""
import os
import re
import subprocess

import pytest

from paper_2501_15021_amd import binding as akvq
from test_kernel_resources import _code_objects
from test_wait_states import OBJDUMP

ACCESS = re.compile(r"^\s+(buffer_(?:load|store|atomic)_\w+)\s+(.*?)\s*(?://.*)?$")
SCALAR_OFFSET = re.compile(r"s\[\d+:\d+\], (\S+)")


def accesses(text):
    """(instruction, scalar offset) of every access through a descriptor."""
    for line in text.splitlines():
        m = ACCESS.match(line)
        if m:
            yield m.group(1), SCALAR_OFFSET.search(m.group(2)).group(1)


def test_the_scan_itself():
    text = ("<k>:\n\tbuffer_load_dwordx4 v[2:5], v1, s[8:11], s65 offen nt // 0001: 00\n\tbuffer_store_dword v1, v2, s[4:7], 0 offen\n"
            "\tbuffer_load_dwordx2 v[2:3], v1, s[8:11], 0 offen offset:512 sc1\n\tglobal_load_dword v1, v2, s[0:1]\n")
    assert list(accesses(text)) == [("buffer_load_dwordx4", "s65"), ("buffer_store_dword", "0"), ("buffer_load_dwordx2", "0")]


def test_no_scalar_offset_where_the_end_may_be_passed(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    with open(akvq.LIB_PATH, "rb") as f:
        blob = f.read()
    found = []
    for i, image in enumerate(_code_objects(blob)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(image)
        found += accesses(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout)
    # (accesses of 8 bytes are the words a head's workgroups exchange: by construction inside their descriptor)
    assert {op for op, _ in found} == {"buffer_load_dwordx2", "buffer_load_dwordx4", "buffer_store_dword", "buffer_store_dwordx2"}
    assert [(op, at) for op, at in found if not op.endswith("x2") and at != "0"] == []
