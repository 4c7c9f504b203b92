"""What the compiler gave the kernels, read from the metadata of the built library (no GPU needed): no kernel reserves
scratch memory, and a decode workgroup of four wavefronts leaves room for three per CU (168 vector registers, 53 KB of
LDS), so that launches of more than two workgroups per CU keep their wavefronts."""
import os
import re
import struct
import subprocess

import pytest

from paper_2501_15021_amd import binding as akvq

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """Device images of the bundles a HIP shared library carries (one bundle per source file)."""
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            offset, size, id_len = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + id_len].decode()
            pos += 24 + id_len
            if "gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    with open(akvq.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {}
    for i, image in enumerate(_code_objects(blob)):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"^  - (?=\.)", notes, flags=re.M)[1:]:
            fields = dict(re.findall(r"^\s*\.(\w+):\s+(\S+)$", entry, flags=re.M))
            if "private_segment_fixed_size" in fields:
                found[fields["symbol"].strip("'").replace(".kd", "")] = fields
    assert sum("decode_gqa_kernel" in n for n in found) == 8 and sum("decode_mha_kernel" in n for n in found) == 8
    return found


def test_no_kernel_reserves_scratch(kernels):
    assert {n: f["private_segment_fixed_size"] for n, f in kernels.items() if f["private_segment_fixed_size"] != "0"} == {}


def test_three_decode_workgroups_per_cu(kernels):
    for n, f in kernels.items():
        if re.search(r"decode_(mha|gqa)_kernel", n) and f["max_flat_workgroup_size"] == "256":
            assert int(f["vgpr_count"]) <= 168, (n, f["vgpr_count"])
            assert int(f["group_segment_fixed_size"]) <= 160 * 1024 // 3, n
