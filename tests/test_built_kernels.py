"""What the built library's own kernel descriptions say: registers that the compiler keeps in memory, instances."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1805_08899_amd import binding

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 code objects of the bundles in a library: magic, count, then (offset, size, length of the name, name) each, eight
    bytes a number, offsets from the magic."""
    at = blob.find(MAGIC)
    while at >= 0:
        number = lambda k: int.from_bytes(blob[k:k + 8], "little")
        k = at + len(MAGIC) + 8
        for _ in range(number(at + len(MAGIC))):
            offset, size, length = number(k), number(k + 8), number(k + 16)
            if blob[k + 24:k + 24 + length].endswith(b"gfx950"):
                yield blob[at + offset:at + offset + size]
            k += 24 + length
        at = blob.find(MAGIC, at + 1)


def _kernels(tmp_path):
    """{mangled name: (registers in memory, bytes of scratch per lane)}"""
    readelf = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf here")
    out = {}
    with open(binding.LIB_PATH, "rb") as f:
        blob = f.read()
    for obj in _code_objects(blob):
        path = tmp_path / "object"
        path.write_bytes(obj)
        notes = subprocess.run([readelf, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in notes.split(".agpr_count:")[1:]:
            value = lambda key: re.search(r"\." + key + r":\s+(\S+)", block).group(1)
            out[value("name")] = (int(value("vgpr_spill_count")), int(value("private_segment_fixed_size")))
    return out


@pytest.mark.parametrize("kernel", ["k_recompute_rows", "k_bwd_pre", "k_bwd_pre_parts"])
def test_no_instance_spills(kernel, tmp_path):
    found = {n: v for n, v in _kernels(tmp_path).items() if re.search(r"\d" + kernel + r"I", n)}
    assert found, "no such kernel in the library"
    assert not {n: v for n, v in found.items() if v != (0, 0)}


def test_every_instance_of_the_recomputation_by_rows_can_be_launched(tmp_path):
    """Lane groups and rows per lane of a sample of Tq rows: two groups up to 100 rows, which four row groups share, then one and passes
    of up to 200 rows, which eight share."""
    reached = set()
    for Tq in range(60, 3000):
        groups = 2 if Tq <= 100 else 1
        passes = -(-Tq // (25 * 8 // groups))
        rows = -(-Tq // passes)
        reached.add((groups, -(-rows // (8 // groups))))
    for dtype in ("f", "NS_6bf16_tE"):
        pattern = re.compile(r"k_recompute_rowsI" + dtype + r"Li(\d)ELi(\d+)EE")
        built = {tuple(int(x) for x in m.groups()) for m in map(pattern.search, _kernels(tmp_path)) if m}
        assert built == reached
