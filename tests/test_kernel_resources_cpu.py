"""Registers and LDS of the propagation kernels as compiled into libcrp.so, from the code objects'
metadata (the library's own kernels, read with llvm-readelf)."""
import os
import re
import struct
import subprocess

import pytest

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LDS = 160 * 1024          # bytes of a compute unit
NODE = 32                 # bytes of a table node in LDS
MAX_NODES = 1024


def _code_objects(lib):
    data = open(lib, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 24)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(precision, grid type, layout, block, trajectory): metadata} of k_propagate."""
    from paper_1307_2643_amd import build as B
    readelf = os.path.join(os.path.dirname(B.hipcc()), "..", "llvm", "bin", "llvm-readelf")
    out = {}
    for i, co in enumerate(_code_objects(B.LIB)):
        p = tmp_path_factory.mktemp("co") / f"{i}.co"
        p.write_bytes(co)
        notes = subprocess.run([readelf, "--notes", str(p)], capture_output=True, text=True,
                               check=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            f = dict(re.findall(r"\.(\w+):\s+(\S+)", block))
            m = re.search(r"k_propagateILi(\d)E([df])Li(\d)ELi(\d+)ELb([01])E", f["name"])
            if m:
                out[int(m[1]), m[2], int(m[3]), int(m[4]), m[5] == "1"] = f
    assert len(out) > 40
    return out


def test_two_blocks_of_256_fit_with_the_largest_tables_on_fp32_records(kernels):
    """Eight waves per compute unit (two per SIMD) with 1024 table nodes: corner records of an FP32
    grid, without and with refinement patches."""
    seen = 0
    for (mode, gt, layout, block, traj), f in kernels.items():
        if gt == "f" and layout in (2, 6) and block == 256:
            need = int(f["group_segment_fixed_size"]) + NODE * MAX_NODES
            assert 2 * need <= LDS, (mode, layout, traj, need)
            seen += 1
    assert seen == 8


def test_no_spills(kernels):
    """No vector register of a propagation kernel is spilled, and none uses scratch."""
    for key, f in kernels.items():
        assert int(f["vgpr_spill_count"]) == 0 and int(f["private_segment_fixed_size"]) == 0, key
