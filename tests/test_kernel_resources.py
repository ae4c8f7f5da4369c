"""What the built kernels take of a compute unit, from the metadata of the library's code object: no kernel has scratch memory (a launch that
needs some makes the runtime provide it for the queue, and the data path allocates nothing), and a workgroup of 1024 leaves room for a second one where it did."""
import re
import struct
import subprocess

import pytest

import paper_2504_17307_amd as pkg

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> metadata of every kernel of the library."""
    lib = open(pkg.LIB_PATH, "rb").read()
    at = lib.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, = struct.unpack_from("<Q", lib, at + 24)
    entry, code = at + 32, None
    for _ in range(n):
        off, size, length = struct.unpack_from("<QQQ", lib, entry)
        if b"gfx950" in lib[entry + 24:entry + 24 + length]:
            code = lib[at + off:at + off + size]
        entry += 24 + length
    path = tmp_path_factory.mktemp("code") / "gfx950.elf"
    path.write_bytes(code)
    notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
    found = {}
    for block in re.split(r"\n  - (?=\.agpr_count|\.args)", notes)[1:]:
        name = re.search(r"\n    \.name: +(\S+)", block).group(1)
        found[name] = {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)\n", block[block.index("\n    .group_segment"):])}
    assert len(found) > 300
    return found


def test_no_kernel_has_scratch_memory(kernels):
    assert {k: v["private_segment_fixed_size"] for k, v in kernels.items() if v["private_segment_fixed_size"]} == {}
    assert {k for k, v in kernels.items() if v["vgpr_spill_count"]} == set()


def test_two_workgroups_of_a_record_fit_on_a_compute_unit(kernels):
    """chunk_few_kernel<1024, 4> of the types whose combination takes no more than 64 registers: f32, i32 and f16."""
    few = {k: v["vgpr_count"] for k, v in kernels.items() if re.search(r"16chunk_few_kernelILi1024ELi4ENS_(5OpF32|5OpI32|4Op16ILi\dENS_8WidenF16)", k)}
    assert len(few) >= 12 and max(few.values()) <= 64, few
