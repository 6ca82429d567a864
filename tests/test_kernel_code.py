"""What the compiler made of the GEMM's stores: the kind of store is part of a kernel's choice, and two
copies of a path that differ in nothing else are easily merged into one."""
import os
import re
import struct
import subprocess

import pytest

from paper_2503_06545_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BF16 = 1   # qc_out


def gfx950_code(path):
    """The gfx950 code objects of a library: bundles of (offset, size, target) with a magic in front."""
    blob, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        entry = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, entry)
            if b"gfx950" in blob[entry + 24:entry + 24 + length]:
                yield blob[at + offset:at + offset + size]
            entry += 24 + length
        at = blob.find(magic, at + 1)


@pytest.fixture(scope="module")
def wide_stores(tmp_path_factory):
    """{kernel's mangled name: [16 B stores through the caches, non-temporal ones]}"""
    if not os.path.exists(OBJDUMP) or not os.path.exists(binding.LIB_PATH):
        pytest.skip("needs the built library and llvm-objdump")
    found, kernel = {}, None
    for i, code in enumerate(gfx950_code(binding.LIB_PATH)):
        path = tmp_path_factory.mktemp("code") / f"{i}.o"
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for line in listing.splitlines():
            name = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if name:
                kernel = found.setdefault(name.group(1), [0, 0])
            elif kernel is not None and "global_store_dwordx4" in line:
                kernel[bool(re.search(r"\bnt\b", line))] += 1
    return found


@pytest.mark.parametrize("kernel,rows", [("gemm_kernel", 16), ("gemm_mid_kernel", 12), ("gemm_half_kernel", 8), ("gemm_split_half_kernel", 4)])
def test_ring_kernels_hold_both_kinds_of_store(wide_stores, kernel, rows):
    """A wavefront stores `rows` rows per lane, two pieces each in 32 bits and one in bf16, on a path for
    whole tiles, non-temporally, and on one for the others: through the caches, for bf16 either way."""
    seen = 0
    for name, counts in wide_stores.items():
        m = re.search(rf"{len(kernel)}{kernel}ILi(\d)ELi(\d)ELi(\d)ELb(\d)E", name)
        if m:
            assert counts == ([rows, 2 * rows] if int(m.group(2)) == BF16 else [2 * rows, 2 * rows]), name
            seen += 1
    assert seen == 2 * (3 * 2 + 3 * 2 + 1)   # weights x (f32: epilogue, zero point; bf16; int32)


@pytest.mark.parametrize("kernel,rows", [("gemm_cached_kernel", 16), ("gemm_mid_cached_kernel", 12), ("gemm_half_cached_kernel", 8)])
def test_ring_kernels_that_keep_their_output_store_through_the_caches(wide_stores, kernel, rows):
    mine = {name: counts for name, counts in wide_stores.items() if f"{len(kernel)}{kernel}I" in name}
    assert len(mine) == 2 * 3 * 2 and all(counts == [4 * rows, 0] for counts in mine.values())
