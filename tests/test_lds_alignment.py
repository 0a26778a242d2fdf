"""Kernels that read their dynamic LDS in 16-byte vectors start it on a
multiple of 16 bytes.  The dynamic part follows the static one, so the built
kernels' static size, from the code objects' metadata, says where it starts."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
VECTOR_LDS = ("k_hold", "k_block_run_staged", "k_batch_staged")


def static_lds(tmp_path):
    """{kernel symbol: bytes of static LDS} of the built library."""
    from paper_2205_01313_amd import _native
    if not os.path.exists(_native.LIB_PATH):
        from paper_2205_01313_amd import build
        build.build()
    lib = tmp_path / "lib.so"
    shutil.copy(_native.LIB_PATH, lib)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", str(lib)], check=True, capture_output=True)
    sizes = {}
    for obj in tmp_path.glob("lib.so.*gfx950"):
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        for size, name in re.findall(r"\.group_segment_fixed_size:\s*(\d+).*?\.name:\s*(\S+)", notes, flags=re.S):
            sizes[name] = int(size)
    return sizes


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="no llvm tools")
def test_vector_lds_starts_aligned(tmp_path):
    sizes = static_lds(tmp_path)
    for kernel in VECTOR_LDS:
        mine = {n: s for n, s in sizes.items() if f"{len(kernel)}{kernel}I" in n}
        assert mine, kernel
        assert all(s % 16 == 0 for s in mine.values()), {n: s for n, s in mine.items() if s % 16}
