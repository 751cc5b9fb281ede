"""No register of the recurrences and projections over kept entries, or of the products on 16-bit planes, is spilled: what the compiler
recorded in the built library about its kernels (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_1901_10997_amd import build

LLVM = "/opt/rocm/llvm/bin"
TARGET = "hipv4-amdgcn-amd-amdhsa--gfx950"
KERNELS = ("persist_batched_q16_kernel", "persist_batched_hlstm_kernel", "proj_q16_kernel", "persist_rows_bf16_kernel", "persist_split_kernel",
           "persist_mfma_bf16_kernel")


def _spills(so, tmp):
    """kernel -> (vector registers spilled, bytes of private memory)"""
    fatbin = os.path.join(tmp, "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fatbin}", so, os.path.join(tmp, "unused")], check=True)
    data = open(fatbin, "rb").read()
    starts = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__|CCOB", data)] + [len(data)]   # a bundle per source file
    found = {}
    for a, b in zip(starts, starts[1:]):
        bundle, obj = os.path.join(tmp, "bundle"), os.path.join(tmp, "object")
        with open(bundle, "wb") as f:
            f.write(data[a:b])
        subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={bundle}", f"--targets={TARGET}", f"--output={obj}"], check=True)
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", obj], check=True, capture_output=True, text=True).stdout
        for text in notes.split("  - .agpr_count")[1:]:
            field = lambda key: re.search(rf"\.{key}:\s+(\S+)", text).group(1)
            found[field("name")] = (int(field("vgpr_spill_count")), int(field("private_segment_fixed_size")))
    return found


@pytest.mark.skipif(not all(os.path.exists(f"{LLVM}/{t}") for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")), reason="no LLVM tools")
def test_no_spilled_registers(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    found = _spills(build.LIB, str(tmp_path))
    for kernel in KERNELS:
        mine = {n: v for n, v in found.items() if kernel in n}
        assert mine, kernel
        assert not {n: v for n, v in mine.items() if v != (0, 0)}
