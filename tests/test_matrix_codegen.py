"""Matrix kernels, as compiled: the 2x2 product's entries are 32-bit multiplies
and additions.  The compiler can merge a product and an addition into a
64-bit multiply-add, and has then let the high half, which nothing wants,
overwrite another entry (kernels.hip dot2); which kernels that hits changes
with any edit, so none may hold the merged form.  Reads the gfx950 code of
the library built from this tree."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2109_12626_amd import dpar

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin",
                       "llvm-objdump")


def test_no_merged_multiply_add(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not available")
    lib = shutil.copy(dpar.LIB_PATH, tmp_path / "l.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True,
                   capture_output=True, cwd=tmp_path)
    code, = tmp_path.glob("l.so*gfx950*")
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(code)],
                          check=True, capture_output=True, text=True).stdout
    merged, products, kernel = {}, {}, None
    for line in text.splitlines():
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            kernel = head[1] if "LaneMat" in head[1] else None
        elif kernel:
            products[kernel] = products.get(kernel, 0) + ("v_mul_lo_u32" in
                                                          line)
            if re.search(r"v_mad_[ui]64_[ui]32", line):
                merged[kernel] = merged.get(kernel, 0) + 1
    # level, subtree, wide, post-order items in every executor, and few ranks
    assert len(products) > 60 and all(n >= 8 for n in products.values())
    assert not merged, merged
