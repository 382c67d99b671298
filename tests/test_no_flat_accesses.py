"""No kernel of the built library reads or writes memory with FLAT instructions (CPU; disassembles the library's own gfx950 code).  A FLAT access counts
among the LDS accesses too, and comes back in no order with the copies to LDS, whose landing several kernels wait for by the number of requests behind
them."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2505_16381_amd as pa

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_global_and_lds_accesses_only(tmp_path):
    pa.load_library()
    lib = shutil.copy(os.path.join(os.path.dirname(pa.__file__), "libpath_attn.so"), tmp_path)      # (its parts are written beside it)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    parts = [p for p in os.listdir(tmp_path) if p.endswith("gfx950")]
    assert len(parts) >= 10
    flat, accesses = [], 0
    for p in parts:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(tmp_path, p)], check=True, capture_output=True, text=True).stdout
        accesses += len(re.findall(r"^\s+global_(?:load|store)", text, re.M))
        fn = "?"
        for line in text.splitlines():
            if line.endswith(">:"):
                fn = line.split("<")[1][:-2]
            elif re.match(r"\s+flat_(?:load|store|atomic)", line):
                flat.append(fn)
    assert accesses > 1000
    assert not flat, sorted(set(flat))
