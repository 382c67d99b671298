"""The waves of the sweep for few workgroups that make the tile copies do not wait for those they have just requested before they multiply (CPU;
disassembles the library's own gfx950 code): the compiler, left to place the wait for the products' operands, waits for all requests there."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2505_16381_amd as pa

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_wait_for_all_between_copies_and_products(tmp_path):
    pa.load_library()
    lib = shutil.copy(os.path.join(os.path.dirname(pa.__file__), "libpath_attn.so"), tmp_path)      # (its parts are written beside it)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    kernels, waits = 0, []
    for p in (p for p in os.listdir(tmp_path) if p.endswith("gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(tmp_path, p)], check=True, capture_output=True, text=True).stdout
        for body in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, code = body.split(">", 1)
            if "attn_few_kernel" not in name:
                continue
            kernels += 1
            requested = False
            ops = [l.split("//")[0].strip() for l in code.splitlines()[1:] if l.startswith("\t")]
            for n, op in enumerate(ops):
                if op.startswith("global_load_lds"):
                    requested = True
                elif op.startswith("s_barrier"):
                    requested = False
                elif requested and re.match(r"s_waitcnt vmcnt\(0\)", op) and any(o.startswith("v_mfma") for o in ops[n + 1:n + 4]):
                    waits.append(name)
    assert kernels >= 20
    assert not waits, sorted(set(waits))
