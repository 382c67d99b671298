"""Which form the forward sweep takes (CPU; the header is plain C++): sizes on both sides of each line of the rule."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16381_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "sweep_form.h"
int main(int, char** v) { printf("%d", path::sweep_form(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0)); }
"""


@pytest.mark.parametrize("chunks,heads,ring,form", [
    (32, 8, False, 1), (33, 8, False, 1), (64, 8, False, 1), (65, 8, False, 2), (32, 8, True, 1), (33, 8, True, 2),      # one round of workgroups, two
    (8, 64, False, 1), (7, 72, False, 0), (4, 96, False, 2), (5, 96, False, 0),                                         # ... two of long chains only
    (34, 24, False, 2), (34, 40, False, 2), (34, 48, False, 0), (31, 48, False, 0), (32, 48, False, 2),                 # three rounds of two chunks
    (47, 24, True, 0), (48, 24, True, 2), (49, 32, True, 0)])
def test_rule(tmp_path, chunks, heads, ring, form):
    src, exe = tmp_path / "form.cpp", tmp_path / "form"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(chunks), str(chunks), str(heads), str(int(ring))], check=True, capture_output=True, text=True)
    assert int(r.stdout) == form
