"""How the far key-side kernel deals the blocks of a super-block's d x d product gradient to its waves (CPU; the header is
plain C++): for every super-block size that builds, each block is written exactly once and nothing outside the matrix is
read or written; other sizes do not compile."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16381_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include "far_blocks.h"
template <int S, int D> void deal() {
    using B = path::FarBlocks<S, D>;
    for (int pos = 0; pos < B::NPOS; ++pos)
        for (int wave = 0; wave < 2; ++wave)
            for (int a = 0; a < B::ROWS; ++a)
                for (int b = 0; b < B::COLS; ++b)
                    printf("%d %d %d\n", B::first_row(pos, wave) + a, B::first_col(pos) + b, (int)B::writes(pos, wave));
}
int main() { deal<CHUNKS, DIM>(); }
"""


def _compile(tmp_path, sbc, d):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(SOURCE)
    r = subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", f"-DCHUNKS={sbc}", f"-DDIM={d}", str(src), "-o", str(exe)], capture_output=True, text=True)
    return r, exe


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sbc", [4, 8, 16, 32])
def test_every_block_is_written_exactly_once(tmp_path, sbc, d):
    r, exe = _compile(tmp_path, sbc, d)
    assert r.returncode == 0, r.stderr
    rows = [tuple(map(int, line.split())) for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines()]
    n = d // 32
    assert all(0 <= a < n and 0 <= b < n for a, b, _ in rows)
    assert sorted((a, b) for a, b, w in rows if w) == [(a, b) for a in range(n) for b in range(n)]


@pytest.mark.parametrize("sbc", [2, 12])
def test_other_sizes_do_not_compile(tmp_path, sbc):
    r, _ = _compile(tmp_path, sbc, 128)
    assert r.returncode != 0 and "a power of two from 4 on" in r.stderr
