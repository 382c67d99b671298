"""Layout of the chunk-transform adjoint's LDS tiles (CPU; the header is plain C++): every element has a place of its own, the lane's shares of
addresses, put together with the constants the kernel uses, are those places, and the two kinds of reads fall on all banks."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16381_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <set>
#include "lds_tile.h"
using namespace path;
#define CHECK(c) do { if (!(c)) { printf("%s, line %d\n", #c, __LINE__); return 1; } } while (0)
int main() {
    constexpr int W = WIDTH, ROWS = 128;
    typedef TurnedTile<W> L;
    std::set<int> places;
    for (int r = 0; r < ROWS; ++r)
        for (int c = 0; c < W; ++c) { const int a = L::at(r, c); CHECK(a >= r * W && a < (r + 1) * W); places.insert(a); }
    CHECK(places.size() == ROWS * W);
    const unsigned tile = 5 * 256;                     // any multiple of 256
    for (int tid = 0; tid < 512; ++tid) {
        const TurnedLane<W> t(tid);
        const int l32 = tid & 31, h = (tid >> 5) & 1, j = l32 & 15;
        auto byte = [&](int r, int c) { return tile + 2 * L::at(r, c); };
        for (int r0 = 0; r0 < ROWS; r0 += 32) {
            for (int c = 0; c < W; c += 16) CHECK(tile + t.nat_at(r0, c) == byte(r0 + l32, c + 8 * h));
            for (int c = 0; c < W; c += 8) CHECK(tile + t.vec_at(r0, c) == byte(r0 + l32, c + 4 * h));
            for (int c = 0; c < W; c += 32)
                for (int q = 0; q < 4; ++q)
                    for (int r = 0; r < 4; ++r) CHECK((TurnedLane<W>::elem_step(tile + t.elem_at(r0, c), q, r)) == byte(r0 + 8 * q + 4 * h + r, c + l32));
        }
        for (int k = 0; k < ROWS; k += 16)
            for (int c = 0; c < W; c += 32)
                for (int four = 0; four < 2; ++four) CHECK(tile + t.tr_at(k, c, four) == byte(k + 8 * h + (j >> 2) + 4 * four, c + (l32 & 16) + 4 * (j & 3)));
        for (int u = 0; u < ROWS * W / 4096; ++u) {
            const int idx = tid + 512 * u;
            CHECK(tile + t.copy_at(u) == byte(idx / (W / 8), idx % (W / 8) * 8));
        }
    }
    // sixteen rows' pieces of 16 bytes, and four rows' 64 bytes: 256 bytes on 64 banks
    for (int r0 = 0; r0 < ROWS; r0 += 16)
        for (int c = 0; c < W; c += 8) {
            std::set<int> b;
            for (int r = 0; r < 16; ++r) b.insert(L::at(r0 + r, c) * 2 % 256 / 16);
            CHECK(b.size() == 16);
        }
    for (int r0 = 0; r0 < ROWS; r0 += 4)
        for (int c = 0; c < W; c += 32) {
            std::set<int> b;
            for (int r = 0; r < 4; ++r)
                for (int e = 0; e < 32; e += 4) b.insert(L::at(r0 + r, c + e) * 2 % 256 / 8);
            CHECK(b.size() == 32);
        }
    return 0;
}
"""


@pytest.mark.parametrize("width", [64, 128])
def test_places_and_banks(tmp_path, width):
    src, exe = tmp_path / "tile.cpp", tmp_path / "tile"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", f"-DWIDTH={width}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
