"""How the kernels that keep a head's or a super-block's workgroups together deal them out to the eight XCDs (CPU; the header is
plain C++): every workgroup of every head exactly once, and of fewer than eight heads equal shares, the first of all heads before the second."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_16381_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "xcd_deal.h"
int main(int c, char** v) {
    const int N = atoi(v[1]), BH = atoi(v[2]);
    if (c == 6) {          // chunks, heads, chunks per super-block, packed, turned
        const int sbc = atoi(v[3]);
        const unsigned grid = path::sb_grid(N, sbc, BH);
        printf("%u\n", grid);
        for (unsigned b = 0; b < grid; ++b) {
            const path::SbPlace p = path::sb_place((int)(b >> 3), b & 7, N, sbc, BH, atoi(v[4]), atoi(v[5]));
            if (p.bh < BH) printf("%u %d %d\n", b & 7, p.bh, p.chunk);
        }
        return 0;
    }
    for (unsigned b = 0; b < path::xcd_deal_grid(N, BH); ++b) {
        const path::XcdDivision q = path::xcd_division((int)(b >> 3), b & 7, N, BH);
        const path::XcdPlace p = path::xcd_place(q.num / q.den, q.num % q.den, b & 7, BH);
        if (p.bh < BH && p.r < N) printf("%u %d %d\n", b & 7, p.bh, p.r);
    }
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    d = tmp_path_factory.mktemp("deal")
    (d / "deal.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(d / "deal.cpp"), "-o", str(d / "deal")], check=True)
    return lambda *a: [tuple(map(int, l.split())) for l in subprocess.run([str(d / "deal"), *map(str, a)], capture_output=True, text=True, check=True).stdout.splitlines()]


@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 64, 127])
@pytest.mark.parametrize("BH", [1, 2, 3, 4, 6, 7, 8, 9, 12, 16, 20, 31, 32, 33, 64, 100])
def test_every_workgroup_once(deal, N, BH):
    got = deal(N, BH)
    assert sorted((bh, r) for _, bh, r in got) == [(bh, r) for bh in range(BH) for r in range(N)]
    if BH < 8:
        share = [sum(x == i for x, _, _ in got) for i in range(8)]
        assert max(share) - min(share) <= 1
        for i in range(8):
            ranks = [r for x, _, r in got if x == i]
            assert ranks == sorted(ranks)
    for x in range(8):                      # a head's workgroups in their order on each XCD
        mine = [(bh, r) for y, bh, r in got if y == x]
        assert all(a[1] < b[1] for a, b in zip(mine, mine[1:]) if a[0] == b[0])


@pytest.mark.parametrize("packed,turn", [(0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("NC,sbc", [(1, 16), (3, 16), (15, 16), (16, 16), (17, 16), (21, 16), (48, 16), (70, 16), (9, 4), (33, 8)])
@pytest.mark.parametrize("BH", [1, 3, 8, 9, 17, 99])
def test_chunks_of_super_blocks(deal, NC, sbc, BH, packed, turn):
    (grid,), *got = deal(NC, BH, sbc, packed, turn)
    assert sorted((bh, c) for _, bh, c in got) == [(bh, c) for bh in range(BH) for c in range(NC)]
    assert grid - len(got) <= 8 * sbc                            # idle workgroups: of pairs that are no multiple of eight
    share = [sum(x == i for x, _, _ in got) for i in range(8)]
    assert max(share) - min(share) <= sbc
    for x in range(8):                      # a pair's chunks one after the other on its XCD
        mine = [(bh, c) for y, bh, c in got if y == x]
        assert all(b == (a[0], a[1] + 1) for a, b in zip(mine, mine[1:]) if a[1] % sbc != sbc - 1 and a[1] != NC - 1)
