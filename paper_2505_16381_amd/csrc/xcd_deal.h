// Numbering of the kernels whose workgroups of one head read the same tiles (plain C++), N workgroups -- or groups of them --
// per head in the order r = 0 .. N-1 in which they should start: workgroup b runs on XCD b % 8, and that XCD takes heads xcd,
// xcd + 8, ... one after the other.  Where there are fewer than XCD_PARTS_BELOW heads and no multiple of eight of them, each
// head is dealt out to two, four or eight XCDs, as many as make the XCDs' shares equal: else one head runs on one XCD of
// eight.  Forward / training step, us, one XCD per head against several, d = 128: one head of 16384 tokens 629 / 2376 -> 346 /
// 1448, two 660 / 2554 -> 382 / 1615, two of 4096 172 / 589 -> 142 / 533; two of 8192, d = 64, 182 / 657 -> 140 / 558 (with the
// sweep's form for few workgroups).  From eight heads on it does not pay: every L2 then fetches every head (training step, 9
// heads of 4096 tokens 740 / 908, 12 787 / 816, 17 1052 / 1520; 20 of 8192 2749 / 2686).
#pragma once

#ifdef __HIP__
#define XCD_FN __host__ __device__ inline
#else
#define XCD_FN inline
#endif

namespace path {

#ifndef XCD_PARTS_BELOW
#define XCD_PARTS_BELOW 8
#endif

// (powers of two as shifts: a division would run on the vector unit and leave everything derived from it there)
XCD_FN int xcd_parts_log2(int BH) { return BH >= XCD_PARTS_BELOW || !(BH & 7) ? 0 : BH & 1 ? 3 : BH & 2 ? 2 : 1; }
XCD_FN int xcd_per_part(int N, int BH) { return (N + (1 << xcd_parts_log2(BH)) - 1) >> xcd_parts_log2(BH); }
XCD_FN unsigned xcd_deal_grid(int N, int BH) { return 8u * (unsigned)(((BH << xcd_parts_log2(BH)) + 7) / 8) * (unsigned)xcd_per_part(N, BH); }

struct XcdPlace { int bh, r; };
// workgroup number `slot` of its XCD, as slot = round * xcd_per_part + rest; bh >= BH or r >= N: nothing to do
XCD_FN XcdPlace xcd_place(int round, int rest, int xcd, int BH) {
    const int s = xcd_parts_log2(BH), v = round * 8 + xcd;
    return {v >> s, (rest << s) + (v & ((1 << s) - 1))};
}

}  // namespace path
