// Numbering of the kernels whose workgroups of one head read the same tiles (plain C++), N workgroups -- or groups of them --
// per head in the order r = 0 .. N-1 in which they should start, heaviest first: workgroup b runs on XCD b % 8, and that XCD takes
// heads xcd, xcd + 8, ... one after the other.  Fewer than eight heads would leave XCDs idle so: theirs are dealt out one by
// one, all heads' r = 0 first, and every XCD gets as many of them (to one), the heavy ones early.  Forward, us, one XCD per head
// against dealt out: d = 128, 4200 tokens, one head 171 / 132, three 172 / 138, five 176 / 144, seven 177 / 147; d = 64, 8192 tokens, one
// 182 / 134, three 185 / 142, five 191 / 181, seven 205 / 196; fp32, d = 64, 7000 tokens, one 761 / 573, seven 832 / 791, d = 128, 6000
// tokens, seven 1252 / 1255.  (Head after head, each dealt out to eight XCDs, gives them the same r of all heads: seven heads, d = 64,
// 223, fp32 at d = 128 1572, and the two groups of the far key sums of 2700 tokens all ran on two XCDs.)  From eight heads on it does
// not pay: every L2 then fetches every head (training step, 9 heads of 4096 tokens 740 / 908, 12 787 / 816, 17 1052 / 1520; 20 of
// 8192 2749 / 2686).
#pragma once

#ifdef __HIP__
#define XCD_FN __host__ __device__ inline
#else
#define XCD_FN inline
#endif

namespace path {

XCD_FN bool xcd_spread(int BH) { return BH < 8; }
XCD_FN unsigned xcd_deal_grid(int N, int BH) { return 8u * (unsigned)(xcd_spread(BH) ? (BH * N + 7) / 8 : (BH + 7) / 8 * N); }

// Workgroup number `slot` of XCD `xcd`: the division that gives its place (one for both forms), and the place from quotient and
// remainder; bh >= BH or r >= N: nothing to do.
struct XcdDivision { int num, den; };
XCD_FN XcdDivision xcd_division(int slot, int xcd, int N, int BH) { return xcd_spread(BH) ? XcdDivision{slot * 8 + xcd, BH} : XcdDivision{slot, N}; }
struct XcdPlace { int bh, r; };
XCD_FN XcdPlace xcd_place(int quotient, int rest, int xcd, int BH) { return xcd_spread(BH) ? XcdPlace{rest, quotient} : XcdPlace{quotient * 8 + xcd, rest}; }

// Numbering of the chunk workgroups of the chunk-transform adjoint: those of a (super-block, head) pair run on one XCD, first
// chunk -- the one with the most queries to its right -- first, and the pairs are dealt to the XCDs in order: head after head, or, in
// a packed batch, super-block after super-block, where the late ones exist in the long sequences only (`turn`: the heads turned by
// one per super-block, see chunk_and_head).  The last, partial super-blocks come behind the whole ones, with as many workgroups as
// they have chunks: an idle workgroup here waits for a CU's LDS like any other.  With sixteen for every pair a training step of
// 144 heads of 63 tokens, d = 128, took 101 us, so 64; 99 heads of 1320, gated, 1302 / 1111; d = 64, 96 heads of 1046, gated, 579 / 456.
// (All chunks dealt out without regard to pairs: 128 heads of 4096, d = 64, 2760 us, so 2650; 64 of 8192, d = 128, 8030 / 7720.)
// Chunk workgroup kk of XCD xcd; sbc chunks per super-block; bh >= BH: nothing to do.
struct SbPlace { int bh, chunk; };
XCD_FN SbPlace sb_place(int kk, int xcd, int NC, int sbc, int BH, bool packed, bool turn) {
    const int full = NC / sbc, rem = NC - full * sbc, P = full * BH;      // whole super-blocks of a head, chunks of the partial one; whole pairs
    const int F = P > xcd ? (P - xcd + 7) >> 3 : 0;                       // ... of this XCD
    const bool tail = kk >= F * sbc;
    if (tail && !rem) return {BH, 0};
    const int n = tail ? rem : sbc, k = tail ? kk - F * sbc : kk, q = k / n;
    const int p = (tail ? F + q : q) * 8 + xcd - (tail ? P : 0);
    if (tail && p >= BH) return {BH, 0};
    const int m = packed ? BH : tail ? 1 : full, hi = p / m, lo = p - hi * m;
    const int sb = tail ? full : packed ? hi : lo;
    int bh = packed ? lo : hi;
    if (packed && turn) bh = (bh + sb) % BH;
    return {bh, sb * sbc + k - q * n};
}
XCD_FN unsigned sb_grid(int NC, int sbc, int BH) {
    const int full = NC / sbc, rem = NC - full * sbc, P = full * BH, A = P + (rem ? BH : 0);
    unsigned most = 0;
    for (int x = 0; x < 8; ++x) {
        const int F = P > x ? (P - x + 7) / 8 : 0, n = A > x ? (A - x + 7) / 8 : 0;
        const unsigned w = (unsigned)(F * sbc + (n - F) * rem);
        if (w > most) most = w;
    }
    return 8 * most;
}

}  // namespace path
