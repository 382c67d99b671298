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

}  // namespace path
