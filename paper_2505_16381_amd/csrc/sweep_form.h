// Form of the forward sweep (plain C++): query chunks per workgroup of attn_few.hip, 0: the general form, attn_fwd2.hip.  n query chunks, NC key
// chunks, BH heads (a packed batch: chunks of its longest sequence, heads of all); fp32 operands, d = 64, have the form with one chunk and the
// general one, d = 128 the general one.
// One chunk where every chunk has a CU, and for two rounds of them, which the chains' different lengths fill evenly if they are not too
// short: forward, d = 128, us with one / two / general form: 16 heads of 1400 tokens 77 / 86 / 95, of 2000 94 / 104 / 121, 128 of 250 40 / 38 / 42;
// not in a ring, whose chains have one length (d = 64, 32 heads of 1024 79 / 70 / 81).  Two where every tile of two has a CU, and for three
// rounds if the chains are long: 32 heads of 2048 155 (general 169), 16 of 4000 177 / 216, of 6000 299 / 315, of 8000 444 / 448, where it ends;
// 64 of 1024 109 / 107; ring, 16 of 4096 350 / 386, d = 64 16 of 3072 150 / 160, 32 of 2048 152 / 150.  With more workgroups the two
// unsynchronised ones that the general form has on a CU fill its pipes better (64 of 8192 tokens 1817 / 1766, d = 64, 128 of 4096 733 / 606).
#pragma once
#include "xcd_deal.h"

namespace path {

XCD_FN int sweep_form(int n, int NC, int BH, bool ring) {
    const unsigned one = xcd_deal_grid(n, BH), two = xcd_deal_grid((n + 1) / 2, BH);
    if (one <= 256 || (one <= 512 && !ring && n >= 8)) return 1;
    return two <= 256 || (two <= 768 && NC >= (ring ? 48 : 32)) ? 2 : 0;
}

}  // namespace path
