// How the far key-side kernel deals the 32x32 blocks of a super-block's dP_superblock ([d][d]) to its workgroups and waves
// (plain C++: the test of the deal compiles it alone).
//
// A super-block has SBC / 2 workgroups of two key waves each (two key chunks per workgroup).  Workgroups form groups of
// GPC that share COLS column blocks; a workgroup stages those rows of the gT tiles, and slot s of the group's 2 GPC waves
// takes row blocks ROWS s .. ROWS s + ROWS - 1.  Where there are more waves than blocks the slots past the last one repeat
// earlier blocks and do not write them.  16 chunks: one block per wave at d = 128, the first two of eight slots at d = 64.
#pragma once

namespace path {

template <int SBC, int D> struct FarBlocks {
    static constexpr int DB = D / 32, NPOS = SBC / 2;
    static_assert(SBC >= 4 && (SBC & (SBC - 1)) == 0, "chunks per super-block: a power of two from 4 on");
    static constexpr int GPC = NPOS > DB ? NPOS / DB : 1;             // workgroups that share column blocks
    static constexpr int COLS = NPOS > DB ? 1 : DB / NPOS;            // column blocks per workgroup
    static constexpr int ROWS = 2 * GPC > DB ? 1 : DB / (2 * GPC);    // row blocks per wave
    static constexpr int SLOTS = DB / ROWS;                           // slots that write
    static constexpr int first_col(int pos) { return pos / GPC * COLS; }
    static constexpr int slot(int pos, int wave) { return 2 * (pos % GPC) + wave; }
    static constexpr int first_row(int pos, int wave) { return slot(pos, wave) % SLOTS * ROWS; }
    static constexpr bool writes(int pos, int wave) { return slot(pos, wave) < SLOTS; }
};

}  // namespace path
