// Argument structs and launchers of the decode-path kernels.
#pragma once
#include "path_common.h"

namespace path {

constexpr int DECODE_MAX_SPLITS = 60;
constexpr int DECODE_SPLIT_ROOM = 64;    // the workspace has room for so many records of d + 2 floats per head

struct PrefillArgs {
    const void *kt2, *dp2;   // second-level tiles of the forward workspace
    const void* v;           // [BH][L][d]
    void *kcache, *vcache;   // [BH][Lmax][d], cache storage type
    int L, NC, Lmax;
};

// The values of a prompt go to their cache unchanged, VROWS rows of a head per workgroup (of the launch that fills the
// key cache: a copy of its own takes 5 us of the stream's time).
constexpr int VROWS = 128;
__host__ __device__ inline int value_row_pieces(int L) { return (L + VROWS - 1) / VROWS; }
template <typename TIO, int D, int NT>
__device__ __forceinline__ void copy_value_rows(const void* v, void* vcache, int L, int Lmax, int bh, int piece, int tid) {
    typedef TIO Vec __attribute__((ext_vector_type(16 / sizeof(TIO))));
    constexpr int VPR = D * (int)sizeof(TIO) / 16;
    const int r0 = piece * VROWS, n = (L - r0 < VROWS ? L - r0 : VROWS) * VPR;
    const Vec* src = reinterpret_cast<const Vec*>(v) + ((size_t)bh * L + r0) * VPR;
    Vec* dst = reinterpret_cast<Vec*>(vcache) + ((size_t)bh * Lmax + r0) * VPR;
#pragma unroll 4
    for (int i = tid; i < n; i += NT) dst[i] = src[i];
}

struct DecodeArgs {
    const void *q, *k, *v, *w, *beta;   // the arriving token: [BH][d], beta [BH]
    void *kcache, *vcache;              // [BH][Lmax][d]
    void* o;                            // [BH][d]
    float* lse;                         // [BH]
    float* partial;                     // the workspace: records of the splits
    int n, Lmax;                        // cached tokens before the step
    float scale;
    // PaTH-FoX (NULL for plain PaTH): the arriving token's log gate [BH] (I/O type) and the running sums
    // c_i = sum_{s<=i} log f_s of the cached tokens, fp32 [BH][Lmax], natural logarithm; the step appends c_n
    const void* log_f;
    float* ccache;
    unsigned long long flag;            // this call's "record is there", set by the launcher; 0: a second launch merges (captured steps)
};

// The same chunk by chunk (16-bit operands): key tiles of the prompt, products of the blocks of cpb chunks.
struct CarryArgs {
    const void *kt, *dp;     // [BH][NC] key tiles at their block's right edge; [BH][ceil(NC/cpb)] tiles of -dP
    const void* v;           // [BH][L][d]
    void *kcache, *vcache;   // [BH][Lmax][d], cache storage type
    int BH, L, NC, Lmax, cpb;
};
// Chunk by chunk for few heads or short prompts: it does every product of a chunk's way for that chunk alone, in a chain of
// light steps on many CUs, where the other kernels run one chain of heavy steps per super-block or head and share the
// products.  The line, in products plus two per workgroup for its start, lies where both take as long; us, chunk by chunk
// against the others: d = 128, 16 heads of 1000 tokens (2432) 14.6 / 37.1, 135 of 500 (5940) 30.2 / 30.0, 132 of 1100 (5940) 33.4 /
// 34.8, 74 of 2048 (5920) 32.4 / 34.9, 14 of 6000 (5922) 29.3 / 40.9; d = 64, 163 of 1500 (9780) 22.7 / 25.3, 198 (11880) 26.6 / 26.7, 79 of
// 3143 (13825) 26.6 / 25.0.  One super-block at d = 64: up to 230 heads the others take as long as their one chain of chunks, 159 of
// 500 (6996) 13.5 / 12.1, 132 of 715 (11880) 17.5 / 16.1, 91 of 1000 (13832) 19.4 / 20.0; above, with a second round of workgroups, 315 of
// 500 (13860) 22.3 / 24.7, 693 of 300 (13860) 25.4 / 46.9.
inline bool carry_pays(int BH, int NC, int blocks, int d) {
    const long long work = (long long)BH * NC * (blocks + 3) / 2;
    if (d == 128) return work <= 6000;
    if (blocks < NC) return work <= 12000;
    return work <= (BH <= 230 && NC > 3 ? 900 * NC - 600 : 14000);
}
hipError_t launch_key_carry(const CarryArgs& a, int d, hipStream_t st);

hipError_t launch_key_prefill(const PrefillArgs& a, int BH, int d, int is_bf16, hipStream_t st);
hipError_t launch_decode_step(DecodeArgs a, int BH, int d, int is_bf16, hipStream_t st);

}  // namespace path
