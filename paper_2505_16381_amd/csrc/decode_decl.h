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
// against the others: d = 128, 16 heads of 1000 tokens (2432) 15.1 / 37.4, of 4000 (3528) 21.8 / 36.1, 32 of 1000 (4864)
// 28.5 / 40.7, 64 of 2048 (5120) 33.5 / 34.4, 32 of 4096 (7168) 40.0 / 37.8, 64 of 1000 (9728) 47.0 / 44.8; d = 64, 64 of
// 1000 (9728) 16.3 / 19.6, 128 of 1000 (19456) 26.5 / 23.9, 32 of 8192 (22528) 32.0 / 27.7.
inline bool carry_pays(int BH, int NC, int blocks, int d) { return (long long)BH * NC * (blocks + 3) / 2 <= (d == 64 ? 14000 : 6000); }
hipError_t launch_key_carry(const CarryArgs& a, int d, hipStream_t st);

hipError_t launch_key_prefill(const PrefillArgs& a, int BH, int d, int is_bf16, hipStream_t st);
hipError_t launch_decode_step(DecodeArgs a, int BH, int d, int is_bf16, hipStream_t st);

}  // namespace path
