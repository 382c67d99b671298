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
inline int value_row_pieces(int L) { return (L + VROWS - 1) / VROWS; }
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
    unsigned long long flag;            // this call's "record is there", set by the launcher
};

hipError_t launch_key_prefill(const PrefillArgs& a, int BH, int d, int is_bf16, hipStream_t st);
hipError_t launch_decode_step(DecodeArgs a, int BH, int d, int is_bf16, hipStream_t st);

}  // namespace path
