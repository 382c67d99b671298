// Shared device-side definitions of the PaTH attention kernels (gfx950 only).
//
// Register/fragment conventions used by every kernel
// --------------------------------------------------
// All contractions run on the 32x32 MFMA tile of a 64-lane wavefront.  Lane
// l = 32*h + c (h = l/32, c = l%32) owns column c of the 32x32 fp32 result;
// its 16 accumulator registers j = 0..15 hold rows
//
//        acc_row(j, h) = 8*(j/4) + 4*h + (j%4).
//
// An operand fragment is 16 bytes per lane: FE = 8 bf16 or 4 fp32 elements.
// One "slab" is what one fragment pair contracts: KW = 2*FE indices
// (bf16: one v_mfma_f32_32x32x16_bf16; fp32: four v_mfma_f32_32x32x2_f32).
//
// Activations (query state X, probabilities P) never leave registers: a
// result in accumulator layout is re-used as the B operand of the next
// contraction by packing registers [s*FE, (s+1)*FE) of a 32-row block into
// slab s.  That fixes which contraction index sits in which fragment element,
//
//        index(block b, slab s, half h, element e) = 32*b + acc_row(s*FE+e, h),
//
// so the other operand (K, V^T, chunk products), which streams through LDS,
// is stored by the preprocessing kernel in exactly that order ("fragment
// order"): fragment ((rb*(Kc/KW) + slab)*64 + lane) of a tile with rows
// 32*rb + c and Kc contraction indices.  Lanes then read consecutive 16-byte
// fragments: conflict-free LDS reads and linear global->LDS copies.  (16-bit
// tiles of keys, -dP, query states, dO, R_c and its gradient exchange lanes
// inside a slab, tile_lane() for lane, so that they can be read transposed too.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xcd_deal.h"

namespace path {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half_t;
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int CHUNK = 64;      // tokens per chunk (UT transform block)
#ifndef PATH_SBC
#define PATH_SBC 16            // a power of two from 4 on.  Training step at B=4, H=16, L=8192, d=128: 8.14 ms; with 8 chunks 8.11, 32 8.79,
                               // 4 11.4; 16 heads of 2048 tokens 498 us, 422, 406, 484 (the path_attn_ring_* contract is stated for 16)
#endif
constexpr int SBC = PATH_SBC;  // chunks per super-block (second blocking level of the forward sweep)

__device__ __forceinline__ int acc_row(int j, int h) { return 8 * (j >> 2) + 4 * h + (j & 3); }

template <typename T> struct Tr;

template <> struct Tr<bf16_t> {
    static constexpr int FE = 8;    // elements per 16-byte fragment
    static constexpr int KW = 16;   // contraction indices per slab
    typedef bf16x8 Frag;
    typedef bf16x4 Vec4;            // 4 consecutive elements
    static __device__ __forceinline__ f32x16 mma(Frag a, Frag b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    // slab s of a 32-row accumulator block as an operand fragment
    template <int S> static __device__ __forceinline__ Frag pack(const f32x16& a) {
        Frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (bf16_t)a[S * 8 + e];
        return f;
    }
    static __device__ __forceinline__ Frag zero() { Frag f; for (int e = 0; e < 8; ++e) f[e] = (bf16_t)0.0f; return f; }
};

template <> struct Tr<half_t> {
    static constexpr int FE = 8;
    static constexpr int KW = 16;
    typedef halfx8 Frag;
    typedef halfx4 Vec4;
    static __device__ __forceinline__ f32x16 mma(Frag a, Frag b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    template <int S> static __device__ __forceinline__ Frag pack(const f32x16& a) {
        Frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (half_t)a[S * 8 + e];
        return f;
    }
    static __device__ __forceinline__ Frag zero() { Frag f; for (int e = 0; e < 8; ++e) f[e] = (half_t)0.0f; return f; }
};

template <> struct Tr<float> {
    static constexpr int FE = 4;
    static constexpr int KW = 8;
    typedef f32x4 Frag;
    typedef f32x4 Vec4;
    static __device__ __forceinline__ f32x16 mma(Frag a, Frag b, f32x16 c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
        return c;
    }
    template <int S> static __device__ __forceinline__ Frag pack(const f32x16& a) {
        Frag f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = a[S * 4 + e];
        return f;
    }
    static __device__ __forceinline__ Frag zero() { Frag f = {0.f, 0.f, 0.f, 0.f}; return f; }
};

// Operand type of the TRANSPORTED quantities (query state, boundary-adjusted
// keys, chunk products and everything inside the chunk transform) for a given
// I/O type.  With bf16 I/O these are carried in fp16: they are not
// representable in the input precision, and their rounding -- not the
// inputs' -- sets the error of the logits; bf16's 8 significand bits leave the
// log-sum-exp about 1.1e-3..2.8e-3 off, fp16's 11 bits about 2e-4, at the same
// MFMA rate.  (The method's transitions are contractions for beta in [0,2],
// |w| <= 1, so these operands are bounded by the norms of q and k, which must
// stay below the fp16 maximum 65504.)  P and V stay in the I/O type.
template <typename TIO> struct Compute { typedef TIO type; };
template <> struct Compute<bf16_t> { typedef half_t type; };

// a * b, element by element, rounded once, to 16 bits.  (Written as a product and a conversion, four at a time, it is rounded to 32 bits first: 6e-5
// of the results then are the other neighbour of a tie.)
__device__ __forceinline__ halfx4 mul_once(f32x4 a, f32x4 b) {
    union { unsigned w[2]; halfx4 v; } u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(u.w[i]) : "v"(a[2 * i]), "v"(b[2 * i]));
        asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(u.w[i]) : "v"(a[2 * i + 1]), "v"(b[2 * i + 1]));
    }
    return u.v;
}

template <typename TO, typename TI>
__device__ __forceinline__ typename Tr<TO>::Frag cvt_frag(const typename Tr<TI>::Frag& f) {
    typename Tr<TO>::Frag o;
#pragma unroll
    for (int e = 0; e < Tr<TI>::FE; ++e) o[e] = (TO)(float)f[e];
    return o;
}

// Number of slabs in a 32-index block / in Kc indices.
template <typename T> constexpr int slabs_per_block() { return 32 / Tr<T>::KW; }

// All slabs of one 32-row accumulator block -> operand fragments dst[0 .. 32/KW).
template <typename T> __device__ __forceinline__ void pack_block(const f32x16& a, typename Tr<T>::Frag* dst);
template <> __device__ __forceinline__ void pack_block<bf16_t>(const f32x16& a, bf16x8* dst) {
    dst[0] = Tr<bf16_t>::pack<0>(a);
    dst[1] = Tr<bf16_t>::pack<1>(a);
}
template <> __device__ __forceinline__ void pack_block<half_t>(const f32x16& a, halfx8* dst) {
    dst[0] = Tr<half_t>::pack<0>(a);
    dst[1] = Tr<half_t>::pack<1>(a);
}
template <> __device__ __forceinline__ void pack_block<float>(const f32x16& a, f32x4* dst) {
    dst[0] = Tr<float>::pack<0>(a);
    dst[1] = Tr<float>::pack<1>(a);
    dst[2] = Tr<float>::pack<2>(a);
    dst[3] = Tr<float>::pack<3>(a);
}

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int j = 0; j < 16; ++j) z[j] = 0.f;
    return z;
}

template <typename T>
__device__ __forceinline__ typename Tr<T>::Frag ld_frag(const T* p) {
    return *reinterpret_cast<const typename Tr<T>::Frag*>(p);
}

// acc += A[arow0 + c][0..Kc) . B[brow0 + c'][0..Kc)  for a 32x32 block; both
// operands are stored with the contraction index contiguous.
template <typename T, int Kc>
__device__ __forceinline__ f32x16 gemm32(const T* A, int lda, int arow0, const T* Bm, int ldb,
                                         int brow0, int l32, int h, f32x16 acc) {
    constexpr int FE = Tr<T>::FE, KW = Tr<T>::KW;
    const T* ap = A + (size_t)(arow0 + l32) * lda + FE * h;
    const T* bp = Bm + (size_t)(brow0 + l32) * ldb + FE * h;
#pragma unroll
    for (int k0 = 0; k0 < Kc; k0 += KW) acc = Tr<T>::mma(ld_frag<T>(ap + k0), ld_frag<T>(bp + k0), acc);
    return acc;
}

// Same with lane-specific row pointers (already offset by the row and by FE*h).
template <typename T, int Kc>
__device__ __forceinline__ f32x16 gemm_rows(const T* ap, const T* bp, f32x16 acc) {
    constexpr int KW = Tr<T>::KW;
#pragma unroll
    for (int k0 = 0; k0 < Kc; k0 += KW) acc = Tr<T>::mma(ld_frag<T>(ap + k0), ld_frag<T>(bp + k0), acc);
    return acc;
}

// Operand fragment of a matrix stored [k][row] (row contiguous) for the lane (l32, h) of a 32x32x16 product:
// the eight values X[kk + 8h + e][r0 + l32], e = 0..7.  Two transposing LDS reads (ds_read_b64_tr_b16): in
// each block of 16 lanes, lane j supplies the address of four consecutive values, and lane i receives
// element i % 4 of the chunks of lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4.  With lane j pointing at
// X[kb + j/4][rb + 4 (j%4)], lane i therefore gets X[kb + e][rb + i], e = 0..3.
template <typename T>
__device__ __forceinline__ typename Tr<T>::Frag ld_frag_tr(const T* X, int ld, int kk, int r0, int l32, int h) {
    static_assert(sizeof(T) == 2, "16-bit transposing reads");
    typedef short v4s __attribute__((ext_vector_type(4)));
    const int j = l32 & 15;
    const T* p = X + (kk + 8 * h + (j >> 2)) * ld + r0 + (l32 & 16) + 4 * (j & 3);
    union { v4s v[2]; typename Tr<T>::Frag f; } u;
    u.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p));
    u.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p + 4 * ld));
    return u.f;
}

// The same with the contraction index in accumulator order: the values X[kk + acc_row(e, h)][r0 + l32], e = 0..7, which
// is how a packed accumulator block orders them.
template <typename T>
__device__ __forceinline__ typename Tr<T>::Frag ld_frag_tr_acc(const T* X, int ld, int kk, int r0, int l32, int h) {
    static_assert(sizeof(T) == 2, "16-bit transposing reads");
    typedef short v4s __attribute__((ext_vector_type(4)));
    const int j = l32 & 15;
    const T* p = X + (kk + 4 * h + (j >> 2)) * ld + r0 + (l32 & 16) + 4 * (j & 3);
    union { v4s v[2]; typename Tr<T>::Frag f; } u;
    u.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p));
    u.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p + 8 * ld));
    return u.f;
}

// acc[m][n] += sum_k A(m,k) B(n,k) as below, fp32 operands: a fragment is four contraction indices 8 s + 4 h + e; where they run along the rows of the stored
// matrix they are four 4-byte reads, of 32 neighbouring columns each.
template <int K, bool TA, bool TB>
__device__ __forceinline__ void mm_f32(f32x16& acc, const float* A, int lda, int ar0, const float* B, int ldb, int br0, int l32, int h) {
    auto frag = [&](const float* X, int ld, int r0, int k, bool tr) {
        f32x4 f;
        if (tr) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = X[(k + e) * ld + r0 + l32];
        } else {
            f = ld_frag<float>(X + (r0 + l32) * ld + k);
        }
        return f;
    };
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 32) {
        f32x4 fa[4], fb[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = k0 + 8 * s + 4 * h;
            fa[s] = frag(A, lda, ar0, k, TA);
            fb[s] = frag(B, ldb, br0, k, TB);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = Tr<float>::mma(fa[s], fb[s], acc);
    }
}

// acc[m][n] += sum_k A(m,k) B(n,k) for one 32x32 block (rows ar0.., columns br0..).
// TA == false: A is stored [m][k] (16-byte fragment reads); TA == true: A is stored [k][m] (transposing reads).  Same for B.
template <typename T, int K, bool TA, bool TB>
__device__ __forceinline__ void mm(f32x16& acc, const T* A, int lda, int ar0, const T* B, int ldb, int br0, int l32, int h) {
    if constexpr (sizeof(T) == 4) { mm_f32<K, TA, TB>(acc, A, lda, ar0, B, ldb, br0, l32, h); return; } else {
    // four slabs (64 contraction indices) at a time: their fragments are fetched ahead of the four products
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 64) {
        typename Tr<T>::Frag fa[4], fb[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = k0 + 16 * s + 8 * h;
            if (TA) {
                fa[s] = ld_frag_tr<T>(A, lda, k0 + 16 * s, ar0, l32, h);
            } else {
                fa[s] = ld_frag<T>(A + (ar0 + l32) * lda + k);
            }
            if (TB) {
                fb[s] = ld_frag_tr<T>(B, ldb, k0 + 16 * s, br0, l32, h);
            } else {
                fb[s] = ld_frag<T>(B + (br0 + l32) * ldb + k);
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(fa[s], fb[s], acc);
    }
    }
}

// Place of lane `lane`'s fragment inside slab s of the tiles that, with 16-bit operands, are also read transposed (see
// below) -- keys and -dP of both levels, query states, dO: half 1 moves by four rows and odd slabs by eight.  A linear
// read of a slab touches the same 1 KB either way.  fp32 tiles keep plain lane order.
template <typename T> __device__ __forceinline__ int tile_lane(int lane, int s) {
    return sizeof(T) == 2 ? lane ^ ((lane >> 5) << 2) ^ ((s & 1) << 3) : lane;
}

// Fragment of the TRANSPOSE of a fragment-order tile (rows q in 32-row halves of DS slabs, contraction c).  Element e
// of a fragment belongs to contraction index 16 s + acc_row(e, h) of its slab s, in both tiles, so the lane needs
// tile[q = 16 qs + acc_row(e, h)][c = 32 b + l32], e = 0..7: two transposing reads, of rows 16 qs + 4 h + 0..3 and the
// same + 8 (in each block of 16 lanes, lane i points at 4 consecutive c of row .. + i/4 and receives column i of the
// four rows).  The 32 lanes of a half-wave point at four rows of two slabs and both halves of each: with fragments
// in plain lane order those would lie 512 bytes apart, on the same banks -- 8.4 LDS cycles per read; the order of
// tile_lane spreads them over all banks -- 2.4 cycles, the rate of a linear read.
template <typename E, int DS>
__device__ __forceinline__ typename Tr<E>::Frag ld_tile_frag_tr(const E* tile, int qs, int b, int l32, int h) {
    static_assert(sizeof(E) == 2, "16-bit transposing reads");
    typedef short v4s __attribute__((ext_vector_type(4)));
    const int i = l32 & 15, sl = l32 >> 4, hh = i & 1;
    const int row = (4 * h + (i >> 2)) ^ (4 * hh), odd = 8 * sl;      // + 16 (qs & 1)
    const E* p = tile + (size_t)((((qs >> 1) * DS + 2 * b) * 64 + 16 * (qs & 1)) * 8) + (sl * 64 + hh * 32 + row) * 8 + 4 * ((i >> 1) & 1);
    union { v4s v[2]; typename Tr<E>::Frag f; } u;
    u.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p + odd * 8));
    u.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p + (8 - odd) * 8));
    return u.f;
}

// Four fragments of the transpose of a tile, (QS0, B0) .. (QS3, B3), as ld_tile_frag_tr gives them, for a wave that has copies
// to LDS in flight: the compiler has a transposing read (the builtin) wait for all of them.  The block waits for its own reads.
struct TileTr { unsigned even, odd; };      // LDS byte addresses of the lane's two reads of fragment (0, 0)
template <typename E>
__device__ __forceinline__ TileTr tile_tr(const E* tile, int l32, int h) {
    const int i = l32 & 15, sl = l32 >> 4, hh = i & 1;
    const int row = (4 * h + (i >> 2)) ^ (4 * hh), odd = 8 * sl;
    const unsigned p = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)tile + (unsigned)(((sl * 64 + hh * 32 + row) * 8 + 4 * ((i >> 1) & 1)) * 2);
    return {p + odd * 16, p + (8 - odd) * 16};
}
template <typename E, int DS, int QS0, int B0, int QS1, int B1, int QS2, int B2, int QS3, int B3>
__device__ __forceinline__ void ld_tile_frags_tr(const TileTr& a, typename Tr<E>::Frag (&f)[4]) {
    static_assert(sizeof(E) == 2, "16-bit transposing reads");
    union U { unsigned long long v[2]; typename Tr<E>::Frag f; } u[4];
#define TILE_TR_OFF(qs, b) ((((qs) >> 1) * DS + 2 * (b)) * 64 + 16 * ((qs) & 1)) * 16
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %9 offset:%10\n\t"
                 "ds_read_b64_tr_b16 %2, %8 offset:%11\n\tds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
                 "ds_read_b64_tr_b16 %4, %8 offset:%12\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
                 "ds_read_b64_tr_b16 %6, %8 offset:%13\n\tds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(u[0].v[0]), "=&v"(u[0].v[1]), "=&v"(u[1].v[0]), "=&v"(u[1].v[1]), "=&v"(u[2].v[0]), "=&v"(u[2].v[1]), "=&v"(u[3].v[0]), "=&v"(u[3].v[1])
                 : "v"(a.even), "v"(a.odd), "n"(TILE_TR_OFF(QS0, B0)), "n"(TILE_TR_OFF(QS1, B1)), "n"(TILE_TR_OFF(QS2, B2)), "n"(TILE_TR_OFF(QS3, B3))
                 : "memory");
#undef TILE_TR_OFF
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = u[k].f;
}

// p, the same for the whole wave, plus a lane's 32-bit offset, as an access takes it from scalar registers and one vector register.  (Left
// to itself the compiler keeps per-lane 64-bit pointers across loops: vector arithmetic, and two address registers per lane.  A pointer to
// global memory: rebuilt from an integer it would otherwise be a generic one, and an access through it FLAT, which has no scalar base,
// counts among the LDS accesses too and is in no order with the copies to LDS.  With the copies
// to LDS this way, us: forward of 128 heads of 4096 tokens, d = 64, 649 -> 614, 64 of 8192, d = 128, 1818 -> 1780, 16 of 1000 51.5 ->
// 50.2; adjoint scan 1919 -> 1903, chunk stage 1472 -> 1447 at the second shape.  Not in the far key sums, whose copying waves have vector
// issue to spare: 64 heads of 8192 tokens, d = 64, 1177 -> 1198, d = 128 1838 -> 1856.)
typedef const __attribute__((address_space(1))) char* GlobalBytes;
__device__ __forceinline__ GlobalBytes scalar_base(const void* p, unsigned lane_offset) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    asm volatile("" : "+v"(lane_offset));        // (its extension to 64 bits stays here, where the access absorbs it)
    return reinterpret_cast<GlobalBytes>((unsigned long long)hi << 32 | lo) + lane_offset;
}

// Linear copy of NFRAG 16-byte fragments global -> LDS, asynchronous (direct-to-LDS), by a workgroup of
// NT threads.  One instruction moves 64 consecutive fragments (lane = fragment); wave wv takes the
// groups wv*NPT .. wv*NPT + NPT-1 (NPT = NFRAG / NT), which are 1 KB apart, so that one
// global address and one LDS base per four groups do: the instruction's immediate offset (added to both
// sides, at most 4095) covers the rest.
template <int NT, int NFRAG, bool SCALAR = true, typename Frag>
__device__ __forceinline__ void async_copy_tile(const Frag* g, Frag* s, int tid, int wv) {
    static_assert(sizeof(Frag) == 16 && NFRAG % 64 == 0 && (NFRAG % NT == 0 || NFRAG < NT), "whole groups of fragments");
    const unsigned lane = (tid & 63) * 16;
    auto at = [&](const Frag* p) { return SCALAR ? scalar_base(p, lane) : (GlobalBytes)(reinterpret_cast<const char*>(p) + lane); };
    if (NFRAG < NT) {          // fewer groups than waves: the first NFRAG/64 waves take one each (wave-uniform test)
        if (wv * 64 < NFRAG)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(at(g + wv * 64)),
                                             (__attribute__((address_space(3))) void*)(s + wv * 64), 16, 0, 0);
        return;
    }
    constexpr int NPT = NFRAG / NT > 0 ? NFRAG / NT : 1;
#pragma unroll
    for (int i0 = 0; i0 < NPT; i0 += 4) {
        const GlobalBytes ga = at(g + (wv * NPT + i0) * 64);
        Frag* sa = s + (wv * NPT + i0) * 64;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)ga, (__attribute__((address_space(3))) void*)sa, 16, 0, 0);
        if (i0 + 1 < NPT) __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)ga, (__attribute__((address_space(3))) void*)sa, 16, 1024, 0);
        if (i0 + 2 < NPT) __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)ga, (__attribute__((address_space(3))) void*)sa, 16, 2048, 0);
        if (i0 + 3 < NPT) __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)ga, (__attribute__((address_space(3))) void*)sa, 16, 3072, 0);
    }
}
__device__ __forceinline__ void wait_async_and_sync() {
    __builtin_amdgcn_s_waitcnt(0x0000);   // vmcnt(0) expcnt(0) lgkmcnt(0): this wave's copies have landed
    __syncthreads();
}

// This wave's LDS writes are done; then everybody's.  Loads and direct-to-LDS copies stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// This wave's direct-to-LDS copies have landed.
__device__ __forceinline__ void copies_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Identity operand for transposing a 32x32 block through the matrix unit: with the block given as
// an A operand (rows r, contraction k; i.e. packed from accumulators that hold it as rows k, lane r),
// D = A * I comes out with rows r, lane k -- the transposed register layout.  Slab s of the identity
// B operand for lane (column l32, half h): element e is 1 where the contraction index equals l32.
template <typename T>
__device__ __forceinline__ void identity_frags(typename Tr<T>::Frag* id, int l32, int h) {
    constexpr int FE = Tr<T>::FE, SPB = 32 / Tr<T>::KW;
#pragma unroll
    for (int s = 0; s < SPB; ++s)
#pragma unroll
        for (int e = 0; e < FE; ++e) id[s][e] = (T)((acc_row(s * FE + e, h) == l32) ? 1.f : 0.f);
}
// out (rows r, lane k) = transpose of the 32x32 block whose operand fragments (rows r, contraction k) are a[0..SPB)
template <typename T>
__device__ __forceinline__ f32x16 transpose32(const typename Tr<T>::Frag* a, const typename Tr<T>::Frag* id) {
    f32x16 o = zero16();
#pragma unroll
    for (int s = 0; s < 32 / Tr<T>::KW; ++s) o = Tr<T>::mma(a[s], id[s], o);
    return o;
}

// Workspace carve-up shared by host launch code and kernels (byte offsets, 256-aligned).
struct FwdWorkspace {
    size_t kt, vt, dp, xinit, sd, kt2, dp2, cum, total;
};

// Layout of the caller's tensors: element strides of the batch, head and token index, for the
// [.,.,.,d] tensors (q, k, v, w, o and the gradients; d contiguous) and for the per-token scalars
// (beta, lse, log f and their gradients).  [B,H,L,d]: {H*L*d, L*d, d | H*L, L, 1};
// [B,L,H,d]: {L*H*d, d, H*d | L*H, 1, H}.  H = heads per batch entry (bh = b * H + h).
// bh0: the kernels of one launch may work on a slice of the heads (a backward that passes over the heads in
// groups to bound its workspace); they number their heads from 0, and head bh of the launch is head bh0 + bh of
// the caller's tensors.
// cu (device pointer, NULL for batches of one length): packed variable-length batches [T,H,d] / [T,H].  Batch
// entry b is the sequence of the tokens cu[b] .. cu[b+1]-1; its length replaces the launch's L in every bound
// (the launch's L and chunk count remain the STRIDES of the workspace arrays, sized for the longest sequence),
// and its tensors start at token cu[b] (vt, st are the token strides; vb, sb are not used).
struct UserLayout {
    long long vb, vh, vt, sb, sh, st;
    int H;
    int bh0;
    const int* cu;
};
__device__ __forceinline__ long long user_vec(const UserLayout& u, int bh, long long t) {
    bh += u.bh0;
    if (u.cu) return ((long long)u.cu[bh / u.H] + t) * u.vt + (bh % u.H) * u.vh;
    return (bh / u.H) * u.vb + (bh % u.H) * u.vh + t * u.vt;
}
__device__ __forceinline__ long long user_scl(const UserLayout& u, int bh, long long t) {
    bh += u.bh0;
    if (u.cu) return ((long long)u.cu[bh / u.H] + t) * u.st + (bh % u.H) * u.sh;
    return (bh / u.H) * u.sb + (bh % u.H) * u.sh + t * u.st;
}
// Numbering of the kernels that run one workgroup per (chunk, head), as a one-dimensional grid of NC * BH
// workgroups.  One length: chunks first, neighbours read neighbouring memory (heads first costs a [B,L,H,d] batch of
// 4 x 3000 tokens 5 % of the chunk transform).  Packed batch: heads first, chunk by chunk -- workgroup n runs on XCD
// n % 8, and with chunks first an XCD would take the same chunk numbers of every sequence, of which the late ones
// exist in the long sequences only.  64 sequences of 256 .. 2048 tokens, 8 heads, d = 128: chunk transform 799 ->
// 584 us, with the backward's outputs 1042 -> 796.
// Where a sequence has no multiple of eight heads, they are turned by one per chunk: else, with a multiple of eight in all,
// the chunks of a head go to one XCD and to half of its CUs, and sequences of different lengths do not balance each other.
// Not if an XCD has a CU for each of its chunks anyway: then a head's chunks had better lie in the L2 of the XCD that its
// sweeps run on (4 sequences of 56 .. 292 tokens, 2 heads, d = 128, forward and backward: turned 127 us, not 118).  Turned / not,
// us: one sequence of 4096 tokens and 31 of 100, 2 heads, d = 128 768 / 1096; the 64 sequences above with 1 head 1003 / 1095;
// 8 of 456 .. 1300, 4 heads, fp32, d = 64 1903 / 1988 (chunks first 1881).
__device__ __forceinline__ void chunk_and_head(const UserLayout& u, int NC, int BH, int& chunk, int& bh) {
    const int n = blockIdx.x, m = u.cu ? BH : NC;
    const int hi = __builtin_amdgcn_readfirstlane(n / m), lo = n - hi * m;       // (the division runs on the vector unit)
    if (!u.cu) { chunk = lo; bh = hi; return; }
    chunk = hi;
    bh = lo;
    if ((u.H & 7) && NC * ((BH + 7) >> 3) > 32) {
        bh += __builtin_amdgcn_readfirstlane(hi % m);
        if (bh >= m) bh -= m;
    }
}
// The workgroup's head and its place among the head's N, see xcd_deal.h (the division runs on the vector unit; its result,
// uniform over the workgroup, goes back to scalar registers, so that everything derived from it -- loop bounds, tile
// addresses -- is scalar arithmetic).
__device__ __forceinline__ bool xcd_deal(int slot, int xcd, int N, int BH, int& bh, int& r) {
    const XcdDivision v = xcd_division(slot, xcd, N, BH);
    const int q = __builtin_amdgcn_readfirstlane(v.num / v.den);
    const XcdPlace p = xcd_place(q, v.num - q * v.den, xcd, BH);
    bh = __builtin_amdgcn_readfirstlane(p.bh);
    r = __builtin_amdgcn_readfirstlane(p.r);
    return bh < BH && r < N;
}
// The workgroup's chunk and head as numbered by sb_place in xcd_deal.h, launched with super_block_grid() workgroups; those past
// the last pair get bh >= BH.
__device__ __forceinline__ void super_block_and_head(const UserLayout& u, int NC, int BH, int& chunk, int& bh) {
    const SbPlace p = sb_place(blockIdx.x >> 3, blockIdx.x & 7, NC, SBC, BH, u.cu != nullptr, (u.H & 7) && NC * ((BH + 7) >> 3) > 32);
    chunk = __builtin_amdgcn_readfirstlane(p.chunk);
    bh = __builtin_amdgcn_readfirstlane(p.bh);
}
__host__ __forceinline__ unsigned super_block_grid(int NC, int BH) { return sb_grid(NC, SBC, BH); }
// length of head bh's sequence: the launch's L, or the head's own in a packed batch
__device__ __forceinline__ int seq_len(const UserLayout& u, int bh, int L) {
    if (!u.cu) return L;
    const int b = (bh + u.bh0) / u.H;
    return u.cu[b + 1] - u.cu[b];
}

struct FwdParams {
    UserLayout ul;
    const void *q, *k, *v, *w, *beta;
    void* o;
    float* lse;
    void *kt, *vt, *dp;   // fragment-order tiles written by prep, read by the sweep
    void *kt2, *dp2;      // second level: keys carried to their super-block's right edge; -(I - P_superblock)
    void *dpt;            // backward only: -dP per chunk in the transposed arrangement (rows a, contraction b) = -dP[a][b]
    float *xinit, *sd;    // accumulator-order fp32 tiles
    const float* cum;     // PaTH-FoX only (else NULL): [BH][64*NC] cumulative log2 of the forget gates, log2(e) * sum_{s<=t} log f_s
    int B, H, L, NC;      // NC = number of 64-token chunks = ceil(L/64)
    float scale;
    // Backward only (NULL in the forward), all in fragment order:
    //   per chunk:  ktT (rows c, contraction s) = Kb[s][c];  vk (rows s, contraction c) = V[s][c] (I/O type);
    //               kt2T: the same arrangement of the second-level keys Kb2;
    //   per super-block: dpt2 (rows a, contraction b) = -(I - P_superblock)[a][b];
    //   per pair (query chunk i, key block), slot block_slot(i, c): xs (rows q, contraction c) and, fp32 operands,
    //               xsT (rows c, contraction q): the query state of chunk i as used against the block.
    void *ktT, *vk, *xs, *xsT, *kt2T, *dpt2;
    int emit_states;      // forward sweep of a training pair: also write xs (and xsT)
    // Backward only: per-chunk matrices of the transform, row-major 64x64 (operand type) --
    // fm = F[t][t'], gktm[s][t'] = strictLower(W K^T)[t'][s], nm = N, aim = A^{-1},
    // ytm[s][t] = Y[t][s]; utm [d][64]: utm[c][t] = U[t][c]; fp32: gm = W W^T, sdm[t][s] = Sd;
    // kbm [Lp][d]: boundary-adjusted keys Kb (rows past L zero; fp32 operands only); rm [d][d] per chunk: R_c of
    // the second level (operand type; fp32 operands row-major, 16-bit operands as a tile with rows a, contraction b).
    void *fm, *gktm, *nm, *aim, *ytm, *utm, *kbm, *rm;
    float *gm, *sdm;
    // Sequence-parallel forward (one device's share of the ring of Sec. 3.5): the sweep's per-query registers --
    // the query state carried to the left edge of what has been attended so far, the unnormalised output, the
    // running maximum and row sum -- kept in memory between the calls.  ring: 0 = ordinary forward; 1 = sweep over
    // the device's own segment, leaving the registers in ring_state; 2 = one hop: the registers are loaded, every
    // key of an earlier segment (whose tiles kt2, vt, dp2 this structure then points at; NC = ITS chunk count) is
    // attended, and they are stored again.  NCq: chunks of the query side (ring = 2 only; else NC).
    float* ring_state;
    int ring, NCq;
    // Key prefill of a prompt of one super-block (second-level kernel only): the decode path's caches [BH][Lmax][d].
    void *kcache, *vcache;
    int Lmax;
};
// ring_state: per (head, query chunk, 32-query half) one record of RING_REC(d) floats, each quantity as the sweep
// holds it: [X: d/32 blocks][O: d/32 blocks] of 1024 floats (register g*4+r of lane l at g*256 + l*4 + r), then the
// running maximum and the row sum per lane (64 + 64), then (PaTH-FoX; zero otherwise) the sum of the gate logarithms
// of the segments passed so far, in base-2 units, once per lane (64).
__host__ __device__ constexpr size_t ring_rec_floats(int d) { return (size_t)2 * (d / 32) * 1024 + 192; }

// The last super-block of a head is never left of a query's own one: no query reads its second-level keys or its
// product, and in the backward no gradient arrives there.  A training step therefore runs neither the second-level
// transform nor its adjoint nor the far sums on it -- one super-block of eight at 8192 tokens, half of the chunks
// of a batch of sequences of 256 to 2048 tokens, everything up to 1024 tokens.  Measured,
// forward + backward: 64 packed sequences of 256 .. 2048 tokens (8 heads, d = 128) 7.50 -> 6.99 ms, one fp32 step of
// 256 tokens 282 -> 253 us (three launches fewer).  (The forward of more than one super-block
// and the ring fill it: the key prefill of the decode path and the ring's hops carry keys beyond the head's end.  A prompt of one
// super-block is prefilled straight from the chunk tiles.)
__host__ __device__ __forceinline__ bool is_last_sb(int sb, int NCown) { return (sb + 1) * SBC >= NCown; }

// Key blocks of the backward, for query chunk i (own super-block I = i / SBC): the chunks
// SBC*I <= j < i one by one ("near"), and the super-blocks J < I as a whole ("far": the state is
// the one at the super-block's right edge, the keys are the second-level keys).  Per head the
// state arrays hold the near slots [0, NC*(SBC-1)) first, then the far slots.
__host__ __device__ __forceinline__ size_t far_base(int i) {
    const size_t I = (size_t)(i / SBC);
    return (size_t)SBC * (I * (I - 1) / 2) + (size_t)(i % SBC) * I;
}
__host__ __device__ __forceinline__ size_t num_block_slots(int NC) { return (size_t)NC * (SBC - 1) + far_base(NC); }
// slot of (query chunk i, block holding key chunk c < i)
__host__ __device__ __forceinline__ size_t block_slot(int i, int c, int NC) {
    const int jsb = (i / SBC) * SBC;
    if (c >= jsb) return (size_t)i * (SBC - 1) + (c - jsb);
    return (size_t)NC * (SBC - 1) + far_base(i) + (size_t)(c / SBC);
}

}  // namespace path
