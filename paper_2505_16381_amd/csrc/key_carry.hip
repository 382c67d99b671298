// Key prefill of the decode caches, 16-bit operands: every chunk's keys carried to the prompt's end on their own,
//
//     K <- K P_j^T = K - K dP_j^T ,     j = the blocks right of the chunk, left to right,
//
// blocks = chunks for a prompt of one super-block (keys and products as the chunk transform left them), super-blocks for a
// longer one (second-level keys, super-block products).  One workgroup per (chunk, head): two waves of 32 keys each keep
// them transposed in registers (fp32, lane = key) with the packed copy as the operand, as the forward sweep keeps its
// queries; -dP_j is wanted with rows a and contraction b and is read out of the sweep's tile (rows b, contraction a) with
// transposing LDS reads.  Four more waves bring the tiles, one (d = 64: three) ahead: a transposing read waits for every copy that
// its own wave has in flight.
//
// What bounds it: the chain of products, 0.8 us each at d = 128 (32 products of one wave are 0.5), and the products' way
// through L2 when there are many heads.  At d = 128 two places for tiles, so that a second workgroup shares the CU, are ahead of four
// throughout: 132 heads of 1100 tokens 33.4 / 40.5 us, 300 of 200 23.1 / 27.0, 19 of 1000 19.2 / 20.2.  The prefill of a prompt of 16 heads and 1000 tokens, d = 128: 37.4 -> 15.1 us (one chain
// of 16 chunks per head before), of 2000 tokens 27.9 -> 9.6.  It rounds once per block the keys where the chains round the
// product of the blocks: against the recurrence in 64 bits 1.727e-3 of the keys' norm instead of 1.807e-3 (1000 tokens; the
// rounding to bf16 alone is 1.652e-3), d = 64 1.737e-3 / 1.916e-3, 2100 tokens 1.815e-3 / 1.831e-3.
#include "path_common.h"
#include "decode_decl.h"

namespace path {

template <typename TIO, int D> struct CarryCfg {
    typedef typename Compute<TIO>::type T;
    static_assert(sizeof(T) == 2, "transposing reads");
    static constexpr int DPF = D * D / Tr<T>::FE, NBUF = D == 128 ? 2 : 4, NT = 384;      // (d = 128: two workgroups per CU)
    static constexpr size_t smem_bytes = (size_t)NBUF * DPF * 16;
};

template <typename TIO, int D>
__global__ __launch_bounds__((CarryCfg<TIO, D>::NT)) void key_carry_kernel(CarryArgs a) {
    using C = CarryCfg<TIO, D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    constexpr int SPB = 2, DB = D / 32, DS = D / 16, DPF = C::DPF, NBUF = C::NBUF, PER = DPF / 256;      // copies per wave and tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* const tiles = reinterpret_cast<Frag*>(smem);

    // longest chains first, then the pieces of the values
    int bh, c;
    if (!xcd_deal(blockIdx.x >> 3, blockIdx.x & 7, a.NC + value_row_pieces(a.L), a.BH, bh, c)) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    if (c >= a.NC) { copy_value_rows<TIO, D, C::NT>(a.v, a.vcache, a.L, a.Lmax, bh, c - a.NC, tid); return; }
    const int nblk = (a.NC + a.cpb - 1) / a.cpb, j0 = c / a.cpb + 1;      // chunks per block; the first block to pass
    const T* dp = reinterpret_cast<const T*>(a.dp) + (size_t)bh * nblk * D * D;

    if (wv >= 2) {                       // ---- copies
        auto issue = [&](int j) {
            async_copy_tile<256, DPF>(reinterpret_cast<const Frag*>(dp + (size_t)j * D * D), tiles + (size_t)((j - j0) % NBUF) * DPF, tid - 128, wv - 2);
        };
        for (int j = j0; j < nblk && j < j0 + NBUF - 1; ++j) issue(j);
        for (int j = j0; j < nblk; ++j) {
            const int ahead = nblk - 1 - j;                      // tile j has landed: so many may be on their way behind it
            if (NBUF > 3 && ahead >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
            else if (NBUF > 2 && ahead >= 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
            else copies_landed();
            lds_barrier();                                       // ... for everybody, and tile j - 1 has been read
            if (j + NBUF - 1 < nblk) issue(j + NBUF - 1);
        }
        return;
    }
    // ---- keys
    f32x16 K[DB];                        // rows feature, lane = key 32 wv + l32
    {
        const Frag* kt = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.kt) + ((size_t)bh * a.NC + c) * CHUNK * D) + (size_t)wv * DS * 64;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            const Frag f = kt[s * 64 + tile_lane<T>(lane, s)];
#pragma unroll
            for (int e = 0; e < 8; ++e) K[s / 2][8 * (s & 1) + e] = (float)f[e];
        }
    }
    for (int j = j0; j < nblk; ++j) {
        lds_barrier();
        const T* t = reinterpret_cast<const T*>(tiles + (size_t)((j - j0) % NBUF) * DPF);
        Frag Kb[DS];
#pragma unroll
        for (int b = 0; b < DB; ++b) pack_block<T>(K[b], Kb + b * SPB);
        // (four fragments at a time, read while the four before are multiplied)
        Frag f[2][4];
        auto read = [&](int g) {
#pragma unroll
            for (int s = 0; s < 4; ++s) f[g & 1][s] = ld_tile_frag_tr<T, DS>(t, 4 * (g % (DS / 4)) + s, g / (DS / 4), l32, h);
        };
        read(0);
#pragma unroll
        for (int g = 0; g < DB * DS / 4; ++g) {
            if (g + 1 < DB * DS / 4) read(g + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) K[g / (DS / 4)] = Tr<T>::mma(f[g & 1][s], Kb[4 * (g % (DS / 4)) + s], K[g / (DS / 4)]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const int tok = c * CHUNK + 32 * wv + l32;
    if (tok >= a.L) return;
    typedef typename Tr<TIO>::Vec4 OVec4;
    TIO* dst = reinterpret_cast<TIO*>(a.kcache) + ((size_t)bh * a.Lmax + tok) * D + 4 * h;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            OVec4 o4;
#pragma unroll
            for (int r = 0; r < 4; ++r) o4[r] = (TIO)K[b][4 * g + r];
            *reinterpret_cast<OVec4*>(dst + 32 * b + 8 * g) = o4;
        }
}

template <int D>
static hipError_t launch_carry_t(const CarryArgs& a, hipStream_t st) {
    using C = CarryCfg<bf16_t, D>;
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&key_carry_kernel<bf16_t, D>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::smem_bytes);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((key_carry_kernel<bf16_t, D>), dim3(xcd_deal_grid(a.NC + value_row_pieces(a.L), a.BH)), dim3(C::NT), C::smem_bytes, st, a);
    return hipGetLastError();
}
hipError_t launch_key_carry(const CarryArgs& a, int d, hipStream_t st) { return d == 64 ? launch_carry_t<64>(a, st) : launch_carry_t<128>(a, st); }

}  // namespace path
