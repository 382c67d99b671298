// Key-side sums of the backward over the FAR query chunks (those right of the key's super-block), 16-bit
// operands: for the keys of two chunks j, j+1, over all query chunks i of the super-blocks to the right,
//
//     S  = Xs Kb2_j^T,  dP = dO V_j^T,  P = exp2(scale2 S - lse2),  dS = P o (dP - delta)
//     dV^T  += dO^T P              dKb2^T += Xs^T dS              dP_superblock += Xs^T g
//
// with the second-level keys Kb2 and the state Xs of chunk i at the super-block's right edge.  (fp32 operands:
// bwd_keyside2_kernel in bwd.hip.)
//
// What bounds it: the chip's power, then the matrix pipes.  Per query chunk a SIMD has 68 products (2176 cycles at 32
// each), 1300 cycles of element-wise work and the operand fragments from LDS.  One wave per SIMD doing all of it in
// turn, with four tiles staged per step, took 5000 cycles at 2.0 GHz.  Here the work is split by kind over eight waves,
// two per SIMD, that meet at one barrier per 32 queries:
//   waves 0..3  32 keys each (keys and values resident): logits, dP, the element-wise part; P and dS leave as
//               operand fragments through LDS, double-buffered;
//   waves 4, 5  dV^T and waves 6, 7 dKb2^T, of 64 keys each, two half-steps behind (the latter also take one each of the
//               sixteen 32x32 blocks of dP_superblock, whose state fragments are in registers anyway: the workgroups of a
//               super-block cover all of it, see far_blocks.h, which saves the pass over the states that it was before).
// The first kind's vector work then runs under the second kind's products.  The second kind, which has issue slots to
// spare, requests the tiles (a direct-to-LDS request holds its wave for about 70 cycles) and reads dO^T and Xs^T out
// of the untransposed ones with transposing LDS reads: a step stages two tiles instead of four, in a ring of three,
// and the transposed states and dO are neither written nor read anywhere.  4200 cycles per chunk, at 1.6 .. 1.8 GHz:
// without any copies it would take 3350, in 1.87 ms instead of 1.97.
// Measured (with the dP_superblock sums, a kernel of its own before): B=4, H=16, L=8192, d=128 2.39 + 0.19 -> 1.97 ms;
// B=8, H=16, L=4096, d=64 0.83 + 0.03 -> 0.64; B=1, H=32, L=32768, d=128, whole training step 50.1 -> 45.5.
#include <type_traits>

#include "path_common.h"
#include "bwd_decl.h"
#include "far_blocks.h"

namespace path {

template <typename TIO, int D> struct FarCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int KVF = CHUNK * D / Tr<T>::FE;                 // fragments of a tile
    static constexpr int GF = CHUNK / Tr<T>::KW * 64;                 // ... of 32 columns of a g tile
    typedef FarBlocks<SBC, D> Blocks;
    static constexpr int GTF = Blocks::COLS * GF;
    static constexpr int STF = 2 * KVF + GTF + 32;                    // a stage: xs | doq | the workgroup's columns of g | lse2, delta
    static constexpr int PDF = 2 * 4 * 2 * 64;                        // a hand-over buffer: (P | dS) x 4 key blocks x 2 slabs
    static constexpr size_t smem_bytes = (size_t)(3 * STF + 2 * PDF) * 16;
    static_assert(smem_bytes <= 160 * 1024, "LDS budget");
};

template <typename TIO, int D, bool FOX>
__global__ __launch_bounds__(512, 2) void bwd_far_kernel(BwdParams p) {
    using C = FarCfg<TIO, D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using FragV = typename Tr<TIO>::Frag;
    constexpr int KW = Tr<T>::KW, SPB = 32 / KW, DB = D / 32, DS = D / KW;
    constexpr int KVF = C::KVF, GTF = C::GTF, STF = C::STF, PDF = C::PDF;
    using Blocks = typename C::Blocks;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* const stages = reinterpret_cast<Frag*>(smem);
    Frag* const hand = stages + 3 * STF;

    // Numbering as in xcd_deal.h, super-block by super-block, the left-most first; the workgroups of a super-block get
    // consecutive numbers on its XCD (they stream the same states and dO tiles at the same time, out of that XCD's L2).
    constexpr int NPOS = Blocks::NPOS;
    const int NC = p.NC, nsb = (NC + SBC - 1) / SBC;
    const int xcd = blockIdx.x & 7, kk = blockIdx.x >> 3, pos = kk % NPOS;
    int J, bh;
    if (!xcd_deal(kk / NPOS, xcd, nsb - 1, p.B * p.H, bh, J)) return;
    const int NCo = (seq_len(p.ul, bh, p.L) + CHUNK - 1) / CHUNK;      // this head's own chunks
    if (is_last_sb(J, NCo)) return;                                    // no queries to the right
    const int j = J * SBC + 2 * pos;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const size_t Lp = (size_t)NC * CHUNK, nslots = num_block_slots(NC);
    const int i0 = (J + 1) * SBC, i1 = NCo;
    const int bb = Blocks::first_col(pos);                             // first column block of the workgroup's blocks of dP_superblock

    if (wv < 4) {
        // ---- logits and the element-wise part of 32 keys ------------------------------------------------------
        const float sl2 = p.scale * 1.44269504088896340736f;
        const int jw = j + (wv >> 1), kh = wv & 1;
        Frag Kb[DS];
        FragV Vb[DS];
        {
            const Frag* kg = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.kt2) + ((size_t)bh * NC + jw) * CHUNK * D);
            const FragV* vg = reinterpret_cast<const FragV*>(reinterpret_cast<const TIO*>(p.vk) + ((size_t)bh * NC + jw) * CHUNK * D);
#pragma unroll
            for (int s = 0; s < DS; ++s) { Kb[s] = kg[((size_t)kh * DS + s) * 64 + tile_lane<T>(lane, s)]; Vb[s] = vg[((size_t)kh * DS + s) * 64 + lane]; }
        }
        const int key_tok = jw * CHUNK + 32 * kh + l32;
        const float ckj = FOX ? p.cum[(size_t)bh * Lp + key_tok] : 0.f;
        float dcol = 0.f;
        // The element-wise part of a half-step runs one half-step after its products, between the products of the
        // next one (two sets of accumulators), and operand fragments are read a batch at a time ahead of their
        // products: those of a tile's second half during the first half's, those of its first half as soon as the
        // tile has landed, under the element-wise part of the half-step before.
        Frag xa[DS];
        FragV da[DS];
        f32x16 S0, P0, S1, P1;                            // logits and dP of the two halves: rows q, lane s
        auto read_ops = [&](int st, int qh) {
            const Frag* sX = stages + st * STF;
            const FragV* sDQ = reinterpret_cast<const FragV*>(sX + KVF);
#pragma unroll
            for (int u = 0; u < DS; ++u) { xa[u] = sX[(qh * DS + u) * 64 + tile_lane<T>(lane, u)]; da[u] = sDQ[(qh * DS + u) * 64 + tile_lane<T>(lane, u)]; }
        };
        // A half-step's work in four slices, each a quarter of its products, a quarter of the element-wise part of the
        // half-step before (half qh of the tile in stage st: P and dS -> its hand-over buffer) and a piece of the copies.
        auto products = [&](f32x16& S, f32x16& dP, int k) {
#pragma unroll
            for (int u = k * DS / 4; u < (k + 1) * DS / 4; ++u) {
                S = Tr<T>::mma(xa[u], Kb[u], S);
                dP = Tr<TIO>::mma(da[u], Vb[u], dP);
            }
        };
        FragV Pb;
        Frag dSb;
        auto element_wise = [&](int st, int qh, const f32x16& S, const f32x16& dP, int g) {
            const float* lse2 = reinterpret_cast<const float*>(stages + st * STF + 2 * KVF + GTF) + 32 * qh + 4 * h;
            const f32x4 ls = *reinterpret_cast<const f32x4*>(lse2 + 8 * g), dls = *reinterpret_cast<const f32x4*>(lse2 + CHUNK + 8 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // Rows past L need no mask: their padded lse2p is huge, so P = exp2(-huge) = 0.
                float arg = __builtin_fmaf(S[4 * g + r], sl2, -ls[r]);
                if (FOX) arg -= ckj;
                const float P = __builtin_amdgcn_exp2f(arg);
                const float dz = P * (dP[4 * g + r] - dls[r]);      // the factor scale is applied to the finished sums
                if (FOX) dcol += dz;
                Pb[(4 * g + r) % 8] = (TIO)P;
                dSb[(4 * g + r) % 8] = (T)dz;
            }
            if (g & 1) {
                Frag* out = hand + qh * PDF;
                reinterpret_cast<FragV*>(out)[(wv * SPB + g / 2) * 64 + lane] = Pb;
                out[(4 * SPB + wv * SPB + g / 2) * 64 + lane] = dSb;
            }
        };
        auto mix = [&]() {                                // a product, then its share of the vector instructions
#pragma unroll
            for (int u = 0; u < DS / 2; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 48 / DS, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        int st = 0;
        lds_barrier();                                    // half-step (i0, 0): tile i0 has landed
        read_ops(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        S0 = zero16(); P0 = zero16();
#pragma unroll
        for (int k = 0; k < 4; ++k) products(S0, P0, k);
        __builtin_amdgcn_sched_barrier(0);
        read_ops(0, 1);
        for (int i = i0; ; ++i) {
            const int st1 = st == 2 ? 0 : st + 1;
            lds_barrier();                                // half-step (i, 1)
            S1 = zero16(); P1 = zero16();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                products(S1, P1, k);
                element_wise(st, 0, S0, P0, k);
                mix();
            }
            if (i + 1 == i1) break;
            lds_barrier();                                // half-step (i + 1, 0): its tile has landed
            read_ops(st1, 0);
            __builtin_amdgcn_sched_barrier(0);
            S0 = zero16(); P0 = zero16();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                element_wise(st, 1, S1, P1, k);
                products(S0, P0, k);
                mix();
            }
            read_ops(st1, 1);
            st = st1;
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 4; ++k) element_wise(st, 1, S1, P1, k);
        lds_barrier();
        if (FOX) {           // the two half-waves hold different query rows of the same keys
            dcol += __shfl_xor(dcol, 32);
            if (h == 0) p.dcol[(size_t)bh * Lp + key_tok] = dcol;
        }
        return;
    }

    // ---- the sums: dV^T (KEYS = false) or dKb2^T (KEYS = true) of the chunk j + (wv & 1) ------------------------
    auto sums = [&](auto keys_tag) {
        constexpr bool KEYS = decltype(keys_tag)::value;
        using E = typename std::conditional<KEYS, T, TIO>::type;      // operand type of the product
        using FragE = typename Tr<E>::Frag;
        const int ck = wv & 1;
        f32x16 acc[DB][2];
#pragma unroll
        for (int b = 0; b < DB; ++b) { acc[b][0] = zero16(); acc[b][1] = zero16(); }
        // dP_superblock: this wave's blocks have row blocks ab ..
        constexpr int NR = Blocks::ROWS, NCB = Blocks::COLS;
        const int ab = Blocks::first_row(pos, ck);
        f32x16 dd[NR][NCB];
#pragma unroll
        for (int a = 0; a < NR; ++a)
#pragma unroll
            for (int b = 0; b < NCB; ++b) dd[a][b] = zero16();
        // the tile's transposed fragments of a half-step, read before the barrier that P and dS wait for
        FragE ta[DB * SPB], td[NR * SPB];
        Frag gf[NCB * SPB];
        auto read_tile = [&](int st, int qh) {
            const E* tile = reinterpret_cast<const E*>(stages + st * STF + (KEYS ? 0 : KVF));
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int u = 0; u < SPB; ++u) ta[b * SPB + u] = ld_tile_frag_tr<E, DS>(tile, qh * SPB + u, b, l32, h);
            if constexpr (KEYS) {
#pragma unroll
                for (int b = 0; b < NCB; ++b)
#pragma unroll
                    for (int u = 0; u < SPB; ++u) gf[b * SPB + u] = ld_tile_frag_tr<T, 2 * NCB>(reinterpret_cast<const T*>(stages + st * STF + 2 * KVF), qh * SPB + u, b, l32, h);
#pragma unroll
                for (int a = 0; a < NR; ++a)
#pragma unroll
                    for (int u = 0; u < SPB; ++u) td[a * SPB + u] = ld_tile_frag_tr<E, DS>(tile, qh * SPB + u, ab + a, l32, h);
            }
        };
        int st = 0;
        auto half = [&](int qh) {
            const FragE* in = reinterpret_cast<const FragE*>(hand + qh * PDF + (KEYS ? 4 * SPB * 64 : 0)) + 2 * ck * SPB * 64;
            FragE f[2][SPB];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int u = 0; u < SPB; ++u) f[k][u] = in[(k * SPB + u) * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < SPB; ++u)
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int k = 0; k < 2; ++k) acc[b][k] = Tr<E>::mma(ta[b * SPB + u], f[k][u], acc[b][k]);
            if constexpr (KEYS) {
#pragma unroll
                for (int u = 0; u < SPB; ++u)
#pragma unroll
                    for (int a = 0; a < NR; ++a)
#pragma unroll
                        for (int b = 0; b < NCB; ++b) dd[a][b] = Tr<T>::mma(td[a * SPB + u], gf[b * SPB + u], dd[a][b]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // These waves, which have time to spare, also request the tiles: a tile in two parts, in the second half-step of
        // the chunk two before it (its stage has then been read for the last time) and the half-step after that.  A
        // transposing read waits for every copy its wave has in flight.  d = 128: requests first in a half-step, reads
        // last (1.98 ms at B=4, H=16, L=8192; the other way round 2.07).  d = 64: a half-step is too short for the copies
        // to land in, so the reads come before the requests (0.64 ms at B=8, H=16, L=4096; the other way round 0.68).
        constexpr bool REQ_FIRST = D == 128;
        const int tid4 = tid - 256, wv4 = wv - 4;
        auto slot_of = [&](int i) { return ((size_t)bh * nslots + block_slot(i, j, NC)) * (size_t)CHUNK * D; };
        auto issue_a = [&](int i, int st) {               // xs, row constants
            if (i >= i1) return;
            Frag* buf = stages + st * STF;
            async_copy_tile<256, KVF, false>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.xs) + slot_of(i)), buf, tid4, wv4);
            if (tid4 < 32) {    // 64 floats of lse2 (lanes 0-15) and of delta (lanes 16-31): 16 bytes per lane
                const float* src = (tid4 < 16 ? p.lse2p : p.delta) + (size_t)bh * Lp + (size_t)i * CHUNK + 4 * (tid4 & 15);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                 (__attribute__((address_space(3))) void*)(buf + 2 * KVF + GTF), 16, 0, 0);
            }
        };
        auto issue_b = [&](int i, int st) {               // doq, g
            if (i >= i1) return;
            Frag* buf = stages + st * STF;
            async_copy_tile<256, KVF, false>(reinterpret_cast<const Frag*>(reinterpret_cast<const TIO*>(p.doq) + ((size_t)bh * NC + i) * CHUNK * D), buf + KVF, tid4, wv4);
            const Frag* g = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.gs) + slot_of(i)) + 2 * bb * 64;      // two slabs per column block of either half
#pragma unroll
            for (int k = 0; k < NCB; ++k) {
                const int n = wv4 * NCB + k;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(g + ((n / (2 * NCB)) * DS + n % (2 * NCB)) * 64 + lane),
                                                 (__attribute__((address_space(3))) void*)(buf + 2 * KVF + n * 64), 16, 0, 0);
            }
        };
        issue_a(i0, 0);
        issue_b(i0, 0);
        copies_landed();
        lds_barrier();                                    // half-steps (i0, 0) and (i0, 1): nothing to add up yet
        issue_a(i0 + 1, 1);
        issue_b(i0 + 1, 1);
        lds_barrier();
        if (REQ_FIRST) issue_a(i0 + 2, 2);
        copies_landed();
        read_tile(0, 0);
        if (!REQ_FIRST) issue_a(i0 + 2, 2);
        for (int i = i0; i < i1; ++i) {
            const int st1 = st == 2 ? 0 : st + 1, st2 = st1 == 2 ? 0 : st1 + 1;
            lds_barrier();                                // half-step (i + 1, 0), or the first of the last two
            if (REQ_FIRST) issue_b(i + 2, st2);
            half(0);
            copies_landed();
            read_tile(st, 1);
            if (!REQ_FIRST) issue_b(i + 2, st2);
            lds_barrier();
            if (REQ_FIRST) issue_a(i + 3, st);
            half(1);
            copies_landed();
            read_tile(st1, 0);                            // (past the end: whatever is there, never used)
            if (!REQ_FIRST) issue_a(i + 3, st);
            st = st1;
        }
        const size_t row = ((size_t)bh * Lp + (j + ck) * CHUNK + l32) * D + 4 * h;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v4;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v4[r] = KEYS ? p.scale * acc[b][k][4 * g + r] : acc[b][k][4 * g + r];
                    *reinterpret_cast<f32x4*>((KEYS ? p.dk2 : p.dvp) + row + (size_t)(32 * k) * D + 32 * b + 8 * g) = v4;
                }
        if (KEYS && Blocks::writes(pos, ck)) {
            // the gradient of P_superblock starts the second level's chain (nothing lies left of super-block 0)
            float* dst = p.dchain + ((size_t)bh * nsb + J) * D * D;
#pragma unroll
            for (int a = 0; a < NR; ++a)
#pragma unroll
                for (int b = 0; b < NCB; ++b)
#pragma unroll
                    for (int jj = 0; jj < 16; ++jj)
                        dst[(size_t)(32 * (ab + a) + acc_row(jj, h)) * D + 32 * (bb + b) + l32] = J >= 1 ? dd[a][b][jj] : 0.f;
        }
    };
    if (wv < 6) sums(std::false_type{});
    else sums(std::true_type{});
}

template <typename TIO, int D, bool FOX>
static hipError_t launch_far_f(const BwdParams& p, hipStream_t st) {
    using C = FarCfg<TIO, D>;
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_far_kernel<TIO, D, FOX>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::smem_bytes);
    if (attr_err != hipSuccess) return attr_err;
    const int nsb = (p.NC + SBC - 1) / SBC;
    hipLaunchKernelGGL((bwd_far_kernel<TIO, D, FOX>), dim3(xcd_deal_grid(nsb - 1, p.B * p.H) * (SBC / 2)), dim3(512), C::smem_bytes, st, p);
    return hipGetLastError();
}
hipError_t launch_bwd_far(const BwdParams& p, int d, hipStream_t st) {
    if (d == 64) return p.cum ? launch_far_f<bf16_t, 64, true>(p, st) : launch_far_f<bf16_t, 64, false>(p, st);
    return p.cum ? launch_far_f<bf16_t, 128, true>(p, st) : launch_far_f<bf16_t, 128, false>(p, st);
}

}  // namespace path
