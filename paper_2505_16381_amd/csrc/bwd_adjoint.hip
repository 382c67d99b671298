// Adjoint scan of the backward, 16-bit operands (fp32 operands: bwd_adjoint2_kernel in bwd.hip).  For the queries of
// chunk i, over the key chunks j = 0 .. i-1 from left to right (second-level keys and one product per super-block left
// of the own one, chunk-level keys and products inside it), everything transposed (64 queries = two MFMA columns):
//
//     S^T = Kb_j Xs^T,   dP^T = V_j dO^T,   dS^T = scale P o (dP^T - delta),   P = exp(scale S^T - lse)
//     g^T <- (I - dP_block) g^T   where a block starts,       g^T += Kb_j^T dS^T
//
// The state after a block is also left, as a tile like the query states' (rows q, contraction b), of
// the pair (i, next block) for the key-side kernels, which read it transposed; what stands at the end is dQb.
//
// One workgroup takes four query chunks with eight waves, two per SIMD, that meet at one barrier per 32 keys:
//   waves 0..3  one chunk each (states and dO resident): logits, dP, the element-wise part; dS leaves as operand
//               fragments through LDS, double-buffered;
//   waves 4..7  one chunk's g each, half a key chunk behind; they request the tiles too.
// The fragments of Kb^T are read out of the key tile itself with transposing LDS reads, likewise those of -dP in the
// arrangement (rows a, contraction b) out of the forward's tile (rows b, contraction a): p.dpt / p.dpt2 point at the
// FORWARD's tiles.  A transposing read waits for every copy its wave has in flight, so all of a chunk's are made in the
// half-step that has none, and the copies are requested and awaited in the other.
//
// What bounds it: power, as for the far keys (0.98 PFLOP/s in both).  A wave of 32 queries that does all of it reads one
// fragment from LDS per product, which keeps the LDS port busy for as long as the matrix pipes (3072 cycles per chunk and
// two waves each); with 64 queries per wave every fragment serves two products, two thirds of that.  d = 64 has half the
// products for the same element-wise part and four of the smaller workgroups on a CU: it stays with those
// (bwd_adjoint2_lite_kernel in bwd.hip; B=8, H=16, L=4096 took 2.89 ms a step with this split, 2.80 without).
// Measured at d = 128: B=4, H=16, L=8192 2.09 -> 1.86 ms, training step 8.22 -> 7.99; L=32768, H=32 42.8 -> 41.5.
#include <type_traits>

#include "path_common.h"
#include "bwd_decl.h"

namespace path {

template <typename TIO, int D> struct AdjCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int KVF = CHUNK * D / Tr<T>::FE, DPF = D * D / Tr<T>::FE;
    static constexpr int STF = 2 * KVF + 16;                          // a stage: keys | values | the keys' gate sums
    static constexpr int HSF = 4 * 4 * 64;                            // a hand-over buffer: dS of 32 keys x four chunks
    static constexpr size_t smem_bytes = (size_t)(2 * STF + DPF + 2 * HSF) * 16;
    static_assert(smem_bytes <= 160 * 1024, "LDS budget");
};
constexpr int ADJ_CPT = 4;      // query chunks per workgroup
static_assert(SBC % ADJ_CPT == 0, "the chunks of a workgroup lie in one super-block");

template <typename TIO, int D, bool FOX>
__global__ __launch_bounds__(512, 2) void bwd_adjoint_kernel(BwdParams p) {
    using C = AdjCfg<TIO, D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using FragV = typename Tr<TIO>::Frag;
    constexpr int KW = Tr<T>::KW, SPB = 32 / KW, DB = D / 32, DS = D / KW;
    constexpr int KVF = C::KVF, DPF = C::DPF, STF = C::STF, HSF = C::HSF;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* const stages = reinterpret_cast<Frag*>(smem);
    Frag* const sDP = stages + 2 * STF;
    Frag* const hand = sDP + DPF;

    // XCD-aware numbering (xcd_deal.h): all tiles of a head together, heaviest first.  They walk the key chunks at the same
    // pace, so a chunk's tiles are fetched once per head into that XCD's L2.
    const int BH = p.B * p.H, NC = p.NC, ntiles = (NC + ADJ_CPT - 1) / ADJ_CPT;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    int bh, rank;
    if (!xcd_deal(slot, xcd, ntiles, BH, bh, rank)) return;
    const int tile = ntiles - 1 - rank;                                    // heaviest first
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int NCo = (seq_len(p.ul, bh, p.L) + CHUNK - 1) / CHUNK;          // this head's own chunks (NC: per head in the workspace arrays)
    if (tile * ADJ_CPT >= NCo) return;
    const int cw = wv & 3, cq = tile * ADJ_CPT + cw;                       // this wave's query chunk
    const bool active = cq < NCo;
    const int nj = (tile * ADJ_CPT + ADJ_CPT < NCo ? tile * ADJ_CPT + ADJ_CPT : NCo) - 1;      // key chunks any wave needs
    const int jsb = tile * ADJ_CPT / SBC * SBC;                            // first chunk of the own super-block
    const int nsb = (NC + SBC - 1) / SBC;
    const size_t Lp = (size_t)NC * CHUNK, nslots = num_block_slots(NC);
    auto block_start = [&](int j) { return j >= jsb || j % SBC == 0; };
    auto tile_of = [&](int j) { return ((size_t)bh * nslots + block_slot(cq, j, NC)) * (size_t)CHUNK * D; };      // the pair (cq, block of j)

    if (wv < 4) {
        // ---- logits, dP and the element-wise part ---------------------------------------------------------------
        const float sl2 = p.scale * 1.44269504088896340736f;
        FragV dOb[2][DS];
        Frag Xb[2][DS];
        float lse2[2] = {0.f, 0.f}, dl[2] = {0.f, 0.f}, drow[2] = {0.f, 0.f};
        auto read_state = [&](int j) {
            const Frag* xg = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.xs) + tile_of(j));
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int s = 0; s < DS; ++s) Xb[qb][s] = __builtin_nontemporal_load(&xg[((size_t)qb * DS + s) * 64 + tile_lane<T>(lane, s)]);
        };
        if (active) {
            const FragV* dq = reinterpret_cast<const FragV*>(reinterpret_cast<const TIO*>(p.doq) + ((size_t)bh * NC + cq) * CHUNK * D);
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
                for (int s = 0; s < DS; ++s) dOb[qb][s] = dq[((size_t)qb * DS + s) * 64 + tile_lane<TIO>(lane, s)];
                const size_t tq = (size_t)bh * Lp + cq * CHUNK + 32 * qb + l32;
                lse2[qb] = p.lse2p[tq] - __builtin_log2f(p.scale);         // the exponential then yields scale * P
                dl[qb] = p.delta[tq];
            }
            if (cq > 0) read_state(0);
        }
        // Fragments are read two slabs ahead of their products; the exponentials go between the products of dP.
        constexpr int W = 2, G = DS / W;
        Frag ka[2][W];
        FragV va[2][W];
        auto read_k = [&](int j, int kb, int g) {
#pragma unroll
            for (int u = 0; u < W; ++u) ka[g & 1][u] = stages[(j & 1) * STF + (kb * DS + W * g + u) * 64 + tile_lane<T>(lane, u)];
        };
        auto read_v = [&](int j, int kb, int g) {
#pragma unroll
            for (int u = 0; u < W; ++u) va[g & 1][u] = reinterpret_cast<const FragV*>(stages + (j & 1) * STF + KVF)[(kb * DS + W * g + u) * 64 + lane];
        };
        if (nj > 0) lds_barrier();
        for (int j = 0; j < nj; ++j) {
            const float* sC = reinterpret_cast<const float*>(stages + (j & 1) * STF + 2 * KVF);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                if (active && j < cq) {
                    f32x16 S[2], dP[2];                                    // rows s (keys), lane q
                    S[0] = zero16(); S[1] = zero16(); dP[0] = zero16(); dP[1] = zero16();
                    read_k(j, kb, 0);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (g + 1 < G) read_k(j, kb, g + 1);
                        else read_v(j, kb, 0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < W; ++u)
#pragma unroll
                            for (int qb = 0; qb < 2; ++qb) S[qb] = Tr<T>::mma(ka[g & 1][u], Xb[qb][W * g + u], S[qb]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (kb == 1 && j + 1 < cq && block_start(j + 1)) read_state(j + 1);      // for the next half-step
                    if (FOX) {      // gate sums of the 16 keys this lane holds (rows 8g + 4h + r of the 32-key block)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const f32x4 c4 = *reinterpret_cast<const f32x4*>(sC + 32 * kb + 8 * g + 4 * h);
#pragma unroll
                            for (int r = 0; r < 4; ++r)
#pragma unroll
                                for (int qb = 0; qb < 2; ++qb) S[qb][4 * g + r] = __builtin_fmaf(S[qb][4 * g + r], sl2, -lse2[qb]) - c4[r];
                        }
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (g + 1 < G) read_v(j, kb, g + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < W; ++u)
#pragma unroll
                            for (int qb = 0; qb < 2; ++qb) {
                                dP[qb] = Tr<TIO>::mma(va[g & 1][u], dOb[qb][W * g + u], dP[qb]);
#pragma unroll
                                for (int e = 0; e < 16 / DS; ++e) {
                                    const int jj = (W * g + u) * (16 / DS) + e;
                                    S[qb][jj] = __builtin_amdgcn_exp2f(FOX ? S[qb][jj] : __builtin_fmaf(S[qb][jj], sl2, -lse2[qb]));
                                }
                            }
#pragma unroll
                        for (int u = 0; u < 2 * W; ++u) {                  // a product, then its share of the vector instructions
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                            if (!FOX) __builtin_amdgcn_sched_group_barrier(0x002, 16 / DS, 0);
                            __builtin_amdgcn_sched_group_barrier(0x400, 16 / DS, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    Frag* out = hand + kb * HSF + cw * (4 * 64) + lane;
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
                        for (int jj = 0; jj < 16; ++jj) {
                            const float ds = S[qb][jj] * (dP[qb][jj] - dl[qb]);              // scale * P * (dP - delta)
                            if (FOX) drow[qb] += ds;
                            S[qb][jj] = ds;
                        }
                        Frag f[SPB];
                        pack_block<T>(S[qb], f);
#pragma unroll
                        for (int u = 0; u < SPB; ++u) out[(qb * SPB + u) * 64] = f[u];
                    }
                }
                lds_barrier();
            }
        }
        if (FOX && active) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                drow[qb] += __shfl_xor(drow[qb], 32);
                if (h == 0) p.drow[(size_t)bh * Lp + cq * CHUNK + 32 * qb + l32] = drow[qb] / p.scale;
            }
        }
        return;
    }

    // ---- g ------------------------------------------------------------------------------------------------------
    const int tid4 = tid - 256;
    auto issue = [&](int j) {                             // keys and values of chunk j
        if (j >= nj) return;
        const size_t bhc = (size_t)bh * NC + j;
        Frag* buf = stages + (j & 1) * STF;
        async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(j < jsb ? p.kt2 : p.kt) + bhc * CHUNK * D), buf, tid4, cw);
        async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const TIO*>(p.vk) + bhc * CHUNK * D), buf + KVF, tid4, cw);
        if (FOX && tid4 < 16)      // 64 floats, 16 bytes per lane
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p.cum + (size_t)bh * Lp + (size_t)j * CHUNK + 4 * tid4),
                                             (__attribute__((address_space(3))) void*)(buf + 2 * KVF), 16, 0, 0);
    };
    auto issue_dp = [&](int j) {                          // the product applied where the block of chunk j starts
        if (j >= nj || !block_start(j)) return;
        const T* src = j < jsb ? reinterpret_cast<const T*>(p.dpt2) + ((size_t)bh * nsb + j / SBC) * (size_t)D * D
                               : reinterpret_cast<const T*>(p.dpt) + ((size_t)bh * NC + j) * (size_t)D * D;
        async_copy_tile<256, DPF>(reinterpret_cast<const Frag*>(src), sDP, tid4, cw);
    };
    f32x16 Gm[DB][2];
#pragma unroll
    for (int b = 0; b < DB; ++b) { Gm[b][0] = zero16(); Gm[b][1] = zero16(); }
    Frag ta[DB * SPB];                                    // Kb^T of 32 keys
    auto read_keys = [&](int j, int kb) {
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int u = 0; u < SPB; ++u) ta[b * SPB + u] = ld_tile_frag_tr<T, DS>(reinterpret_cast<const T*>(stages + (j & 1) * STF), kb * SPB + u, b, l32, h);
    };
    auto add = [&](int kb) {                              // g^T += Kb^T dS^T
        const Frag* in = hand + kb * HSF + cw * (4 * 64) + lane;
        Frag f[2][SPB];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int u = 0; u < SPB; ++u) f[qb][u] = in[(qb * SPB + u) * 64];
#pragma unroll
        for (int u = 0; u < SPB; ++u)
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) Gm[b][qb] = Tr<T>::mma(ta[b * SPB + u], f[qb][u], Gm[b][qb]);
    };
    if (nj > 0) {
        issue(0);
        copies_landed();
        lds_barrier();                                    // half-step 0: nothing to add yet
        issue(1);
        copies_landed();
        lds_barrier();
    }
    auto apply_dp = [&]() {                               // g <- g (I - dP_blk)^T: the product with the state before this step
        // (each fragment of -dP serves both halves of the queries; two at a time, the registers are full)
        Frag Gb[2][DS];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int b = 0; b < DB; ++b) pack_block<T>(Gm[b][qb], Gb[qb] + b * SPB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int s0 = 0; s0 < DS; s0 += 4) {
                Frag pa[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) pa[u] = ld_tile_frag_tr<T, DS>(reinterpret_cast<const T*>(sDP), s0 + u, b, l32, h);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int qb = 0; qb < 2; ++qb) Gm[b][qb] = Tr<T>::mma(pa[u], Gb[qb][s0 + u], Gm[b][qb]);
            }
    };
    auto step = [&](int j, auto near_tag) {               // NEAR: a block starts at every chunk
        constexpr bool NEAR = decltype(near_tag)::value;
        const bool mine = active && j < cq;
        // half-step 2j + 1
        if (mine) {
            if (NEAR || (j > 0 && j % SBC == 0)) apply_dp();
            read_keys(j, 0);
            add(0);
            read_keys(j, 1);
        }
        lds_barrier();
        // half-step 2j + 2: the stage of chunk j and the product have been read for the last time
        issue_dp(j + 1);
        issue(j + 2);
        if (mine) add(1);
        copies_landed();
        if (active && j + 1 < cq && block_start(j + 1)) {             // g after this block: tile (rows q, contraction b) of the pair (cq, next block)
            Frag* gt = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.gs) + tile_of(j + 1));
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    Frag fr[SPB];
                    pack_block<T>(Gm[b][qb], fr);
#pragma unroll
                    for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &gt[((size_t)qb * DS + b * SPB + s2) * 64 + tile_lane<T>(lane, s2)]);
                }
        }
        if (j + 1 < nj) lds_barrier();
    };
    const int jn = nj < jsb ? nj : (jsb > 0 ? jsb : 1);   // (nothing stands left of chunk 0)
    int j = 0;
    for (; j < jn && j < nj; ++j) step(j, std::false_type{});
    for (; j < nj; ++j) step(j, std::true_type{});
    if (!active) return;
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float* dst = p.dqb + ((size_t)bh * Lp + cq * CHUNK + 32 * qb + l32) * D + 4 * h;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 v4;
#pragma unroll
                for (int r = 0; r < 4; ++r) v4[r] = Gm[b][qb][4 * g + r];
                *reinterpret_cast<f32x4*>(dst + 32 * b + 8 * g) = v4;
            }
    }
}

template <typename TIO, int D, bool FOX>
static hipError_t launch_adjoint_f(const BwdParams& p, hipStream_t st) {
    using C = AdjCfg<TIO, D>;
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_adjoint_kernel<TIO, D, FOX>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::smem_bytes);
    if (attr_err != hipSuccess) return attr_err;
    const unsigned ntiles = (unsigned)((p.NC + ADJ_CPT - 1) / ADJ_CPT);
    hipLaunchKernelGGL((bwd_adjoint_kernel<TIO, D, FOX>), dim3(xcd_deal_grid((int)ntiles, p.B * p.H)), dim3(512), C::smem_bytes, st, p);
    return hipGetLastError();
}
hipError_t launch_bwd_adjoint(const BwdParams& p, hipStream_t st) {
    return p.cum ? launch_adjoint_f<bf16_t, 128, true>(p, st) : launch_adjoint_f<bf16_t, 128, false>(p, st);
}

}  // namespace path
