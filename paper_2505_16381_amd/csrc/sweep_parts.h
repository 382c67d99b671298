// Parts of the forward sweep that its two forms share (attn_fwd2.hip, attn_few.hip): both yield the same bits.
#pragma once
#include "path_common.h"

namespace path {

// Block b (32 columns) of a query state (operand copy, query half qb) into the tile xs of a pair (query chunk, key block) -- fp32
// operands: and its transpose xsT -- in the arrangement of the backward's own states sweep (states_bwd.hip).  Streamed: the key and
// value tiles stay in L2.
template <typename T, int D>
__device__ __forceinline__ void emit_state_block(T* xs, T* xsT, const typename Tr<T>::Frag* Xb, int b, int qb, int lane) {
    using Frag = typename Tr<T>::Frag;
    constexpr int KW = Tr<T>::KW, SPB = 32 / KW, DS = D / KW, QS = CHUNK / KW;
    Frag* xd = reinterpret_cast<Frag*>(xs);
#pragma unroll
    for (int s = 0; s < SPB; ++s) __builtin_nontemporal_store(Xb[s], &xd[((size_t)qb * DS + b * SPB + s) * 64 + tile_lane<T>(lane, b * SPB + s)]);
    if (sizeof(T) == 4) {                // (16-bit operands: the consumers transpose xs themselves)
        Frag* xt = reinterpret_cast<Frag*>(xsT);
        Frag idf[SPB], fr[SPB];
        identity_frags<T>(idf, lane & 31, lane >> 5);
        pack_block<T>(transpose32<T>(Xb, idf), fr);       // rows q, lane c (block b)
#pragma unroll
        for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &xt[((size_t)b * QS + qb * SPB + s2) * 64 + lane]);
    }
}
template <typename T, int D>
__device__ __forceinline__ void emit_state(T* xs, T* xsT, const typename Tr<T>::Frag* Xh, int qb, int lane) {
#pragma unroll
    for (int b = 0; b < D / 32; ++b) emit_state_block<T, D>(xs, xsT, Xh + b * (32 / Tr<T>::KW), b, qb, lane);
}

// PaTH-FoX: logits in base-2 units minus the keys' gate sums (ck: those of the lane's first four keys); softmax_step then goes on with scale 1.
template <int RING>
__device__ __forceinline__ void gate_logits(f32x16& S, const float* ck, float sl2, float koff) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 c4 = *reinterpret_cast<const f32x4*>(ck + 8 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) S[4 * g + r] = __builtin_fmaf(S[4 * g + r], sl2, (RING == 2 ? koff : 0.f) - c4[r]);
    }
}

// ---- online softmax of 32 keys: S becomes P.  Fast path: exponentiate against the current reference maximum
// without looking at the block's own maximum; only if a lane's partial row sum is not
// below 2^16 (a logit beat the reference by more than ~16 bits, or overflowed), or on
// the wave's first block, take the slow path: find the block maximum, move the
// reference, rescale O and l, and exponentiate again.  Probabilities may thus be as
// large as 2^16, which bf16/fp32 operands and the fp32 sums hold without loss.
template <bool FOX> __device__ __forceinline__ float softmax_element(float S, float sl2, float mneg) {
    return __builtin_amdgcn_exp2f(FOX ? S + mneg : __builtin_fmaf(S, sl2, mneg));
}
// E, rs: the fast path's probabilities and their sum; slow: what it comes to, or the wave's first block (no reference yet).
template <bool FOX, int DB>
__device__ __forceinline__ void softmax_settle(f32x16& S, f32x16& E, float rs, bool slow, f32x16 (&O)[DB], float& m_run, float& l_run, float sl2) {
    if (slow) {
        float mloc = fmaxf(S[0], S[1]);
#pragma unroll
        for (int jj = 2; jj < 16; jj += 2) mloc = fmaxf(mloc, fmaxf(S[jj], S[jj + 1]));
        mloc = fmaxf(mloc, __shfl_xor(mloc, 32)) * (FOX ? 1.f : sl2);
        const float m_new = fmaxf(m_run, mloc);     // finite: the first block holds the diagonal
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) O[b][jj] *= alpha;
        rs = 0.f;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            E[jj] = softmax_element<FOX>(S[jj], sl2, -m_new);
            rs += E[jj];
        }
    }
    l_run += rs;
    S = E;
}
__device__ __forceinline__ bool softmax_exceeded(float rs) { return __builtin_amdgcn_ballot_w64(!(rs < 65536.f)) != 0; }
template <bool FOX, int DB>
__device__ __forceinline__ void softmax_step(f32x16& S, f32x16 (&O)[DB], float& m_run, float& l_run, float sl2, bool first) {
    f32x16 E;
    float rs = 0.f;
    bool slow = first;
    if (!slow) {
        const float mneg = -m_run;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            E[jj] = softmax_element<FOX>(S[jj], sl2, mneg);
            rs += E[jj];
        }
        slow = softmax_exceeded(rs);
    }
    softmax_settle<FOX, DB>(S, E, rs, slow, O, m_run, l_run, sl2);
}

// ---- epilogue: normalise, store o and lse (paper Sec. 3.3, last step) ---------------------
// A lane holds pieces of four components, 4h of every eight; with 16-bit results the two halves of the wave exchange
// every other one, so that each stores eight at a time (16 bytes: half as many stores.  Whole forward, 512 heads of 300
// tokens, d = 128 211.4 -> 207.7 us; 128 heads of 2048, d = 64 273.0 -> 270.1, within what two runs differ by).
template <typename TIO, int D, bool FOX>
__device__ __forceinline__ void store_result(const FwdParams& p, const f32x16 (&O)[D / 32], float m_run, float l_run, int bh, int tq, int L, int h) {
    using Vec4 = typename Tr<TIO>::Vec4;
    constexpr int DB = D / 32;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = 1.f / l_tot;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    union { Vec4 v4[4]; u32x4 v8[2]; unsigned w[8]; } out[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[b].v4[g][r] = (TIO)(O[b][4 * g + r] * inv);
        if constexpr (sizeof(TIO) == 2) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                unsigned* w = out[b].w + 4 * g;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const auto x = __builtin_amdgcn_permlane32_swap(w[e], w[2 + e], false, false);
                    w[e] = x[0]; w[2 + e] = x[1];
                }
            }
        }
    }
    if (tq < L) {
        TIO* orow = reinterpret_cast<TIO*>(p.o) + user_vec(p.ul, bh, tq);
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            if constexpr (sizeof(TIO) == 2) {
#pragma unroll
                for (int g = 0; g < 2; ++g) *reinterpret_cast<u32x4*>(orow + 32 * b + 16 * g + 8 * h) = out[b].v8[g];
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g) *reinterpret_cast<Vec4*>(orow + 32 * b + 8 * g + 4 * h) = out[b].v4[g];
            }
        }
        const float ci = FOX ? p.cum[(size_t)bh * p.NC * CHUNK + tq] : 0.f;
        if (h == 0) p.lse[user_scl(p.ul, bh, tq)] = (m_run + __builtin_amdgcn_logf(l_tot) + ci) * 0.69314718055994530942f;
    }
}

}  // namespace path
