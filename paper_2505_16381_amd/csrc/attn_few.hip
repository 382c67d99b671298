// Forward sweep where a chip's worth of workgroups, or a little more, is all there is: the sweep of attn_fwd2.hip -- the same
// products and sums in the same order, bit for bit -- cut by kind of work over the eight waves of a CU, one or two query chunks
// per workgroup.
//
// What bounds it is the length of a chunk's chain: 16-bit operands, d = 128, a wave of 32 queries has 32 products for the
// logits and P V and 32 for the state's update per key chunk, with its exponentials and its reads from LDS in between, and little
// else on its SIMD.  But the state does not depend on the softmax.  So, per query chunk,
//   two waves    32 queries each: logits, online softmax, O.  In a stage of 32 keys they have the softmax of these keys between the products
//                of the logits of the next 32 and of P V of the 32 before, one exponential and one read from LDS per product.
//   two waves    half of the columns of the query state each, a stage and a half ahead; its operand copy goes to the former, and to the other
//                one, through LDS.  The fragments of the chunk products come straight from memory, each read once per query chunk.  They
//                also write the states that a training pair's backward starts from.
//   waves 4..7   the copies of keys and values to LDS, two stages ahead (with two chunks per workgroup these are the states' waves).
// One barrier per stage.  The form of attn_fwd2.hip with copying waves that ran before, with at most 256 tiles of two chunks, took,
// us: sweep of 16 heads of 1000 tokens, d = 128, 33.2, now 21.0, d = 64 20.9 / 14.6; one head of 8000, d = 128, 139 / 94; fp32 (general
// form), d = 64, 4 heads of 900, 90 / 64.  Whole forward, against the general form: two heads of 14000 tokens, d = 128, 364 / 218, d = 64
// 248 / 150; 16 of 4000 235 / 191 and 141 / 113.  Of the 21 us 6 are the start (arguments, first tiles, own chunk), then 0.7 to 1.1 a chunk, of which
// the products alone would take 0.5: reads and writes of LDS (1150 cycles a chunk) and L2 are what is left.
#include <type_traits>

#include "path_common.h"
#include "sweep_form.h"
#include "sweep_parts.h"

namespace path {

template <typename TIO, int D, int CPT> struct FewCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int FE = Tr<T>::FE;
    static constexpr int HF = 32 * D / FE, XF = 32 * D / FE;      // fragments of 32 keys, of 32 queries' states
    static constexpr int NST = 4, NSC = 8;                        // stages of keys and values, of gate sums
    static constexpr size_t smem_bytes = (size_t)(2 * NST * HF + 2 * CPT * XF) * 16 + NSC * 32 * 4;
    static_assert(smem_bytes <= 160 * 1024, "LDS budget");
};

// FOX, EMIT, RING: as in attn_fwd2.hip.  CPT: query chunks per workgroup.
template <typename TIO, int D, bool FOX, bool EMIT, int RING, int CPT>
__global__ __launch_bounds__(512, 2) void attn_few_kernel(FwdParams p) {
    using C = FewCfg<TIO, D, CPT>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using FragV = typename Tr<TIO>::Frag;
    constexpr int KW = Tr<T>::KW;
    constexpr int SPB = 32 / KW, DB = D / 32, DS = D / KW;
    constexpr int HF = C::HF, NST = C::NST, NSC = C::NSC;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* sK = reinterpret_cast<Frag*>(smem);                   // [NST stages] keys
    Frag* sV = sK + NST * HF;                                   // [NST stages] values
    Frag* sX = sV + NST * HF;                                   // [CPT chunks][2 query halves] states
    float* sC = reinterpret_cast<float*>(sX + 2 * CPT * C::XF); // FOX: [NSC stages][32] gate sums of the stage's keys

    const int BH = p.B * p.H, NC = p.NC, NCq = RING == 2 ? p.NCq : NC;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    int bh, rank;
    const int ntiles = (NCq + CPT - 1) / CPT;
    if (!xcd_deal(slot, xcd, ntiles, BH, bh, rank)) return;
    const int cq0 = (ntiles - 1 - rank) * CPT;                  // heaviest first
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int L = seq_len(p.ul, bh, p.L);
    const int NCown = RING == 2 ? NCq : (L + CHUNK - 1) / CHUNK;     // this head's own length (packed batches: may be shorter)
    if (cq0 >= NCown) return;
    // Of the waves 0 .. 2 CPT - 1 (logits) and the next 2 CPT (states) two each have a query chunk.
    const int cw = CPT == 2 ? (wv >> 1) & 1 : 0, cq = cq0 + cw, qb = wv & 1;
    const bool active = cq < NCown;
    const int ctop = cq0 + CPT - 1 < NCown ? cq0 + CPT - 1 : NCown - 1;
    static_assert(SBC % CPT == 0, "the chunks of a workgroup lie in one super-block");
    const int jtop = RING == 2 ? NC - 1 : ctop;                 // (a hop sweeps every chunk of the other segment, all of them as far blocks)
    const int jsb = RING == 2 ? NC : (cq0 / SBC) * SBC;         // first chunk of the own super-block
    const int nsb = (NC + SBC - 1) / SBC;
    // Stage u = 0, 1, ...: chunk jtop - u / 2, key half u % 2, place u % NST.  Iterations W0 .. nstage - 1, a barrier before each: in
    // iteration u the softmax of stage u, between the products of stage u - 1's P V and stage u + 1's logits; then the keys of stage u + 2
    // and, u even, the state for the next chunk are read.  The product after chunk j is applied in iterations v - 2 and v - 1, v = 2 (jtop - j).
    // (A hop needs the first two stages' logits, and may have a product after its first chunk.)
    const int nstage = 2 * (jtop + 1);
    constexpr int W0 = RING == 2 ? -2 : 0;
    float* const rec = RING ? p.ring_state + ((size_t)bh * NCq + cq) * 2 * ring_rec_floats(D) : nullptr;      // of both query halves

    // Copies, by waves 4 .. 7.  Group w, requested in iteration w: the keys of stage w + 4 (read from iteration w + 2 on; their place until
    // iteration w - 2) and the values of stage w + 2 (w + 3; w - 1).  In iteration w, group w - 2 has landed.
    constexpr int CV = HF / 256, CK = CV + (FOX ? 1 : 0);      // a wave's copies: values, keys
    static_assert(HF % 256 == 0, "every wave makes as many copies");
    auto copies_of = [&](int w) { return (w + 4 < nstage ? CK : 0) + (w + 2 >= 0 && w + 2 < nstage ? CV : 0); };
    auto issue_gates = [&](int u) {
        const int j = jtop - (u >> 1), cwv = wv - 4;
        if (FOX && u < nstage && lane < 2)       // 8 floats per wave
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(p.cum + (size_t)bh * NC * CHUNK + (size_t)j * CHUNK + 32 * (u & 1) + 8 * cwv + 4 * lane),
                                             (__attribute__((address_space(3))) void*)(sC + (u & (NSC - 1)) * 32 + 8 * cwv), 16, 0, 0);
    };
    auto issue = [&](int w) {
        const int uk = w + 4, uv = w + 2, jk = jtop - (uk >> 1), jv = jtop - (uv >> 1);
        if (uk < nstage) {
            const T* kg = reinterpret_cast<const T*>(jk >= jsb ? p.kt : p.kt2) + ((size_t)bh * NC + jk) * CHUNK * D;
            async_copy_tile<256, HF>(reinterpret_cast<const Frag*>(kg) + (uk & 1) * HF, sK + (size_t)(uk & (NST - 1)) * HF, tid - 256, wv - 4);
            issue_gates(uk);
        }
        if (uv >= 0 && uv < nstage) {
            const TIO* vg = reinterpret_cast<const TIO*>(p.vt) + ((size_t)bh * NC + jv) * CHUNK * D;
            async_copy_tile<256, HF>(reinterpret_cast<const Frag*>(vg) + (uv & 1) * HF, sV + (size_t)(uv & (NST - 1)) * HF, tid - 256, wv - 4);
        }
    };
    if (wv >= 4) {
        if (W0 == 0) { issue_gates(0); issue_gates(1); }      // (the own chunk's logits are there)
        issue(W0 - 2);
        issue(W0 - 1);
    }
    // All but `most` of this wave's requests, or a few more, have come back.
    auto wait_but = [&](int most) {
#define WAIT_BUT(N) else if (most >= N) asm volatile("s_waitcnt vmcnt(" #N ")" ::: "memory")
        if (most >= 40) asm volatile("s_waitcnt vmcnt(40)" ::: "memory");
        WAIT_BUT(28);
        WAIT_BUT(20);
        WAIT_BUT(12);
        WAIT_BUT(10);
        WAIT_BUT(8);
        WAIT_BUT(5);
        WAIT_BUT(4);
        WAIT_BUT(3);
        WAIT_BUT(2);
        WAIT_BUT(1);
        else copies_landed();
#undef WAIT_BUT
    };
    if (CPT == 1 && wv >= 4) {
        for (int w = W0; w < nstage; ++w) {
            wait_but(copies_of(w - 1));
            lds_barrier();
            issue(w);
        }
        return;
    }

    if (wv >= 2 * CPT) {
        // ---- the query state: fp32 master; its operand copy, in registers, and in LDS for the logits and for the other wave, which has the
        // other half of the columns.  The products' fragments come straight from memory, a chunk ahead: each is read once per query chunk.
        auto state = [&](auto second) {
            constexpr int HX = decltype(second)::value, HB = DB / 2, HS = DS / 2;      // this wave's half; blocks and slabs of a half
            int iter = W0, before = 0, last = 0;          // CPT 2: requests behind the copies of the iteration before the last, in the last one
            // KEPT: requests, at least, behind the fragments that this iteration's products are with, < 0: no products.  The compiler takes a copy to
            // LDS for an access of both memories and, with one on its way, would wait for all requests where the fragments are used, the copies just
            // requested included: us, forward of 16 heads of 4000 tokens, d = 128, 195.6, so 193.8, of 6000 317.7 / 315.2, ring of 32 heads of 1024,
            // d = 64, 73.2 / 72.0.
            const std::integral_constant<int, -1> none;
            auto next_iteration = [&](auto kept) {
                constexpr int KEPT = decltype(kept)::value;
                if constexpr (CPT == 2 && KEPT >= 0) __builtin_amdgcn_s_waitcnt((KEPT & 15) | (KEPT >> 4) << 14 | 0x0f70);
                if constexpr (CPT == 2) wait_but(before + copies_of(iter - 1) + last);
                lds_barrier();
                if constexpr (CPT == 2) issue(iter);
                ++iter;
                before = last;
                last = 0;
            };
            if (!active) {
                while (iter < nstage) next_iteration(none);
                return;
            }
            f32x16 Xm[2][HB];                             // [query half][block]
            Frag own[2][HS], other[2][HS];
            Frag* const sXc = sX + cw * 2 * C::XF;
            auto pack = [&]() {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int b = 0; b < HB; ++b) pack_block<T>(Xm[q][b], own[q] + b * SPB);
            };
            auto publish = [&]() {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int s = 0; s < HS; ++s) sXc[q * C::XF + (HX * HS + s) * 64 + lane] = own[q][s];
            };
            auto read_other = [&]() {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int s = 0; s < HS; ++s) other[q][s] = sXc[q * C::XF + ((1 - HX) * HS + s) * 64 + lane];
            };
            // The chunk of the next product left of chunk j, if any (< 0): the next chunk in the own super-block, then the first of each.
            auto next = [&](int j) {
                if (j <= 0) return -1;
                const int n = j - 1 >= jsb ? j - 1 : (j - 1) / SBC * SBC;
                return n > 0 || RING ? n : -1;
            };
            Frag pa[HB][DS];                              // fragments of a product: each block's in the place of its predecessor's
            auto read_dp = [&](int j, int block, bool used) {
                const Frag* src = (j >= jsb ? reinterpret_cast<const Frag*>(p.dp) + ((size_t)bh * NC + j) * (D * D / C::FE)
                                            : reinterpret_cast<const Frag*>(p.dp2) + ((size_t)bh * nsb + j / SBC) * (D * D / C::FE)) + (HX * HB + block) * DS * 64;
#pragma unroll
                for (int s = 0; s < DS; ++s) pa[block][s] = *(const __attribute__((address_space(1))) Frag*)(scalar_base(src + (s & ~3) * 64, tile_lane<T>(lane, s) * 16) + (s & 3) * 1024);
                if (used) last += DS;                     // (requests that nobody waits for may have gone)
            };
            auto mul = [&](int block) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int s = 0; s < DS; ++s) Xm[q][block] = Tr<T>::mma(pa[block][s], s / HS == HX ? own[q][s % HS] : other[q][s % HS], Xm[q][block]);
            };
            const float* xs = RING == 2 ? rec : p.xinit + ((size_t)bh * NC + cq) * 2 * (size_t)DB * 1024;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int b = 0; b < HB; ++b)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 v4 = *reinterpret_cast<const f32x4*>(xs + q * (RING == 2 ? ring_rec_floats(D) : (size_t)DB * 1024) + (size_t)(HX * HB + b) * 1024 + g * 256 + lane * 4);
#pragma unroll
                        for (int r = 0; r < 4; ++r) Xm[q][b][4 * g + r] = v4[r];
                    }
            pack();
            publish();
            int j = RING == 2 ? jtop : cq - 1;
            const int first = next(j + 1);
            if (first >= 0) {
#pragma unroll
                for (int b = 0; b < HB; ++b) read_dp(first, b, true);
            }
            last = 0;
            while (iter < 2 * (jtop - j) - 2) next_iteration(none);      // (stages of the chunk to the right)
            auto emit = [&](int j) {
                const size_t slot = ((size_t)bh * num_block_slots(NC) + block_slot(cq, j >= jsb ? j : j - (SBC - 1), NC)) * (size_t)CHUNK * D;
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int b = 0; b < HB; ++b) emit_state_block<T, D>(reinterpret_cast<T*>(p.xs) + slot, reinterpret_cast<T*>(p.xsT) + slot, own[q] + b * SPB, HX * HB + b, q, lane);
                last += sizeof(T) == 4 ? 2 * DS : DS;
            };
            auto update = [&](int j, auto near) {
                constexpr int EM = decltype(near)::value ? (sizeof(T) == 4 ? 2 * DS : DS) : 0;
                const int jl = next(j), js = jl >= 0 ? jl : j;      // (no branch around the requests: how many there are is known)
                next_iteration(std::integral_constant<int, HB == 2 ? DS : 0>{});
                read_other();
                mul(0);
                __builtin_amdgcn_sched_barrier(0);
                read_dp(js, 0, jl >= 0);
                if (decltype(near)::value) emit(j);
                next_iteration(std::integral_constant<int, HB == 2 ? DS + EM : -1>{});
                if constexpr (HB == 2) {
                    mul(1);
                    __builtin_amdgcn_sched_barrier(0);
                    read_dp(js, 1, jl >= 0);
                }
                pack();
                publish();
            };
            for (; j >= jsb && (j > 0 || RING); --j) update(j, std::integral_constant<bool, EMIT>{});
            for (; j >= 0; --j) {
                if (j < jsb && j % SBC == 0 && (j > 0 || RING)) { update(j, std::false_type{}); continue; }
                next_iteration(none);
                if (EMIT && (j >= jsb || (j % SBC) == SBC - 1)) emit(j);
                next_iteration(none);
            }
            next_iteration(none);                         // the last two
            next_iteration(none);
            if (RING)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int b = 0; b < HB; ++b)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            f32x4 x4;
#pragma unroll
                            for (int r = 0; r < 4; ++r) x4[r] = Xm[q][b][4 * g + r];
                            *reinterpret_cast<f32x4*>(rec + q * ring_rec_floats(D) + (size_t)(HX * HB + b) * 1024 + g * 256 + lane * 4) = x4;
                        }
        };
        if (qb == 0) state(std::integral_constant<int, 0>{});
        else state(std::integral_constant<int, 1>{});
        return;
    }

    // ---- logits, online softmax, output ---------------------------------------------------------------------------------
    if (!active) {
        for (int w = W0; w < nstage; ++w) lds_barrier();
        return;
    }
    float* const recq = RING ? rec + qb * ring_rec_floats(D) : nullptr;
    const float sl2 = p.scale * 1.44269504088896340736f;
    f32x16 O[DB], S, Sn;
    Frag Xh[DS];
    float m_run = -INFINITY, l_run = 0.f, koff = 0.f;     // m in base-2 logit units; koff: gates in a hop, see attn_fwd2.hip
    f32x4 diag[RING != 2 ? 2 : 1][4];
#pragma unroll
    for (int b = 0; b < DB; ++b) {
        O[b] = zero16();
        if (RING == 2)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 o4 = *reinterpret_cast<const f32x4*>(recq + (size_t)(DB + b) * 1024 + g * 256 + lane * 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) O[b][4 * g + r] = o4[r];
            }
    }
    if (RING == 2) {
        m_run = recq[2 * DB * 1024 + lane]; l_run = recq[2 * DB * 1024 + 64 + lane];
        if (FOX) koff = recq[2 * DB * 1024 + 128 + lane] + p.cum[(size_t)bh * NC * CHUNK + (size_t)NC * CHUNK - 1];
    } else {
#pragma unroll
        for (int kb = 0; kb < (RING != 2 ? 2 : 1); ++kb)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                diag[kb][g] = *reinterpret_cast<const f32x4*>(p.sd + ((size_t)bh * NC + cq) * 4096 + ((size_t)qb * 2 + kb) * 1024 + g * 256 + lane * 4);
    }
    auto read_state = [&]() {
#pragma unroll
        for (int s = 0; s < DS; ++s) Xh[s] = sX[(cw * 2 + qb) * C::XF + s * 64 + lane];
    };
    Frag ka[DS];
    FragV va[DB * SPB], Pb[SPB];
    constexpr int NV = DB * SPB, N = DS + NV;
    auto read_key = [&](int u, int s) { ka[s] = sK[(u & (NST - 1)) * HF + s * 64 + tile_lane<T>(lane, s)]; };
    auto read_value = [&](int u, int n) { va[n] = reinterpret_cast<const FragV*>(sV)[(u & (NST - 1)) * HF + (n % DB * SPB + n / DB) * 64 + lane]; };
    auto add_value = [&](int n) { O[n % DB] = Tr<TIO>::mma(va[n], Pb[n / DB], O[n % DB]); };
    auto logits = [&](f32x16& Sn) {
        Sn = zero16();
#pragma unroll
        for (int s = 0; s < DS; ++s) Sn = Tr<T>::mma(ka[s], Xh[s], Sn);
    };
    // Slice by slice: a product, its share of the exponentials (added up a slice later), and reads from LDS -- the values that the later
    // products are with, then, in the registers of what the first products were with, the keys and maybe the state for the next ones
    // (past the last stage: whatever is there, never used).
    auto stage = [&](int u, auto even, auto first, f32x16& S, f32x16& Sn) {      // S: the stage's logits, Sn: the next one's
        constexpr bool EVEN = decltype(even)::value, FIRST = decltype(first)::value;
        constexpr bool EARLY = FIRST && RING != 2 && !FOX;      // own chunk: nothing to wait for
        if (EARLY) softmax_step<FOX, DB>(S, O, m_run, l_run, sl2, true);
        lds_barrier();
        if (FOX) gate_logits<RING>(S, sC + (u & (NSC - 1)) * 32 + 4 * h, sl2, koff);
        if constexpr (FIRST) {
#pragma unroll
            for (int s = 0; s < DS; ++s) read_key(u + 2, s);
            read_state();
            if (!EARLY) softmax_step<FOX, DB>(S, O, m_run, l_run, sl2, RING != 2);
        } else {
            constexpr int EV = 16 / N;
            static_assert(N * EV == 16 && (DS % NV == 0 || NV % DS == 0), "whole shares");
            f32x16 E;
            float rs = 0.f;
            const float mneg = -m_run;
            Sn = zero16();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < N; ++n) {
                if (n < DS) {
#pragma unroll
                    for (int r = n * NV / DS; r < (n + 1) * NV / DS; ++r) read_value(u - 1, r);
                    Sn = Tr<T>::mma(ka[n], Xh[n], Sn);
                } else {
                    add_value(n - DS);
#pragma unroll
                    for (int r = (n - DS) * DS / NV; r < (n - DS + 1) * DS / NV; ++r) {
                        read_key(u + 2, r);
                        if (EVEN) Xh[r] = sX[(cw * 2 + qb) * C::XF + r * 64 + lane];
                    }
                }
#pragma unroll
                for (int e = 0; e < EV; ++e) {
                    E[n * EV + e] = softmax_element<FOX>(S[n * EV + e], sl2, mneg);
                    if (n > 0) rs += E[(n - 1) * EV + e];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int e = 0; e < EV; ++e) rs += E[(N - 1) * EV + e];
            softmax_settle<FOX, DB>(S, E, rs, softmax_exceeded(rs), O, m_run, l_run, sl2);
        }
        pack_block<TIO>(S, Pb);
    };
    int u = 0;
    if (RING == 2) {
        lds_barrier();                                    // iteration -2
        read_state();                                     // (the next one may be published in iteration -1)
        lds_barrier();
#pragma unroll
        for (int s = 0; s < DS; ++s) read_key(0, s);
        logits(S);
#pragma unroll
        for (int s = 0; s < DS; ++s) read_key(1, s);
        logits(Sn);                                       // (stage 0 has no products of a stage before to stand among)
    } else {                                              // own chunk: precomputed Q K^T - F Y, causal mask
        for (; u < 2 * (jtop - cq); ++u) lds_barrier();   // (stages of the chunk to the right)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[4 * g + r] = 8 * g + 4 * h + r <= 32 * qb + l32 ? diag[0][g][r] : -INFINITY;
                Sn[4 * g + r] = 32 + 8 * g + 4 * h + r <= 32 * qb + l32 ? diag[RING != 2][g][r] : -INFINITY;
            }
    }
    stage(u, std::true_type{}, std::true_type{}, S, Sn);
    stage(u + 1, std::false_type{}, std::false_type{}, Sn, S);
    for (u += 2; u < nstage; u += 2) {
        stage(u, std::true_type{}, std::false_type{}, S, Sn);
        stage(u + 1, std::false_type{}, std::false_type{}, Sn, S);
    }
#pragma unroll
    for (int n = 0; n < NV; ++n) { read_value(nstage - 1, n); add_value(n); }
    if (RING) {
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 o4;
#pragma unroll
                for (int r = 0; r < 4; ++r) o4[r] = O[b][4 * g + r];
                *reinterpret_cast<f32x4*>(recq + (size_t)(DB + b) * 1024 + g * 256 + lane * 4) = o4;
            }
        recq[2 * DB * 1024 + lane] = m_run;
        recq[2 * DB * 1024 + 64 + lane] = l_run;
        recq[2 * DB * 1024 + 128 + lane] = (RING == 2 && FOX) ? koff : 0.f;
        return;
    }
    store_result<TIO, D, FOX>(p, O, m_run, l_run, bh, cq * CHUNK + 32 * qb + l32, L, h);
}

static int few_chunks(const FwdParams& p) { return sweep_form(p.ring == 2 ? p.NCq : p.NC, p.NC, p.B * p.H, p.ring != 0); }

template <typename TIO, int D, bool FOX, bool EMIT, int RING, int CPT>
hipError_t launch_attn_few_c(const FwdParams& p, hipStream_t stream) {
    constexpr size_t bytes = FewCfg<TIO, D, CPT>::smem_bytes;
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_few_kernel<TIO, D, FOX, EMIT, RING, CPT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (attr_err != hipSuccess) return attr_err;
    const int ntiles = ((RING == 2 ? p.NCq : p.NC) + CPT - 1) / CPT;
    hipLaunchKernelGGL((attn_few_kernel<TIO, D, FOX, EMIT, RING, CPT>), dim3(xcd_deal_grid(ntiles, p.B * p.H)), dim3(512), bytes, stream, p);
    return hipGetLastError();
}
template <typename TIO, int D, bool FOX, bool EMIT, int RING>
hipError_t launch_attn_few_f(const FwdParams& p, hipStream_t stream) {
    if constexpr (sizeof(TIO) == 2) {
        if (few_chunks(p) == 2) return launch_attn_few_c<TIO, D, FOX, EMIT, RING, 2>(p, stream);
    }
    return launch_attn_few_c<TIO, D, FOX, EMIT, RING, 1>(p, stream);
}
template <typename TIO, int D>
hipError_t launch_attn_few_t(const FwdParams& p, hipStream_t stream) {
    if (p.ring == 1) return p.cum ? launch_attn_few_f<TIO, D, true, false, 1>(p, stream) : launch_attn_few_f<TIO, D, false, false, 1>(p, stream);
    if (p.ring == 2) return p.cum ? launch_attn_few_f<TIO, D, true, false, 2>(p, stream) : launch_attn_few_f<TIO, D, false, false, 2>(p, stream);
    if (p.emit_states) return p.cum ? launch_attn_few_f<TIO, D, true, true, 0>(p, stream) : launch_attn_few_f<TIO, D, false, true, 0>(p, stream);
    return p.cum ? launch_attn_few_f<TIO, D, true, false, 0>(p, stream) : launch_attn_few_f<TIO, D, false, false, 0>(p, stream);
}
bool attn_few_runs(const FwdParams& p, int d, int is_bf16) { return is_bf16 ? few_chunks(p) > 0 : d == 64 && few_chunks(p) == 1; }
hipError_t launch_attn_few(const FwdParams& p, int d, int is_bf16, hipStream_t stream) {
    if (!is_bf16) return launch_attn_few_t<float, 64>(p, stream);
    return d == 64 ? launch_attn_few_t<bf16_t, 64>(p, stream) : launch_attn_few_t<bf16_t, 128>(p, stream);
}

}  // namespace path
