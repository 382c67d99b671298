// Decode path of PaTH attention (paper Sec. 3.4 "Efficient Inference").
//
//  * Key prefill (the section's second formula): the cache a prompt leaves behind holds
//    k_i^(l) = H_l ... H_{i+1} k_i.  Blockwise with suffix products, on top of what the forward's
//    preprocessing already wrote: Kb2_c (keys carried to their super-block's right edge) and
//    -dP2_J = -(I - P_superblock J).  With E = I - R (R = P2_last ... P2_{J+1}) kept transposed in
//    fp32 registers,
//        K^(l)_c = Kb2_c - Kb2_c E^T ,      E <- E + dP2_J - E dP2_J ,
//    exactly the second level's own recurrence one level up (see prep2_fwd.hip), so the cost is
//    linear in l.  One workgroup per (head, super-block): it runs the d x d recurrence from the
//    right end down to its own super-block (a few small products per step, the same for every
//    workgroup of the head, hence the same E) and carries only its own super-block's keys.
//    Results go row-major into the key cache, in the cache's storage type.  (A prompt of one super-block
//    has nothing to carry beyond it: its keys take the second level's own step straight to the cache,
//    see prep2_fwd.hip.  16-bit operands, few heads or short prompts: every chunk by itself, see key_carry.hip.)
//    Further workgroups copy the values.
//
//  * Decode step (the section's first equation): when token t arrives every cached key is
//    refreshed in place, k_i <- k_i - beta_t (w_t . k_i) w_t, and attention of q_t over the
//    refreshed cache is ordinary softmax attention.  Both happen in ONE pass over the key cache
//    (read k, write k, read v: 3 n d elements per head -- HBM-bound), split over the cached
//    positions; the split that ends last merges them, adds the arriving token's own key and
//    value, and appends them to the caches.  Short caches are not split.
//
//  * PaTH-FoX at decode time (Sec. 2.2 extension): with the running sums c_i of the log gates kept beside the
//    caches, key i's logit gets c_t - c_i, c_t = c_{t-1} + log f_t; the arriving token's own logit gets nothing
//    and its sum is appended (GATES instantiations).
#include <atomic>
#include <type_traits>

#include "path_common.h"
#include "decode_decl.h"

namespace path {

// ---------------------------------------------------------------------------------------
template <typename TIO, int D> struct PrefillCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int KV_FRAGS = CHUNK * D / Tr<T>::FE, DP_FRAGS = D * D / Tr<T>::FE;
    // operand copy of E | -dP2 tile of the super-block | one key tile
    static constexpr size_t smem_bytes = (size_t)(2 * DP_FRAGS + KV_FRAGS) * 16;
};

template <typename TIO, int D>
__global__ __launch_bounds__(256) void key_prefill_kernel(PrefillArgs a) {
    using T = typename Compute<TIO>::type;
    using Frag = typename Tr<T>::Frag;
    typedef typename Tr<TIO>::Vec4 OVec4;
    constexpr int FE = Tr<T>::FE, KW = Tr<T>::KW;
    constexpr int SPB = 32 / KW, DB = D / 32, DS = D / KW, NE = DB * DB / 4, NK = 2 * DB / 4;
    constexpr int KVF = PrefillCfg<TIO, D>::KV_FRAGS, DPF = PrefillCfg<TIO, D>::DP_FRAGS;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* Es = reinterpret_cast<Frag*>(smem);      // tile (rows a, contraction b) of E
    Frag* sDP = Es + DPF;                          // -dP2 tile (rows b, contraction a)
    Frag* sK = sDP + DPF;                          // Kb2 tile of the current chunk (rows s, contraction c)

    const int bh = blockIdx.x, Jme = blockIdx.y;   // this workgroup carries the keys of super-block Jme
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, h = lane >> 5, l32 = lane & 31;
    const int NC = a.NC, L = a.L, nsb = (NC + SBC - 1) / SBC;
    if (Jme >= nsb) { copy_value_rows<TIO, D, 256>(a.v, a.vcache, L, a.Lmax, bh, Jme - nsb, tid); return; }

    Frag idf[SPB];
    identity_frags<T>(idf, l32, h);
    f32x16 Fm[NE];      // E^T: block o = (rows b-block bb, lane a-block ab), blk = wv + 4*o

    for (int J = nsb - 1; J >= Jme; --J) {
        const bool lastsb = J == nsb - 1;          // E = 0: plain copy
        const int c0 = J * SBC, c1 = (c0 + SBC < NC) ? c0 + SBC : NC;
        if (J > Jme) {                             // on the way down: only the product of super-block J
            __syncthreads();                       // sDP is free
            async_copy_tile<256, DPF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.dp2) + ((size_t)bh * nsb + J) * (size_t)D * D), sDP, tid, wv);
            wait_async_and_sync();
        }
        for (int c = c0; c < c1 && J == Jme; ++c) {
            const size_t bhc = (size_t)bh * NC + c;
            __syncthreads();                       // sK is free (and, first time round, Es is written)
            async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.kt2) + bhc * (size_t)CHUNK * D), sK, tid, wv);
            wait_async_and_sync();
            // K^(l)^T[cc][s] = Kb2^T[cc][s] - sum_b E[cc][b] Kb2[s][b]   (registers rows cc, lane s)
#pragma unroll
            for (int o = 0; o < NK; ++o) {
                const int blk = wv + 4 * o, cb = blk >> 1, sb2 = blk & 1;
                f32x16 acc = zero16();
                if (!lastsb) {
#pragma unroll
                    for (int s = 0; s < DS; ++s) acc = Tr<T>::mma(Es[(cb * DS + s) * 64 + lane], sK[((size_t)sb2 * DS + s) * 64 + tile_lane<T>(lane, s)], acc);
                }
                const int s = 32 * sb2 + l32, tok = c * CHUNK + s;
                if (tok < L) {
                    TIO* dst = reinterpret_cast<TIO*>(a.kcache) + ((size_t)bh * a.Lmax + tok) * D + 32 * cb + 4 * h;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        // accumulator register jj = 4g + r holds column 32cb + 8g + 4h + r of key s; the tile's
                        // fragment order keeps that same element at slab jj / FE, position jj % FE of this lane
                        OVec4 o4;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int jj = 4 * g + r;
                            const Frag kf = sK[((size_t)sb2 * DS + cb * SPB + jj / FE) * 64 + tile_lane<T>(lane, jj / FE)];
                            o4[r] = (TIO)((float)kf[jj % FE] - acc[jj]);
                        }
                        *reinterpret_cast<OVec4*>(dst + 8 * g) = o4;
                    }
                }
            }
        }
        if (J == Jme) break;
        // E^T <- E^T + dP2^T - dP2^T E^T   (registers rows b, lane a)
#pragma unroll
        for (int o = 0; o < NE; ++o) {
            const int blk = wv + 4 * o, bb = blk / DB, ab = blk % DB;
            f32x16 acc = zero16();
            if (!lastsb) {
#pragma unroll
                for (int s = 0; s < DS; ++s) acc = Tr<T>::mma(sDP[((size_t)bb * DS + s) * 64 + tile_lane<T>(lane, s)], Es[(ab * DS + s) * 64 + lane], acc);
            }
            Frag dfr[SPB];
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) dfr[s2] = sDP[((size_t)bb * DS + ab * SPB + s2) * 64 + tile_lane<T>(lane, s2)];
            const f32x16 dpT = transpose32<T>(dfr, idf);
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) {
                const float prev = lastsb ? 0.f : Fm[o][jj];
                Fm[o][jj] = prev - dpT[jj] + acc[jj];
            }
        }
        __syncthreads();      // every read of the old operand copy is done
#pragma unroll
        for (int o = 0; o < NE; ++o) {
            const int blk = wv + 4 * o, bb = blk / DB, ab = blk % DB;
            Frag fr[SPB];
            pack_block<T>(Fm[o], fr);
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) Es[(ab * DS + bb * SPB + s2) * 64 + lane] = fr[s2];
        }
    }
}

// ---------------------------------------------------------------------------------------
// The last part of a step, by D threads (whole waves), thread c for component c: the arriving token's own key and value
// join the cached keys' maximum M, row sum Ls and unnormalised output O; the caches grow by one.
template <typename TIO, int D, bool GATES>
struct DecodeTail {
    TIO kt, vt;
    float qk, gate;
    __device__ __forceinline__ void load(const DecodeArgs& a, int bh, int c) {
        const TIO* q = reinterpret_cast<const TIO*>(a.q) + (size_t)bh * D;
        const TIO* k = reinterpret_cast<const TIO*>(a.k) + (size_t)bh * D;
        kt = k[c];
        vt = reinterpret_cast<const TIO*>(a.v)[(size_t)bh * D + c];
        qk = 0.f;
#pragma unroll
        for (int b = 0; b < D; b += 64) qk = __builtin_fmaf((float)q[b + (c & 63)], (float)k[b + (c & 63)], qk);
        // the token's running gate sum, which joins the cache (its own logit carries no gate)
        gate = GATES ? (a.n > 0 ? a.ccache[(size_t)bh * a.Lmax + a.n - 1] : 0.f) + (float)reinterpret_cast<const TIO*>(a.log_f)[bh] : 0.f;
    }
    // The token's own logit.  Every wave of the head takes it -- all of q and k -- before a barrier, and no wave writes o
    // before that barrier: o may be one of the inputs.
    __device__ __forceinline__ void logit(float scale) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) qk += __shfl_xor(qk, off);
        qk *= scale;
    }
    __device__ __forceinline__ void finish(const DecodeArgs& a, int bh, int c, float M, float Ls, float O) const {
#pragma clang fp contract(off)
        const float s_new = qk;
        const float Mn = fmaxf(M, s_new);
        const float old = M == -INFINITY ? 0.f : __expf(M - Mn), own = __expf(s_new - Mn);
        Ls = __builtin_fmaf(Ls, old, own);
        O = __builtin_fmaf(O, old, own * (float)vt);
        reinterpret_cast<TIO*>(a.o)[(size_t)bh * D + c] = (TIO)(O / Ls);
        if (c == 0) a.lse[bh] = Mn + __logf(Ls);
        reinterpret_cast<TIO*>(a.kcache)[((size_t)bh * a.Lmax + a.n) * D + c] = kt;
        reinterpret_cast<TIO*>(a.vcache)[((size_t)bh * a.Lmax + a.n) * D + c] = vt;
        if (GATES && c == 0) a.ccache[(size_t)bh * a.Lmax + a.n] = gate;
    }
};

// One pass over the cached keys of a split: refresh, logit, online softmax, P V.  DIRECT: the split is the whole head
// and the workgroup ends the step itself; else every split leaves its partial results in the
// workspace, and the last one (MERGED) or decode_merge_kernel (RECORDS) merges them.
// A key is handled by LPK = D/8 consecutive lanes (8 elements each); a wave takes 64/LPK keys at a time and UN such
// rounds per step, whose rows it has requested a step ahead.  The sums over a key's lanes are DPP moves (a shuffle
// through LDS costs its latency eight times per key).
// What bounds it: HBM (3 n d elements per head), for few heads the latency of a step.  Values are read and refreshed
// keys written past the caches' replacement (non-temporal), which leaves the Infinity Cache (256 MB) to the keys, the
// one stream that is both read and written; the same hint on the key reads costs 15 %.  d = 128, replayed from a graph,
// against a pass without prefetch, hints and DPP sums: B=4, H=16, n=8192 with one cache step after step, whose keys stay in
// that cache, 81.6 -> 65.3 us (without the hints a third slower), with six caches in turn, as a model's layers have them, 96.6
// -> 84.0 (4.8 TB/s); 16 heads of 32768 keys 101.8 -> 67.3 and 117.6 -> 85.6.
template <int LPK> __device__ __forceinline__ float group_sum(float x) {      // over the LPK lanes of a key, in all of them
    static_assert(LPK == 8 || LPK == 16, "within a row of 16 lanes");
    auto add = [&](auto ctrl) { x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    add(std::integral_constant<int, 0xB1>{});                     // quad_perm [1,0,3,2]
    add(std::integral_constant<int, 0x4E>{});                     // quad_perm [2,3,0,1]
    add(std::integral_constant<int, 0x141>{});                    // row_half_mirror: the other quad of the eight
    if (LPK == 16) add(std::integral_constant<int, 0x140>{});     // row_mirror: the other eight
    return x;
}

template <typename T> __device__ __forceinline__ void agent_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ T agent_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Merge of the splits inside the same launch, without a counter that would have to start at zero: every split leaves its
// record and then its flag, and then looks at all flags of the head; a split that finds them all set merges.  The last one
// to set its flag does; so may others that look at that moment, which write the same bits.  Nobody waits for another.  A
// merge clears the flags behind it, by when every split has set its own, so that the next step finds none; a workspace that
// has been anything else holds the call's 64-bit pattern with probability 2^-64 (a pattern per call, so that flags of a call
// that raced with another on its workspace mean nothing later).  All inputs of the token are in registers before a flag is
// set (o may be one of them).  It takes as long as a second launch on the GPU, and 2.8 us less on the host.  (A tag
// beside every value instead of the flag, one trip to memory less: 1024 keys, 64 heads, d = 128 16.3 us against 14.2.)
// A captured step would carry one pattern through all its replays, and flags that a replay left standing would be taken for
// the next one's: its splits leave records only, and a second launch merges them, whatever the workspace held.  (Both forms
// give the same bits: what may be rounded once is written as __builtin_fmaf, and the compiler fuses nothing by itself.)
enum DecodeMode { DECODE_DIRECT, DECODE_MERGED, DECODE_RECORDS };
struct DecodeRecord {            // of one split and 64 components
    float o[64], m, l;
    unsigned long long flag;
};

// One wave: the records of its 64 components (at most 64 splits: lane s holds the maximum and the row sum of split s), then the
// step's last part, component c of D per lane.
template <typename TIO, int D, bool GATES, bool AGENT, typename F>
__device__ __forceinline__ void decode_merge(const DecodeArgs& a, const DecodeRecord* rec, int nsplit, const DecodeTail<TIO, D, GATES>& tail, int bh, int c, F meanwhile) {
#pragma clang fp contract(off)
    static_assert(DECODE_MAX_SPLITS <= 64, "one split per lane");
    const int lane = c & 63;
    auto get = [](const float* p) { return AGENT ? agent_load(p) : *p; };
    constexpr int NB = 16;                            // outputs of so many splits requested at once
    float on[NB];
    auto request_o = [&](int s0) {                    // (splits past the last one repeat it, and count as zero)
#pragma unroll
        for (int r = 0; r < NB; ++r) on[r] = get(&rec[s0 + r < nsplit ? s0 + r : nsplit - 1].o[lane]);
    };
    const float ms = lane < nsplit ? get(&rec[lane].m) : -INFINITY;
    float Ls = lane < nsplit ? get(&rec[lane].l) : 0.f;
    request_o(0);
    meanwhile();
    float M = ms;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float wt = ms == -INFINITY ? 0.f : __expf(ms - M);
    Ls *= wt;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) Ls += __shfl_xor(Ls, off);
    float O = 0.f;
    for (int s0 = 0; s0 < nsplit; s0 += NB) {
        float oc[NB];
#pragma unroll
        for (int r = 0; r < NB; ++r) oc[r] = s0 + r < nsplit ? on[r] : 0.f;
        if (s0 + NB < nsplit) request_o(s0 + NB);
#pragma unroll
        for (int r = 0; r < NB; ++r) O = __builtin_fmaf(oc[r], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), s0 + r)), O);
    }
    tail.finish(a, bh, c, M, Ls, O);
}

template <typename TIO, int D, bool GATES, int NT, DecodeMode MODE>
__global__ __launch_bounds__(NT) void decode_partial_kernel(DecodeArgs a) {
#pragma clang fp contract(off)
    constexpr int LPK = D / 8, KPW = 64 / LPK, NW = NT / 64, UN = 4 / (int)sizeof(TIO), STEP = NW * UN * KPW;
    typedef TIO Vec8 __attribute__((ext_vector_type(8)));
    __shared__ float red_m[NW], red_l[NW];
    __shared__ float red_o[NW][D];

    const int split = blockIdx.x, bh = blockIdx.y, nsplit = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane / LPK, sub = lane % LPK;                 // key within the wave's round; 8-element slice
    const int n = a.n;
    const int i_begin = (int)((long long)n * split / nsplit), i_end = (int)((long long)n * (split + 1) / nsplit);

    TIO* kc = reinterpret_cast<TIO*>(a.kcache) + (size_t)bh * a.Lmax * D + 8 * sub;
    const TIO* vc = reinterpret_cast<const TIO*>(a.vcache) + (size_t)bh * a.Lmax * D + 8 * sub;
    const float* cc = GATES ? a.ccache + (size_t)bh * a.Lmax : nullptr;
    Vec8 kn[UN], vn[UN];                              // the next step's rows, requested a step ahead
    float cn[UN];
    auto request = [&](int i0) {                      // (positions past the end repeat the last one)
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            int i = i0 + r * KPW + grp;
            i = i < i_end ? i : i_end - 1;
            kn[r] = *reinterpret_cast<const Vec8*>(kc + (size_t)i * D);
            vn[r] = __builtin_nontemporal_load(reinterpret_cast<const Vec8*>(vc + (size_t)i * D));
            cn[r] = GATES ? cc[i] : 0.f;
        }
    };
    int i0 = i_begin + wv * (UN * KPW);
    if (i0 < i_end) request(i0);
    DecodeTail<TIO, D, GATES> tail;
    if (MODE != DECODE_RECORDS && tid < D) tail.load(a, bh, tid);

    float q8[8], w8[8];
    {
        const Vec8 qv = *reinterpret_cast<const Vec8*>(reinterpret_cast<const TIO*>(a.q) + (size_t)bh * D + 8 * sub);
        const Vec8 wv8 = *reinterpret_cast<const Vec8*>(reinterpret_cast<const TIO*>(a.w) + (size_t)bh * D + 8 * sub);
#pragma unroll
        for (int e = 0; e < 8; ++e) { q8[e] = (float)qv[e]; w8[e] = (float)wv8[e]; }
    }
    const float beta = (float)reinterpret_cast<const TIO*>(a.beta)[bh];
    const float c_t = GATES ? (n > 0 ? cc[n - 1] : 0.f) + (float)reinterpret_cast<const TIO*>(a.log_f)[bh] : 0.f;
    float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;

    for (; i0 < i_end; i0 += STEP) {
        Vec8 kv[UN], vv[UN];
        float ci[UN], s[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) { kv[r] = kn[r]; vv[r] = vn[r]; ci[r] = cn[r]; }
        if (i0 + STEP < i_end) request(i0 + STEP);
        float wk[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            wk[r] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) wk[r] = __builtin_fmaf(w8[e], (float)kv[r][e], wk[r]);
        }
#pragma unroll
        for (int r = 0; r < UN; ++r) wk[r] = group_sum<LPK>(wk[r]);
        // refreshed keys, rounded to the cache's storage type: the stored value is the state, and
        // the logit is taken against it
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            const int i = i0 + r * KPW + grp;
            s[r] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                kv[r][e] = (TIO)__builtin_fmaf(-beta * wk[r], w8[e], (float)kv[r][e]);
                s[r] = __builtin_fmaf(q8[e], (float)kv[r][e], s[r]);
            }
            if (i < i_end) __builtin_nontemporal_store(kv[r], reinterpret_cast<Vec8*>(kc + (size_t)i * D));
        }
        float mn = m;
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            s[r] = GATES ? __builtin_fmaf(a.scale, group_sum<LPK>(s[r]), c_t - ci[r]) : a.scale * group_sum<LPK>(s[r]);
        }
        if (i0 + UN * KPW > i_end) {                      // past the end: weight zero, and a zero to weigh (the repeated row may hold infinities)
#pragma unroll
            for (int r = 0; r < UN; ++r)
                if (i0 + r * KPW + grp >= i_end) { s[r] = -INFINITY; vv[r] = Vec8{}; }
        }
#pragma unroll
        for (int r = 0; r < UN; ++r) mn = fmaxf(mn, s[r]);
        const float ref = mn == -INFINITY ? 0.f : mn;             // nothing yet: every weight below is exp(-inf)
        const float alpha = __expf(m - ref);
        m = mn;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= alpha;
#pragma unroll
        for (int r = 0; r < UN; ++r) {
            const float pr = __expf(s[r] - ref);
            l = r == 0 ? __builtin_fmaf(l, alpha, pr) : l + pr;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(pr, (float)vv[r][e], acc[e]);
        }
    }
    // merge the keys of the wave's lanes, then the waves
    {
        float M = m;
#pragma unroll
        for (int off = LPK; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
        const float sc = m == -INFINITY ? 0.f : __expf(m - M);
        l *= sc;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= sc;
#pragma unroll
        for (int off = LPK; off < 64; off <<= 1) {
            l += __shfl_xor(l, off);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off);
        }
        if (lane == 0) { red_m[wv] = M; red_l[wv] = l; }
        if (grp == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) red_o[wv][8 * sub + e] = acc[e];
        }
    }
    if (MODE != DECODE_RECORDS && wv < D / 64) {
        tail.logit(a.scale);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // all that this wave reads of the token's inputs is in registers
    }
    __syncthreads();
    if (tid >= D) return;
    float M = -INFINITY;
#pragma unroll
    for (int g = 0; g < NW; ++g) M = fmaxf(M, red_m[g]);
    float Ls = 0.f, O = 0.f;
#pragma unroll
    for (int g = 0; g < NW; ++g) {
        const float sc = red_m[g] == -INFINITY ? 0.f : __expf(red_m[g] - M);
        Ls = __builtin_fmaf(red_l[g], sc, Ls);
        O = __builtin_fmaf(red_o[g][tid], sc, O);
    }
    if constexpr (MODE == DECODE_DIRECT) { tail.finish(a, bh, tid, M, Ls, O); return; }
    // The record of this wave's 64 components, past the L2s (agent scope); once it is there, the flag.
    DecodeRecord* const rec = reinterpret_cast<DecodeRecord*>(a.partial) + (size_t)(bh * (D / 64) + wv) * nsplit;
    DecodeRecord* const own = rec + split;
    if constexpr (MODE == DECODE_RECORDS) {
        own->o[lane] = O;
        if (lane == 0) { own->m = M; own->l = Ls; }
        return;
    }
    agent_store(&own->o[lane], O);
    if (lane == 0) { agent_store(&own->m, M); agent_store(&own->l, Ls); }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) agent_store(&own->flag, a.flag);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const unsigned long long flag = lane < nsplit ? agent_load(&rec[lane].flag) : a.flag;
    if (__builtin_amdgcn_ballot_w64(flag != a.flag) != 0) return;      // another split will find them all set
    asm volatile("" ::: "memory");
    decode_merge<TIO, D, GATES, true>(a, rec, nsplit, tail, bh, tid, []() {});
    if (lane < nsplit) agent_store(&rec[lane].flag, 0ull);
}

template <typename TIO, int D, bool GATES>
__global__ __launch_bounds__(D) void decode_merge_kernel(DecodeArgs a, int nsplit) {
    const int bh = blockIdx.x, c = threadIdx.x;
    const DecodeRecord* rec = reinterpret_cast<const DecodeRecord*>(a.partial) + (size_t)(bh * (D / 64) + (c >> 6)) * nsplit;
    DecodeTail<TIO, D, GATES> tail;
    decode_merge<TIO, D, GATES, false>(a, rec, nsplit, tail, bh, c, [&]() {
        tail.load(a, bh, c);
        tail.logit(a.scale);
        if (D > 64) __syncthreads();
    });
}

// ---------------------------------------------------------------------------------------
template <typename TIO, int D>
static hipError_t launch_prefill_t(const PrefillArgs& a, int BH, hipStream_t st) {
    const size_t bytes = PrefillCfg<TIO, D>::smem_bytes;
    static const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&key_prefill_kernel<TIO, D>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((key_prefill_kernel<TIO, D>), dim3(BH, (a.NC + SBC - 1) / SBC + value_row_pieces(a.L)), dim3(256), bytes, st, a);
    return hipGetLastError();
}
hipError_t launch_key_prefill(const PrefillArgs& a, int BH, int d, int is_bf16, hipStream_t st) {
    if (is_bf16) return d == 64 ? launch_prefill_t<bf16_t, 64>(a, BH, st) : launch_prefill_t<bf16_t, 128>(a, BH, st);
    return d == 64 ? launch_prefill_t<float, 64>(a, BH, st) : launch_prefill_t<float, 128>(a, BH, st);
}

// Splits of the cached positions.  Bound by HBM, a step takes as long as the fullest CU: what counts is the share of a head's
// keys that its workgroups have, ceil(splits * heads / 256) / splits.  Eight waves, one or two workgroups per CU (registers
// leave room for sixteen waves): 34 heads of 12825 keys, d = 128, 15 splits (510 workgroups) 55.5 us, 16 (544) 64.1; 62 of 2152
// 8 (496) 20.8, 9 (558) 25.2; fp32, 10 of 6441 25 (250) 22.9, 32 (320) 29.2.  Two only up to 16 splits -- one batch of the
// merge: 16 heads of 8192 keys 16 20.8, 32 21.2 -- and otherwise if they are the better ones.  Four waves, up to four
// workgroups, where that divides better from 96 heads on: gated, 140 of 1827 7 (980) 36.3, eight waves 3 (420) 37.1; 200 of 2000 5
// (1000) 52.8, 2 (400) 54.8.
// Where keys and values are as large as the Infinity Cache, four workgroups per CU in two rounds: in one round some lengths bring
// the workgroups' addresses into step: three caches in turn, 64 heads of 8192 keys in caches of 8256 88 us, of 8000 in 8256 88, in two
// 84 both; else they are level (8192 in 8200 84.6 / 83.1, in 9192 85.5 / 85.0; of 7000 keys 70.6 / 72.1).  One cache step after step, part of
// which stays in the Infinity Cache, is ahead in one round (66 / 68.4), and so is everything smaller (64 heads of 4096 36 / 41).
// A split has a step of its waves to do, 16 KB of keys, and no more of them are taken than pay for their merge: one head,
// replayed, 350 KB of keys 15 splits 7.0 us, 32 7.2; fp32 1400 KB 32 8.1, 44 8.2; 8 MB 60 12.9, 32 15.8.  Short and few heads: splits of
// four waves and 64 keys, which start on more CUs (one head of 577 keys, d = 64, 10 of four waves 6.5 us, 5 of eight 6.9), unless they
// fill them less evenly.
// More than 256 heads: a step takes 50 us and more of the GPU, a second launch costs none of it, and without the merge the
// kernel has 91 registers and not 99, five waves per SIMD: 300 heads of 1500 keys 59.0 us, merged in the launch 63.8.
struct DecodeSplits { int n, waves; bool merged; };
static DecodeSplits decode_splits(int BH, int n, size_t key_bytes) {
    const int len4 = (n + 63) / 64, steps = (int)((key_bytes + 16383) / 16384);
    if (BH > 256) { const int s = (1024 + BH - 1) / BH; return {s < 1 ? 1 : s < len4 ? s : len4, 4, false}; }
    const int most = key_bytes < 400 * 1024 ? 16 : key_bytes < 2560 * 1024 ? 32 : DECODE_MAX_SPLITS, lim = most < steps ? most : steps;
    if (BH >= 64 && BH * key_bytes >= (size_t)120 << 20) return {1024 / BH, 8, true};
    auto load = [&](int s) { return (s * BH + 255) / 256; };                   // workgroups of the fullest CU
    int s8 = 256 / BH < lim ? 256 / BH : lim;
    if (len4 <= 16 && len4 * BH <= 512) return load(len4) * s8 <= load(s8) * len4 ? DecodeSplits{len4, 4, true} : DecodeSplits{s8, 8, true};
    const int two = 512 / BH < lim ? 512 / BH : lim;
    if (two <= 16 && load(two) * s8 <= load(s8) * two) s8 = two;
    if (BH >= 96) {
        int s4 = 1;
        for (int j = 1; j <= 4; ++j) {
            const int s = 256 * j / BH < len4 ? 256 * j / BH : len4;
            if (load(s) * s4 < load(s4) * s) s4 = s;
        }
        if (10 * load(s4) * s8 <= 9 * load(s8) * s4) return {s4, 4, true};
    }
    return {s8, 8, true};
}

// Short heads are not split: one workgroup of sixteen waves (up to 128 keys four: 512 heads of 100 keys, d = 64, 7.9 us against
// 10.7), which has nothing to merge but one CU for a head.  The line holds for steps replayed from a graph (eager ones are bound by
// their one launch, 9.3 us, on either side): bf16 64 KB of keys up to 40 heads, 88 for 64, 120 for 96, 128 from 104 on; fp32, whose
// keys a wave is done with sooner, 88 KB up to 40 heads, 112 for 64, 128 from 80 on.  Above 128 KB it never is ahead.  us, one
// workgroup against splits, bf16: 16 heads, d = 128, 56 KB 6.7 / 7.1, 72 7.3 / 7.0, 120 9.4 / 7.1; 48 heads, d = 64, 72 KB 7.6 / 7.9, 88 8.4 / 8.2;
// 96 heads, d = 64, 72 KB 8.0 / 9.1, 104 9.7 / 10.1, 120 11.0 / 10.5; 200 heads, d = 64, 104 KB 12.8 / 15.0.  fp32: 4 heads, d = 128, 72 KB 6.4 /
// 6.9, 88 7.0 / 7.1; 48 heads, d = 128, 72 KB 6.9 / 7.8, 88 7.7 / 7.9, 104 8.3 / 7.8; d = 64, 88 KB 7.6 / 8.0.
static bool decode_one_workgroup(int BH, size_t key_bytes, bool f32) {
    const int least = f32 ? 88 : 64, kb = BH + (f32 ? 48 : 24);
    return key_bytes <= (size_t)(kb < least ? least : kb > 128 ? 128 : kb) * 1024;
}

template <typename TIO, int D, bool GATES>
static hipError_t launch_decode_g(const DecodeArgs& a, int BH, hipStream_t st) {
    if (decode_one_workgroup(BH, (size_t)a.n * D * sizeof(TIO), sizeof(TIO) == 4)) {
        if (a.n <= 128) hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 256, DECODE_DIRECT>), dim3(1, BH), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 1024, DECODE_DIRECT>), dim3(1, BH), dim3(1024), 0, st, a);
        return hipGetLastError();
    }
    static_assert(DECODE_MAX_SPLITS * (D / 64) * sizeof(DecodeRecord) <= DECODE_SPLIT_ROOM * (D + 2) * 4, "the workspace holds the records");
    const DecodeSplits s = decode_splits(BH, a.n, (size_t)a.n * D * sizeof(TIO));
    if (s.merged && a.flag != 0) {
        if (s.waves == 4) hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 256, DECODE_MERGED>), dim3(s.n, BH), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 512, DECODE_MERGED>), dim3(s.n, BH), dim3(512), 0, st, a);
        return hipGetLastError();
    }
    if (s.waves == 4) hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 256, DECODE_RECORDS>), dim3(s.n, BH), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((decode_partial_kernel<TIO, D, GATES, 512, DECODE_RECORDS>), dim3(s.n, BH), dim3(512), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_merge_kernel<TIO, D, GATES>), dim3(BH), dim3(D), 0, st, a, s.n);
    return hipGetLastError();
}
template <typename TIO, int D>
static hipError_t launch_decode_t(const DecodeArgs& a, int BH, hipStream_t st) {
    return a.ccache ? launch_decode_g<TIO, D, true>(a, BH, st) : launch_decode_g<TIO, D, false>(a, BH, st);
}
hipError_t launch_decode_step(DecodeArgs a, int BH, int d, int is_bf16, hipStream_t st) {
    static std::atomic<unsigned long long> calls{0};
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(st, &cs) == hipSuccess;
    if (!known) (void)hipGetLastError();              // (the null stream while another one is captured; the launch says whether that is allowed)
    a.flag = !known || cs != hipStreamCaptureStatusNone ? 0 : (calls.fetch_add(1, std::memory_order_relaxed) + 1) * 0x9e3779b97f4a7c15ull;      // (odd factor: 2^64 calls before one recurs; never 0 before)
    if (is_bf16) return d == 64 ? launch_decode_t<bf16_t, 64>(a, BH, st) : launch_decode_t<bf16_t, 128>(a, BH, st);
    return d == 64 ? launch_decode_t<float, 64>(a, BH, st) : launch_decode_t<float, 128>(a, BH, st);
}

}  // namespace path
