// Chunk preprocessing of PaTH attention (paper Sec. 3.2: UT transform of a
// chunk, boundary-adjusted queries and keys, chunk transition product).
//
// One workgroup (4 waves) per (batch*head, chunk of 64 tokens).  With
// Q, K, W the chunk's rows and beta its transition strengths:
//
//   G   = W W^T                       A = I + strictLower(diag(beta) G)
//   N   = A^{-1} diag(beta)           (the chunk's "T^{-1}", Sec. 3 UT paragraph)
//   U   = N W                         dP = W^T U   (chunk product P = I - dP)
//   F   = tril(Q W^T)                 Y  = N strictLower(W K^T)
//   Qb  = Q - F U                     Kb = K - Y^T W            (Sec. 3.2 matrix forms)
//   Sd  = Q K^T - F Y                 (diagonal block logits, Sec. 3.2 case i = j)
//
// The triangular system is solved by forward substitution in fp32 (never
// through 1/beta, so beta = 0 is regular); everything else is MFMA.
// This file: fp32 operands (16-bit operands: prep16_fwd.hip).
// Outputs go to the workspace in the layouts the sweep kernel consumes
// without any shuffling: K-tile, V^T-tile and -dP-tile in fragment order,
// Qb and Sd in accumulator order (fp32).  Rows past L are treated as
// beta = 0, w = k = q = v = 0.
#include "path_common.h"

namespace path {

template <int D> struct PrepCfg {
    typedef float T;
    static constexpr int FE = Tr<T>::FE;
    static constexpr int KW = Tr<T>::KW;
    static constexpr int LDD = D + FE;                 // padded length-D rows
    static constexpr int LDC = CHUNK + FE;             // padded length-64 rows
    static constexpr int LDA = CHUNK + 4;              // solve matrix
    static constexpr int LDH = 32 + 4;                 // 32x32 helpers of the blocked inverse
    // Q and K are not staged: their operand fragments come straight from global memory (the chunk's rows are
    // read a few times, out of L2).  One workgroup per CU.
    static constexpr int WSUT = (CHUNK * LDD > D * LDC) ? CHUNK * LDD : D * LDC;   // U^T re-uses W's rows
    // element offsets -- every block is a multiple of 16 bytes
    static constexpr size_t off_ws = 0;                               // W rows, later U^T
    static constexpr size_t off_wt = off_ws + WSUT;                   // W^T
    static constexpr size_t off_f = off_wt + (size_t)D * LDC;         // F
    static constexpr size_t off_gk = off_f + (size_t)CHUNK * LDC;     // (strictLower(W K^T))^T
    static constexpr size_t off_yt = off_gk + (size_t)CHUNK * LDC;    // Y^T
    static constexpr size_t off_af = off_yt + (size_t)CHUNK * LDC;    // A / solve
    static constexpr size_t off_beta = off_af + (size_t)CHUNK * LDA;
    static constexpr size_t off_xf = off_beta + CHUNK;                // A^{-1}, overwritten by N (same shape)
    static constexpr size_t smem_bytes = (off_xf + (size_t)CHUNK * LDA) * 4;
    // the two 32x32 helpers, (A^{-1})_11^T and (A_21 (A^{-1})_11)^T, lie in Y^T's space (Y^T is written only after the inverse is done)
    static constexpr size_t off_xt1 = off_yt, off_tt = off_xt1 + (size_t)32 * LDH;
    static_assert(2 * 32 * LDH <= CHUNK * LDC, "helpers must fit in Y^T");
    static_assert(LDC == LDA, "in-place N needs equal row pitch");
};

// BWD: also write the backward-only outputs (all of them; their pointers are set).  A compile-time
// switch, so that the forward's instantiation carries none of that code.
template <int D, bool BWD, bool STRIDED>
__global__ __launch_bounds__(256, 1) void prep_fwd_kernel(FwdParams p) {
    using C = PrepCfg<D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using Vec4 = typename Tr<T>::Vec4;
    constexpr int FE = C::FE, KW = C::KW, LDD = C::LDD, LDC = C::LDC, LDA = C::LDA;
    constexpr int SPB = 32 / KW;   // slabs per 32-index block

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T* sT = reinterpret_cast<T*>(smem);
    T* Ws = sT + C::off_ws;
    // W^T is written out, element by element, while the chunk is staged, and U^T re-uses W's rows once phase 1 is over.
    T* Wt = sT + C::off_wt;
    T* Ut = Ws;
    T* Fs = sT + C::off_f;
    T* Gk = sT + C::off_gk;
    T* Yt = sT + C::off_yt;
    float* Af = sT + C::off_af;
    float* bs = sT + C::off_beta;
    float* Xf = sT + C::off_xf;
    T* Nt = Xf;
    float* XT1 = sT + C::off_xt1;
    float* TT = sT + C::off_tt;
    constexpr int LDH = C::LDH;

    int chunk, bh;
    chunk_and_head(p.ul, p.NC, p.B * p.H, chunk, bh);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, h = lane >> 5, l32 = lane & 31;
    const int L = seq_len(p.ul, bh, p.L), NC = p.NC;      // this head's own length; NC: chunks per head in the workspace arrays
    const int t0 = chunk * CHUNK;
    if (t0 >= L) return;                                   // (packed batch: a shorter sequence has fewer chunks)
    const int nvalid = (L - t0 < CHUNK) ? (L - t0) : CHUNK;
    const long long rowbase = user_vec(p.ul, bh, t0);       // the caller's layout: token stride TS between rows
    // token stride of the caller's tensors; a compile-time constant unless the layout interleaves heads
    // (then every row address costs vector arithmetic instead of an immediate offset)
    const int TS = STRIDED ? (int)p.ul.vt : D;
    const T* Qg = reinterpret_cast<const T*>(p.q) + rowbase;
    const T* Kg = reinterpret_cast<const T*>(p.k) + rowbase;
    const T* Vg = reinterpret_cast<const T*>(p.v) + rowbase;
    const T* Wg = reinterpret_cast<const T*>(p.w) + rowbase;
    const T* Bg = reinterpret_cast<const T*>(p.beta) + user_scl(p.ul, bh, t0);

    // V is only re-arranged (tiles V^T and, for the backward, V): the wave's elements of both, fetched at the
    // start and held in registers until the output phase.
    constexpr int NBV = (D / 32) * 2 / 4;           // 32x32 blocks of a 64 x d tile per wave
    T vt_r[NBV][16];                              // V^T blocks: registers rows s, lane c
    Vec4 vk_r[BWD ? NBV : 1][4];                  // V blocks: registers rows c (4 consecutive per load), lane s
    auto load_v = [&]() {
#pragma unroll
        for (int i = 0; i < NBV; ++i) {
            const int blk = wv + 4 * i;
            const int cb = blk >> 1, sb = blk & 1;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int s = 32 * sb + acc_row(j, h);
                vt_r[i][j] = (s < nvalid) ? Vg[s * TS + 32 * cb + l32] : (T)0.f;
            }
            if (BWD && p.ktT) {
                const int s = 32 * sb + l32;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) vk_r[i][g][r] = (T)0.f;
                    if (s < nvalid) vk_r[i][g] = *reinterpret_cast<const Vec4*>(Vg + s * TS + 32 * cb + 8 * g + 4 * h);
                }
            }
        }
    };

    // ---- phase 0: stage the chunk (zero rows past L) ---------------------------
    // All of a thread's loads are issued before the first conversion, so their latencies overlap.
    {
        constexpr int NIT = CHUNK * (D / FE) / 256;
        Frag wr[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = tid + it * 256, row = idx / (D / FE), cf = idx % (D / FE);
            if (row < nvalid) wr[it] = ld_frag<T>(Wg + row * TS + cf * FE);
        }
        load_v();                     // needed only at the very end: in flight during everything in between
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = tid + it * 256, row = idx / (D / FE), cf = idx % (D / FE);
            Frag wv_ = Tr<T>::zero();
            if (row < nvalid) wv_ = wr[it];
            *reinterpret_cast<Frag*>(Ws + row * LDD + cf * FE) = wv_;
#pragma unroll
            for (int e = 0; e < FE; ++e) Wt[(cf * FE + e) * LDC + row] = wv_[e];
        }
    }
    if (tid < CHUNK) bs[tid] = (tid < nvalid) ? (float)Bg[tid * (int)p.ul.st] : 0.f;
    __syncthreads();

    // Q and K are read from global memory.  Rows past L must not be touched: those lanes are redirected to
    // row 0 and their products masked out by the zero W / the explicit masks below.

    const int bi = wv >> 1, bj = wv & 1;   // this wave's 32x32 block of a 64x64 result
    const size_t bhc = (size_t)bh * NC + chunk;

    // Row of Q/K this lane supplies as an operand row (clamped for the global path).
    auto qk_row = [&](int r) { return r < nvalid ? r : 0; };
    auto qk_ok = [&](int r) { return r < nvalid; };
    // operand fragment of row r of Q or K: the FE elements from column k on
    auto qk_frag = [&](const T* base, int r, int k) { return ld_frag<T>(base + (size_t)qk_row(r) * TS + k); };
    // F block: rows t (Q), cols t' (W); keep t' <= t.
    auto f_block = [&]() {
        const int ar = 32 * (wv >> 1) + l32, bjj = wv & 1;
        f32x16 acc = zero16();
        const T* bp = Ws + (size_t)(32 * bjj + l32) * LDD + FE * h;
#pragma unroll
        for (int k0 = 0; k0 < D; k0 += KW) acc = Tr<T>::mma(qk_frag(Qg, ar, k0 + FE * h), ld_frag<T>(bp + k0), acc);
        const int tp = 32 * bjj + l32;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int t = 32 * (wv >> 1) + acc_row(j, h);
            Fs[t * LDC + tp] = (tp <= t && t < nvalid) ? (T)acc[j] : (T)0.f;
        }
    };

    // (W^T block cb) x (rows xr0.. of X)^T and (rows xr0.. of X) x (W^T block cb)^T, contraction over the chunk's tokens
    auto wt_times = [&](int cb, const T* X, int xr0) { return gemm32<T, CHUNK>(Wt, LDC, 32 * cb, X, LDC, xr0, l32, h, zero16()); };
    auto times_wt = [&](const T* X, int xr0, int cb) { return gemm32<T, CHUNK>(X, LDC, xr0, Wt, LDC, 32 * cb, l32, h, zero16()); };

    // ---- phase 1: products of the inputs ----------------------------------------
    // G block -> Af[t][s] = beta_t G[t][s] for s < t, else 0.
    {
        f32x16 acc = gemm32<T, D>(Ws, LDD, 32 * bi, Ws, LDD, 32 * bj, l32, h, zero16());
        const int s = 32 * bj + l32;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int t = 32 * bi + acc_row(j, h);
            Af[t * LDA + s] = (s < t) ? bs[t] * acc[j] : 0.f;
            if (BWD && p.gm) p.gm[bhc * 4096 + t * 64 + s] = acc[j];
        }
    }
    f_block();
    // Gk block: rows t' (W), cols s (K); stored transposed Gk[s][t'], keep t' > s.
    {
        f32x16 acc = zero16();
        {
            const T* ap = Ws + (size_t)(32 * bi + l32) * LDD + FE * h;
#pragma unroll
            for (int k0 = 0; k0 < D; k0 += KW) acc = Tr<T>::mma(ld_frag<T>(ap + k0), qk_frag(Kg, 32 * bj + l32, k0 + FE * h), acc);
        }
        const int s = 32 * bj + l32;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            Vec4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int tp = 32 * bi + 8 * g + 4 * h + r;
                v4[r] = (tp > s && qk_ok(s)) ? (T)acc[4 * g + r] : (T)0.f;
            }
            *reinterpret_cast<Vec4*>(Gk + s * LDC + 32 * bi + 8 * g + 4 * h) = v4;
        }
    }
    // K Q^T block (rows s = keys, cols t = queries): first term of Sd^T, kept in registers.
    f32x16 accS = zero16();
    {
#pragma unroll
        for (int k0 = 0; k0 < D; k0 += KW) accS = Tr<T>::mma(qk_frag(Kg, 32 * bi + l32, k0 + FE * h), qk_frag(Qg, 32 * bj + l32, k0 + FE * h), accS);
    }
    __syncthreads();

    // ---- phase 2: X = A^{-1} (A unit lower triangular), then N = X diag(beta) --------------
    // Blocked: the two 32x32 diagonal blocks by forward substitution (waves 0 and 1, one
    // lane per column -- a column of the inverse depends only on itself), the off-diagonal
    // block X_21 = -X_22 (A_21 X_11) by two fp32 MFMA products.
    if (wv < 2) {
        if (lane < 32) {
            const int c = lane, r0 = wv ? 32 * LDA + 32 : 0;       // the wave's diagonal block
            float n[32];
#pragma unroll
            for (int t = 0; t < 32; ++t) n[t] = 0.f;
#pragma unroll
            for (int t = 0; t < 32; ++t) {
                float a0 = (t == c) ? 1.f : 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
                for (int s4 = 0; s4 < (t + 3) / 4; ++s4) {
                    const f32x4 a4 = *reinterpret_cast<const f32x4*>(Af + r0 + t * LDA + 4 * s4);   // zeros for s >= t
                    a0 -= a4[0] * n[4 * s4 + 0];
                    a1 -= a4[1] * n[4 * s4 + 1];
                    a2 -= a4[2] * n[4 * s4 + 2];
                    a3 -= a4[3] * n[4 * s4 + 3];
                }
                const float acc = (a0 + a1) + (a2 + a3);
                n[t] = acc;
                Xf[r0 + t * LDA + c] = acc;
                if (wv == 0) XT1[c * LDH + t] = acc;
            }
        }
    } else if (wv == 2) {
        for (int idx = lane; idx < 32 * 32; idx += 64) Xf[(idx >> 5) * LDA + 32 + (idx & 31)] = 0.f;   // upper-right block
    }
    __syncthreads();
    if (wv == 0) {      // T = A_21 X_11, stored transposed
        f32x16 acc = gemm32<float, 32>(Af + 32 * LDA, LDA, 0, XT1, LDH, 0, l32, h, zero16());
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = acc[4 * g + r];
            *reinterpret_cast<f32x4*>(TT + l32 * LDH + 8 * g + 4 * h) = v4;
        }
    }
    __syncthreads();
    if (wv == 0) {      // X_21 = -X_22 T
        f32x16 acc = gemm32<float, 32>(Xf + 32 * LDA + 32, LDA, 0, TT, LDH, 0, l32, h, zero16());
#pragma unroll
        for (int j = 0; j < 16; ++j) Xf[32 * LDA + acc_row(j, h) * LDA + l32] = -acc[j];
    }
    __syncthreads();
    {
        constexpr int NX = CHUNK * CHUNK / 256;
        float x[NX];
        const int c = tid & 63;
#pragma unroll
        for (int it = 0; it < NX; ++it) {
            const int t = (tid >> 6) + 4 * it;
            x[it] = Xf[t * LDA + c];
        }
#pragma unroll
        for (int it = 0; it < NX; ++it) {
            const int t = (tid >> 6) + 4 * it;
            Nt[t * LDC + c] = (T)(x[it] * bs[c]);
            if (BWD && p.aim) reinterpret_cast<T*>(p.aim)[bhc * 4096 + t * 64 + c] = (T)x[it];
        }
    }
    __syncthreads();

    // ---- phase 3: U^T = W^T N^T  and  Y^T -----------------------------------------
    // Y block: rows t (N), cols s (Gk rows); stored transposed Yt[s][t].
    {
        f32x16 acc = gemm32<T, CHUNK>(Nt, LDC, 32 * bi, Gk, LDC, 32 * bj, l32, h, zero16());
        const int s = 32 * bj + l32;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            Vec4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = (T)acc[4 * g + r];
            *reinterpret_cast<Vec4*>(Yt + s * LDC + 32 * bi + 8 * g + 4 * h) = v4;
        }
    }
    // U^T blocks: rows c (W^T), cols t (N rows).  (Ut aliases Ws, all reads of Ws are done.)
    {
        f32x16 accU[D / 64];
#pragma unroll
        for (int i = 0; i < D / 64; ++i) {
            const int blk = wv + 4 * i;                 // (D/32)*2 blocks over 4 waves
            const int cb = blk >> 1, tb = blk & 1;
            accU[i] = wt_times(cb, Nt, 32 * tb);
        }
        __syncthreads();                                 // nobody still reads Ws (phase 1) -- and keeps phases apart
#pragma unroll
        for (int i = 0; i < D / 64; ++i) {
            const int blk = wv + 4 * i;
            const int cb = blk >> 1, tb = blk & 1;
#pragma unroll
            for (int j = 0; j < 16; ++j) Ut[(32 * cb + acc_row(j, h)) * LDC + 32 * tb + l32] = (T)accU[i][j];
        }
    }
    __syncthreads();

    // ---- phase 4: outputs -----------------------------------------------------------
    // 16 bytes per lane (the LDS rows are 16-byte aligned: LDC * sizeof(T) is a multiple of 16)
    typedef T RowVec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int VE = 16 / (int)sizeof(T), VPR = 64 / VE;
    static_assert((LDC * sizeof(T)) % 16 == 0, "aligned rows");
    if (BWD && p.fm) {
        T* gk = reinterpret_cast<T*>(p.gktm) + bhc * 4096;
        for (int idx = tid; idx < 64 * VPR; idx += 256) {
            const int r = idx / VPR, c = (idx % VPR) * VE;
            __builtin_nontemporal_store(*reinterpret_cast<const RowVec*>(Gk + r * LDC + c), reinterpret_cast<RowVec*>(gk + r * 64 + c));
        }
    }
    if (BWD && p.fm) {   // backward: keep the chunk's matrices (row-major, operand type)
        T* fm = reinterpret_cast<T*>(p.fm) + bhc * 4096;
        T* nm = reinterpret_cast<T*>(p.nm) + bhc * 4096;
        T* yt = reinterpret_cast<T*>(p.ytm) + bhc * 4096;
        T* ut = reinterpret_cast<T*>(p.utm) + bhc * (size_t)D * 64;
        for (int idx = tid; idx < 64 * VPR; idx += 256) {
            const int r = idx / VPR, c = (idx % VPR) * VE;
            __builtin_nontemporal_store(*reinterpret_cast<const RowVec*>(Fs + r * LDC + c), reinterpret_cast<RowVec*>(fm + r * 64 + c));
            __builtin_nontemporal_store(*reinterpret_cast<const RowVec*>(Nt + r * LDC + c), reinterpret_cast<RowVec*>(nm + r * 64 + c));
            __builtin_nontemporal_store(*reinterpret_cast<const RowVec*>(Yt + r * LDC + c), reinterpret_cast<RowVec*>(yt + r * 64 + c));
        }
        for (int idx = tid; idx < D * VPR; idx += 256) {
            const int r = idx / VPR, c = (idx % VPR) * VE;
            __builtin_nontemporal_store(*reinterpret_cast<const RowVec*>(Ut + r * LDC + c), reinterpret_cast<RowVec*>(ut + r * 64 + c));
        }
    }
    // (a) Sd^T = K Q^T - Y^T F^T, accumulator order: [bhc][qb][kb][g][lane][4]
    {
        f32x16 corr = gemm32<T, CHUNK>(Yt, LDC, 32 * bi, Fs, LDC, 32 * bj, l32, h, zero16());
        float* dst = p.sd + (bhc * 4 + (size_t)(bj * 2 + bi)) * 1024;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = accS[4 * g + r] - corr[4 * g + r];
            __builtin_nontemporal_store(v4, reinterpret_cast<f32x4*>(dst + (g * 64 + lane) * 4));
            if (BWD && p.sdm) *reinterpret_cast<f32x4*>(p.sdm + bhc * 4096 + (32 * bj + l32) * 64 + 32 * bi + 8 * g + 4 * h) = v4;
        }
    }
    // (b) -dP tile (rows = output column b of dP, contraction = a): acc rows a, cols b.
    {
        Frag* dst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.dp) + bhc * (size_t)D * D);
        constexpr int NB = (D / 32) * (D / 32);
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
            const int blk = wv + 4 * i;
            const int ab = blk / (D / 32), bb = blk % (D / 32);
            f32x16 acc = wt_times(ab, Ut, 32 * bb);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = -acc[j];
            Frag fr[SPB];
            pack_block<T>(acc, fr);
#pragma unroll
            for (int s = 0; s < SPB; ++s) __builtin_nontemporal_store(fr[s], &dst[((size_t)bb * (D / KW) + ab * SPB + s) * 64 + tile_lane<T>(lane, s)]);
        }
    }
    // (c) Kb tile (rows = key s, contraction = c): acc rows c, cols s;  Kb^T = K^T - W^T Y.
    // (d) Qb in accumulator order (rows c, cols t): Qb^T = Q^T - U^T F^T.
    {
        Frag* kdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.kt) + bhc * (size_t)CHUNK * D);
        constexpr int NB = (D / 32) * 2;
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
            const int blk = wv + 4 * i;
            const int cb = blk >> 1, sb = blk & 1;
            f32x16 acc = wt_times(cb, Yt, 32 * sb);
            const int s = 32 * sb + l32;
            const T* krow = Kg + (size_t)qk_row(s) * TS + 32 * cb + 4 * h;
            const bool ok = qk_ok(s);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const Vec4 k4 = *reinterpret_cast<const Vec4*>(krow + 8 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[4 * g + r] = (ok ? (float)k4[r] : 0.f) - acc[4 * g + r];
            }
            Frag fr[SPB];
            pack_block<T>(acc, fr);
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &kdst[((size_t)sb * (D / KW) + cb * SPB + s2) * 64 + tile_lane<T>(lane, s2)]);
            if (BWD) {       // the same keys row-major [token][c]
                T* kb = reinterpret_cast<T*>(p.kbm) + (bhc * CHUNK + s) * (size_t)D + 32 * cb + 4 * h;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    Vec4 o4;
#pragma unroll
                    for (int r = 0; r < 4; ++r) o4[r] = (T)acc[4 * g + r];
                    *reinterpret_cast<Vec4*>(kb + 8 * g) = o4;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
            const int blk = wv + 4 * i;
            const int cb = blk >> 1, tb = blk & 1;
            f32x16 acc = gemm32<T, CHUNK>(Ut, LDC, 32 * cb, Fs, LDC, 32 * tb, l32, h, zero16());
            const int t = 32 * tb + l32;
            const T* qrow = Qg + (size_t)qk_row(t) * TS + 32 * cb + 4 * h;
            const bool ok = qk_ok(t);
            // xinit: [bh][query block of 32][d block][g][lane][4]
            float* xdst = p.xinit + ((((size_t)bh * NC + chunk) * 2 + tb) * (D / 32) + cb) * 1024;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const Vec4 q4 = *reinterpret_cast<const Vec4*>(qrow + 8 * g);
                f32x4 v4;
#pragma unroll
                for (int r = 0; r < 4; ++r) v4[r] = (ok ? (float)q4[r] : 0.f) - acc[4 * g + r];
                __builtin_nontemporal_store(v4, reinterpret_cast<f32x4*>(xdst + (g * 64 + lane) * 4));
            }
        }
        // (e) V^T tile (rows = c, contraction = key s): plain re-layout of V.
        Frag* vdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.vt) + bhc * (size_t)CHUNK * D);
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) {
            const int blk = wv + 4 * i;
            const int cb = blk >> 1, sb = blk & 1;
            f32x16 acc;
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = (float)vt_r[i][j];
            Frag fr[SPB];
            pack_block<T>(acc, fr);
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &vdst[(((size_t)sb * (D / 32) + cb) * SPB + s2) * 64 + lane]);   // [key half][d block][slab]
        }
        if (BWD && p.dpt) {
            // -dP in the transposed arrangement (rows c, contraction b) = -dP[c][b]: accumulate with rows b,
            // lane c.  Read by the backward's adjoint scan.
            Frag* pdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.dpt) + bhc * (size_t)D * D);
            constexpr int NBP = (D / 32) * (D / 32);
#pragma unroll
            for (int i = 0; i < NBP / 4; ++i) {
                const int blk = wv + 4 * i;
                const int bb = blk / (D / 32), cb = blk % (D / 32);
                f32x16 acc = times_wt(Ut, 32 * bb, cb);
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[j] = -acc[j];
                Frag fr[SPB];
                pack_block<T>(acc, fr);
#pragma unroll
                for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &pdst[((size_t)cb * (D / KW) + bb * SPB + s2) * 64 + lane]);
            }
        }
        if (BWD && p.ktT) {
            // ---- backward-only tiles ------------------------------------------------------------
            constexpr int QS = CHUNK / KW;
            // ktT (rows c, contraction s) = Kb[s][c]: accumulate with rows s, lane c.
            Frag* tdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.ktT) + bhc * (size_t)CHUNK * D);
#pragma unroll
            for (int i = 0; i < NB / 4; ++i) {
                const int blk = wv + 4 * i;
                const int cb = blk >> 1, sb = blk & 1;
                f32x16 acc = times_wt(Yt, 32 * sb, cb);
                const int c = 32 * cb + l32;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int s = 32 * sb + acc_row(j, h);
                    const float kv = qk_ok(s) ? (float)Kg[(size_t)qk_row(s) * TS + c] : 0.f;
                    acc[j] = kv - acc[j];
                }
                Frag fr[SPB];
                pack_block<T>(acc, fr);
#pragma unroll
                for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &tdst[((size_t)cb * QS + sb * SPB + s2) * 64 + lane]);
            }
            // vk (rows s, contraction c) = V[s][c] (I/O type): registers rows c, lane s
            Frag* vkd = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.vk) + bhc * (size_t)CHUNK * D);
#pragma unroll
            for (int i = 0; i < NB / 4; ++i) {
                const int blk = wv + 4 * i;
                const int cb = blk >> 1, sb = blk & 1;
                f32x16 acc;
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[j] = (float)vk_r[i][j >> 2][j & 3];
                Frag fr[SPB];
                pack_block<T>(acc, fr);
#pragma unroll
                for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &vkd[((size_t)sb * (D / KW) + cb * SPB + s2) * 64 + lane]);
            }
        }
    }
}

template <int D, bool BWD, bool STRIDED>
hipError_t launch_prep_fwd_s(const FwdParams& p, hipStream_t stream) {
    using C = PrepCfg<D>;
    // set once per process; a function-local static is initialised under the language's own lock
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&prep_fwd_kernel<D, BWD, STRIDED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::smem_bytes);
    if (attr_err != hipSuccess) return attr_err;
    dim3 grid((unsigned)(p.NC * p.B * p.H));
    hipLaunchKernelGGL((prep_fwd_kernel<D, BWD, STRIDED>), grid, dim3(256), C::smem_bytes, stream, p);
    return hipGetLastError();
}
template <int D, bool BWD>
hipError_t launch_prep_fwd_b(const FwdParams& p, hipStream_t stream) {
    return p.ul.vt != D ? launch_prep_fwd_s<D, BWD, true>(p, stream) : launch_prep_fwd_s<D, BWD, false>(p, stream);
}
template <int D>
hipError_t launch_prep_fwd_t(const FwdParams& p, hipStream_t stream) {
    return p.fm ? launch_prep_fwd_b<D, true>(p, stream) : launch_prep_fwd_b<D, false>(p, stream);
}

hipError_t launch_prep16_fwd(const FwdParams& p, int d, hipStream_t stream);      // 16-bit operands
hipError_t launch_prep_fwd(const FwdParams& p, int d, int is_bf16, hipStream_t stream) {
    if (is_bf16) return launch_prep16_fwd(p, d, stream);
    return d == 64 ? launch_prep_fwd_t<64>(p, stream) : launch_prep_fwd_t<128>(p, stream);
}

}  // namespace path
