// Chunk preprocessing (see prep_fwd.hip for the quantities and their layouts) for 16-bit operands.
//
// One workgroup of four waves per (chunk, head).  Q, K, V, W are fetched whole rows at a time and staged; everything the
// later phases need of Q, K and V is taken out of LDS before the fp32 matrices of the inverse come to lie in their place:
//
//   0  W (converted), Q, K, V -> LDS
//   1  the lower 32x32 blocks of F^T, S = K Q^T and Gk by three waves, which share their operand fragments, those of
//      G by the fourth; V^T (and V) tiles out; the wave's pieces of Q and K for the outputs -> registers
//   2  A, Gk -> LDS;  A^-1;  N
//   3  Y^T, U^T
//   4  outputs: a wave takes one 32-column block of W^T for all its products with it
//
// Blocks that the triangular shapes make zero are neither multiplied nor, in the diagonal logits, stored: both readers mask them.
//
// What bounds it: memory, where there are several workgroups per CU (512 heads of 1024 tokens, d = 128: 1.4 GB in 286 us = 4.9 TB/s,
// what a plain copy of such blocks reaches; d = 64 153 us), the chain of its phases where there are few (16 heads of 1000 tokens
// 14.3 us, launch after launch; d = 64 10.8.  A single launch among others takes 17 to 18).  With operand fragments of Q and K read from global memory by each wave that needs them -- 32 rows per
// request -- and V element by element, 426, 195, 18.6 and 14.0 us: requests, not bytes, were what it waited for.
#include "path_common.h"

namespace path {

template <typename TIO, int D> struct Prep16Cfg {
    typedef typename Compute<TIO>::type T;
    static_assert(sizeof(TIO) == 2 && sizeof(T) == 2, "16-bit operands");
    static constexpr int LDD = D + 8, LDC = CHUNK + 8, LDH = 36;      // pitches: length-D rows, length-64 rows, fp32 32x32 blocks
    static constexpr int BLK = 32 * LDH;                              // one such block (floats)
    // bytes.  W | U^T, Y^T, N -- before them Q and K, then the three blocks each of A and its inverse | Gk, before it V | F (d = 128;
    // at d = 64, where three workgroups share a CU, F passes through registers to Gk's place) | helper of the inverse | beta
    static constexpr bool OWN_F = D == 128;
    static constexpr int W_ = 0, UT = W_ + CHUNK * LDD * 2, YT = UT + D * LDC * 2, NT = YT + CHUNK * LDC * 2, GK = NT + CHUNK * LDC * 2;
    static constexpr int FS = OWN_F ? GK + CHUNK * LDC * 2 : GK, HELP = FS + CHUNK * LDC * 2, BETA = HELP + BLK * 4, TOTAL = BETA + CHUNK * 4;
    static constexpr int KR = UT, QR = KR + CHUNK * LDD * 2, VR = GK, AF = UT, XF = AF + 3 * BLK * 4;
    static constexpr int WGS_PER_CU = D == 64 ? 3 : 2;
    static_assert(QR + CHUNK * LDD * 2 <= GK && XF + 3 * BLK * 4 <= GK && VR + CHUNK * LDD * 2 <= BETA, "what lies in turn in one place fits");
    static_assert(WGS_PER_CU * TOTAL <= 160 * 1024, "LDS budget");
};

template <typename TIO, int D, bool BWD, bool STRIDED>
__global__ __launch_bounds__(256, (Prep16Cfg<TIO, D>::WGS_PER_CU)) void prep16_fwd_kernel(FwdParams p) {
    using C = Prep16Cfg<TIO, D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using FragV = typename Tr<TIO>::Frag;
    using Vec4 = typename Tr<T>::Vec4;
    typedef typename Tr<TIO>::Vec4 VecIO4;
    constexpr int LDD = C::LDD, LDC = C::LDC, LDH = C::LDH, BLK = C::BLK, DB = D / 32, DS = D / 16;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *Ws = reinterpret_cast<T*>(smem + C::W_), *Ut = reinterpret_cast<T*>(smem + C::UT), *Yt = reinterpret_cast<T*>(smem + C::YT);
    T *Nt = reinterpret_cast<T*>(smem + C::NT), *Gk = reinterpret_cast<T*>(smem + C::GK), *Fs = reinterpret_cast<T*>(smem + C::FS);
    TIO *Kr = reinterpret_cast<TIO*>(smem + C::KR), *Qr = reinterpret_cast<TIO*>(smem + C::QR), *Vr = reinterpret_cast<TIO*>(smem + C::VR);
    // A and A^-1: 32x32 blocks (0,0), (1,0), (1,1)
    float *Af = reinterpret_cast<float*>(smem + C::AF), *Xf = reinterpret_cast<float*>(smem + C::XF);
    float *help = reinterpret_cast<float*>(smem + C::HELP), *bs = reinterpret_cast<float*>(smem + C::BETA);

    int chunk, bh;
    chunk_and_head(p.ul, p.NC, p.B * p.H, chunk, bh);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int L = seq_len(p.ul, bh, p.L), NC = p.NC;      // this head's own length; NC: chunks per head in the workspace arrays
    const int t0 = chunk * CHUNK;
    if (t0 >= L) return;                                   // (packed batch: a shorter sequence has fewer chunks)
    const int nvalid = (L - t0 < CHUNK) ? (L - t0) : CHUNK;
    const long long rowbase = user_vec(p.ul, bh, t0);
    const int TS = STRIDED ? (int)p.ul.vt : D;             // token stride of the caller's tensors (a compile-time constant unless the layout interleaves heads)
    const size_t bhc = (size_t)bh * NC + chunk;

    // ---- phase 0: stage the chunk (zero rows past L), all loads ahead of the first store ------------------------
    {
        constexpr int NIT = CHUNK * D / 8 / 256;
        const TIO* src[4] = {reinterpret_cast<const TIO*>(p.w) + rowbase, reinterpret_cast<const TIO*>(p.k) + rowbase,
                             reinterpret_cast<const TIO*>(p.q) + rowbase, reinterpret_cast<const TIO*>(p.v) + rowbase};
        FragV r[4][NIT];
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int idx = tid + it * 256, row = idx / (D / 8), c = (idx % (D / 8)) * 8;
                r[x][it] = Tr<TIO>::zero();
                if (row < nvalid) r[x][it] = ld_frag<TIO>(src[x] + row * TS + c);
            }
        if (tid < CHUNK) bs[tid] = tid < nvalid ? (float)(reinterpret_cast<const TIO*>(p.beta) + user_scl(p.ul, bh, t0))[tid * (int)p.ul.st] : 0.f;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = tid + it * 256, row = idx / (D / 8), c = (idx % (D / 8)) * 8;
            *reinterpret_cast<Frag*>(Ws + row * LDD + c) = cvt_frag<T, TIO>(r[0][it]);
            *reinterpret_cast<FragV*>(Kr + row * LDD + c) = r[1][it];
            *reinterpret_cast<FragV*>(Qr + row * LDD + c) = r[2][it];
            *reinterpret_cast<FragV*>(Vr + row * LDD + c) = r[3][it];
        }
    }
    __syncthreads();

    // ---- phase 1 -------------------------------------------------------------------------------------------------
    // a wave's blocks of the [64][d] outputs: columns 32 cb .., rows 32 (sb0 + i) ..
    constexpr int NBV = DB / 2;
    const int cb = wv % DB, sb0 = D == 64 ? wv / DB : 0;
    VecIO4 kr[NBV][4], qr[NBV][4];
#pragma unroll
    for (int i = 0; i < NBV; ++i) {
        const int row = 32 * (sb0 + i) + l32, c = 32 * cb + 4 * h;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            kr[i][g] = *reinterpret_cast<const VecIO4*>(Kr + row * LDD + c + 8 * g);
            qr[i][g] = *reinterpret_cast<const VecIO4*>(Qr + row * LDD + c + 8 * g);
        }
    }
    // V^T tile (rows c, contraction = key) and, for the backward, V tile (rows s, contraction c)
    if (!BWD || p.vt) {
        FragV* vdst = reinterpret_cast<FragV*>(reinterpret_cast<TIO*>(p.vt) + bhc * (size_t)CHUNK * D);
#pragma unroll
        for (int i = 0; i < NBV; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int sb = sb0 + i;
                __builtin_nontemporal_store(ld_frag_tr_acc<TIO>(Vr, LDD, 32 * sb + 16 * s, 32 * cb, l32, h), &vdst[((size_t)(sb * DB + cb) * 2 + s) * 64 + lane]);      // [key half][d block][slab]
            }
    }
    if (BWD) {
        FragV* vkd = reinterpret_cast<FragV*>(reinterpret_cast<TIO*>(p.vk) + bhc * (size_t)CHUNK * D);
#pragma unroll
        for (int i = 0; i < NBV; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int sb = sb0 + i;
                const TIO* v = Vr + (32 * sb + l32) * LDD + 32 * cb + 16 * s + 4 * h;
                union { VecIO4 v4[2]; FragV f; } u;
                u.v4[0] = *reinterpret_cast<const VecIO4*>(v);
                u.v4[1] = *reinterpret_cast<const VecIO4*>(v + 8);
                __builtin_nontemporal_store(u.f, &vkd[((size_t)sb * DS + cb * 2 + s) * 64 + lane]);
            }
    }
    // Wave (x, y) = (wv / 2, wv % 2): block of queries x and keys y of F^T (rows t', lane t), S (rows s, lane t) and Gk (rows t', lane s).
    // Wave 1, whose blocks are zero, takes G (rows s, lane t): blocks (0,0), (1,0), (1,1) of A.
    const int x = wv >> 1, y = wv & 1;
    f32x16 a0 = zero16(), a1 = zero16(), a2 = zero16();
    if (wv != 1) {
        const TIO *qp = Qr + (32 * x + l32) * LDD + 8 * h, *kp = Kr + (32 * y + l32) * LDD + 8 * h;
        const T *wx = Ws + (32 * x + l32) * LDD + 8 * h, *wy = Ws + (32 * y + l32) * LDD + 8 * h;
#pragma unroll
        for (int k = 0; k < D; k += 16) {
            const Frag q = cvt_frag<T, TIO>(ld_frag<TIO>(qp + k)), kk = cvt_frag<T, TIO>(ld_frag<TIO>(kp + k));
            a0 = Tr<T>::mma(ld_frag<T>(wy + k), q, a0);
            a1 = Tr<T>::mma(kk, q, a1);
            a2 = Tr<T>::mma(ld_frag<T>(wx + k), kk, a2);
        }
    } else {
        const T *w0 = Ws + l32 * LDD + 8 * h, *w1 = w0 + 32 * LDD;
#pragma unroll
        for (int k = 0; k < D; k += 16) {
            const Frag f0 = ld_frag<T>(w0 + k), f1 = ld_frag<T>(w1 + k);
            a0 = Tr<T>::mma(f0, f0, a0);
            a1 = Tr<T>::mma(f0, f1, a1);
            a2 = Tr<T>::mma(f1, f1, a2);
        }
    }
    const f32x16 accS = a1;
    Vec4 fr[4];                                            // F[t = 32 x + l32][t' = 32 y + 8 g + 4 h + r]: zero right of the diagonal
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) fr[g][r] = wv != 1 && 32 * y + 8 * g + 4 * h + r <= 32 * x + l32 ? (T)a0[4 * g + r] : (T)0.f;
    auto store_f = [&]() {
#pragma unroll
        for (int g = 0; g < 4; ++g) *reinterpret_cast<Vec4*>(Fs + (32 * x + l32) * LDC + 32 * y + 8 * g + 4 * h) = fr[g];
    };
    __syncthreads();                                       // Q, K, V have been read

    // ---- phase 2: A, Gk;  X = A^-1 (A unit lower triangular), N = X diag(beta) -----------------------------------------
    if (wv == 1) {
        const float b0 = bs[l32], b1 = bs[32 + l32];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v0, v1, v2;                              // strictly lower part of diag(beta) G, rows t = l32
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool low = 8 * g + 4 * h + r < l32;
                v0[r] = low ? b0 * a0[4 * g + r] : 0.f;
                v1[r] = b1 * a1[4 * g + r];
                v2[r] = low ? b1 * a2[4 * g + r] : 0.f;
            }
            float* d = Af + l32 * LDH + 8 * g + 4 * h;
            *reinterpret_cast<f32x4*>(d) = v0;
            *reinterpret_cast<f32x4*>(d + BLK) = v1;
            *reinterpret_cast<f32x4*>(d + 2 * BLK) = v2;
        }
    }
    // Gk[s][t'], t' > s
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        Vec4 v4;
#pragma unroll
        for (int r = 0; r < 4; ++r) v4[r] = wv != 1 && 32 * x + 8 * g + 4 * h + r > 32 * y + l32 ? (T)a2[4 * g + r] : (T)0.f;
        *reinterpret_cast<Vec4*>(Gk + (32 * y + l32) * LDC + 32 * x + 8 * g + 4 * h) = v4;
    }
    if (C::OWN_F) store_f();
    __syncthreads();
    // Blocked: the two 32x32 diagonal blocks by forward substitution (waves 0 and 1, one lane per column -- a column of the
    // inverse depends only on itself), the off-diagonal block X_21 = -X_22 (A_21 X_11) by two fp32 MFMA products.
    if (wv < 2) {
        if (lane < 32) {
            const int c = lane, r0 = wv ? 2 * BLK : 0;     // the wave's diagonal block
            float n[32];
#pragma unroll
            for (int t = 0; t < 32; ++t) n[t] = 0.f;
#pragma unroll
            for (int t = 0; t < 32; ++t) {
                float s0 = (t == c) ? 1.f : 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
                for (int s4 = 0; s4 < (t + 3) / 4; ++s4) {
                    const f32x4 a4 = *reinterpret_cast<const f32x4*>(Af + r0 + t * LDH + 4 * s4);   // zeros for s >= t
                    s0 -= a4[0] * n[4 * s4 + 0];
                    s1 -= a4[1] * n[4 * s4 + 1];
                    s2 -= a4[2] * n[4 * s4 + 2];
                    s3 -= a4[3] * n[4 * s4 + 3];
                }
                const float acc = (s0 + s1) + (s2 + s3);
                n[t] = acc;
                Xf[r0 + t * LDH + c] = acc;
                if (wv == 0) help[c * LDH + t] = acc;
            }
        }
    }
    __syncthreads();
    if (wv == 0) {      // A_21 X_11, stored transposed in X_11^T's place, then X_21 = -X_22 (A_21 X_11): the wave's own
        f32x16 acc = gemm32<float, 32>(Af + BLK, LDH, 0, help, LDH, 0, l32, h, zero16());
#pragma unroll
        for (int g = 0; g < 4; ++g) *reinterpret_cast<f32x4*>(help + l32 * LDH + 8 * g + 4 * h) = f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        acc = gemm32<float, 32>(Xf + 2 * BLK, LDH, 0, help, LDH, 0, l32, h, zero16());
#pragma unroll
        for (int j = 0; j < 16; ++j) Xf[BLK + acc_row(j, h) * LDH + l32] = -acc[j];
    }
    __syncthreads();
    {
        f32x4 v[4];
        const int c = 4 * (tid & 15), c32 = c >> 5;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int t = (tid >> 4) + 16 * it, t32 = it >> 1;
            v[it] = t32 >= c32 ? *reinterpret_cast<const f32x4*>(Xf + (t32 + c32) * BLK + (t & 31) * LDH + (c & 31)) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (C::XF + 3 * BLK * 4 > C::NT) __syncthreads();  // (N takes the inverse's place)
        const f32x4 b = *reinterpret_cast<const f32x4*>(bs + c);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int t = (tid >> 4) + 16 * it;
            Vec4 x4;
#pragma unroll
            for (int r = 0; r < 4; ++r) x4[r] = (T)v[it][r];
            *reinterpret_cast<Vec4*>(Nt + t * LDC + c) = mul_once(v[it], b);
            if (BWD) __builtin_nontemporal_store(x4, reinterpret_cast<Vec4*>(reinterpret_cast<T*>(p.aim) + bhc * 4096 + t * 64 + c));
        }
    }
    __syncthreads();

    // ---- phase 3: Y^T and U^T = W^T N^T -----------------------------------------------------------------------------------
    {       // Y block: rows t (N), lane s (Gk rows)
        const f32x16 acc = gemm32<T, CHUNK>(Nt, LDC, 32 * x, Gk, LDC, 32 * y, l32, h, zero16());
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            Vec4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = (T)acc[4 * g + r];
            *reinterpret_cast<Vec4*>(Yt + (32 * y + l32) * LDC + 32 * x + 8 * g + 4 * h) = v4;
        }
    }
    Frag wt[4];                                            // W^T, rows 32 cb .., contraction over the tokens
#pragma unroll
    for (int s = 0; s < 4; ++s) wt[s] = ld_frag_tr<T>(Ws, LDD, 16 * s, 32 * cb, l32, h);
#pragma unroll
    for (int i = 0; i < NBV; ++i) {                        // U blocks: rows t (N), lane c
        const int tb = sb0 + i;
        f32x16 acc = zero16();
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (s < 2 * (tb + 1)) acc = Tr<T>::mma(ld_frag<T>(Nt + (32 * tb + l32) * LDC + 16 * s + 8 * h), wt[s], acc);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            Vec4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = (T)acc[4 * g + r];
            *reinterpret_cast<Vec4*>(Ut + (32 * cb + l32) * LDC + 32 * tb + 8 * g + 4 * h) = v4;
        }
    }
    // backward: the chunk's matrices, row-major
    auto keep = [&](void* dst, const T* src, int rows) {
        T* d = reinterpret_cast<T*>(dst) + bhc * (size_t)rows * 64;
        for (int idx = tid; idx < rows * 8; idx += 256) {
            const int r = idx >> 3, c = (idx & 7) * 8;
            __builtin_nontemporal_store(ld_frag<T>(src + r * LDC + c), reinterpret_cast<Frag*>(d + r * 64 + c));
        }
    };
    if (BWD) {
        keep(p.gktm, Gk, 64);
        keep(p.nm, Nt, 64);
    }
    if (!C::OWN_F) {
        __syncthreads();
        store_f();
    }
    __syncthreads();

    // ---- phase 4: outputs -----------------------------------------------------------------------------------------------
    // K tile (rows = key s, contraction = c): Kb^T = K^T - W^T Y
    {
        Frag* kdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.kt) + bhc * (size_t)CHUNK * D);
#pragma unroll
        for (int i = 0; i < NBV; ++i) {
            const int sb = sb0 + i;
            f32x16 acc = zero16();
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s >= 2 * sb) acc = Tr<T>::mma(wt[s], ld_frag<T>(Yt + (32 * sb + l32) * LDC + 16 * s + 8 * h), acc);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = (float)kr[i][j >> 2][j & 3] - acc[j];
            Frag f[2];
            pack_block<T>(acc, f);
#pragma unroll
            for (int s = 0; s < 2; ++s) __builtin_nontemporal_store(f[s], &kdst[((size_t)sb * DS + cb * 2 + s) * 64 + tile_lane<T>(lane, s)]);
        }
    }
    // -dP tile (rows = output column b of dP, contraction = a): acc rows a, lane b
    {
        Frag* dst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.dp) + bhc * (size_t)D * D);
#pragma unroll
        for (int i = 0; i < DB * DB / 4; ++i) {
            const int bb = D == 64 ? wv / DB : i;
            f32x16 acc = zero16();
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(wt[s], ld_frag<T>(Ut + (32 * bb + l32) * LDC + 16 * s + 8 * h), acc);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = -acc[j];
            Frag f[2];
            pack_block<T>(acc, f);
#pragma unroll
            for (int s = 0; s < 2; ++s) __builtin_nontemporal_store(f[s], &dst[((size_t)bb * DS + cb * 2 + s) * 64 + tile_lane<T>(lane, s)]);
        }
    }
    // Qb in accumulator order (rows c, lane t): Qb^T = Q^T - U^T F^T.  xinit: [bh][query block of 32][d block][g][lane][4]
    {
        Frag uf[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) uf[s] = ld_frag<T>(Ut + (32 * cb + l32) * LDC + 16 * s + 8 * h);
#pragma unroll
        for (int i = 0; i < NBV; ++i) {
            const int tb = sb0 + i;
            f32x16 acc = zero16();
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s < 2 * (tb + 1)) acc = Tr<T>::mma(uf[s], ld_frag<T>(Fs + (32 * tb + l32) * LDC + 16 * s + 8 * h), acc);
            float* xdst = p.xinit + ((bhc * 2 + tb) * DB + cb) * 1024;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 v4;
#pragma unroll
                for (int r = 0; r < 4; ++r) v4[r] = (float)qr[i][g][r] - acc[4 * g + r];
                __builtin_nontemporal_store(v4, reinterpret_cast<f32x4*>(xdst + (g * 64 + lane) * 4));
            }
        }
    }
    // Sd^T = K Q^T - Y^T F^T, accumulator order: [bhc][query block][key block][g][lane][4]
    if (wv != 1) {
        f32x16 corr = zero16();
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (s >= 2 * y && s < 2 * (x + 1)) corr = Tr<T>::mma(ld_frag<T>(Yt + (32 * y + l32) * LDC + 16 * s + 8 * h), ld_frag<T>(Fs + (32 * x + l32) * LDC + 16 * s + 8 * h), corr);
        float* dst = p.sd + (bhc * 4 + (size_t)(x * 2 + y)) * 1024;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 v4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = accS[4 * g + r] - corr[4 * g + r];
            __builtin_nontemporal_store(v4, reinterpret_cast<f32x4*>(dst + (g * 64 + lane) * 4));
        }
    }
    if (BWD) {
        keep(p.fm, Fs, 64);
        keep(p.ytm, Yt, 64);
        keep(p.utm, Ut, D);
    }
}

template <typename TIO, int D, bool BWD, bool STRIDED>
static hipError_t launch_prep16_s(const FwdParams& p, hipStream_t stream) {
    using C = Prep16Cfg<TIO, D>;
    // set once per process; a function-local static is initialised under the language's own lock
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&prep16_fwd_kernel<TIO, D, BWD, STRIDED>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::TOTAL);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((prep16_fwd_kernel<TIO, D, BWD, STRIDED>), dim3((unsigned)(p.NC * p.B * p.H)), dim3(256), (size_t)C::TOTAL, stream, p);
    return hipGetLastError();
}
template <int D, bool BWD>
static hipError_t launch_prep16_b(const FwdParams& p, hipStream_t stream) {
    return p.ul.vt != D ? launch_prep16_s<bf16_t, D, BWD, true>(p, stream) : launch_prep16_s<bf16_t, D, BWD, false>(p, stream);
}
template <int D>
static hipError_t launch_prep16_t(const FwdParams& p, hipStream_t stream) {
    return p.fm ? launch_prep16_b<D, true>(p, stream) : launch_prep16_b<D, false>(p, stream);
}
hipError_t launch_prep16_fwd(const FwdParams& p, int d, hipStream_t stream) { return d == 64 ? launch_prep16_t<64>(p, stream) : launch_prep16_t<128>(p, stream); }

}  // namespace path
