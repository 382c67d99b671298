// Second blocking level of the forward (not in the paper; it follows from the
// associativity the paper uses in Sec. 3.2 for the cross-block term): inside a
// super-block of SBC chunks the boundary-adjusted keys are carried further, to
// the super-block's right edge, and the chunk products are multiplied up,
//
//     R_c = P_last ... P_{c+1}         (R_last = I),      R_{c-1} = R_c P_c
//     Kb2_c = Kb_c R_c^T ,             P_superblock = R_{first-1} ,
//
// so that the sweep applies ONE d x d product per super-block instead of one
// per chunk.  With E_c = I - R_c:  E_{c-1} = E_c + dP_c - E_c dP_c  and
// Kb2_c = Kb_c - Kb_c E_c^T.
//
// One workgroup per (batch*head, super-block), one wave per 32 rows of E: the rows of E do not depend on each other
// (E dP takes a row of E to a row), and column c of Kb2 needs row c of E alone.  A wave keeps its rows transposed in
// fp32 registers (rows b, lane = row a); those registers packed are the operand of both products, so the waves share
// nothing but the chunk's key and -dP tiles, copied to LDS as the chunk kernel wrote them.  Where -dP is needed
// element-wise in the transposed register layout it is transposed through the matrix unit.  (fp32 operands at d = 64: two
// waves per 32 rows, half of the columns and half of the keys each, that pass each other their half of E through LDS.  With
// two waves in all, half of the CU's matrix pipes idle: transform and key prefill of 16 heads of 2000 tokens 184 us,
// with four 150.)
//
// What bounds it: memory where there are many super-blocks (64 KB per chunk at d = 128, 96 with the backward's
// outputs), the chain of 16 chunks where there are few.  Hence two shapes: more than one workgroup per CU, one stage of
// tiles each, and a single workgroup per CU with the next two chunks' tiles on their way during the current one's products,
// brought by waves of their own (a copy takes the wave that makes it 70 cycles).
// At d = 128: 64 heads of 7 super-blocks with the backward's outputs 160 us (4.3 TB/s), 512 heads of 2 without them
// 154 us, one super-block per head into the cache 38 us.  (Waves that each took all of E's blocks from LDS, two
// fragments per product: 171, 226 and, with the rows turned and copied afterwards, 84 us.)  With the backward's outputs and
// one stage, d = 128 keeps 8 registers in scratch.
#include "path_common.h"
#include "decode_decl.h"

namespace path {

enum { P2_FWD = 0, P2_BWD = 1, P2_CACHE = 2 };
// P2_BWD: also write the backward-only outputs.  P2_CACHE: the key prefill of a prompt of one super-block -- the keys,
// carried to the super-block's right edge, which is the prompt's end, go to the decode path's cache (row-major, its
// storage type), and further workgroups copy the values.
template <typename TIO, int D, int NBUF> struct Prep2Cfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int KV_FRAGS = CHUNK * D / Tr<T>::FE, DP_FRAGS = D * D / Tr<T>::FE;
    static constexpr int SPLIT = sizeof(T) == 4 && D == 64 ? 2 : 1;      // waves per 32 rows of E
    static constexpr int NT = 64 * (D / 32) * SPLIT;
    static constexpr int XCH_FRAGS = SPLIT == 1 ? 0 : DP_FRAGS;          // E as operand fragments
    static constexpr size_t smem_bytes = ((size_t)NBUF * (KV_FRAGS + DP_FRAGS) + XCH_FRAGS) * 16;      // stages of (key tile | -dP tile)
    static constexpr bool COPIERS = NBUF == 3;                           // as many waves again make the copies, two stages ahead
    static constexpr int THREADS = COPIERS ? 2 * NT : NT;
    static constexpr int WAVES_PER_SIMD = COPIERS ? 2 : sizeof(T) == 2 && NBUF == 1 ? (D == 64 ? 3 : 2) : 1;
};

template <typename TIO, int D, int MODE, int NBUF>
__global__ __launch_bounds__((Prep2Cfg<TIO, D, NBUF>::THREADS), (Prep2Cfg<TIO, D, NBUF>::WAVES_PER_SIMD)) void prep2_fwd_kernel(FwdParams p) {
    using C = Prep2Cfg<TIO, D, NBUF>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    constexpr int FE = Tr<T>::FE, KW = Tr<T>::KW;
    constexpr int SPB = 32 / KW, DB = D / 32, DS = D / KW, KVF = C::KV_FRAGS, DPF = C::DP_FRAGS, NT = C::NT;
    constexpr bool BWD = MODE == P2_BWD;
    constexpr int SPLIT = C::SPLIT, NB = DB / SPLIT, NKH = 2 / SPLIT;      // the wave's column blocks of E and halves of the key tile
    static_assert(SPLIT == 1 || NBUF == 1, "the exchange takes its barriers from the single stage");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Frag* const stage = reinterpret_cast<Frag*>(smem);
    Frag* const xch = stage + NBUF * (KVF + DPF);

    const int sb = blockIdx.x, bh = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    if (MODE == P2_CACHE && sb > 0) {
        copy_value_rows<TIO, D, NT>(p.v, p.vcache, p.L, p.Lmax, bh, sb - 1, tid);
        return;
    }
    const int NC = p.NC, nsb = (NC + SBC - 1) / SBC;                       // chunks and super-blocks per head in the workspace arrays
    const int NCown = (seq_len(p.ul, bh, p.L) + CHUNK - 1) / CHUNK;        // this head's own (packed batches: may be fewer)
    const int c0 = sb * SBC;
    if (c0 >= NCown) return;
    if (BWD && is_last_sb(sb, NCown)) return;         // (a training step never looks at it from the right: see is_last_sb)
    const int clast = (c0 + SBC - 1 < NCown) ? c0 + SBC - 1 : NCown - 1;

    const int ra = wv / SPLIT, part = SPLIT == 1 ? 0 : wv % SPLIT;         // row block of E; which half of the work on it
    const int b0 = part * NB, h0 = part * NKH;                             // first column block, first half of the key tile

    Frag idf[SPB], Eb[DS];
    identity_frags<T>(idf, l32, h);
    f32x16 Fm[NB];      // E^T of the wave's rows: rows b of column block b0 + o, lane a = 32 ra + l32
#pragma unroll
    for (int o = 0; o < NB; ++o) Fm[o] = zero16();

    auto place = [&](int c) { return stage + (size_t)(NBUF == 3 ? (clast - c) % 3 : c & (NBUF - 1)) * (KVF + DPF); };
    auto issue = [&](int c, int ctid, int cwv) {
        const size_t bhc = (size_t)bh * NC + c;
        Frag* buf = place(c);
        async_copy_tile<NT, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.kt) + bhc * (size_t)CHUNK * D), buf, ctid, cwv);
        async_copy_tile<NT, DPF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(p.dp) + bhc * (size_t)D * D), buf + KVF, ctid, cwv);
    };
    if constexpr (C::COPIERS) {
        if (wv >= NT / 64) {
            const int ctid = tid - NT, cwv = wv - NT / 64;
            issue(clast, ctid, cwv);
            if (clast > c0) issue(clast - 1, ctid, cwv);
            for (int c = clast; c >= c0; --c) {
                if (c > c0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((KVF + DPF) / NT) : "memory");      // chunk c has landed, the next one may be on its way
                else copies_landed();
                lds_barrier();                 // ... for everybody, and chunk c + 1 has been read
                if (c - 2 >= c0) issue(c - 2, ctid, cwv);
            }
            return;
        }
    }
    if (NBUF == 2) issue(clast, tid, wv);
    for (int c = clast; c >= c0; --c) {
        const size_t bhc = (size_t)bh * NC + c;
        if (C::COPIERS) {
            lds_barrier();
        } else if (NBUF == 2) {
            wait_async_and_sync();             // chunk c has landed; everyone is done with chunk c+1
            if (c > c0) issue(c - 1, tid, wv);
        } else {
            __syncthreads();
            issue(c, tid, wv);
            if (SPLIT > 1) {
#pragma unroll
                for (int o = 0; o < NB; ++o) {
                    Frag fr[SPB];
                    pack_block<T>(Fm[o], fr);
#pragma unroll
                    for (int s2 = 0; s2 < SPB; ++s2) xch[(ra * DS + (b0 + o) * SPB + s2) * 64 + lane] = fr[s2];
                }
            }
            wait_async_and_sync();
        }
        const Frag* k1 = place(c);
        const Frag* dpn = k1 + KVF;                                                                                  // (rows b, contr a) = -dP[a][b]
        if constexpr (SPLIT == 1) {
#pragma unroll
            for (int b = 0; b < DB; ++b) pack_block<T>(Fm[b], Eb + b * SPB);
        } else {
#pragma unroll
            for (int s = 0; s < DS; ++s) Eb[s] = xch[(ra * DS + s) * 64 + lane];
        }
        if (BWD) {      // backward only: R_c = I - E_c (16-bit operands: a tile with rows a, contraction b; fp32: row-major [a][b])
#pragma unroll
            for (int o = 0; o < NB; ++o) {
                const int b = b0 + o;
                int diag = b == ra ? l32 - 4 * h : -1;
                asm volatile("" : "+v"(diag));            // compared here: sixteen masks kept over the loop would spill
                f32x16 rc;
#pragma unroll
                for (int jj = 0; jj < 16; ++jj) rc[jj] = (acc_row(jj, 0) == diag ? 1.f : 0.f) - Fm[o][jj];
                if (sizeof(T) == 2) {
                    Frag* rdst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.rm) + bhc * (size_t)D * D);
                    Frag fr[SPB];
                    pack_block<T>(rc, fr);
#pragma unroll
                    for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &rdst[((size_t)ra * DS + b * SPB + s2) * 64 + tile_lane<T>(lane, s2)]);
                } else {
                    float* rdst = reinterpret_cast<float*>(p.rm) + bhc * (size_t)D * D + (size_t)(32 * ra + l32) * D + 32 * b + 4 * h;
#pragma unroll
                    for (int g = 0; g < 4; ++g) *reinterpret_cast<f32x4*>(rdst + 8 * g) = f32x4{rc[4 * g], rc[4 * g + 1], rc[4 * g + 2], rc[4 * g + 3]};
                }
            }
        }
        // The last chunk has E = 0.  fp32 products take so long that they are left out there (the own segment of a ring, 3 heads
        // of one chunk, d = 128: 62.0 us, without them 52.2); 16-bit products take a sixteenth of that.
        const bool products = sizeof(T) == 2 || c != clast;
        // The products in groups of DS fragments (halves of the key tile, then row blocks of -dP), each group's
        // read from LDS while the one before is multiplied; the scheduling barriers keep it to two groups in registers.
        Frag f[2][DS], dfr[2][SPB];
        auto read_group = [&](int g) {
            const Frag* src = g < NKH ? k1 + (size_t)(h0 + g) * DS * 64 : dpn + (size_t)(b0 + g - NKH) * DS * 64;
#pragma unroll
            for (int s = 0; s < DS; ++s) f[g & 1][s] = src[s * 64 + tile_lane<T>(lane, s)];
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) dfr[g & 1][s2] = src[(ra * SPB + s2) * 64 + tile_lane<T>(lane, s2)];
        };
        read_group(0);
        // Kb2^T[cc][s] = Kb^T[cc][s] - sum_b E[cc][b] Kb[s][b]   (registers rows cc of the wave, lane s)
        Frag* k2 = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.kt2) + bhc * (size_t)CHUNK * D);
#pragma unroll
        for (int g = 0; g < NKH; ++g) {
            const int sb2 = h0 + g;
            read_group(g + 1);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 acc = zero16();
            if (products) {
#pragma unroll
                for (int s = 0; s < DS; ++s) acc = Tr<T>::mma(Eb[s], f[g][s], acc);
            }
            if (MODE == P2_CACHE) {
                typedef typename Tr<TIO>::Vec4 OVec4;
                const int tok = c * CHUNK + 32 * sb2 + l32;
                if (tok < p.L) {
                    TIO* dst = reinterpret_cast<TIO*>(p.kcache) + ((size_t)bh * p.Lmax + tok) * D + 32 * ra + 4 * h;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        OVec4 o4;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int jj = 4 * q + r;
                            o4[r] = (TIO)((float)dfr[g][jj / FE][jj % FE] - acc[jj]);
                        }
                        *reinterpret_cast<OVec4*>(dst + 8 * q) = o4;
                    }
                }
                continue;
            }
            Frag fr[SPB];
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) {
#pragma unroll
                for (int e = 0; e < FE; ++e) fr[s2][e] = (T)((float)dfr[g][s2][e] - acc[s2 * FE + e]);
            }
#pragma unroll
            for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(fr[s2], &k2[((size_t)sb2 * DS + ra * SPB + s2) * 64 + tile_lane<T>(lane, s2)]);
            if (BWD && sizeof(T) == 4) {     // backward with fp32 operands only: the arrangement (rows cc, contraction s)
                Frag* k2T = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.kt2T) + bhc * (size_t)CHUNK * D);
                const f32x16 tr = transpose32<T>(fr, idf);      // rows s, lane cc
                Frag ft[SPB];
                pack_block<T>(tr, ft);
#pragma unroll
                for (int s2 = 0; s2 < SPB; ++s2) __builtin_nontemporal_store(ft[s2], &k2T[((size_t)ra * (CHUNK / KW) + sb2 * SPB + s2) * 64 + lane]);
            }
        }
        if (MODE == P2_CACHE && c == c0) break;
        // E^T <- E^T + dP^T - dP^T E^T   (registers rows b, lane a)
#pragma unroll
        for (int o = 0; o < NB; ++o) {
            const int g = NKH + o;
            if (o + 1 < NB) read_group(g + 1);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 acc = zero16();
            if (products) {
#pragma unroll
                for (int s = 0; s < DS; ++s) acc = Tr<T>::mma(f[g & 1][s], Eb[s], acc);
            }
            // -dP[a][b] in this block's register layout (rows b, lane a): the tile piece (rows b,
            // contraction a) transposed through the matrix unit
            const f32x16 dpT = transpose32<T>(dfr[g & 1], idf);
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) Fm[o][jj] = Fm[o][jj] - dpT[jj] + acc[jj];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (MODE == P2_CACHE) return;
    // -(I - P_superblock) as the sweep's tile (rows b, contraction a): E itself (rows a, lane b) is the
    // transpose of what the registers hold -- taken through the matrix unit.
    Frag* dst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.dp2) + ((size_t)bh * nsb + sb) * (size_t)D * D);
#pragma unroll
    for (int o = 0; o < NB; ++o) {
        const int b = b0 + o;
        Frag fin[SPB];
        pack_block<T>(Fm[o], fin);                              // tile piece (rows a, contraction b)
        if (BWD && sizeof(T) == 4) {      // backward, fp32 operands only: -(I - P_superblock) in the arrangement (rows a, contraction b)
            Frag* dt = reinterpret_cast<Frag*>(reinterpret_cast<T*>(p.dpt2) + ((size_t)bh * nsb + sb) * (size_t)D * D);
#pragma unroll
            for (int s = 0; s < SPB; ++s) {
                Frag ng;
#pragma unroll
                for (int e = 0; e < FE; ++e) ng[e] = (T)(-(float)fin[s][e]);
                __builtin_nontemporal_store(ng, &dt[((size_t)ra * DS + b * SPB + s) * 64 + lane]);
            }
        }
        f32x16 tr = transpose32<T>(fin, idf);                   // rows a, lane b
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) tr[jj] = -tr[jj];
        Frag fr[SPB];
        pack_block<T>(tr, fr);
#pragma unroll
        for (int s = 0; s < SPB; ++s) __builtin_nontemporal_store(fr[s], &dst[((size_t)b * DS + ra * SPB + s) * 64 + tile_lane<T>(lane, s)]);
    }
}

template <typename TIO, int D, int MODE, int NBUF>
hipError_t launch_prep2_b(const FwdParams& p, dim3 grid, hipStream_t stream) {
    using C = Prep2Cfg<TIO, D, NBUF>;
    // set once per process; a function-local static is initialised under the language's own lock
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&prep2_fwd_kernel<TIO, D, MODE, NBUF>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::smem_bytes);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((prep2_fwd_kernel<TIO, D, MODE, NBUF>), grid, dim3(C::THREADS), C::smem_bytes, stream, p);
    return hipGetLastError();
}
template <typename TIO, int D, int MODE>
hipError_t launch_prep2_m(const FwdParams& p, hipStream_t stream) {
    const int BH = p.B * p.H, nsb = (p.NC + SBC - 1) / SBC - (MODE == P2_BWD ? 1 : 0);      // (training: every super-block but the last)
    if (nsb < 1) return hipSuccess;
    if constexpr (MODE == P2_CACHE) {
        const dim3 grid(1 + value_row_pieces(p.L), BH);
        return launch_prep2_b<TIO, D, MODE, sizeof(TIO) == 2 ? 2 : 1>(p, grid, stream);
    } else {
        const dim3 grid(nsb, BH);
        // (fp32 operands: two stages of tiles do not fit)
        if constexpr (sizeof(TIO) == 2) {
            // one workgroup for every CU or less; above that the second workgroup hides more than the second stage does
            // (one stage against two, us: d = 128, 128 workgroups 59 / 52, 192 59 / 50, 512 106 / 127; d = 64, 256 30 / 24, 384 47 / 50).
            // With copying waves and three stages another 4 to 9 us less (128 workgroups, d = 128: both transforms 144 -> 135, 32
            // workgroups 66.9 -> 59.7; d = 64, 6 workgroups 32.2 -> 28.3)
            if ((long long)nsb * BH <= 256) return launch_prep2_b<TIO, D, MODE, 3>(p, grid, stream);
        }
        return launch_prep2_b<TIO, D, MODE, 1>(p, grid, stream);
    }
}
template <typename TIO, int D>
hipError_t launch_prep2_fwd_t(const FwdParams& p, hipStream_t stream) {
    if (p.kcache) return launch_prep2_m<TIO, D, P2_CACHE>(p, stream);
    return p.rm ? launch_prep2_m<TIO, D, P2_BWD>(p, stream) : launch_prep2_m<TIO, D, P2_FWD>(p, stream);
}

hipError_t launch_prep2_fwd(const FwdParams& p, int d, int is_bf16, hipStream_t stream) {
    if (is_bf16) return d == 64 ? launch_prep2_fwd_t<bf16_t, 64>(p, stream) : launch_prep2_fwd_t<bf16_t, 128>(p, stream);
    return d == 64 ? launch_prep2_fwd_t<float, 64>(p, stream) : launch_prep2_fwd_t<float, 128>(p, stream);
}

}  // namespace path
