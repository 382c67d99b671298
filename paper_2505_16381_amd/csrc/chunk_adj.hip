// Near key-side sums and adjoint of the chunk transform (the UT transform of Sec. 3.2 and the diagonal block of
// Sec. 3.3), fused: one workgroup per (chunk, head), for 2-byte operand types and for
// fp32 operands at d = 64.  The paper gives
// no backward; with the chunk's matrices (rows = the 64 tokens of the chunk)
//
//   F   strictly-lower part of the boundary-adjusted query transform,  Y = solved W-side block,
//   N, Gk, A^-1 from the UT transform,  U = T^-1-transformed W (dP = W^T U),  Sd the raw diagonal logits,
//
// the gradients that arrive are dQb, dKb (boundary-adjusted queries / keys), ddP (chunk product),
// dV' (off-diagonal part of dV), and the steps are
//
//   dPd = dO V^T;  P = exp(scale Sd - lse) (key <= query);  dSd = scale P o (dPd - delta)
//   dV  = dV' + P^T dO
//   dF  = tril(-dSd Y^T - dQb U^T)            dY = -F^T dSd - W dKb^T
//   dU  = -F^T dQb + W ddP                     dN = dY Gk^T + dU W^T
//   (ddP, dKb: the near sums, which this kernel takes first, plus the second level's share, see sb_chain_kernel below)
//   dGk = sl(N^T dY)     R = A^-T dN     M = sl(-R N^T)     dGs = diag(beta) M + (diag(beta) M)^T
//   dbeta_a = R_aa + sum_s M_as G_as
//   dQ  = dQb + dSd K + dF W
//   dK  = dKb + dSd^T Q + dGk^T W
//   dW  = -Y dKb + U ddP^T + dF^T Q + dGk K + N^T dU + dGs W
//
// (sl = strictly lower part).  Every matrix is staged ONCE into LDS in the layout it has in
// memory (converted to the operand type); a product whose contraction runs along the rows of a
// stored matrix takes its 16-byte fragments with two transposing LDS reads instead of keeping a
// transposed copy.  dK and dW accumulate in registers across the whole kernel; the 64 x 64
// intermediates never leave LDS.  fp32 operands: the near sums and the second level's share come from memory, transposed
// operands are 4-byte LDS reads; d = 128 does not fit and stays a list of staged products (chunk_adjoint_kernel in bwd.hip), 24
// of them one after the other, each through memory.  Training step of 2 heads of 256 tokens, d = 64: that kernel 132 -> 37 us, the
// step 253.5 -> 156.7; 16 heads of 1000 tokens 577 -> 465; 64 of 2048 4219 -> 3792.
//
// What bounds it: latency -- chains of short dependent phases between barriers, at d = 128 with one workgroup per CU -- and
// then memory: at d = 128 the states and adjoint states of 7.5 pairs on average (0.24 MB), 0.3 MB of the chunk's matrices and
// the four gradients (0.06 MB) per chunk.  The near sums as a kernel of its own left dV, dKb and ddP in memory, 128 KB
// written and read again per chunk: 743 + 1027 -> 1450 us at B=4, H=16, L=8192, d=128, 357 + 417 -> 671 at B=8, H=16, L=4096,
// d=64, packed batch of 64 sequences of 256 .. 2048 tokens (8 heads, d = 128) 700 + 1267 -> 1460.  (Near sums alone 681 us, the
// rest alone 892, at the first of these shapes.  With a third stage of states for the pairs the near sums take as long, and at
// d = 64 longer.)  Of what follows the near sums most is vector instructions, in a chain: addresses, conversions, LDS stores of two
// bytes.  With tiles turned instead of padded (lds_tile.h; 64 heads of 8192 tokens, d = 128: 60 million cycles of bank conflicts, now
// 11), addresses that leave one exclusive or per access,
// 64 x 64 results multiplied out transposed, so that they are stored four at a time, dGs formed where M is and whole chunks stored without
// checks of the row, the chunk stage (with sb_chain_kernel) went, us, at d = 128 from 1594 to 1499 (64 heads of 8192 tokens), 1288 to 1163
// (512 of 1024), 42.2 to 38.2 (8 of 1000), at d = 64 from 711 to 675 (128 of 4096).  The turned tiles alone, with addresses left to the compiler,
// gave nothing: what they saved in conflicts they cost in vector instructions.
#include <type_traits>

#include "path_common.h"
#include "bwd_decl.h"
#include "lds_tile.h"

namespace path {
namespace {

constexpr int CA_NT = 512;       // threads per workgroup (8 waves)

// Near key-side sums (the first part of the kernel): stages of tiles and hand-over buffers, in fragments.
template <typename TIO, int D> struct NearCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int KVF = CHUNK * D / Tr<T>::FE;                 // fragments of a tile
    static constexpr int STF = 3 * KVF + 32;                          // a stage: xs | doq | g | lse2, delta
    static constexpr int PDF = 2 * 2 * 4 * 64;                        // a hand-over buffer: (P | dS) x 2 key halves x 4 slabs
    // d = 64: one hand-over buffer (and a second barrier per pair), so that two workgroups share a CU.  (The 128 registers that
    // this leaves do; with gates 16 more, 17 with interleaved heads, lie in scratch, none of them inside the loop over pairs.)
    static constexpr int HB = D == 64 ? 1 : 2;
    static constexpr int smem_bytes = (2 * STF + HB * PDF) * 16;
    // dV | dKb on their way to the waves that go on with them, fp32 [key][D + 4]
    static constexpr int LDX = D + 4, XV = 0, XK = CHUNK * LDX, xch_bytes = 2 * CHUNK * LDX * 4;
};

// A tile of rows of W elements in LDS: 16-bit types as in lds_tile.h, 32-bit types padded.
template <typename T, int W> struct Tile {
    static constexpr int PITCH = sizeof(T) == 2 ? W : W + 4;
    static __device__ __forceinline__ int at(int row, int col) { return sizeof(T) == 4 ? row * PITCH + col : TurnedTile<W>::at(row, col); }
};
struct TileLanes {      // a lane's share of addresses in tiles of both widths
    int l32, h;
    TurnedLane<64> w64;
    TurnedLane<128> w128;
    __device__ __forceinline__ TileLanes(int tid) : l32(tid & 31), h((tid >> 5) & 1), w64(tid), w128(tid) {}
    template <int W> __device__ __forceinline__ const TurnedLane<W>& of() const {
        if constexpr (W == 64) return w64; else return w128;
    }
};
typedef __attribute__((address_space(3))) unsigned char LdsByte;
template <typename V> __device__ __forceinline__ V lds_read(unsigned a) { return *(__attribute__((address_space(3))) const V*)(LdsByte*)(uintptr_t)a; }
template <typename V> __device__ __forceinline__ void lds_write(unsigned a, V v) { *(__attribute__((address_space(3))) V*)(LdsByte*)(uintptr_t)a = v; }
template <typename T> __device__ __forceinline__ unsigned lds_addr(const T* p) { return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void*)p; }

template <typename TIO, int D> struct CaCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int ES = sizeof(T);
    static constexpr bool NEAR_SUMS = ES == 2;      // fp32 operands: the near sums and the second level's share are taken before
    static_assert(ES == 2 || D == 64, "fp32 tiles of d = 128 do not fit");
    typedef Tile<T, D> TileD;
    typedef Tile<T, CHUNK> TileC;
    static constexpr int LDD = D + 16 / ES;          // pitch of the second level's dKb2 rows (elements)
    static constexpr int SMALL = 64 * TileC::PITCH * ES, BIG_ = 64 * TileD::PITCH * ES, BIG = BIG_ > D * TileC::PITCH * ES ? BIG_ : D * TileC::PITCH * ES;   // bytes of a 64 x 64, of a 64 x D or D x 64 tile
    // byte offsets.  d = 128: W | X0 X3 (adjacent: ddP spans both) | X1 | X2 | Y0 Y1 Y2 | N | misc.
    // d = 64, where all tiles have one size: W | X0 | Y0 | X1 | X2 | X3 = N | Y1 | Y2 | misc: two
    // workgroups per CU (with ten tiles, 92 KB and one workgroup what follows the near sums took 0.63 ms at B=8, H=16, L=4096, not
    // 0.42).
    static constexpr int XW = 0, X0 = BIG, X3 = D == 64 ? 5 * BIG : 2 * BIG, X1 = 3 * BIG, X2 = 4 * BIG;
    static constexpr int Y0 = D == 64 ? 2 * BIG : 5 * BIG, Y1 = D == 64 ? 6 * BIG : Y0 + SMALL, Y2 = Y1 + SMALL, YN = D == 64 ? X3 : Y2 + SMALL;
    static constexpr int TILES = D == 64 ? Y2 + SMALL : YN + SMALL, NEAR = NEAR_SUMS ? NearCfg<TIO, D>::smem_bytes : 0;
    // between the near sums and the chunk's tiles: R | D of the second level | dV, dKb | dKb2
    static constexpr int SR = 0, SD = D * D * 2, XCH = 2 * SD, SK2 = XCH + NearCfg<TIO, D>::xch_bytes, MID = NEAR_SUMS ? SK2 + 64 * LDD * 2 : 0;
    static constexpr int MISC = MID > NEAR ? (MID > TILES ? MID : TILES) : (NEAR > TILES ? NEAR : TILES);
    static constexpr int TOTAL = MISC + 2048;
    static constexpr int WGS_PER_CU = D == 64 && ES == 2 ? 2 : 1;
    static_assert(D == 64 ? BIG == SMALL : D * TileD::PITCH * ES <= 2 * BIG, "ddP tile must fit X0 (d = 64) or X0 and X3");
    static_assert(WGS_PER_CU * TOTAL <= 160 * 1024, "LDS budget");
};

// ROWS x COLS elements of type S from global memory (row-major, `stride` elements between rows), 8 per
// thread and step, held in registers between load() and store(); rows >= nvalid are zero.
template <typename S, int ROWS, int COLS, int NT = CA_NT> struct GTile {
    static constexpr int NV = ROWS * COLS / 8 / NT;
    static_assert(NV >= 1 && NV * 8 * NT == ROWS * COLS, "tile must be a multiple of the workgroup's reach");
    typedef S Vec8 __attribute__((ext_vector_type(8)));
    Vec8 v[NV];
    __device__ __forceinline__ void load(const S* src, int stride, int nvalid, int tid) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int idx = tid + u * NT, r = idx / (COLS / 8), c = (idx % (COLS / 8)) * 8;
            if (r < nvalid) v[u] = *reinterpret_cast<const Vec8*>(src + r * stride + c);
            else
#pragma unroll
                for (int e = 0; e < 8; ++e) v[u][e] = (S)0.f;
        }
    }
    template <typename T, bool NEG> __device__ __forceinline__ auto converted(int u) const {
        typedef T TVec8 __attribute__((ext_vector_type(8)));
        TVec8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (T)(NEG ? -(float)v[u][e] : (float)v[u][e]);
        return o;
    }
    template <typename T, bool NEG> __device__ __forceinline__ void store(T* dst, int ld, int tid) const {      // padded rows
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int idx = tid + u * NT, r = idx / (COLS / 8), c = (idx % (COLS / 8)) * 8;
            const auto o = converted<T, NEG>(u);
            *reinterpret_cast<decltype(converted<T, NEG>(0))*>(dst + r * ld + c) = o;
        }
    }
    template <typename T, bool NEG> __device__ __forceinline__ void store(T* dst, int tid, const TileLanes& t) const {      // a Tile
        if constexpr (sizeof(T) == 4) { store<T, NEG>(dst, Tile<T, COLS>::PITCH, tid); return; } else {
        static_assert(NT == 512, "copy_at's threads");
#pragma unroll
        for (int u = 0; u < NV; ++u) lds_write(lds_addr(dst) + t.of<COLS>().copy_at(u), converted<T, NEG>(u));
        }
    }
};

// One 32x32 accumulator block (rows m, lane n) -> rows r0 .., columns c0 .. of a tile [m][n], in the operand type.
template <typename T, int W>
__device__ __forceinline__ void st_block(T* dst, int r0, int c0, const f32x16& acc, const TileLanes& t) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) dst[Tile<T, W>::at(r0 + acc_row(jj, t.h), c0 + t.l32)] = (T)acc[jj];
    } else {
        const unsigned a = lds_addr(dst) + t.of<W>().elem_at(r0, c0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) lds_write(TurnedLane<W>::elem_step(a, q, r), (T)acc[4 * q + r]);
    }
}
// The same of a block with rows n, lane m (the product with its operands exchanged): a quarter of the stores.
template <typename T, int W>
__device__ __forceinline__ void st_block_t(T* dst, int r0, int c0, const f32x16& acc, const TileLanes& t) {
    typedef typename Tr<T>::Vec4 TVec4;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        TVec4 v4;
#pragma unroll
        for (int r = 0; r < 4; ++r) v4[r] = (T)acc[4 * g + r];
        if constexpr (sizeof(T) == 4) *reinterpret_cast<TVec4*>(dst + Tile<T, W>::at(r0 + t.l32, c0 + 8 * g + 4 * t.h)) = v4;
        else lds_write(lds_addr(dst) + t.of<W>().vec_at(r0, c0 + 8 * g), v4);
    }
}

// The four fragments of 64 contraction indices from k0 on, of rows (TR: columns) r0 + l32 of a tile.
template <typename T, int W, bool TR>
__device__ __forceinline__ void tile_frags(typename Tr<T>::Frag (&f)[4], const T* X, int r0, int k0, const TileLanes& t) {
    if constexpr (!TR) {
#pragma unroll
        for (int s = 0; s < 4; ++s) f[s] = lds_read<typename Tr<T>::Frag>(lds_addr(X) + t.of<W>().nat_at(r0, k0 + 16 * s));
    } else {
        typedef short v4s __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            union { v4s v[2]; typename Tr<T>::Frag f; } u;
            u.v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(LdsByte*)(uintptr_t)(lds_addr(X) + t.of<W>().tr_at(k0 + 16 * s, r0, 0)));
            u.v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(LdsByte*)(uintptr_t)(lds_addr(X) + t.of<W>().tr_at(k0 + 16 * s, r0, 1)));
            f[s] = u.f;
        }
    }
}
// acc[m][n] += sum_k A(m,k) B(n,k) as mm() in path_common.h, for operands in tiles of WA and WB columns.
template <typename T, int K, bool TA, int WA, bool TB, int WB>
__device__ __forceinline__ void mmt(f32x16& acc, const T* A, int ar0, const T* B, int br0, const TileLanes& t) {
    if constexpr (sizeof(T) == 4) { mm_f32<K, TA, TB>(acc, A, Tile<T, WA>::PITCH, ar0, B, Tile<T, WB>::PITCH, br0, t.l32, t.h); return; } else {
    // four slabs (64 contraction indices) at a time: their fragments are fetched ahead of the four products
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 64) {
        typename Tr<T>::Frag fa[4], fb[4];
        tile_frags<T, WA, TA>(fa, A, ar0, k0, t);
        tile_frags<T, WB, TB>(fb, B, br0, k0, t);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(fa[s], fb[s], acc);
    }
    }
}

// Near key-side sums, over the query chunks i right of the key's chunk j inside its own super-block, with the
// chunk-level keys Kb and the chunk's own product,
//
//     S = Xs Kb_j^T,  dP = dO V_j^T,  ...       dV^T += dO^T P      dKb^T += Xs^T dS      ddP_j -= Xs^T g
//
// split by kind of work as for the far keys (bwd_keys.hip), one barrier per pair (64 queries):
//   waves 0..3  (key half w & 1) x (query half w >> 1): logits, dP, element-wise part of the pair;
//   waves 4..7  a quarter of each sum: ddP_j of this pair, dV^T and dKb^T of the pair before (its transposed fragments
//               stay in registers, so that two stages of tiles do).
// The former request the next pair's tiles.  The sums stay in the registers of waves 4..7 (dV^T, dKb^T row blocks NA rb + a
// of key half kb, -ddP blocks (NA rb + a, NA kb + b), rows = second index; rb = (wave - 4) / 2, kb = wave % 2), the keys' part of the gate
// gradient, one query half each, in dcol of waves 0..3.  tiles_read(): run by all waves when the tiles have been read for
// the last time; the hand-over buffer of the last pair is read after that.
template <typename TIO, int D, bool FOX, typename F>
__device__ __forceinline__ void near_sums(const ChunkFusedArgs& a, unsigned char* smem, int j, int bh, int NCown, F tiles_read,
                                          f32x16 (&dV)[D / 64], f32x16 (&dK)[D / 64], f32x16 (&dd)[D / 64][D / 64], float& dcol) {
    using C = NearCfg<TIO, D>;
    using T = typename C::T;
    using Frag = typename Tr<T>::Frag;
    using FragV = typename Tr<TIO>::Frag;
    constexpr int KW = Tr<T>::KW, SPB = 32 / KW, DB = D / 32, DS = D / KW, QS = CHUNK / KW;
    constexpr int KVF = C::KVF, STF = C::STF, PDF = C::PDF, HB = C::HB;
    Frag* const stages = reinterpret_cast<Frag*>(smem);
    Frag* const hand = stages + 2 * STF;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int NC = a.NC;
    const size_t Lp = (size_t)NC * CHUNK, nslots = num_block_slots(NC);
    const int i0 = j + 1, i1 = (j / SBC + 1) * SBC < NCown ? (j / SBC + 1) * SBC : NCown;
    constexpr int NA = DB / 2;
#pragma unroll
    for (int a2 = 0; a2 < NA; ++a2) {
        dV[a2] = zero16(); dK[a2] = zero16();
#pragma unroll
        for (int b = 0; b < NA; ++b) dd[a2][b] = zero16();
    }
    dcol = 0.f;
    if (i0 >= i1) { tiles_read(); return; }               // the super-block's last chunk: no such queries
    auto issue = [&](int i) {                             // into stage i & 1, by waves 0..3: a transposing read, as the others make, waits for
                                                          // every copy its own wave has in flight (by all eight waves: 1630 us, d = 64 945)
        Frag* buf = stages + (i & 1) * STF;
        const size_t slot = ((size_t)bh * nslots + block_slot(i, j, NC)) * (size_t)CHUNK * D;
        async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.xs) + slot), buf, tid, wv);
        async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const TIO*>(a.doq) + ((size_t)bh * NC + i) * CHUNK * D), buf + KVF, tid, wv);
        async_copy_tile<256, KVF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.gs) + slot), buf + 2 * KVF, tid, wv);
        if (tid < 32) {         // 64 floats of lse2 (lanes 0-15) and of delta (lanes 16-31): 16 bytes per lane
            const float* src = (tid < 16 ? a.lse2p : a.delta) + (size_t)bh * Lp + (size_t)i * CHUNK + 4 * (tid & 15);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(buf + 3 * KVF), 16, 0, 0);
        }
    };
    if (wv < 4) {
        issue(i0);
        // ---- logits and the element-wise part -----------------------------------------------------------------
        const float sl2 = a.scale * 1.44269504088896340736f;
        const int kh = wv & 1, qh = wv >> 1;
        Frag Kb[DS];
        FragV Vb[DS];
        {
            const Frag* kg = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.kt) + ((size_t)bh * NC + j) * CHUNK * D);
            const FragV* vg = reinterpret_cast<const FragV*>(reinterpret_cast<const TIO*>(a.vk) + ((size_t)bh * NC + j) * CHUNK * D);
#pragma unroll
            for (int s = 0; s < DS; ++s) { Kb[s] = kg[((size_t)kh * DS + s) * 64 + tile_lane<T>(lane, s)]; Vb[s] = vg[((size_t)kh * DS + s) * 64 + lane]; }
        }
        const int key_tok = j * CHUNK + 32 * kh + l32;
        const float ckj = FOX ? a.cum[(size_t)bh * Lp + key_tok] : 0.f;
        for (int i = i0; i < i1; ++i) {
            copies_landed();
            lds_barrier();                                // pair i has landed; pair i - 1 has been read
            const Frag* sX = stages + (i & 1) * STF;
            const FragV* sDQ = reinterpret_cast<const FragV*>(sX + KVF);
            Frag xa[DS];
            FragV da[DS];
#pragma unroll
            for (int u = 0; u < DS; ++u) { xa[u] = sX[(qh * DS + u) * 64 + tile_lane<T>(lane, u)]; da[u] = sDQ[(qh * DS + u) * 64 + tile_lane<T>(lane, u)]; }
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < i1) issue(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 S = zero16(), dP = zero16();           // rows q, lane s
#pragma unroll
            for (int u = 0; u < DS; ++u) {
                S = Tr<T>::mma(xa[u], Kb[u], S);
                dP = Tr<TIO>::mma(da[u], Vb[u], dP);
            }
            const float* lse2 = reinterpret_cast<const float*>(sX + 3 * KVF) + 32 * qh + 4 * h;
            Frag* out = hand + (i & (HB - 1)) * PDF + (kh * QS + qh * SPB) * 64;
            FragV Pb[SPB];
            Frag dSb[SPB];
#pragma unroll
            for (int u = 0; u < SPB; ++u) {
#pragma unroll
                for (int g = 2 * u; g < 2 * u + 2; ++g) {
                    const f32x4 ls = *reinterpret_cast<const f32x4*>(lse2 + 8 * g), dls = *reinterpret_cast<const f32x4*>(lse2 + CHUNK + 8 * g);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // Rows past L need no mask: their padded lse2p is huge, so P = exp2(-huge) = 0.
                        float arg = __builtin_fmaf(S[4 * g + r], sl2, -ls[r]);
                        if (FOX) arg -= ckj;
                        const float P = __builtin_amdgcn_exp2f(arg);
                        const float dz = P * (dP[4 * g + r] - dls[r]);      // the factor scale is applied to the finished sums
                        if (FOX) dcol += dz;
                        Pb[u][(4 * g + r) % 8] = (TIO)P;
                        dSb[u][(4 * g + r) % 8] = (T)dz;
                    }
                }
            }
            if (HB == 1) lds_barrier();                   // the pair before has been read
#pragma unroll
            for (int u = 0; u < SPB; ++u) {
                reinterpret_cast<FragV*>(out)[u * 64 + lane] = Pb[u];
                out[(2 * QS + u) * 64 + lane] = dSb[u];
            }
        }
        lds_barrier();
        tiles_read();
        return;
    }

    // ---- the sums: row blocks NA rb .. of dV^T and dKb^T for key half kb, blocks (NA rb .., NA kb ..) of ddP ---------
    const int rb = (wv - 4) >> 1, kb = wv & 1;
    Frag xt[NA * QS];
    FragV dt[NA * QS];
    auto pair_sums = [&](int i) {                         // dV^T, dKb^T of pair i
        const Frag* in = hand + (i & (HB - 1)) * PDF + kb * QS * 64;
        FragV pf[QS];
        Frag sf[QS];
#pragma unroll
        for (int s = 0; s < QS; ++s) { pf[s] = reinterpret_cast<const FragV*>(in)[s * 64 + lane]; sf[s] = in[(2 * QS + s) * 64 + lane]; }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < QS; ++s)
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                dV[a] = Tr<TIO>::mma(dt[a * QS + s], pf[s], dV[a]);
                dK[a] = Tr<T>::mma(xt[a * QS + s], sf[s], dK[a]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pair_tile = [&](int i) {                         // ddP of pair i; its transposed fragments
        const Frag* sX = stages + (i & 1) * STF;
        Frag gf[NA * QS];
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int s = 0; s < QS; ++s) {
                xt[a * QS + s] = ld_tile_frag_tr<T, DS>(reinterpret_cast<const T*>(sX), s, NA * rb + a, l32, h);
                gf[a * QS + s] = ld_tile_frag_tr<T, DS>(reinterpret_cast<const T*>(sX + 2 * KVF), s, NA * kb + a, l32, h);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < QS; ++s)
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NA; ++b) dd[a][b] = Tr<T>::mma(gf[b * QS + s], xt[a * QS + s], dd[a][b]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int s = 0; s < QS; ++s) dt[a * QS + s] = ld_tile_frag_tr<TIO, DS>(reinterpret_cast<const TIO*>(sX + KVF), s, NA * rb + a, l32, h);
    };
    lds_barrier();
    pair_tile(i0);
    if (HB == 1) lds_barrier();
    for (int i = i0 + 1; i < i1; ++i) {
        lds_barrier();
        pair_sums(i - 1);
        pair_tile(i);
        if (HB == 1) lds_barrier();
    }
    lds_barrier();
    tiles_read();
    pair_sums(i1 - 1);
}

template <typename TIO, int D, bool FOX, bool STRIDED>
__global__ __launch_bounds__(CA_NT, 2 * (CaCfg<TIO, D>::WGS_PER_CU)) void chunk_fused_kernel(ChunkFusedArgs args) {
    using C = CaCfg<TIO, D>;
    typedef typename C::T T;
    constexpr int LDD = C::LDD;
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    T* XW = reinterpret_cast<T*>(smem + C::XW);
    T* X0 = reinterpret_cast<T*>(smem + C::X0);
    T* X1 = reinterpret_cast<T*>(smem + C::X1);
    T* X2 = reinterpret_cast<T*>(smem + C::X2);
    T* X3 = reinterpret_cast<T*>(smem + C::X3);
    T* Y0 = reinterpret_cast<T*>(smem + C::Y0);
    T* Y1 = reinterpret_cast<T*>(smem + C::Y1);
    T* Y2 = reinterpret_cast<T*>(smem + C::Y2);
    T* YN = reinterpret_cast<T*>(smem + C::YN);
    float* misc = reinterpret_cast<float*>(smem + C::MISC);
    float *beta_s = misc, *rdiag = misc + 64, *rowsum = misc + 128, *colsum = misc + 256, *nearcol = misc + 384;

    int chunk, bh;
    super_block_and_head(args.ul, args.NC, args.BH, chunk, bh);
    if (bh >= args.BH) return;
    const int L = seq_len(args.ul, bh, args.L), NC = args.NC;      // this head's own length; NC: chunks per head in the workspace arrays
    if (chunk * CHUNK >= L) return;                        // (packed batch: a shorter sequence has fewer chunks)
    const int NCown = (L + CHUNK - 1) / CHUNK;

    const bool right = !is_last_sb(chunk / SBC, NCown);          // there are queries right of the super-block

    // ---- near key-side sums: dV, dKb, ddP over the query chunks right of this one in its super-block -----------
    // (behind them, the second level's tiles of the chunk: R_c and the gradient of R_{c-1})
    constexpr int NA = D / 64;
    f32x16 nV[NA], nK[NA], dd[NA][NA];
    float ncol;
    if constexpr (C::NEAR_SUMS) near_sums<TIO, D, FOX>(args, smem, chunk, bh, NCown, [&]() {
        if (!right) return;
        typedef typename Tr<T>::Frag Frag;
        constexpr int DPF = D * D / 8;
        const size_t o = ((size_t)bh * NC + chunk) * D * D;
        const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6);
        async_copy_tile<CA_NT, DPF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(args.rm) + o), reinterpret_cast<Frag*>(smem + C::SR), t, w);
        async_copy_tile<CA_NT, DPF>(reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(args.dr) + o), reinterpret_cast<Frag*>(smem + C::SD), t, w);
    }, nV, nK, dd, ncol);

    // (from here on nothing is shared with the above, or the compiler would keep addresses and arguments in registers
    // across both)
    typedef const __attribute__((address_space(4))) void* KernArg;
    KernArg ka = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka));
    const ChunkFusedArgs& a = *(const ChunkFusedArgs*)ka;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid), "+v"(bh), "+v"(chunk));
    bh = __builtin_amdgcn_readfirstlane(bh);
    chunk = __builtin_amdgcn_readfirstlane(chunk);
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int ntok = (L - chunk * CHUNK < CHUNK) ? L - chunk * CHUNK : CHUNK;
    const size_t Lp = (size_t)NC * CHUNK;
    const long long ubase = user_vec(a.ul, bh, (long long)chunk * CHUNK);    // the caller's tensors: row of the chunk's first token
    const int TS = STRIDED ? (int)a.ul.vt : D;                                // ... and their token stride (a compile-time
                                                                              // constant unless the layout interleaves heads)
    const size_t pbase = ((size_t)bh * Lp + (size_t)chunk * CHUNK) * D;      // padded [Lp][d] workspace tensors
    const size_t cbase = ((size_t)bh * NC + chunk) * 4096;                   // 64 x 64 per chunk
    const size_t tpad = (size_t)bh * Lp + (size_t)chunk * CHUNK;             // per-token, padded
    const TIO* qg = reinterpret_cast<const TIO*>(a.q) + ubase;
    const TIO* kg = reinterpret_cast<const TIO*>(a.k) + ubase;
    const TIO* vg = reinterpret_cast<const TIO*>(a.v) + ubase;
    const TIO* wg = reinterpret_cast<const TIO*>(a.w) + ubase;
    const TIO* dog = reinterpret_cast<const TIO*>(a.d_o) + ubase;
    const T* utmg = reinterpret_cast<const T*>(a.utm) + ((size_t)bh * NC + chunk) * D * CHUNK;

    // wave -> 32x32 block of a 64 x D result (all 8 waves for D = 128; waves 0..3 for D = 64) and of a 64 x 64 result
    // (waves 0..3; waves 4..7 for D = 64)
    constexpr int NBD = D / 32;
    const bool actD = wv < 2 * NBD, act6 = D == 64 ? wv >= 4 : wv < 4;
    const int mbD = wv / NBD, cbD = wv % NBD, mb6 = (wv >> 1) & 1, cb6 = wv & 1;

    // (the lane's part of an address apart, as an unsigned offset: the rest stays in scalar registers)
    const unsigned lane_in = 4 * h * D + l32, lane_out = 4 * h * TS + l32;
    auto cin = [&](const float* g, f32x16& acc) {       // accumulator block (mbD, cbD) from a padded fp32 [64][D] tensor
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) acc[jj] = (g + (32 * mbD + acc_row(jj, 0)) * D + 32 * cbD)[lane_in];
    };
    auto out_user = [&](void* base, const f32x16& acc) {   // ... to a user gradient, rows of existing tokens only
        TIO* g = reinterpret_cast<TIO*>(base) + ubase + 32 * mbD * TS + 32 * cbD;
        if (ntok == CHUNK) {
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) (g + acc_row(jj, 0) * TS)[lane_out] = (TIO)acc[jj];
        } else {
#pragma unroll
            for (int jj = 0; jj < 16; ++jj)
                if (32 * mbD + acc_row(jj, h) < ntok) (g + acc_row(jj, 0) * TS)[lane_out] = (TIO)acc[jj];
        }
    };

    // blocks of ddP: NA x NA on each of the waves 4..7, as the near sums left them
    const bool actP = wv >= 4;
    const int rb = (wv >> 1) & 1, kb = wv & 1;
    f32x16 accV = zero16(), accQ, accK = zero16();
    // (d = 64: waves 0..3 and 4..7 hold different things, and two workgroups per CU leave 128 registers: one place for dQ / dY)
    f32x16 y_own;
    f32x16& accY = D == 64 ? accQ : y_own;

    // ---- the second level's share: ddP -= R^T D, dKb += dKb2 R (D = gradient of R_{c-1}); dV, dKb change hands ----
    GTile<TIO, 64, D> tW, tdO, tV;
    if constexpr (!C::NEAR_SUMS) {
        tW.load(wg, TS, ntok, tid);
        tdO.load(dog, TS, ntok, tid);
        tV.load(vg, TS, ntok, tid);
        if (actD) { cin(a.dvp + pbase, accV); cin(a.dkb + pbase, accK); }
        if (actP) {
            const float* g = a.ddp + ((size_t)bh * NC + chunk) * D * D;
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {
                const f32x4 v4 = *reinterpret_cast<const f32x4*>(g + (size_t)(32 * rb + l32) * D + 32 * kb + 8 * gg + 4 * h);
#pragma unroll
                for (int r = 0; r < 4; ++r) dd[0][0][4 * gg + r] = v4[r];
            }
        }
    } else {
        constexpr int DS = D / 16;
        typedef typename Tr<T>::Frag Frag;
        using N = NearCfg<TIO, D>;
        const T *sR = reinterpret_cast<const T*>(smem + C::SR), *sD = reinterpret_cast<const T*>(smem + C::SD);
        T* sK2 = reinterpret_cast<T*>(smem + C::SK2);
        float* x = reinterpret_cast<float*>(smem + C::XCH);
        GTile<float, 64, D> tK2;
        f32x16 far = zero16();
        if (right) {
            tK2.load(a.dk2 + ((size_t)bh * NC + chunk) * CHUNK * D, D, 64, tid);
            if (actD) cin(a.dvp + pbase, far);
        }
        tW.load(wg, TS, ntok, tid);
        tdO.load(dog, TS, ntok, tid);
        tV.load(vg, TS, ntok, tid);
        if (FOX) {           // summed over the half-waves here and over the two query halves through LDS
            ncol += __shfl_xor(ncol, 32);
            if (wv < 4 && (wv >> 1) == 1 && h == 0) nearcol[32 * (wv & 1) + l32] = ncol;
        }
        lds_barrier();                                    // the last hand-over buffer has been read
        if (FOX && wv < 2 && h == 0) nearcol[32 * wv + l32] += ncol;
        if (actP) {
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v4, k4;
#pragma unroll
                    for (int r = 0; r < 4; ++r) { v4[r] = nV[i][4 * g + r]; k4[r] = a.scale * nK[i][4 * g + r]; }
                    float* y = x + (32 * kb + l32) * N::LDX + 32 * (NA * rb + i) + 8 * g + 4 * h;
                    *reinterpret_cast<f32x4*>(y + N::XV) = v4;
                    *reinterpret_cast<f32x4*>(y + N::XK) = k4;
                }
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int b = 0; b < NA; ++b)
#pragma unroll
                    for (int jj = 0; jj < 16; ++jj) dd[i][b][jj] = chunk >= 1 ? -dd[i][b][jj] : 0.f;      // (chunk 0 has no transform to the left of it)
        }
        if (right) tK2.template store<T, false>(sK2, LDD, tid);
        wait_async_and_sync();
        if (actD) {
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) {
                const int r = (32 * mbD + acc_row(jj, h)) * N::LDX + 32 * cbD + l32;
                accV[jj] = x[N::XV + r] + far[jj];
                accK[jj] = x[N::XK + r];
            }
        }
        if (right) {
            if (actP) {
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int b = 0; b < NA; ++b) {
                        f32x16 acc = zero16();
#pragma unroll
                        for (int s0 = 0; s0 < DS; s0 += 4) {
                            Frag fa[4], fb[4];
#pragma unroll
                            for (int s = 0; s < 4; ++s) { fa[s] = ld_tile_frag_tr<T, DS>(sR, s0 + s, NA * rb + i, l32, h); fb[s] = ld_tile_frag_tr<T, DS>(sD, s0 + s, NA * kb + b, l32, h); }
#pragma unroll
                            for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(fb[s], fa[s], acc);
                        }
#pragma unroll
                        for (int jj = 0; jj < 16; ++jj) dd[i][b][jj] -= acc[jj];
                    }
            }
            if (actD) {
                typedef typename Tr<T>::Vec4 TVec4;
                f32x16 acc = zero16();
#pragma unroll
                for (int s0 = 0; s0 < DS; s0 += 4) {
                    Frag fa[4], fb[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const T* kp = sK2 + (32 * mbD + l32) * LDD + 16 * (s0 + s) + 4 * h;        // contraction index in accumulator order
                        const TVec4 lo = *reinterpret_cast<const TVec4*>(kp), hi = *reinterpret_cast<const TVec4*>(kp + 8);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { fa[s][e] = lo[e]; fa[s][4 + e] = hi[e]; }
                        fb[s] = ld_tile_frag_tr<T, DS>(sR, s0 + s, cbD, l32, h);
                    }
#pragma unroll
                    for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(fa[s], fb[s], acc);
                }
#pragma unroll
                for (int jj = 0; jj < 16; ++jj) accK[jj] += acc[jj];
            }
        }
        __syncthreads();
    }

    const TileLanes tl(tid);

    // ---- stage W, dO, V; per-token scalars ---------------------------------------------------
    if (tid < CHUNK) {
        beta_s[tid] = tid < ntok ? (float)reinterpret_cast<const TIO*>(a.beta)[user_scl(a.ul, bh, chunk * CHUNK + tid)] : 0.f;
        if (FOX) { colsum[tid] = 0.f; colsum[CHUNK + tid] = 0.f; }
    }
    // the diagonal block is taken transposed (rows s = keys in registers, lane = query t = 32 cb6 + l32), as the chunk
    // transform left its raw logits for the sweep
    f32x4 sd[4];
    const int tq = 32 * cb6 + l32;
    float lse_t = 0.f, delta_t = 0.f;
    if (act6) {
#pragma unroll
        for (int g = 0; g < 4; ++g) sd[g] = *reinterpret_cast<const f32x4*>(a.sd + (((size_t)bh * NC + chunk) * 4 + cb6 * 2 + mb6) * 1024 + (g * 64 + lane) * 4);
        if (tq < ntok) lse_t = a.lse[user_scl(a.ul, bh, chunk * CHUNK + tq)];
        delta_t = a.delta[tpad + tq];
    }
    tW.template store<T, false>(XW, tid, tl);
    tdO.template store<T, false>(X0, tid, tl);
    tV.template store<T, false>(X1, tid, tl);
    f32x16 accW = zero16();
    GTile<TIO, 64, D> tQ;
    tQ.load(qg, TS, ntok, tid);
    GTile<T, 64, 64> tY;
    tY.load(reinterpret_cast<const T*>(a.ytm) + cbase, 64, 64, tid);
    GTile<T, D, 64> tU;
    tU.load(utmg, 64, D, tid);
    __syncthreads();

    // ---- dPd = dO V^T; P, dSd (diagonal block) -> Y0 = P, Y1 = dSd, both [query][key] ----------
    if (act6) {
        f32x16 acc = zero16();
        mmt<T, D, false, D, false, D>(acc, X1, 32 * mb6, X0, 32 * cb6, tl);
        const float cum_t = FOX ? a.cum[tpad + tq] : 0.f;
        float rsum = 0.f;
        typedef typename Tr<T>::Vec4 TVec4;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int s0 = 32 * mb6 + 8 * g + 4 * h;
            f32x4 cum_s4 = {0.f, 0.f, 0.f, 0.f};
            if (FOX) cum_s4 = *reinterpret_cast<const f32x4*>(a.cum + tpad + s0);
            TVec4 p4, d4;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float P = 0.f, ds = 0.f;
                if (s0 + r <= tq && tq < ntok) {
                    float z = a.scale * sd[g][r] - lse_t;
                    if (FOX) z += (cum_t - cum_s4[r]) * 0.69314718055994530942f;     // gate sums are kept in base-2 units
                    P = __expf(z);
                    const float dz = P * (acc[4 * g + r] - delta_t);
                    ds = a.scale * dz;
                    if (FOX) { rsum += dz; atomicAdd(colsum + s0 + r, dz); }
                }
                p4[r] = (T)P;
                d4[r] = (T)ds;
            }
            *reinterpret_cast<TVec4*>(Y0 + C::TileC::at(tq, s0)) = p4;
            *reinterpret_cast<TVec4*>(Y1 + C::TileC::at(tq, s0)) = d4;
        }
        if (FOX) atomicAdd(colsum + CHUNK + tq, rsum);
    }
    if (actD) cin(a.dqb + pbase, accQ);
    __syncthreads();
    if (FOX && tid < CHUNK) {        // the diagonal block's column and row sums of the logit gradient
        a.dcol[tpad + tid] = (C::NEAR_SUMS ? nearcol[tid] + (right ? a.dcol[tpad + tid] : 0.f) : a.dcol[tpad + tid]) + colsum[tid];
        a.drow[tpad + tid] += colsum[CHUNK + tid];
    }

    // ---- dV = dV' + P^T dO ---------------------------------------------------------------------
    if (actD) {
        mmt<T, 64, true, 64, true, D>(accV, Y0, 32 * mbD, X0, 32 * cbD, tl);
        out_user(a.dv, accV);
    }
    __syncthreads();                 // dO (X0), V (X1), P (Y0) are free
    tQ.template store<T, false>(X0, tid, tl);
    tY.template store<T, true>(Y0, tid, tl);          // -Y^T as stored ([r][s])
    if (actD) {
        f32x16 neg;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) neg[jj] = -accQ[jj];
        st_block<T, D>(X1, 32 * mbD, 32 * cbD, neg, tl);                // -dQb
        st_block<T, D>(X3, 32 * mbD, 32 * cbD, accK, tl);               // dKb
    }
    tU.template store<T, false>(X2, tid, tl);         // U as stored: [feature][token]
    GTile<TIO, 64, D> tK;
    tK.load(kg, TS, ntok, tid);
    GTile<T, 64, 64> tF;
    tF.load(reinterpret_cast<const T*>(a.fm) + cbase, 64, 64, tid);
    __syncthreads();

    // ---- dK = dKb + dSd^T Q (kept open);  dF = tril(-dSd Y^T - dQb U^T) -> Y2 --------------------
    if (actD) mmt<T, 64, true, 64, true, D>(accK, Y1, 32 * mbD, X0, 32 * cbD, tl);
    if (act6) {
        f32x16 acc = zero16();
        mmt<T, 64, true, 64, false, 64>(acc, Y0, 32 * cb6, Y1, 32 * mb6, tl);
        mmt<T, D, true, 64, false, D>(acc, X2, 32 * cb6, X1, 32 * mb6, tl);
#pragma unroll
        for (int jj = 0; jj < 16; ++jj)
            if (32 * cb6 + acc_row(jj, h) > 32 * mb6 + l32) acc[jj] = 0.f;
        st_block_t<T, 64>(Y2, 32 * mb6, 32 * cb6, acc, tl);
    }
    __syncthreads();

    // ---- dW = dF^T Q - Y dKb (kept open) ----------------------------------------------------------
    if (actD) {
        mmt<T, 64, true, 64, true, D>(accW, Y2, 32 * mbD, X0, 32 * cbD, tl);
        mmt<T, 64, true, 64, true, D>(accW, Y0, 32 * mbD, X3, 32 * cbD, tl);
    }
    __syncthreads();                 // Q (X0) and Y (Y0) are free
    tK.template store<T, false>(X0, tid, tl);
    tF.template store<T, false>(Y0, tid, tl);
    GTile<T, 64, 64> tN, tG;
    tN.load(reinterpret_cast<const T*>(a.nm) + cbase, 64, 64, tid);
    tG.load(reinterpret_cast<const T*>(a.gktm) + cbase, 64, 64, tid);
    __syncthreads();

    // ---- dQ = dQb + dSd K + dF W;  dY = -(F^T dSd + W dKb^T) ----------------------------------------
    if (actD) {
        mmt<T, 64, false, 64, true, D>(accQ, Y1, 32 * mbD, X0, 32 * cbD, tl);
        mmt<T, 64, false, 64, true, D>(accQ, Y2, 32 * mbD, XW, 32 * cbD, tl);
        out_user(a.dq, accQ);
    }
    if (act6) {
        accY = zero16();
        mmt<T, 64, true, 64, true, 64>(accY, Y1, 32 * cb6, Y0, 32 * mb6, tl);
        mmt<T, D, false, D, false, D>(accY, X3, 32 * cb6, XW, 32 * mb6, tl);
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) accY[jj] = -accY[jj];
    }
    GTile<T, 64, 64> tA;
    tA.load(reinterpret_cast<const T*>(a.aim) + cbase, 64, 64, tid);
    tK.load(kg, TS, ntok, tid);       // K once more, for dGk K at the end
    __syncthreads();                 // K (X0), dKb (X3), dSd (Y1), dF (Y2) are free
    if (act6) st_block_t<T, 64>(Y2, 32 * mb6, 32 * cb6, accY, tl);     // dY
    if (actP) {                      // ddP [a][b] (d = 128: spans X0 and X3)
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int b = 0; b < NA; ++b) st_block_t<T, D>(X0, 32 * (NA * rb + i), 32 * (NA * kb + b), dd[i][b], tl);
    }
    tN.template store<T, false>(YN, tid, tl);
    tG.template store<T, false>(Y1, tid, tl);
    __syncthreads();

    // ---- dU = -F^T dQb + W ddP;  dW += U ddP^T ---------------------------------------------------
    f32x16 accU = zero16();
    if (actD) {
        mmt<T, 64, true, D, true, 64>(accU, X1, 32 * cbD, Y0, 32 * mbD, tl);
        mmt<T, D, true, D, false, D>(accU, X0, 32 * cbD, XW, 32 * mbD, tl);
        mmt<T, D, true, 64, false, D>(accW, X2, 32 * mbD, X0, 32 * cbD, tl);
    }
    __syncthreads();                 // every wave is done with dQb (X1), U (X2)
    if (actD) st_block_t<T, D>(X1, 32 * mbD, 32 * cbD, accU, tl);       // dU [token][feature]
    tK.template store<T, false>(X2, tid, tl);
    __syncthreads();

    // ---- dW += N^T dU;  dN = dY Gk^T + dU W^T -> Y0 ------------------------------------------------
    if (actD) mmt<T, 64, true, 64, true, D>(accW, YN, 32 * mbD, X1, 32 * cbD, tl);
    if (act6) {
        f32x16 acc = zero16();
        mmt<T, 64, true, 64, false, 64>(acc, Y1, 32 * cb6, Y2, 32 * mb6, tl);
        mmt<T, D, false, D, false, D>(acc, XW, 32 * cb6, X1, 32 * mb6, tl);
        st_block_t<T, 64>(Y0, 32 * mb6, 32 * cb6, acc, tl);
    }
    __syncthreads();                 // dN visible; Gk (Y1) is free

    // ---- dGk = sl(N^T dY) -> Y1 ----------------------------------------------------------------------
    if (act6) {
        f32x16 acc = zero16();
        mmt<T, 64, true, 64, true, 64>(acc, Y2, 32 * cb6, YN, 32 * mb6, tl);
#pragma unroll
        for (int jj = 0; jj < 16; ++jj)
            if (32 * cb6 + acc_row(jj, h) >= 32 * mb6 + l32) acc[jj] = 0.f;
        st_block_t<T, 64>(Y1, 32 * mb6, 32 * cb6, acc, tl);
    }
    __syncthreads();                 // dY (Y2) is free
    tA.template store<T, false>(Y2, tid, tl);
    __syncthreads();

    // ---- R = A^-T dN -> X1 (operand) and its diagonal (fp32) ----------------------------------------
    if (act6) {
        f32x16 acc = zero16();
        mmt<T, 64, true, 64, true, 64>(acc, Y0, 32 * cb6, Y2, 32 * mb6, tl);
        st_block_t<T, 64>(X1, 32 * mb6, 32 * cb6, acc, tl);
        if (mb6 == cb6) {
#pragma unroll
            for (int jj = 0; jj < 16; ++jj)
                if (acc_row(jj, h) == l32) rdiag[32 * mb6 + l32] = acc[jj];
        }
    }
    __syncthreads();

    // ---- M = sl(-R N^T);  dGs = diag(beta) M + (diag(beta) M)^T -> Y2;  row sums of M o G for dbeta ----------------
    if (act6 && mb6 >= cb6) {
        f32x16 acc = zero16(), gacc = zero16();           // rows n, lane m
        mmt<T, 64, false, 64, false, 64>(acc, YN, 32 * cb6, X1, 32 * mb6, tl);
        mmt<T, D, false, D, false, D>(gacc, XW, 32 * cb6, XW, 32 * mb6, tl);          // G = W W^T, as the transform forms it
        const int m = 32 * mb6 + l32;
        const float bm = beta_s[m];
        float mv[16], mg[16];
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            mv[jj] = (32 * cb6 + acc_row(jj, h) >= m) ? 0.f : -acc[jj];
            mg[jj] = gacc[jj] * mv[jj];
        }
        {       // the row's sum by halves, columns 16 apart first; products are rounded before they are added
#pragma clang fp contract(off)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) mg[jj] = mg[jj] + mg[jj + 8];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                mg[jj] = mg[jj] + mg[jj + 4];
                mg[jj] = mg[jj] + __shfl_xor(mg[jj], 32);
            }
            const float sum = (mg[0] + mg[2]) + (mg[1] + mg[3]);
            if (h == 0) rowsum[cb6 * CHUNK + m] = sum;
        }
        // left of the diagonal beta M is rounded once, its mirror image to 32 bits first
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 m4 = {mv[4 * g], mv[4 * g + 1], mv[4 * g + 2], mv[4 * g + 3]};
            const f32x4 b4 = {bm, bm, bm, bm};
            if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4*>(Y2 + C::TileC::at(m, 32 * cb6 + 8 * g + 4 * h)) = b4 * m4;
            else lds_write(lds_addr(Y2) + tl.of<64>().vec_at(32 * mb6, 32 * cb6 + 8 * g), mul_once(m4, b4));
        }
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            const int n = 32 * cb6 + acc_row(jj, h);
            float bmv = bm * mv[jj];
            asm("" : "+v"(bmv));
            if (n < m) Y2[C::TileC::at(n, m)] = (T)bmv;
        }
    }
    __syncthreads();

    // ---- dbeta -----------------------------------------------------------------------------------------------------
    if (tid < ntok)
        reinterpret_cast<TIO*>(a.dbeta)[user_scl(a.ul, bh, chunk * CHUNK + tid)] = (TIO)(rowsum[tid] + (tid >= 32 ? rowsum[CHUNK + tid] : 0.f) + rdiag[tid]);

    // ---- dK += dGk^T W;  dW += dGs W + dGk K ------------------------------------------------------------
    if (actD) {
        mmt<T, 64, true, 64, true, D>(accK, Y1, 32 * mbD, XW, 32 * cbD, tl);
        out_user(a.dk, accK);
        mmt<T, 64, false, 64, true, D>(accW, Y2, 32 * mbD, XW, 32 * cbD, tl);
        mmt<T, 64, false, 64, true, D>(accW, Y1, 32 * mbD, X2, 32 * cbD, tl);
        out_user(a.dw, accW);
    }
}

template <typename TIO, int D, bool FOX, bool STRIDED>
hipError_t launch_s(const ChunkFusedArgs& a, int BH, hipStream_t st) {
    using C = CaCfg<TIO, D>;
    // set once per process; a function-local static is initialised under the language's own lock
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&chunk_fused_kernel<TIO, D, FOX, STRIDED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::TOTAL);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((chunk_fused_kernel<TIO, D, FOX, STRIDED>), dim3(super_block_grid(a.NC, BH)), dim3(CA_NT), (size_t)C::TOTAL, st, a);
    return hipGetLastError();
}
template <typename TIO, int D, bool FOX>
hipError_t launch_t(const ChunkFusedArgs& a, int BH, hipStream_t st) {
    return a.ul.vt != D ? launch_s<TIO, D, FOX, true>(a, BH, st) : launch_s<TIO, D, FOX, false>(a, BH, st);
}


// ---------------------------------------------------------------------------------------
// The chain of the second blocking level's adjoint (Kb2_c = Kb_c R_c^T, R_{c-1} = R_c P_c with R_last = I,
// P_superblock = R_{first-1}; P_c = I - dP_c, dP_c = W_c^T U_c): with G the gradient of R_{c-1}, starting from the
// gradient of P_superblock (far key-side kernel), chunks first .. last,
//     G <- G - (G U_c^T) W_c + dKb2_c^T Kb_c .
// G before chunk c is left as a tile; what it is for -- ddP_c -= R_c^T G, dKb_c += dKb2_c R_c -- the chunk-transform
// adjoint does, where ddP_c and dKb_c are read anyway.  The rows of G do not depend on each other: a wave keeps 32 of
// them, transposed, in accumulator registers (lane = row), its operand copy is those registers packed, and the only
// thing the waves share is the tiles of U, W and Kb, fetched one chunk ahead.
// What bounds it: memory (112 KB per chunk at d = 128), and the chain's latency when there are few heads.  (At d = 128 it keeps
// 8 to 14 registers in scratch: two workgroups per CU leave 256.)  As one
// workgroup of eight waves that exchanged G through LDS and updated ddP and dKb in memory itself (304 KB per chunk)
// it took 0.50 ms at B=4, H=16, L=8192, d=128.
template <typename TIO, int D> struct SbCfg {
    typedef typename Compute<TIO>::type T;
    static constexpr int NT = 64 * (D / 32);                          // one wave per 32 rows of G
    static constexpr int LDD = D + 8, LDC = CHUNK + 8;
    static constexpr int U_ = 0, W_ = D * LDC * 2, KB = W_ + 64 * LDD * 2, TOTAL = KB + 64 * D * 2;    // bytes: U | W | Kb tile
};

template <typename TIO, int D, bool STRIDED>
__global__ __launch_bounds__((SbCfg<TIO, D>::NT), 2) void sb_chain_kernel(SbChainArgs a) {
    using C = SbCfg<TIO, D>;
    typedef typename C::T T;
    using Frag = typename Tr<T>::Frag;
    constexpr int LDD = C::LDD, LDC = C::LDC, DB = D / 32, DS = D / 16, NT = C::NT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T* sU = reinterpret_cast<T*>(smem + C::U_);       // U_c as stored: [feature][token]
    T* sW = reinterpret_cast<T*>(smem + C::W_);       // W_c [t][b]
    T* sKb = reinterpret_cast<T*>(smem + C::KB);      // Kb_c, a tile (rows s, contraction b)

    const int J = blockIdx.x, bh = blockIdx.y, NC = a.NC;           // NC: chunks per head in the workspace arrays
    const int L = seq_len(a.ul, bh, a.L), NCo = (L + CHUNK - 1) / CHUNK, nsb = (NC + SBC - 1) / SBC;   // this head's own length and chunks
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int c0 = J * SBC;
    if (is_last_sb(J, NCo)) return;                   // no gradient arrives there (packed batch: a shorter sequence has fewer super-blocks)
    const int TS = STRIDED ? (int)a.ul.vt : D;        // token stride of W

    f32x16 G[DB];                                     // G^T: rows b, lane = row a = 32 wv + l32
    {
        const float* src = a.dchain + (((size_t)bh * nsb + J) * D + 32 * wv + l32) * D + 4 * h;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 v4 = *reinterpret_cast<const f32x4*>(src + 32 * b + 8 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) G[b][4 * g + r] = v4[r];
            }
    }
    GTile<T, D, 64, NT> tU;
    GTile<TIO, 64, D, NT> tW;
    Frag tKb[64 * D / 8 / NT];
    auto fetch = [&](int c) {
        const size_t bhc = (size_t)bh * NC + c;
        tU.load(reinterpret_cast<const T*>(a.utm) + bhc * D * CHUNK, 64, D, tid);
        tW.load(reinterpret_cast<const TIO*>(a.w) + user_vec(a.ul, bh, (long long)c * CHUNK), TS, 64, tid);     // (a whole chunk: not the head's last)
        const Frag* kg = reinterpret_cast<const Frag*>(reinterpret_cast<const T*>(a.kt) + bhc * CHUNK * D);
#pragma unroll
        for (int u = 0; u < 64 * D / 8 / NT; ++u) tKb[u] = kg[tid + u * NT];
    };
    fetch(c0);
    for (int c = c0; ; ++c) {
        Frag Gb[DS];
#pragma unroll
        for (int b = 0; b < DB; ++b) pack_block<T>(G[b], Gb + 2 * b);
        Frag* dst = reinterpret_cast<Frag*>(reinterpret_cast<T*>(a.dr) + ((size_t)bh * NC + c) * D * D) + (size_t)wv * DS * 64;
#pragma unroll
        for (int s = 0; s < DS; ++s) __builtin_nontemporal_store(Gb[s], &dst[s * 64 + tile_lane<T>(lane, s)]);
        if (c == c0 + SBC - 1) break;
        __syncthreads();                              // the previous chunk's reads are done
        tU.template store<T, false>(sU, LDC, tid);
        tW.template store<T, false>(sW, LDD, tid);
#pragma unroll
        for (int u = 0; u < 64 * D / 8 / NT; ++u) reinterpret_cast<Frag*>(sKb)[tid + u * NT] = tKb[u];
        float k2[32];                                 // dKb2_c[s][a], s = 16 i + acc_row(e, h): needed after T1
        const float* kp = a.dk2 + (((size_t)bh * NC + c) * CHUNK + 4 * h) * D + 32 * wv + l32;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) k2[8 * i + e] = kp[(16 * i + acc_row(e, 0)) * D];
        __syncthreads();
        // T1^T[t][a] = -sum_k U[t][k] G[a][k]
        Frag t1[4];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            f32x16 acc = zero16();
#pragma unroll
            for (int s0 = 0; s0 < DS; s0 += 4) {
                Frag f[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) f[s] = ld_frag_tr_acc<T>(sU, LDC, 16 * (s0 + s), 32 * tb, l32, h);
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = Tr<T>::mma(f[s], Gb[s0 + s], acc);
            }
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) acc[jj] = -acc[jj];
            pack_block<T>(acc, t1 + 2 * tb);
        }
        if (c + 1 < c0 + SBC - 1) fetch(c + 1);
        Frag kf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) kf[i][e] = (T)k2[8 * i + e];
        // G^T += W^T T1^T + Kb^T dKb2
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            Frag f[4], k[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) { k[s] = ld_tile_frag_tr<T, DS>(sKb, s, b, l32, h); f[s] = ld_frag_tr_acc<T>(sW, LDD, 16 * s, 32 * b, l32, h); }
#pragma unroll
            for (int s = 0; s < 4; ++s) G[b] = Tr<T>::mma(k[s], kf[s], G[b]);
#pragma unroll
            for (int s = 0; s < 4; ++s) G[b] = Tr<T>::mma(f[s], t1[s], G[b]);
        }
    }
}

template <typename TIO, int D, bool STRIDED>
hipError_t launch_sb_s(const SbChainArgs& a, int BH, hipStream_t st) {
    using C = SbCfg<TIO, D>;
    // set once per process; a function-local static is initialised under the language's own lock
    static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&sb_chain_kernel<TIO, D, STRIDED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::TOTAL);
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((sb_chain_kernel<TIO, D, STRIDED>), dim3((a.NC + SBC - 1) / SBC - 1, BH), dim3(C::NT), (size_t)C::TOTAL, st, a);      // (NC > SBC)
    return hipGetLastError();
}
template <typename TIO, int D>
hipError_t launch_sb_t(const SbChainArgs& a, int BH, hipStream_t st) {
    return a.ul.vt != D ? launch_sb_s<TIO, D, true>(a, BH, st) : launch_sb_s<TIO, D, false>(a, BH, st);
}

}  // namespace

hipError_t launch_bwd_sb_chain(const SbChainArgs& a, int BH, int d, hipStream_t st) {
    return d == 64 ? launch_sb_t<bf16_t, 64>(a, BH, st) : launch_sb_t<bf16_t, 128>(a, BH, st);
}

hipError_t launch_chunk_fused(const ChunkFusedArgs& a, int BH, int d, int is_bf16, hipStream_t st) {
    const bool fox = a.cum != nullptr;
    if (!is_bf16) return fox ? launch_t<float, 64, true>(a, BH, st) : launch_t<float, 64, false>(a, BH, st);
    if (d == 64) return fox ? launch_t<bf16_t, 64, true>(a, BH, st) : launch_t<bf16_t, 64, false>(a, BH, st);
    return fox ? launch_t<bf16_t, 128, true>(a, BH, st) : launch_t<bf16_t, 128, false>(a, BH, st);
}

}  // namespace path
