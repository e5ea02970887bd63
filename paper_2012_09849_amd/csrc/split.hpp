// Tile kernel for binary32 problems on the bfloat16 matrix instruction: gemm.hpp's contractions with operands cut into
// pieces (see Pieces there), for the same problem structs.
//
// As in gemm.hpp a workgroup's operand tiles go global -> registers -> LDS -> matrix instruction, cut into pieces on the way
// into LDS (5.5 vector instructions an operand, 6 bytes of LDS an operand).  What bounds it: with six matrix instructions
// per 16 k and 32x32 tile the cutting and the LDS traffic take about as long as the products, and in one wavefront they
// add up; several workgroups per compute unit overlap them.  Hence small tiles (64x64, four wavefronts, 30 KB of LDS) and
// no second LDS buffer.  Measured, conv2 forward / weight gradient / input gradient at 1024 rows of 84x84 frames (200 rows):
// 50 / 71 / 72 us (15 / 17 / 20) so, 50 / 81 / 123 (17 / 22 / 37) with 8 wavefronts on 128-row tiles and two LDS buffers,
// the cutting placed between the matrix instructions; 61 / 89 / 90 (26 / 26 / 30 at 256 rows) on the binary32 instruction.
#pragma once
#include "gemm.hpp"

namespace hts {

// k-tiles of loads in flight in registers: two, or `static constexpr int SPLIT_DEPTH = 1` for problems whose gathers cost many
// registers (weight gradients: 71 against 83 us)
template <class P, class = void> struct SplitDepth { static constexpr int value = 2; };
template <class P> struct SplitDepth<P, std::void_t<decltype(P::SPLIT_DEPTH)>> { static constexpr int value = P::SPLIT_DEPTH; };

// workgroup barrier that orders LDS accesses only (__syncthreads() would also wait for the loads in flight)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class P>
__global__ __launch_bounds__(P::WAVES_M * P::WAVES_N * 64) void gemm_split_kernel(const P p)
{
    const int zb = blockIdx.z, M = rows_of(p, zb);
    constexpr int BM = P::BM, BN = P::BN, BK = P::BK, D = SplitDepth<P>::value;
    constexpr int WM = P::WAVES_M, WN = P::WAVES_N, NT = WM * WN * 64;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int LS = BK + 8;                           // row pitch 80 bytes: 16-byte aligned, 16 rows on 16 different bank groups
    constexpr int VA = P::VA, VB = P::VB, NPA = PiecesA<P>::value, NPB = PiecesB<P>::value;
    constexpr bool NAT_A = !P::A_ALONG_K, NAT_B = !P::B_ALONG_K;
    constexpr int LSNA = BM + (BM % 64 == 0 ? 32 : 0), LSNB = BN + (BN % 64 == 0 ? 32 : 0);
    constexpr int CA = NAT_A ? BK * (BM / VA) : BM * BK / VA, CB = NAT_B ? BK * (BN / VB) : BN * BK / VB;
    constexpr int NA = (CA + NT - 1) / NT, NB = (CB + NT - 1) / NT;        // vectors per thread
    constexpr int PLA = NAT_A ? BK * LSNA : BM * LS, PLB = NAT_B ? BK * LSNB : BN * LS;     // elements of one piece's tile
    constexpr int SEG = SegOf<P>::value, GROUP = GroupOf<P>::value;
    constexpr bool SWAP = OwnsRow<P>::value;
    static_assert(sizeof(typename P::T) == 4 && !F32Mfma<P>::value && BK == 32 && SEG % BK == 0 && (GROUP == 0 || GROUP % SEG == 0), "binary32 problem");
    static_assert(TM >= 1 && TN >= 1 && TM * 32 * WM == BM && TN * 32 * WN == BN && BM % VA == 0 && BN % VB == 0, "tile shape");
    __shared__ __attribute__((aligned(16))) bf16_t As[NPA * PLA];
    __shared__ __attribute__((aligned(16))) bf16_t Bs[NPB * PLB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM, lrow = lane & 31, lk = lane >> 5;
    int m0, n0, z;
    if (!tile_of(p, M, m0, n0, z)) return;       // the whole workgroup leaves
    const int kbeg = z * p.klen;
    const int kend = min(p.K, kbeg + p.klen);

    // fixed assignment of operand vectors to threads (spare threads repeat others' vectors); the row part of every gather is resolved once
    typename P::CtxA ca[NA];
    typename P::CtxB cb[NB];
    int ka[NA], kb[NB], la[NA], lb[NB];          // k offset inside the tile, LDS offset
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int id = CA % NT == 0 ? tid + i * NT : (tid + i * NT) % CA;
        const int r = NAT_A ? (id % (BM / VA)) * VA : id / (BK / VA);
        ka[i] = NAT_A ? id / (BM / VA) : (id % (BK / VA)) * VA;
        la[i] = NAT_A ? ka[i] * LSNA + r : r * LS + ka[i];
        ca[i] = make_ctx_a(p, m0 + r, zb);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int id = CB % NT == 0 ? tid + i * NT : (tid + i * NT) % CB;
        const int r = NAT_B ? (id % (BN / VB)) * VB : id / (BK / VB);
        kb[i] = NAT_B ? id / (BN / VB) : (id % (BK / VB)) * VB;
        lb[i] = NAT_B ? kb[i] * LSNB + r : r * LS + kb[i];
        cb[i] = make_ctx_b(p, n0 + r, zb);
    }
    const int ntiles = (kend - kbeg + BK - 1) / BK;
    Vec<float, VA> ra[D][NA];
    Vec<float, VB> rb[D][NB];
    // (a tile behind the last one fetches the last one again and is never used: loads stay unconditional)
    auto fetch = [&](int t, Vec<float, VA> (&xa)[NA], Vec<float, VB> (&xb)[NB]) {
        const int k0 = kbeg + min(t, ntiles - 1) * BK;
#pragma unroll
        for (int i = 0; i < NA; ++i) xa[i] = tile_load_a(p, ca[i], k0, ka[i], kend);
#pragma unroll
        for (int i = 0; i < NB; ++i) xb[i] = tile_load_b(p, cb[i], k0, kb[i], kend);
    };
    auto cut = [&](const Vec<float, VA> (&xa)[NA], const Vec<float, VB> (&xb)[NB]) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            Vec<bf16_t, VA> pc[NPA];
            to_pieces<float, VA>(xa[i], pc);
#pragma unroll
            for (int q = 0; q < NPA; ++q) *reinterpret_cast<Vec<bf16_t, VA> *>(As + q * PLA + la[i]) = pc[q];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            Vec<bf16_t, VB> pc[NPB];
            to_pieces<float, VB>(xb[i], pc);
#pragma unroll
            for (int q = 0; q < NPB; ++q) *reinterpret_cast<Vec<bf16_t, VB> *>(Bs + q * PLB + lb[i]) = pc[q];
        }
    };
    // (lane layouts of the operand reads: see gemm.hpp)
    const int nat_k = 8 * (lane >> 5) + ((lane & 15) >> 2), nat_row = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const int a_off = NAT_A ? wm * TM * 32 + nat_k * LSNA + nat_row : (wm * TM * 32 + lrow) * LS + 8 * lk;
    const int b_off = NAT_B ? wn * TN * 32 + nat_k * LSNB + nat_row : (wn * TN * 32 + lrow) * LS + 8 * lk;
    auto read_a = [&](int pc, int i, int kk) {
        const bf16_t *q = As + pc * PLA + a_off;
        if constexpr (NAT_A) return tr8(q + kk * LSNA + i * 32, LSNA);
        else return *reinterpret_cast<const bf16x8 *>(q + i * 32 * LS + kk);
    };
    auto read_b = [&](int pc, int j, int kk) {
        const bf16_t *q = Bs + pc * PLB + b_off;
        if constexpr (NAT_B) return tr8(q + kk * LSNB + j * 32, LSNB);
        else return *reinterpret_cast<const bf16x8 *>(q + j * 32 * LS + kk);
    };
    f32x16 acc[TM][TN], small[TM][TN];           // the segment's sums of the p0 q0 products and of the small ones
    auto clear = [&](f32x16 (&x)[TM][TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) x[i][j][r] = 0.0f;
    };
    auto add = [&](f32x16 (&x)[TM][TN], const f32x16 (&y)[TM][TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) x[i][j] += y[i][j];
    };
    clear(acc);
    clear(small);
    f32x16 seg_tot[SEG > 0 ? TM : 1][SEG > 0 ? TN : 1], grp_tot[GROUP > 0 ? TM : 1][GROUP > 0 ? TN : 1];
    if constexpr (SEG > 0) clear(seg_tot);
    if constexpr (GROUP > 0) clear(grp_tot);

    auto close = [&](int t) {                    // end of a segment (and group): fixed places in k, so every kernel adds alike
        if constexpr (SEG > 0) {
            if ((t + 1) % (SEG / BK) == 0 || t + 1 == ntiles) {
                add(acc, small);
                add(seg_tot, acc);
                clear(acc);
                clear(small);
                if constexpr (GROUP > 0) {
                    if ((t + 1) % (GROUP / BK) == 0 || t + 1 == ntiles) { add(grp_tot, seg_tot); clear(seg_tot); }
                }
            }
        }
    };
    auto step = [&](int t, Vec<float, VA> (&xa)[NA], Vec<float, VB> (&xb)[NB]) {
        cut(xa, xb);
        lds_barrier();
        fetch(t + D, xa, xb);
        bf16x8 av[NPA][2][TM], bv[NPB][2][TN];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int pc = 0; pc < NPA; ++pc)
#pragma unroll
                for (int i = 0; i < TM; ++i) av[pc][h][i] = read_a(pc, i, 16 * h);
#pragma unroll
            for (int pc = 0; pc < NPB; ++pc)
#pragma unroll
                for (int j = 0; j < TN; ++j) bv[pc][h][j] = read_b(pc, j, 16 * h);
        }
        for_piece_pairs<NPA, NPB>([&](auto pa, auto pb, auto is_small) {
            constexpr int ia = decltype(pa)::value, ib = decltype(pb)::value;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        f32x16 &d = decltype(is_small)::value ? small[i][j] : acc[i][j];
                        d = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[ib][h][j], av[ia][h][i], d, 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[ia][h][i], bv[ib][h][j], d, 0, 0, 0);
                    }
        });
        lds_barrier();
        close(t);
    };
    static_assert(D == 1 || D == 2, "depth");
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, ra[d], rb[d]);
    EpiInputs<P, TM, TN, SWAP> epi;
    if constexpr (EpiEarly<P>::value) epi_fetch(p, epi, m0, n0, M, zb, wm, wn, lane);
    int t = 0;
    for (; t + D <= ntiles; t += D) {            // (no branch between the steps: the compiler then knows which loads are in flight)
#pragma unroll
        for (int d = 0; d < D; ++d) step(t + d, ra[d], rb[d]);
    }
    if (D == 2 && t < ntiles) step(t, ra[0], rb[0]);
    if constexpr (SEG == 0) add(acc, small);
    if constexpr (GROUP > 0) epi_store(p, grp_tot, epi, m0, n0, M, z, zb, wm, wn, lane);
    else if constexpr (SEG > 0) epi_store(p, seg_tot, epi, m0, n0, M, z, zb, wm, wn, lane);
    else epi_store(p, acc, epi, m0, n0, M, z, zb, wm, wn, lane);
}

}  // namespace hts
