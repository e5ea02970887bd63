// Tile kernel for bfloat16 problems whose operands are contiguous along k and need no masking, for large batches:
// gemm.hpp's contractions with the operand tiles copied from memory straight into LDS (buffer_load ... lds, 16 bytes a lane),
// up to DMA_STAGES - 1 k-tiles ahead, one barrier per k-tile.  The register-staged kernel writes every operand byte to LDS
// from registers (the slowest LDS operation), keeps one k-tile in flight and takes two barriers per k-tile; this one has
// no staging registers, so larger tiles fit, and the address of a copy is a fixed lane offset plus a scalar.  Same k order
// and segments, hence the same bits.  A lane's LDS addresses are formed once (a wavefront may be alone on its SIMD, where every vector
// instruction beside the matrix instructions counts) and a k-tile's operands are all read before its first product: FC at 4096 rows
// of 84x84 frames 28.0 -> 26.0 us, conv2 at 2048 of 72x96 23.3 -> 22.3.  Masked rows (FC's input gradient) leave through LDS as whole lines, which is
// how their masks come in: 2048 rows of 72x96 frames 18.5 -> 14.2 us, 1024 of 84x84 11.8 -> 10.0 (without any store 9.1: the rest is the masks and the
// rows, 21 MB).  What bounds it now: batches of a few hundred rows by the memory latency of the first
// k-tiles; large ones by the segments' sums (16 additions for four matrix instructions, 17.9 of FC's 26 us at 4096 rows without copies and
// reads) with the copies' way through the L1, and, conv2, by HBM (4096 rows: 147 MB in 41.5 us).  Not kept: a k-tile's operands in registers one tile
// ahead (205 registers: conv2 23.3 -> 27.6 us, FC at 4096 rows 28.9); conv2's rows through LDS as well (13.6 -> 14.1 us at 1024 rows of 84x84); 4 to 8 stages (128 KB of LDS: 6.6-7.2 us where 3
// stages take 5.5-5.8), 256-row tiles of conv2 (44 us against 41.5 at 4096 rows), 128x128 tiles of FC (11.4 against 10.4 at 1024).
#pragma once
#include "gemm.hpp"

namespace hts {

typedef __attribute__((address_space(3))) void *lds_void;

// A problem offers `int dma_k(int k0) const`: where k-tile k0 starts in an A row, in elements from ctx_a(row).p; a B row is
// contiguous.  K and klen are whole numbers of k-tiles of 64, rows start at multiples of 16 bytes, and ctx_a(row).p does not
// decrease with the row (a tile's rows are addressed from its first one with 32 bits).

// 16 bytes per lane, memory -> LDS: lane l's bytes land at dst + 16 l (dst: one address for the wavefront)
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t src, uint32_t lane_off, uint32_t wave_off, const bf16_t *dst)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void)dst, 16, (int)lane_off, (int)wave_off, 0, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_source(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// problem P on tiles of another shape
template <class P, int BM_, int BN_, int WM_, int WN_, int STAGES_, int GROUP_ = 0> struct DmaTiles : P {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = WM_, WAVES_N = WN_, DMA_STAGES = STAGES_, GROUP = GROUP_;
    explicit DmaTiles(const P &p) : P(p) {}
};

// A problem with `static constexpr bool MASKED_ROWS = true` has a row-major output [M][N] of its operand type, `T *out_rows()` (N a multiple
// of 8), that is zero where the entry of `const T *mask_rows()` is not above zero.
template <class P, class = void> struct MaskedRows : std::false_type {};
template <class P> struct MaskedRows<P, std::void_t<decltype(P::MASKED_ROWS)>> : std::integral_constant<bool, P::MASKED_ROWS> {};

// vmcnt(VM) lgkmcnt(0)
template <int VM> constexpr int wait_imm()
{
    static_assert(VM >= 0 && VM < 64, "vmcnt has six bits");
    return (VM & 15) | ((VM >> 4) << 14) | (7 << 4);
}

// waits until at most min(ahead, AHEAD) k-tiles' copies (PER a tile) of this wavefront are under way, and for its LDS reads
template <int AHEAD, int PER> __device__ __forceinline__ void wait_tiles(int ahead)
{
    if constexpr (AHEAD > 0) {
        if (ahead < AHEAD) { wait_tiles<AHEAD - 1, PER>(ahead); return; }
    }
    __builtin_amdgcn_s_waitcnt(wait_imm<AHEAD * PER>());
}

// step(t + U) for U = 0, 1, ... while there are k-tiles left
template <class Step, int... U> __device__ __forceinline__ void dma_steps(const Step &step, int t, int nt, std::integer_sequence<int, U...>)
{
    (void)((t + U < nt ? (step(t + U, std::integral_constant<int, U>{}), true) : false) && ...);
}

template <class P>
__global__ __launch_bounds__(P::WAVES_M * P::WAVES_N * 64, 2) void gemm_dma_kernel(const P p)
{
    constexpr int BM = P::BM, BN = P::BN, BK = 64, NS = P::DMA_STAGES;
    constexpr int WM = P::WAVES_M, WN = P::WAVES_N, NT = WM * WN * 64, NW = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int SEG = SegOf<P>::value, GROUP = GroupOf<P>::value;
    constexpr bool ROWS = MaskedRows<P>::value, SWAP = OwnsRow<P>::value;
    constexpr int NA = BM / 8 / NW, NB = BN / 8 / NW;          // copies of 8 rows per wavefront and k-tile
    constexpr int STAGE = (BM + BN) * BK;                       // elements
    static_assert(sizeof(typename P::T) == 2 && P::A_ALONG_K && P::B_ALONG_K && (SEG == 0 || SEG == BK) && (GROUP == 0 || GROUP % BK == 0), "problem");
    static_assert(NA * 8 * NW == BM && NB * 8 * NW == BN && TM * 32 * WM == BM && TN * 32 * WN == BN, "tile shape");
    __shared__ __attribute__((aligned(1024))) bf16_t tile[NS * STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM, lrow = lane & 31, lk = lane >> 5;
    int m0, n0, z;
    if (!tile_of(p, launch_at(), p.M, m0, n0, z)) return;       // the whole workgroup leaves
    const int kbeg = z * p.klen, nt = (min(p.K, kbeg + p.klen) - kbeg) / BK;

    // LDS rows of 64 k: 16-byte slot s of row r holds k-vector s ^ ((r >> 1) & 7), so the sixteen rows of an operand read
    // fall into different banks; a copy of 8 rows is contiguous in LDS and takes whole 128-byte lines from memory
    const bf16_t *abase = p.ctx_a(m0).p, *bbase = p.ctx_b(n0).p;
    const __amdgpu_buffer_rsrc_t ra = dma_source(abase, 0xfffffffcu), rb = dma_source(bbase, 0xfffffffcu);
    uint32_t oa[NA], ob[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = (wave * NA + i) * 8 + (lane >> 3);
        oa[i] = (uint32_t)((const char *)p.ctx_a(m0 + r).p - (const char *)abase) + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int r = (wave * NB + i) * 8 + (lane >> 3);
        ob[i] = (uint32_t)((const char *)p.ctx_b(n0 + r).p - (const char *)bbase) + 16u * ((lane & 7) ^ ((r >> 1) & 7));
    }
    auto fetch = [&](int t, int s) {
        const int k0 = kbeg + t * BK;
        const uint32_t wa = 2u * (uint32_t)p.dma_k(k0), wb = 2u * (uint32_t)k0;
#pragma unroll
        for (int i = 0; i < NA; ++i) dma16(ra, oa[i], wa, tile + s * STAGE + (wave * NA + i) * 8 * BK);
#pragma unroll
        for (int i = 0; i < NB; ++i) dma16(rb, ob[i], wb, tile + s * STAGE + BM * BK + (wave * NB + i) * 8 * BK);
    };
    // A segment is one k-tile.  Its sums are added to the running ones while the next k-tile's products are formed, hence two
    // sets of accumulators, taken in turn.
    f32x16 acc[SEG > 0 ? 2 : 1][TM][TN], tot[SEG > 0 ? TM : 1][SEG > 0 ? TN : 1], grp[GROUP > 0 ? TM : 1][GROUP > 0 ? TN : 1];
    auto clear = [&](auto &x) {
        for (auto &r : x) for (auto &c : r)
#pragma unroll
            for (int q = 0; q < 16; ++q) c[q] = 0.0f;
    };
    clear(acc[0]);
    if constexpr (SEG > 0) { clear(acc[1]); clear(tot); }
    if constexpr (GROUP > 0) clear(grp);
    auto add = [&](auto &x, const auto &y) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) x[i][j] += y[i][j];
    };
    // LDS addresses of a lane's operands, one for each 16 k; stage and tile are the instruction's offset
    typedef const bf16x8 __attribute__((address_space(3))) *lds_operand;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t *)tile;
    uint32_t ak[4], bk[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const uint32_t slot = 16u * ((2 * kk + lk) ^ ((lrow >> 1) & 7));
        ak[kk] = base + (wm * TM * 32 + lrow) * 128u + slot;
        bk[kk] = base + (BM + wn * TN * 32 + lrow) * 128u + slot;
        asm volatile("" : "+v"(ak[kk]), "+v"(bk[kk]));
    }
    EpiInputs<P, TM, TN, SWAP && !ROWS> epi;
    if constexpr (!ROWS && EpiEarly<P>::value) epi_fetch(p, epi, m0, n0, p.M, 0, wm, wn, lane);
    // ROWS: what this thread stores, and its ReLU masks: 8 columns of every (NT / VPR)-th row
    constexpr int VPR = BN / 8, PASSES = BM * VPR / NT, PITCH = BN + 8;
    static_assert(!ROWS || (SWAP && BM * VPR % NT == 0 && BM * PITCH <= NS * STAGE), "the output tile takes the place of the operands'");
    const int orow = tid / VPR, ocol = (tid % VPR) * 8;
    bf16x8 mask[ROWS ? PASSES : 1];
    if constexpr (ROWS)
#pragma unroll
        for (int q = 0; q < PASSES; ++q)
            mask[q] = *reinterpret_cast<const bf16x8 *>(p.mask_rows() + (long long)min(m0 + orow + q * (NT / VPR), p.M - 1) * p.N + min(n0 + ocol, p.N - 8));
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) if (s < nt) fetch(s, s);
    auto step = [&](int t, auto uc) {
        constexpr int U = decltype(uc)::value, S = U % NS, PAR = SEG > 0 ? U & 1 : 0;
        // this wavefront's copies of tile t have landed (later tiles' may be in flight); its reads of tile t-1 are done
        wait_tiles<NS - 2, NA + NB>(nt - 1 - t);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();               // everybody's
        asm volatile("" ::: "memory");
        if (t + NS - 1 < nt) fetch(t + NS - 1, (S + NS - 1) % NS);
        const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        bf16x8 av[4][TM], bv[4][TN];                // all of the k-tile's reads are issued before its products
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int i = 0; i < TM; ++i) av[kk][i] = *(lds_operand)(uintptr_t)(ak[kk] + (uint32_t)(S * STAGE * 2 + i * 32 * 128));
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[kk][j] = *(lds_operand)(uintptr_t)(bk[kk] + (uint32_t)(S * STAGE * 2 + j * 32 * 128));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const f32x16 &c = SEG > 0 && kk == 0 ? zero : acc[PAR][i][j];
                    acc[PAR][i][j] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv[kk][j], av[kk][i], c, 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kk][i], bv[kk][j], c, 0, 0, 0);
                }
            if constexpr (SEG > 0) if (kk == 0) add(tot, acc[1 - PAR]);
        }
        if constexpr (GROUP > 0) if (t > 0 && t % (GROUP / BK) == 0) { add(grp, tot); clear(tot); }
    };
    constexpr int UNROLL = NS % 2 ? 2 * NS : NS;
    for (int t = 0; t < nt; t += UNROLL) dma_steps(step, t, nt, std::make_integer_sequence<int, UNROLL>{});
    if constexpr (SEG > 0) { if (nt & 1) add(tot, acc[0]); else add(tot, acc[1]); }
    if constexpr (GROUP > 0) add(grp, tot);
    auto &out = [&]() -> auto & { if constexpr (GROUP > 0) return grp; else if constexpr (SEG > 0) return tot; else return acc[0]; }();
    if constexpr (ROWS) {
        // Through LDS, so that rows leave as whole lines: straight from the accumulators a lane stores 8 bytes of a row at a time, a
        // 32-column tile's instruction touches 32 lines for 16 bytes each, and so do its masks' loads.
        __syncthreads();                            // everybody's operand reads are done
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = (wn * TN + j) * 32 + 8 * g + 4 * lk;
                    Vec<bf16_t, 4> y;
#pragma unroll
                    for (int q = 0; q < 4; ++q) y[q] = from_f32<bf16_t>(out[i][j][4 * g + q]);
                    *reinterpret_cast<Vec<bf16_t, 4> *>(tile + ((wm * TM + i) * 32 + lrow) * PITCH + n) = y;
                }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PASSES; ++q) {
            const int r = orow + q * (NT / VPR);
            bf16x8 y = *reinterpret_cast<const bf16x8 *>(tile + r * PITCH + ocol);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = to_f32(mask[q][e]) > 0.0f ? y[e] : from_f32<bf16_t>(0.0f);
            if (m0 + r < p.M && n0 + ocol < p.N) *reinterpret_cast<bf16x8 *>(p.out_rows() + (long long)(m0 + r) * p.N + n0 + ocol) = y;
        }
    } else epi_store(p, out, epi, m0, n0, p.M, z, 0, wm, wn, lane);
}

template <class P> inline int dma_workgroups(const P &p, int bm, int bn) { return ((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn) * ((p.K + p.klen - 1) / p.klen); }
template <class P> inline hipError_t launch_dma(const P &p, hipStream_t stream)
{
    const int tiles = ((p.M + P::BM - 1) / P::BM) * ((p.N + P::BN - 1) / P::BN), nz = (p.K + p.klen - 1) / p.klen;
    hipLaunchKernelGGL(gemm_dma_kernel<P>, dim3(((tiles + 7) / 8) * 8, nz), dim3(P::WAVES_M * P::WAVES_N * 64), 0, stream, p);
    return hipGetLastError();
}

}  // namespace hts
