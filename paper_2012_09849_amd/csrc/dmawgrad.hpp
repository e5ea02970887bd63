// bfloat16 weight gradients of conv2, conv3 and FC:  D[n][col] = sum over positions m of dy[m][n] * in[m][col].
//
// Both operands lie in memory with the reduction index as their slow one, in rows of at least 64 neighbouring values.  A workgroup
// takes 64 rows of D and HALVES x 64 columns over a reduction chunk, 64 positions (a k-tile) at a time: the k-tile's rows are copied
// straight into LDS (buffer_load ... lds: eight lanes a 128-byte row, so a gather costs an address per row and no conversion),
// up to STAGES - 1 k-tiles ahead, one barrier per k-tile, and reach the matrix instruction's lane layout by the transposing LDS read.
// 16-byte slot s of LDS row r holds column vector s ^ 4 (r / 2 % 2): the four rows that sixteen lanes read at once fall into
// different banks.  The register-staged tile kernel wrote every byte to LDS from registers, computed two position decompositions per 16
// bytes and padded the bias to a tile of columns; here the bias is one more matrix instruction against ones in the wavefronts of the
// first columns.  The chunks and the order inside them are the same, and so are the bits.
// us, tile kernel -> this one (conv2, conv3, FC): 1024 rows of 84x84 frames 22.5 -> 13.7, 16.6 -> 11.6, 14.4 -> 9.0; 2048 rows of 72x96
// 34.7 -> 21.5, 21.9 -> 16.5, 25.6 -> 16.7; 16 rows of 84x84 5.7 -> 5.5, 5.6 -> 4.7, 6.0 -> 5.1.  What bounds it now: the operands' way
// into LDS (conv2 at 1024 rows: 127 MB in 13.7 us, 9.3 TB/s out of the L2s).  Not kept: 4 stages (the same time), 2 (conv2 16.4); tiles of
// 128 columns by four wavefronts (conv2 16.3, FC 11.1) or of 192 (conv3 14.0).
#pragma once
#include "dmagemm.hpp"
#include "problems.hpp"

namespace hts {

constexpr int DW_ROW = 128, DW_TILE = 64 * DW_ROW;       // bytes of a row of 64 values; of 64 of them

// A buffer as the instruction takes it, and the copy itself: written out, because the compiler makes every transposing LDS read wait
// for all copies under way (it cannot tell their tiles apart), which leaves nothing of the stages.  The copy has no result; the kernel
// waits for it before the barrier that hands the tile over.  The compiler keeps no distances to what is inside: m0, the LDS address, is
// written one wait state ahead; a buffer's words, which lane reads write, have their five wait states where they are made; the offsets come
// from scalar instructions, which need none.  (Five wait states in every copy: conv2's weight gradient 21.1 -> 21.7 us at 2048 rows of
// 72x96 frames.  A value brought back from a spill by a lane read would need them; tests/test_copy_wait_states.py finds one in the built library.)
typedef __attribute__((ext_vector_type(4))) int rsrc_words;
__device__ __forceinline__ rsrc_words copy_source(const void *p, uint32_t bytes)
{
    const unsigned long long a = (unsigned long long)p;
    rsrc_words r = {__builtin_amdgcn_readfirstlane((int)a), __builtin_amdgcn_readfirstlane((int)(a >> 32) & 0xffff), __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
    asm volatile("s_nop 4" : "+s"(r));
    return r;
}
__device__ __forceinline__ void copy16(const rsrc_words &src, uint32_t lane_off, uint32_t wave_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :: "v"(lane_off), "s"(src), "s"(wave_off), "s"(lds) : "memory", "m0");
}

// WN: wavefronts along the columns, two of them along the rows.  Conv2's eight halves go in pairs, with eight wavefronts; conv3's nine and
// FC's few one by one, for more workgroups.  block: index in the grid; tile: wgrad_dma_lds bytes of LDS.
// W offers: A_PITCH, bytes between its rows of dy; `From from(kbeg, kend, rt)`, the chunk's buffers; halves(), how many 64-column halves
// there are; outer(HALVES) and inner(HALVES): sets of workgroups, each of them on one XCD, and workgroups of a set, with
// place(outer, inner, &rt, &ct, &z); b_source(k0, From), the buffer of the k-tile from k0 on, b_row(k0, r, kend, From) and b_half(half),
// byte offsets of its row r and of a half's columns in it;
// store(n, col, value, z), store_bias(n, value, z).
template <class W, int HALVES, int STAGES, int WN> __device__ __forceinline__ void wgrad_dma_tile(const W &p, const int block, unsigned char *tile)
{
    constexpr int TN = 2 * HALVES / WN, ROWS = 32 / WN, STAGE = (1 + HALVES) * DW_TILE, PER = ROWS / 8 * (1 + HALVES);      // columns of 32 a wavefront; copies a k-tile
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w & 1, wn = w >> 1;
    const int per = p.inner(HALVES), slot = block >> 3, outer = (slot / per) * 8 + (block & 7), inner = slot - (slot / per) * per;
    if (outer >= p.outer(HALVES)) return;
    int rt, ct, z;
    p.place(outer, inner, rt, ct, z);
    const int kbeg = z * p.klen, kend = min(p.K, kbeg + p.klen), nt = (kend - kbeg + 63) / 64;
    const int h0 = ct * HALVES;

    const typename W::From from = p.from(kbeg, kend, rt);
    // copies: this lane's 16 bytes of row ROWS w + 8 i + lane / 8 of every k-tile
    const int lr = lane >> 3;
    const uint32_t src16 = 16u * (uint32_t)((lane & 7) ^ (4 * ((lr >> 1) & 1)));
    uint32_t half_off[HALVES];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) half_off[h] = p.b_half(min(h0 + h, p.halves() - 1));
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)tile;
    auto fetch = [&](int t, int s) {
        const uint32_t dst = lds0 + (uint32_t)(s * STAGE + ROWS * w * DW_ROW);
        const rsrc_words b = p.b_source(kbeg + t * 64, from);
#pragma unroll
        for (int i = 0; i < ROWS / 8; ++i) {
            const int r = ROWS * w + 8 * i + lr;
            copy16(from.a, (uint32_t)(r * W::A_PITCH) + src16, (uint32_t)(t * 64 * W::A_PITCH), dst + 8 * i * DW_ROW);
            const uint32_t row = p.b_row(kbeg + t * 64, r, kend, from) + src16;
#pragma unroll
            for (int h = 0; h < HALVES; ++h) copy16(b, row, half_off[h], dst + (1 + h) * DW_TILE + 8 * i * DW_ROW);
        }
    };
    // transposing reads: lane 4j + q of a 16-lane group points at four columns of reduction row j and receives the four rows of its column
    const int kg = lane >> 5, g1 = (lane >> 4) & 1, jj = (lane & 15) >> 2, q = lane & 3;
    auto place32 = [&](int c32) { return (uint32_t)((8 * kg + jj) * DW_ROW + 16 * ((c32 / 8 + 2 * g1 + (q >> 1)) ^ (4 * ((jj >> 1) & 1))) + 8 * (q & 1)); };
    const uint32_t a_off = place32(32 * wm);
    uint32_t b_off[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) { const int c = (wn * TN + j) * 32; b_off[j] = (uint32_t)((1 + c / 64) * DW_TILE) + place32(c % 64); }
    f32x16 acc[TN], bias;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        bias[r] = 0.0f;
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j][r] = 0.0f;
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = from_f32<bf16_t>(1.0f);
    const bool sums = ct == 0 && wn == 0;
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) if (s < nt) fetch(s, s);
    auto loop = [&](auto with_bias) {
        int s = 0;
        for (int t = 0; t < nt; ++t) {
            wait_tiles<STAGES - 2, PER>(nt - 1 - t);  // this wavefront's copies of k-tile t have landed; its reads of t - 1 are done
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (t + STAGES - 1 < nt) fetch(t + STAGES - 1, s == 0 ? STAGES - 1 : s - 1);
            const unsigned char *base = tile + s * STAGE;
            bf16x8 av[4], bv[4][TN];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                auto read = [&](uint32_t off) { return tr8(reinterpret_cast<const bf16_t *>(base + off + kk * 16 * DW_ROW), DW_ROW / 2); };
                av[kk] = read(a_off);
#pragma unroll
                for (int j = 0; j < TN; ++j) bv[kk][j] = read(b_off[j]);
            }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kk], bv[kk][j], acc[j], 0, 0, 0);
                if constexpr (decltype(with_bias)::value) bias = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kk], ones, bias, 0, 0, 0);
            }
            s = s + 1 == STAGES ? 0 : s + 1;
        }
    };
    if (sums) loop(std::true_type{}); else loop(std::false_type{});
    const int lrow = lane & 31;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int n = rt * 64 + 32 * wm + 8 * (r / 4) + 4 * kg + (r % 4);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = h0 * 64 + (wn * TN + j) * 32 + lrow;
            if (col < p.halves() * 64) p.store(n, col, acc[j][r], z);
        }
        if (sums && lrow == 0) p.store_bias(n, bias[r], z);
    }
}

template <int HALVES, int STAGES> constexpr size_t wgrad_dma_lds() { return (size_t)STAGES * (1 + HALVES) * DW_TILE; }
template <class W, int HALVES, int STAGES, int WN> __global__ __launch_bounds__(128 * WN, 2) void wgrad_dma_kernel(const W p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char tile[wgrad_dma_lds<HALVES, STAGES>()];
    wgrad_dma_tile<W, HALVES, STAGES, WN>(p, (int)blockIdx.x, tile);
}

template <class L> struct DmaConvWgrad {
    static constexpr int A_PITCH = DW_ROW;
    struct From { rsrc_words a, b; int b0; };
    ConvWgrad<bf16_t, L> w;
    int K, klen;
    explicit DmaConvWgrad(const ConvWgrad<bf16_t, L> &p) : w(p), K(p.K), klen(p.klen) {}
    HTS_HD int outer(int) const { return (K + klen - 1) / klen; }
    HTS_HD int inner(int per) const { return (halves() + per - 1) / per; }
    HTS_HD int halves() const { return L::K / 64; }
    __device__ __forceinline__ void place(int outer, int inner, int &rt, int &ct, int &z) const { rt = 0; ct = inner; z = outer; }
    // (both buffers give zeros behind the chunk: a chunk's samples span less than 2 GB)
    __device__ __forceinline__ From from(int kbeg, int kend, int) const
    {
        const int b0 = w.dPo.div(kbeg);
        return {copy_source(w.dy + (long long)kbeg * 64, (uint32_t)(kend - kbeg) * DW_ROW), copy_source(w.in + (long long)b0 * w.Hin * w.Win * L::CIN, 0x80000000u), b0};
    }
    __device__ __forceinline__ rsrc_words b_source(int, const From &f) const { return f.b; }
    __device__ __forceinline__ uint32_t b_row(int k0, int r, int kend, const From &f) const
    {
        const int k = k0 + r, m = min(k, kend - 1), b = w.dPo.div(m), pos = m - b * w.Po, oy = w.dWo.div(pos), ox = pos - oy * w.Wo;
        return k < kend ? 2u * (((uint32_t)(b - f.b0) * w.Hin + oy * L::STRIDE) * w.Win + ox * L::STRIDE) * L::CIN : 0x80000000u;
    }
    __device__ __forceinline__ uint32_t b_half(int h) const
    {
        static_assert(L::KSZ * L::CIN % 64 == 0, "halves inside a tap row");
        const int u = h * 64 / (L::KSZ * L::CIN);
        return 2u * (uint32_t)(u * w.Win * L::CIN + h * 64 - u * (L::KSZ * L::CIN));
    }
    __device__ __forceinline__ void store(int n, int col, float v, int z) const { w.part[((long long)z * 64 + n) * w.N + col] = v; }
    __device__ __forceinline__ void store_bias(int n, float v, int z) const { w.part[((long long)z * 64 + n) * w.N + L::K] = v; }
};

struct DmaFcWgrad {
    static constexpr int A_PITCH = 1024;
    struct From { rsrc_words a; };
    FcWgrad<bf16_t> w;
    int K, klen;
    explicit DmaFcWgrad(const FcWgrad<bf16_t> &p) : w(p), K(p.K), klen(p.K) {}
    HTS_HD int outer(int per) const { return (halves() + per - 1) / per; }
    HTS_HD int inner(int) const { return 8; }
    HTS_HD int halves() const { return w.F / 64; }
    __device__ __forceinline__ void place(int outer, int inner, int &rt, int &ct, int &z) const { rt = inner; ct = outer; z = 0; }
    // (both buffers end with the last sample.  The activations can be more than 4 GB, 43008 rows of 256x256 frames, say: a buffer for
    // every k-tile, of at most 2 GB, as a frame of at most 2^24 values leaves at most as many features)
    __device__ __forceinline__ From from(int, int, int rt) const { return {copy_source(w.dh + rt * 64, (uint32_t)K * A_PITCH - (uint32_t)rt * DW_ROW)}; }
    __device__ __forceinline__ rsrc_words b_source(int k0, const From &) const
    {
        return copy_source(w.a3 + (long long)k0 * w.F, (uint32_t)min(K - k0, 64) * (uint32_t)w.F * 2u);
    }
    __device__ __forceinline__ uint32_t b_row(int, int r, int, const From &) const { return (uint32_t)r * (uint32_t)w.F * 2u; }
    __device__ __forceinline__ uint32_t b_half(int h) const { return (uint32_t)h * DW_ROW; }
    __device__ __forceinline__ void store(int j, int f, float v, int) const { w.g[w.fcw + (long long)j * w.F + f] = v; }
    __device__ __forceinline__ void store_bias(int j, float v, int) const { w.g[w.fcb + j] = v; }
};

template <int HALVES, class W> inline int wgrad_dma_blocks(const W &p) { return 8 * ((p.outer(HALVES) + 7) / 8) * p.inner(HALVES); }
template <int HALVES, int STAGES, int WN, class W> inline hipError_t launch_wgrad_dma(const W &p, hipStream_t stream)
{
    const int blocks = wgrad_dma_blocks<HALVES>(p);
    hipLaunchKernelGGL((wgrad_dma_kernel<W, HALVES, STAGES, WN>), dim3(blocks), dim3(128 * WN), 0, stream, p);
    return hipGetLastError();
}

}  // namespace hts
