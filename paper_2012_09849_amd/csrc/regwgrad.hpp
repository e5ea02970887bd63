// binary32 weight gradients with both operands straight from memory into registers.
//
// v_mfma_f32_* does not overlap vector instructions, neither its own wavefront's nor another's: a 16x16x4 takes 32 cycles of its
// SIMD and every vector instruction beside it about 5 more (a stand-alone probe; bfloat16's hides four).  The tile kernel issues 5.3 of
// them per 64-cycle instruction of these contractions -- gather addresses, for the most part -- and reaches 60 % of the pipe.  Here a
// wavefront owns a 32 x 64 block of the gradient over a reduction chunk.  A step is four positions: lane group q of
// 16 fetches position q, lane i of it two (four) neighbouring columns of an operand, which serve two (four) 16-column tiles at
// once (tile j has columns 4i + j: the block comes out with its rows and columns in that order, which the store undoes).  No LDS
// tiles, no barriers, no conversions of layout: per step two fetches, an addition and eight matrix instructions.
// Addresses: the row operand advances by a constant (a scalar), the gathered one takes its positions' offsets from a table of 32 that
// the wavefront fills for itself, one per lane, a block ahead.  What lies behind the end of the chunk reads as zero (the row
// operand's buffer ends there).
//
// The matrix instruction is a sequential fma chain, lowest k first, whatever its tile shape: the same bits as the tile
// kernel's, chunk by chunk.  1024 rows of 84x84 frames, conv1, conv2, conv3, FC and the heads in one launch: 215 us on the tile kernel, 183
// now (122 at the matrix pipes' peak of 157.3 TFLOP/s).  Not kept: 64 x 64 blocks (fewer vector instructions, but tasks so long that a third of
// the compute units end early: 208 us); blocks of 32 x 32 in segments of 64 for small minibatches (80 rows: 33.5 us against 31.5 of the
// wave-per-segment bodies: chains of up to 192 steps).
#pragma once
#include "problems.hpp"

namespace hts {

constexpr int RW_BLOCK = 32, RW_STEPS = RW_BLOCK / 4, RW_DEPTH = 8;      // positions and steps of a block; steps in flight

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));      // at any multiple of four bytes
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// A problem W offers: ROW_TILES (of 32 rows), col_tiles() (of 64, without
// the bias), K, klen, CHUNKED (more than one chunk), BIAS; `const float *a_row(int k)` and A_PITCH (bytes between rows of the row operand); From from(kbeg, c, li):
// what the fetches of the other operand need, advance(From) after a block; fill(table, i, k, From) where GATHER; load_b, expand_b;
// store(n, kcol, four values, z) and store_bias(n, value, z).
template <class W, bool BIAS_ONLY>
__device__ __forceinline__ void regwgrad_task(const W &p, int rt, int c, int z, uint32_t *table)
{
    constexpr int TM = 2, TN = 4;
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    const int kbeg = z * p.klen, kend = min(p.K, kbeg + p.klen);
    const int nblocks = (kend - kbeg + RW_BLOCK - 1) / RW_BLOCK;

    const uint32_t a_lane = (uint32_t)(q * W::A_PITCH + (rt * 16 * TM + li * TM) * 4);
    __amdgpu_buffer_rsrc_t ra;
    const char *abase = reinterpret_cast<const char *>(p.a_row(kbeg));
    uint32_t aleft;
    typename W::From from = p.from(kbeg, c, li);
    auto fill = [&](int blk) {             // this lane's entry of the block's table
        if constexpr (W::GATHER) {
            const int k = min(kbeg + blk * RW_BLOCK + (lane & 31), kend - 1);
            p.fill(table, lane & 31, k, from);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // (other lanes read it; a wavefront's LDS operations execute in order)
            __builtin_amdgcn_wave_barrier();
        }
    };
    auto point = [&](int blk) {            // row operand's buffer: from this block on, to the end of the chunk
        const char *b = abase + (long long)blk * RW_BLOCK * W::A_PITCH;
        const long long left = (long long)(kend - kbeg - blk * RW_BLOCK) * W::A_PITCH;
        aleft = left < 0 ? 0u : left > 0x7fffffffll ? 0x7fffffffu : (uint32_t)left;
        ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(b), 0, (int)aleft, 0x00020000);
    };
    typedef typename W::Raw Raw;
    f32x2_t av[RW_DEPTH];
    Raw bv[RW_DEPTH];
    auto load_a = [&](int step) -> f32x2_t {
        return __builtin_bit_cast(f32x2_t, __builtin_amdgcn_raw_buffer_load_b64(ra, (int)a_lane, step * 4 * W::A_PITCH, 0));
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    fill(0);
    point(0);
    if constexpr (!BIAS_ONLY) {
#pragma unroll
        for (int s = 0; s < RW_DEPTH; ++s) { av[s] = load_a(s); bv[s] = p.load_b(table, s, q, from); }
        for (int blk = 0; blk < nblocks; ++blk) {
#pragma unroll
            for (int s = 0; s < RW_STEPS; ++s) {
                if (s == (RW_STEPS - RW_DEPTH) % RW_STEPS) { fill(blk + 1); point(blk + 1); from = p.advance(from); }      // the block's own fetches are out
                const f32x4 b = p.expand_b(bv[s % RW_DEPTH]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s % RW_DEPTH][i], b[j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);      // (each step's fetches here, behind its products, whose registers they take; or the compiler gathers them)
                av[s % RW_DEPTH] = load_a((s + RW_DEPTH) % RW_STEPS);
                bv[s % RW_DEPTH] = p.load_b(table, (s + RW_DEPTH) % RW_STEPS, q, from);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // tile (i, j), register r of lane (q, li): row TM (4q + r) + i, column TN li + j
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                f32x4 v;
#pragma unroll
                for (int j = 0; j < TN; ++j) v[j] = acc[i][j][r];
                p.store(rt * 16 * TM + TM * (4 * q + r) + i, c * 16 * TN + TN * li, v, z);
            }
        return;
    }
    // the bias column: products against a constant
#pragma unroll
    for (int s = 0; s < RW_DEPTH; ++s) av[s] = load_a(s);
    for (int blk = 0; blk < nblocks; ++blk) {
#pragma unroll
        for (int s = 0; s < RW_STEPS; ++s) {
            if (s == (RW_STEPS - RW_DEPTH) % RW_STEPS) point(blk + 1);
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s % RW_DEPTH][i], W::BIAS, acc[i][0], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            av[s % RW_DEPTH] = load_a((s + RW_DEPTH) % RW_STEPS);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (li == 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) p.store_bias(rt * 16 * TM + TM * (4 * q + r) + i, acc[i][0][r], z);
    }
}

// conv2 / conv3: a tile of 64 columns is one tap of 64 channels or two neighbouring taps of 32, contiguous in the layer's input
template <class L> struct RegConvWgrad {
    static constexpr int ROW_TILES = 2, A_PITCH = 256;
    static constexpr bool CHUNKED = true;
    static constexpr bool GATHER = true;
    static constexpr float BIAS = 1.0f;
    static_assert(L::KSZ * L::CIN % 64 == 0, "column tiles inside a tap row");
    typedef f32x4 Raw;
    struct From { __amdgpu_buffer_rsrc_t r; uint32_t lane; int b0; };
    ConvWgrad<float, L> w;
    int K, klen;
    explicit RegConvWgrad(const ConvWgrad<float, L> &p) : w(p), K(p.K), klen(p.klen) {}
    HTS_HD int col_tiles() const { return L::K / 64; }
    __device__ __forceinline__ const float *a_row(int k) const { return w.dy + (long long)k * 64; }
    __device__ __forceinline__ From from(int kbeg, int c, int li) const
    {
        const int b0 = w.dPo.div(kbeg), kc = c * 64, u = kc / (L::KSZ * L::CIN);
        const float *base = w.in + (long long)b0 * w.Hin * w.Win * L::CIN;
        return {__builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, -4, 0x00020000),
                (uint32_t)(4 * (u * w.Win * L::CIN + kc - u * (L::KSZ * L::CIN) + 4 * li)), b0};
    }
    __device__ __forceinline__ From advance(const From &f) const { return f; }
    // (a chunk's samples span less than 4 GB: it is a 64th of a batch whose activations fit the card beside their gradients)
    __device__ __forceinline__ void fill(uint32_t *table, int i, int k, const From &f) const
    {
        const int b = w.dPo.div(k), pos = k - b * w.Po, oy = w.dWo.div(pos), ox = pos - oy * w.Wo;
        table[i] = 4u * (((uint32_t)(b - f.b0) * w.Hin + oy * L::STRIDE) * w.Win + ox * L::STRIDE) * L::CIN;
    }
    __device__ __forceinline__ Raw load_b(const uint32_t *table, int step, int q, const From &f) const
    {
        return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b128(f.r, (int)(table[step * 4 + q] + f.lane), 0, 0));
    }
    __device__ __forceinline__ Raw expand_b(const Raw &v) const { return v; }
    __device__ __forceinline__ void store(int n, int kcol, const Raw &v, int z) const { *reinterpret_cast<f32x4_u *>(w.part + ((long long)z * 64 + n) * w.N + kcol) = v; }
    __device__ __forceinline__ void store_bias(int n, float v, int z) const { w.part[((long long)z * 64 + n) * w.N + L::K] = v; }
};

// FC: rows of both operands are samples
struct RegFcWgrad {
    static constexpr int ROW_TILES = 16, A_PITCH = 2048;
    static constexpr bool CHUNKED = false;
    static constexpr bool GATHER = false;
    static constexpr float BIAS = 1.0f;
    typedef f32x4 Raw;
    struct From { const char *base; __amdgpu_buffer_rsrc_t r; uint32_t lane; int k; };
    FcWgrad<float> w;
    int K, klen;
    explicit RegFcWgrad(const FcWgrad<float> &p) : w(p), K(p.K), klen(p.klen) {}
    HTS_HD int col_tiles() const { return w.F / 64; }
    __device__ __forceinline__ const float *a_row(int k) const { return w.dh + (long long)k * 512; }
    __device__ __forceinline__ From at(const char *base, uint32_t lane, int k) const      // (rows behind the last sample read as zero)
    {
        const long long left = (long long)(K - k) * w.F * 4 - (base - reinterpret_cast<const char *>(w.a3 + (long long)k * w.F));
        return {base, __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, (int)(left < 0 ? 0 : left > 0x7fffffffll ? 0x7fffffffll : left), 0x00020000), lane, k};
    }
    __device__ __forceinline__ From from(int kbeg, int c, int li) const
    {
        return at(reinterpret_cast<const char *>(w.a3 + (long long)kbeg * w.F + (c < col_tiles() ? c : 0) * 64), (uint32_t)(16 * li), kbeg);
    }
    __device__ __forceinline__ From advance(const From &f) const { return at(f.base + (long long)RW_BLOCK * w.F * 4, f.lane, f.k + RW_BLOCK); }
    __device__ __forceinline__ Raw load_b(const uint32_t *, int step, int q, const From &f) const
    {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(f.r, (int)(f.lane + (uint32_t)(q * w.F * 4)), step * w.F * 16, 0));
    }
    __device__ __forceinline__ f32x4 expand_b(const Raw &v) const { return v; }
    __device__ __forceinline__ void store(int j, int f, const f32x4 &v, int) const { *reinterpret_cast<f32x4_u *>(w.g + w.fcw + (long long)j * w.F + f) = v; }
    __device__ __forceinline__ void store_bias(int j, float v, int) const { w.g[w.fcb + j] = v; }
};

// conv1: four neighbouring pixels per lane; a tile of 64 columns is an input channel's 8x8 window
template <bool INDEXED> struct RegConv1Wgrad {
    static constexpr int ROW_TILES = 1, A_PITCH = 128;
    static constexpr bool CHUNKED = true;
    static constexpr bool GATHER = true;
    static constexpr float BIAS = 255.0f;
    typedef uint32_t Raw;
    struct From { uint32_t lane; };
    Conv1Wgrad<float, INDEXED> w;
    int K, klen;
    explicit RegConv1Wgrad(const Conv1Wgrad<float, INDEXED> &p) : w(p), K(p.K), klen(p.klen) {}
    HTS_HD int col_tiles() const { return w.C; }
    __device__ __forceinline__ const float *a_row(int k) const { return w.dy + (long long)k * 32; }
    __device__ __forceinline__ From from(int, int c, int li) const { return {(uint32_t)((c * w.H + (li >> 1)) * w.W + 4 * (li & 1))}; }
    __device__ __forceinline__ From advance(const From &f) const { return f; }
    __device__ __forceinline__ void fill(uint32_t *table, int i, int k, const From &) const
    {
        const int b = w.dP1.div(k), pos = k - b * w.P1, oy = w.dW1.div(pos), ox = pos - oy * w.W1;
        const long long row = INDEXED ? (long long)w.index[b] : (long long)b;
        const unsigned long long at = (unsigned long long)(uintptr_t)w.obs + (unsigned long long)((row * w.C * w.H + oy * 4) * w.W + ox * 4);
        table[2 * i] = (uint32_t)at; table[2 * i + 1] = (uint32_t)(at >> 32);
    }
    __device__ __forceinline__ Raw load_b(const uint32_t *table, int step, int q, const From &f) const
    {
        const uint32_t *e = table + 2 * (step * 4 + q);
        typedef const Raw __attribute__((address_space(1))) *global_raw;
        return *(global_raw)((((unsigned long long)e[1] << 32) | e[0]) + f.lane);
    }
    __device__ __forceinline__ f32x4 expand_b(Raw x) const
    {
        f32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (float)((x >> (8 * j)) & 0xFFu);
        return v;
    }
    __device__ __forceinline__ void store(int n, int kcol, const f32x4 &v, int z) const { *reinterpret_cast<f32x4_u *>(w.part + ((long long)z * 32 + n) * w.N + kcol) = v; }
    __device__ __forceinline__ void store_bias(int n, float v, int z) const { w.part[((long long)z * 32 + n) * w.N + w.Kc] = v; }
};

}  // namespace hts
