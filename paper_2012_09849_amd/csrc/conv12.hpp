// conv1 and conv2 forward of bf16 batches of 4x84x84 frames in one kernel: conv1's output of a sample goes to conv2 through LDS.
//
// One workgroup per compute unit walks a share of the samples, twelve wavefronts, three kinds of them, one of each kind on a SIMD:
//   4-7  (producers) fetch a frame two samples ahead into registers and convert the next one's pixels to bf16, once, into one of two images
//   0-3  conv1: position tiles w, w + 4, ... of 32, weights in registers, the position operand straight from the image (see conv1_slab_kernel)
//   8-11 conv2 of the sample before: 16 output channels each, their 512 x 16 weights in registers, 16x16x32 products, one a tap
// A sample takes two barriers: while conv2 reads the sample before, conv1's wavefronts keep what they have formed in registers; then
// it goes to LDS, over that.  There a sample lies as two planes, its even and its odd columns, so that neighbouring outputs read neighbouring
// pixels, and 16-byte slot s of a pixel holds channel vector s ^ c12_swizzle(its row, its column in the plane).
// Same k order, segments and epilogues as the other kernels, hence the same bits.
// Conv1's 25 KB of a sample are not written and read again (actor), or not read (learner), and there is one launch and one first fetch less.
// Medians of kernel traces, us, a launch each / this: 1024 rows 20 + 13.7 / 24.8, 4096 62 to 65 + 41 to 43 / 73 to 78; learner, which keeps conv1's output
// for its backward pass, 1024 rows 20.3 + 14.1 / 26.9.  What bounds it, by the counters at 4096 rows: a sample takes 8.4 thousand of a unit's cycles, of which
// the LDS is active for 4.5 (position operands of both layers, 1 KB an instruction; 0.95 of them bank conflicts), the matrix units for 3.2 and the vector units,
// four cycles an instruction, for 3.8 (segment sums, conversions, epilogues).  168 registers a wavefront are what three to a SIMD leave, and all are in use.  Not kept: conv2's reads two segments
// ahead (the same time), the next tile's reads ahead of a tile's sums (spills, 80 to 94 us at 4096 rows), the thirteenth tile by one of conv1's wavefronts (76).
#pragma once
#include "dmagemm.hpp"

namespace hts {

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

struct Conv12Args {
    const uint8_t *obs;
    const int32_t *index;
    const bf16_t *w1, *w2;  // [32][256], [64][512]
    const float *b1, *b2;
    bf16_t *out1, *out2;    // [B][400][32] (learner: kept for the backward pass), [B][81][64]
    int B;
};
constexpr int C12_THREADS = 768, C12_MAX_SAMPLES = 64;       // observations per workgroup (their row indices are read once, into LDS)
constexpr int C12_H = 84, C12_IMG = 4 * C12_H * C12_H * 2, C12_W1 = 20, C12_P1 = 400, C12_W2 = 9, C12_P2 = 81;
constexpr int C12_PLANE_W = 10, C12_PLANE = 200, C12_ACT = C12_P1 * 64;        // pixels; bytes
constexpr int C12_WPITCH = 528, C12_LDS = 2 * C12_IMG + C12_ACT + 32 * C12_WPITCH + 128 + C12_MAX_SAMPLES * 4;

// Sixteen lanes of a 16-byte LDS read are served at once, and they are not neighbours: 0-3, 12-15, 20-23 and 24-27 (and so on).  conv2's
// lanes 8 r + x take pixels x of two rows and every 16 lanes the next channel vector: with this the sixteen fall into different banks
HTS_HD int c12_swizzle(int y, int xp) { return (2 * (y >> 1 & 1)) ^ (3 * (xp >> 2 & 1)); }

// one tile of 32 positions of conv1: the 32 channels, 16 consecutive ones of a lane's position.  at: where its position's patch begins in the
// image (LDS); weight(t): operand t of 16
template <bool WEIGHTS_AHEAD, class Weight> __device__ __forceinline__ void c12_tile(const uint32_t at, const Weight &weight, const float *lbias, const int lk, uint4 (&d)[2])
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef const volatile u32x2 __attribute__((address_space(3))) *lds_u32x2;
    // two channels at a time, a chain of products each; 8 pixels (8-byte aligned) as two single reads (see conv1_slab_kernel)
    constexpr int PD = 4;
    bf16x8 q[PD], wq[PD];
    auto step_of = [](int e) { return 4 * (2 * (e >> 3) + (e & 1)) + ((e >> 1) & 3); };      // step e: operand 4 channel + (patch rows 2t, 2t + 1)
    auto read = [&](int e, int slot) {
        const int ch = step_of(e) >> 2, t = step_of(e) & 3;
        const uint32_t o = (uint32_t)(2 * (ch * C12_H + 2 * t) * C12_H);
        const u32x2 lw = *(lds_u32x2)(uintptr_t)(at + o), hw = *(lds_u32x2)(uintptr_t)(at + o + 8u);
        const Vec<bf16_t, 4> lo = __builtin_bit_cast(Vec<bf16_t, 4>, lw), hi = __builtin_bit_cast(Vec<bf16_t, 4>, hw);
#pragma unroll
        for (int i = 0; i < 4; ++i) { q[slot][i] = lo[i]; q[slot][4 + i] = hi[i]; }
        if constexpr (WEIGHTS_AHEAD) wq[slot] = weight(step_of(e));
    };
    f32x16 acc[2], tot, zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
#pragma unroll
    for (int e = 0; e < PD; ++e) read(e, e);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const bf16x8 av = q[e % PD], wv = WEIGHTS_AHEAD ? wq[e % PD] : weight(step_of(e));
        if (e + PD < 16) read(e + PD, e % PD);
        __builtin_amdgcn_sched_barrier(0);
        acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, av, (step_of(e) & 3) == 0 ? zero : acc[e & 1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // a channel's segment sum joins the total, in channel order (it is never -0, so the total starts as the first)
        if (e == 7) {
#pragma unroll
            for (int r = 0; r < 16; ++r) tot[r] = acc[0][r] + acc[1][r];
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) tot[r] += acc[0][r];
#pragma unroll
    for (int r = 0; r < 16; ++r) tot[r] += acc[1][r];
    // register 4g + j is channel 8g + 4 lk + j: the two lanes of a position trade halves
    uint2 p[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 bias = *reinterpret_cast<const f32x4 *>(lbias + 8 * g + 4 * lk);
        Vec<bf16_t, 4> o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float y = __builtin_fmaf(tot[4 * g + j], 1.0f / 255.0f, bias[j]);
            o[j] = from_f32<bf16_t>(y > 0.0f ? y : 0.0f);
        }
        p[g] = __builtin_bit_cast(uint2, o);
    }
    const uint2 s0 = lk ? p[0] : p[2], s1 = lk ? p[1] : p[3];
    uint2 r0, r1;
    r0.x = __shfl_xor(s0.x, 32, 64); r0.y = __shfl_xor(s0.y, 32, 64);
    r1.x = __shfl_xor(s1.x, 32, 64); r1.y = __shfl_xor(s1.y, 32, 64);
    d[0] = lk ? make_uint4(r0.x, r0.y, p[2].x, p[2].y) : make_uint4(p[0].x, p[0].y, r0.x, r0.y);
    d[1] = lk ? make_uint4(r1.x, r1.y, p[3].x, p[3].y) : make_uint4(p[1].x, p[1].y, r1.x, r1.y);
}
// what a lane of conv1 knows of position m
struct C12Position {
    uint32_t patch;        // offset in an image
    int m;                 // 2^24: none
    uint32_t slot[2];      // offsets of its two channel vectors in conv2's input
    __device__ __forceinline__ C12Position(int tile, int lane)
    {
        const int lrow = lane & 31, lk = lane >> 5, mm = tile * 32 + lrow, mc = min(mm, C12_P1 - 1), y = mc / C12_W1, x = mc - y * C12_W1, xp = x >> 1, sw = c12_swizzle(y, xp);
        m = mm < C12_P1 ? mm : 1 << 24;
        patch = (uint32_t)(2 * ((4 * y + lk) * C12_H + 4 * x));
        const int px = ((x & 1) * C12_PLANE + y * C12_PLANE_W + xp) * 64;
        slot[0] = (uint32_t)(px + 16 * ((2 * lk) ^ sw)); slot[1] = (uint32_t)(px + 16 * ((2 * lk + 1) ^ sw));
    }
    __device__ __forceinline__ void place(unsigned char *act, const uint4 (&d)[2]) const
    {
        if (m < C12_P1) { *reinterpret_cast<uint4 *>(act + slot[0]) = d[0]; *reinterpret_cast<uint4 *>(act + slot[1]) = d[1]; }
    }
    __device__ __forceinline__ void keep(bf16_t *out, int b, int lk, const uint4 (&d)[2]) const
    {
        const __amdgpu_buffer_rsrc_t to = dma_source(out + (long long)b * (C12_P1 * 32), C12_P1 * 64);
        const int at = m * 64 + 32 * lk;                       // (no position: behind the buffer's end, not stored)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, d[0]), to, at, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, d[1]), to, at + 16, 0, 0);
    }
};

template <bool KEEP> __global__ __launch_bounds__(C12_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void conv12_kernel(const Conv12Args a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char c12_smem[];
    unsigned char *act = c12_smem + 2 * C12_IMG;
    unsigned char *wl = act + C12_ACT;
    float *lbias = reinterpret_cast<float *>(wl + 32 * C12_WPITCH);
    int *rowid = reinterpret_cast<int *>(lbias + 32);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lk = lane >> 5;
    const uint32_t smem0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)c12_smem;
    const int b0 = blockIdx.x, bstep = gridDim.x, nsamp = (a.B - b0 + bstep - 1) / bstep;
    if (tid < nsamp) { const int b = b0 + tid * bstep; rowid[tid] = a.index ? a.index[b] : b; }
    if (tid >= 64 && tid < 96) lbias[tid - 64] = a.b1[tid - 64];
    __syncthreads();
    if (w >= 4 && w < 8) {
        // ---- producers ----
        // (8 pixels a lane, so that the lanes of a write to the image are neighbours)
        constexpr int NV = 4 * C12_H * C12_H / 8, NP = (NV + 255) / 256;
        const int pt = tid - 256;
        const uint32_t own = 8u * (uint32_t)pt, end = 8u * (uint32_t)min(pt, NV - 1 - 256 * (NP - 1));
        uint2 raw[2][NP];
        auto fetch = [&](int s, uint2 (&r)[NP]) {
            const uint8_t *src = a.obs + (long long)__builtin_amdgcn_readfirstlane(rowid[s]) * (4 * C12_H * C12_H);
#pragma unroll
            for (int i = 0; i < NP; ++i) r[i] = *reinterpret_cast<const uint2 *>(src + 2048 * i + (i + 1 < NP ? own : end));
        };
        auto convert = [&](const uint2 (&r)[NP], int buf) {
            unsigned char *dst = c12_smem + buf * C12_IMG + 16 * pt;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (pt + 256 * i >= NV) continue;
                bf16x8 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = from_f32<bf16_t>((float)((r[i].x >> (8 * e)) & 0xFFu));
                    v[4 + e] = from_f32<bf16_t>((float)((r[i].y >> (8 * e)) & 0xFFu));
                }
                *reinterpret_cast<bf16x8 *>(dst + i * 4096) = v;
            }
        };
        fetch(0, raw[0]);
        if (nsamp > 1) fetch(1, raw[1]);
        // one of them forms conv1's thirteenth tile (half a tile), its weights in LDS: rows of 512 bytes and 16, so that they start four banks apart
        const C12Position last(12, lane);
        const unsigned char *wrow = wl + (lane & 31) * C12_WPITCH + 16 * lk;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = pt + 256 * i;
            *reinterpret_cast<uint4 *>(wl + (v >> 5) * C12_WPITCH + (v & 31) * 16) = *reinterpret_cast<const uint4 *>(a.w1 + v * 8);
        }
        convert(raw[0], 0);
        if (nsamp > 2) fetch(2, raw[0]);
        __syncthreads();
        for (int s0 = 0; s0 < nsamp; s0 += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {                      // sample s + 1 sits in register set 1 - j
                const int s = s0 + j;
                if (s >= nsamp) break;                         // (the same for the whole workgroup)
                if (s + 1 < nsamp) convert(raw[1 - j], 1 - j);
                if (s + 3 < nsamp) fetch(s + 3, raw[1 - j]);
                uint4 held[2];
                if (w == 7) {
                    c12_tile<true>(smem0 + j * C12_IMG + last.patch, [&](int t) { return *reinterpret_cast<const bf16x8 *>(wrow + 32 * t); }, lbias, lk, held);
                    if constexpr (KEEP) last.keep(a.out1, b0 + s * bstep, lk, held);
                }
                __syncthreads();
                if (w == 7) last.place(act, held);
                __syncthreads();
            }
        }
        return;
    }
    if (w < 4) {
        // ---- conv1 ----
        bf16x8 wreg[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) wreg[t] = *reinterpret_cast<const bf16x8 *>(a.w1 + (lane & 31) * 256 + 16 * t + 8 * lk);
        const C12Position pos[3] = {C12Position(w, lane), C12Position(w + 4, lane), C12Position(w + 8, lane)};
        __syncthreads();
        for (int s = 0; s < nsamp; ++s) {
            uint4 held[3][2];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                c12_tile<false>(smem0 + (s & 1) * C12_IMG + pos[i].patch, [&](int t) { return wreg[t]; }, lbias, lk, held[i]);
                if constexpr (KEEP) pos[i].keep(a.out1, b0 + s * bstep, lk, held[i]);
            }
            __syncthreads();                                   // conv2 has read the sample before
#pragma unroll
            for (int i = 0; i < 3; ++i) pos[i].place(act, held[i]);
            __syncthreads();
        }
        return;
    }
    // ---- conv2 ----
    const int li = lane & 15, kq = lane >> 4, ch = 16 * (w - 8);
    bf16x8 wreg[16];                                           // tap t: row ch + li, channels 8 kq .. + 7
#pragma unroll
    for (int t = 0; t < 16; ++t) wreg[t] = *reinterpret_cast<const bf16x8 *>(a.w2 + (ch + li) * 512 + 32 * t + 8 * kq);
    const f32x4 bias = *reinterpret_cast<const f32x4 *>(a.b2 + ch + 4 * kq);
    // Six tiles of 16 positions: eight of each of two rows, whose pixels lie in different banks; the ninth column at the end.
    // Where the window's pixels (u, v) lie, v = 2x, 2x + 1, u < 2 (u >= 2: 32 bytes exchanged, and a constant); where the output goes
    typedef const bf16x8 __attribute__((address_space(3))) *lds_operand;
    const uint32_t act0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)act;
    uint32_t at[6][2], to[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int q = min(16 * i + li, C12_P2 - 1), oy = q < 72 ? q >> 3 : q - 72, ox = q < 72 ? q & 7 : 8;
#pragma unroll
        for (int x = 0; x < 2; ++x) at[i][x] = act0 + (uint32_t)((2 * oy * C12_PLANE_W + ox + x) * 64 + 16 * (c12_swizzle(2 * oy, ox + x) ^ kq));
        to[i] = 16 * i + li < C12_P2 ? (uint32_t)((oy * C12_W2 + ox) * 128 + 2 * (ch + 4 * kq)) : 0x80000000u;      // (behind the buffer's end: not stored)
    }
    __syncthreads();
    for (int s = 0; s <= nsamp; ++s) {
        if (s > 0) {
            const __amdgpu_buffer_rsrc_t out = dma_source(a.out2 + (long long)(b0 + (s - 1) * bstep) * (C12_P2 * 64), C12_P2 * 128);
#pragma unroll
            for (int i0 = 0; i0 < 6; i0 += 2) {                // two tiles at a time
                bf16x8 av[2][2][2];                            // two segments in turn: tile, tap of the segment
                auto read = [&](int sg) {                      // segment sg: taps (u, v) and (u, v + 1), u = sg / 2, v = 2 (sg % 2)
                    const int u = sg >> 1, x = sg & 1;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int v = 0; v < 2; ++v)
                            av[sg & 1][i][v] = *(lds_operand)(uintptr_t)((at[i0 + i][x] ^ (u & 2 ? 32u : 0u)) + (uint32_t)((v * C12_PLANE + u * C12_PLANE_W) * 64));
                };
                const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                f32x4 tot[2] = {zero, zero}, acc[2][2];
                auto add = [&](int set) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r) tot[i][r] += acc[set][i][r];
                };
                read(0);
#pragma unroll
                for (int sg = 0; sg < 8; ++sg) {
                    if (sg < 7) read(sg + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int v = 0; v < 2; ++v)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            acc[sg & 1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wreg[2 * sg + v], av[sg & 1][i][v], v == 0 ? zero : acc[sg & 1][i], 0, 0, 0);
                    if (sg > 0) add((sg - 1) & 1);             // (the segment before: this one's products are under way)
                    __builtin_amdgcn_sched_barrier(0);
                }
                add(1);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    Vec<bf16_t, 4> y;
#pragma unroll
                    for (int r = 0; r < 4; ++r) { const float v = tot[i][r] + bias[r]; y[r] = from_f32<bf16_t>(v > 0.0f ? v : 0.0f); }
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, y), out, (int)to[i0 + i], 0, 0);
                }
            }
        }
        if (s < nsamp) { __syncthreads(); __syncthreads(); }
    }
}

inline hipError_t launch_conv12(const Conv12Args &a, int cus, hipStream_t stream)
{
    if (a.B <= 0) return hipSuccess;
    void (*kern)(const Conv12Args) = a.out1 ? conv12_kernel<true> : conv12_kernel<false>;
    static std::atomic<bool> attr_set[2] = {};      // raise the dynamic-LDS limit once per instantiation (setting it twice is harmless)
    std::atomic<bool> &set = attr_set[a.out1 ? 1 : 0];
    if (!set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C12_LDS);
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    int grid = a.B < cus ? a.B : cus;                                    // one workgroup per compute unit (its LDS), walking the batch
    const int least = (a.B + C12_MAX_SAMPLES - 1) / C12_MAX_SAMPLES;
    if (grid < least) grid = least;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(C12_THREADS), C12_LDS, stream, a);
    return hipGetLastError();
}

}  // namespace hts
