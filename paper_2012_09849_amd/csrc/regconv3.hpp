// conv3 forward of large bf16 batches on known grids: weights in registers, samples copied into LDS ahead of their products.
//
// A workgroup, one per compute unit, walks groups of G samples.  Four of its eight wavefronts keep the 576 x 32 weights of output channels 0-31 in
// registers, four those of 32-63, read once in fragment order (see frag16); the samples come straight into LDS (buffer_load ... lds), up to two
// groups ahead.  A pixel's 128 bytes lie 144 apart, and rows and samples so that the windows of sixteen neighbouring positions begin in different
// banks also where they wrap (lanes in between copy nothing); every offset within a window is a constant of the instruction.  The output is channel-major: it goes through LDS and leaves as whole vectors.
// Same k order and segments as the other kernels, hence the same bits.
// What bounds it: each further group of two 84x84 samples, 33 KB, takes 2.1 us on every unit, 4.1 TB/s where a plain copy reaches 4.8; in front
// of the first products lie 5 us, of which the weights' way through the L1, 36 KB to each wavefront, 1.9.  4096 rows of 84x84 frames 26.7 -> 24.5 us, 256
// 10.4 -> 8.8 (brackets, 3.3 of each).  Not kept: the second group ahead of the weights (1024 rows 12.4 -> 12.6).
#pragma once
#include "dmawgrad.hpp"

namespace hts {

struct RegConv3Args {
    const bf16_t *in;      // [B][HIN*WIN][64]
    const bf16_t *w;       // [64][576], k = (tap, c), in fragment order
    const float *bias;
    bf16_t *out;           // [B][64][PO]
    bf16_t *out2;          // learner: [B][PO][64]
    int B;
};

template <int HIN_, int WIN_, int G_, int SEG_> struct RegConv3 {
    static constexpr int HIN = HIN_, WIN = WIN_, G = G_, HO = HIN - 2, WO = WIN - 2, PIN = HIN * WIN, PO = HO * WO;
    static constexpr int next(int least, int like) { return least + ((like - least) % 16 + 16) % 16; }
    static constexpr int STEPS = 36, SEGSTEPS = SEG_ / 16;
    // 16-byte slots: nine a pixel, and as many more behind a row and a sample as make output position i's window begin at 9 i modulo 16
    static constexpr int PIX = 9, ROW = next(PIX * WIN, PIX * WO), SAMPLE = next(HIN * ROW, PIX * PO);
    static constexpr int COPIES = (G * SAMPLE + 63) / 64, STAGE = COPIES * 1024, PER = (COPIES + 7) / 8, STAGES = 3;
    static constexpr int ROWS = G * PO, TILES = (ROWS + 31) / 32, OUT = G * PO * 128, STORES = (OUT / 16 + 511) / 512, LDS = STAGES * STAGE + OUT + 256;
    static_assert(STEPS % SEGSTEPS == 0 && PO * 128 % 16 == 0, "whole segments and vectors");
    static_assert(LDS <= 160 * 1024, "shape");
};

template <class C, bool LEARN> __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv3_regconv_kernel(const RegConv3Args a)
{
    constexpr int STEPS = C::STEPS, SS = C::SEGSTEPS, PER = C::PER, PD = 6;
    constexpr uint32_t NONE = 0x80000000u;
    extern __shared__ __attribute__((aligned(1024))) unsigned char rc3_smem[];
    unsigned char *outl = rc3_smem + C::STAGES * C::STAGE;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), half = w & 1, lrow = lane & 31, kg = lane >> 5;
    const int groups = (a.B + C::G - 1) / C::G, step = gridDim.x;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)rc3_smem;
    // this lane's source of copy w + 8 i of a group (excess copies repeat the last one)
    uint32_t src[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int slot = min(w + 8 * i, C::COPIES - 1) * 64 + lane, g = slot / C::SAMPLE, r = slot - g * C::SAMPLE, y = r / C::ROW, r9 = r - y * C::ROW, x = r9 / C::PIX, c = r9 - x * C::PIX;
        src[i] = g < C::G && y < C::HIN && x < C::WIN && c < 8 ? 16u * (uint32_t)(8 * (g * C::PIN + y * C::WIN + x) + c) : NONE;
    }
    auto fetch = [&](int grp, int s) {                          // beyond the batch: zeros
        const long long left = grp < groups ? (long long)(a.B - grp * C::G) * C::PIN * 128 : 0;
        const rsrc_words from = copy_source(a.in + (left ? (long long)grp * C::G * C::PIN * 64 : 0), (uint32_t)(left < (long long)NONE ? left : (long long)NONE));
#pragma unroll
        for (int i = 0; i < PER; ++i) copy16(from, src[i], 0u, lds0 + (uint32_t)(s * C::STAGE + min(w + 8 * i, C::COPIES - 1) * 1024));
    };
    fetch(blockIdx.x, 0);
    bf16x8 wt[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k)
        wt[k] = *reinterpret_cast<const bf16x8 *>(a.w + (((2 * half + (lrow >> 4)) * 18 + (k >> 1)) * 64 + (2 * (k & 1) + kg) * 16 + (lrow & 15)) * 8);
    float *biasl = reinterpret_cast<float *>(outl + C::OUT);   // (registers are short)
    if (tid < 64) biasl[tid] = a.bias[tid];
#pragma unroll
    for (int k = 0; k < STEPS; ++k) asm volatile("" : "+v"(wt[k]));      // (the first group's copies, asked for before, are there too)
    fetch(blockIdx.x + step, 1);
    int s = 0, done = 0;
    for (int grp = blockIdx.x; grp < groups; grp += step, ++done) {
        // This wavefront's copies of the group have landed.  Behind them in order: of the last two groups worked on at least STORES stores each,
        // and the next group's copies.
        if (done == 0) __builtin_amdgcn_s_waitcnt(wait_imm<PER>());
        else if (done == 1) __builtin_amdgcn_s_waitcnt(wait_imm<PER + C::STORES>());
        else __builtin_amdgcn_s_waitcnt(wait_imm<PER + 2 * C::STORES>());
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch(grp + 2 * step, s == 0 ? 2 : s - 1);
        const int ng = min(C::G, a.B - grp * C::G);             // samples of the group that exist
        for (int t = w >> 1; t < C::TILES; t += 4) {
            const int idx = t * 32 + lrow, ic = min(idx, C::ROWS - 1), g = ic / C::PO, p = ic - g * C::PO, oy = p / C::WO, ox = p - oy * C::WO;
            const unsigned char *at = rc3_smem + s * C::STAGE + 16 * (g * C::SAMPLE + oy * C::ROW + ox * C::PIX + kg);
            auto read = [&](int k) {                            // k: tap k / 4, channels 16 (k % 4) + 8 kg .. + 7
                return *reinterpret_cast<const bf16x8 *>(at + 16 * (k / 12 * C::ROW + k / 4 % 3 * C::PIX + 2 * (k % 4)));
            };
            bf16x8 av[PD];
#pragma unroll
            for (int k = 0; k < PD; ++k) av[k] = read(k);
            f32x16 tot, acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) tot[r] = 0.0f;
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                const bf16x8 x = av[k % PD];
                if (k + PD < STEPS) av[k % PD] = read(k + PD);
                __builtin_amdgcn_sched_barrier(0);
                if (k % SS == 0) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt[k], x, acc, 0, 0, 0);
                if (k % SS == SS - 1) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[r] += acc[r];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // register 4 q + e: channel 32 half + 8 q + 4 kg + e of position p of sample g
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x2 pk[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 bias = *reinterpret_cast<const f32x4 *>(biasl + half * 32 + 8 * q + 4 * kg);
                Vec<bf16_t, 4> y;
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float v = tot[4 * q + e] + bias[e]; y[e] = from_f32<bf16_t>(v > 0.0f ? v : 0.0f); }
                if (idx < C::ROWS) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) *reinterpret_cast<bf16_t *>(outl + 2 * ((g * 64 + half * 32 + 8 * q + 4 * kg + e) * C::PO + p)) = y[e];
                }
                pk[q] = __builtin_bit_cast(u32x2, y);
            }
            if constexpr (LEARN) {
                // the two lanes of a position trade halves: one has channels 0-15 and the other 16-31 of the 32
                const __amdgpu_buffer_rsrc_t to = dma_source(a.out2 + (long long)grp * C::ROWS * 64, (uint32_t)(ng * C::PO * 128));
                const uint32_t o = idx < C::ROWS ? (uint32_t)(idx * 128 + half * 64 + 32 * kg) : NONE;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x2 mine = kg ? pk[2 + h] : pk[h], send = kg ? pk[h] : pk[2 + h];
                    u32x2 got;
                    got.x = __shfl_xor(send.x, 32, 64);
                    got.y = __shfl_xor(send.y, 32, 64);
                    const u32x4 v = kg ? u32x4{got.x, got.y, mine.x, mine.y} : u32x4{mine.x, mine.y, got.x, got.y};
                    __builtin_amdgcn_raw_buffer_store_b128(v, to, (int)(o + 16 * h), 0, 0);
                }
            }
        }
        __syncthreads();
        // (STORES of them in every case, what does not exist beyond the buffer's end: the waits above count them)
        typedef int i32x4s __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t to = dma_source(a.out + (long long)grp * C::ROWS * 64, (uint32_t)(ng * C::PO * 128));
#pragma unroll
        for (int i = 0; i < C::STORES; ++i) {
            const int v = tid + 512 * i;
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const i32x4s *>(outl + 16 * min(v, C::OUT / 16 - 1)), to, v < C::OUT / 16 ? 16 * v : (int)NONE, 0, 0);
        }
        s = s + 1 == C::STAGES ? 0 : s + 1;
    }
    __builtin_amdgcn_s_waitcnt(wait_imm<0>());       // no copy is under way when the workgroup's LDS is given back
}

template <class C> inline hipError_t launch_regconv3(const RegConv3Args &a, int cus, hipStream_t stream)
{
    if (a.B <= 0) return hipSuccess;
    void (*kern)(const RegConv3Args) = a.out2 ? conv3_regconv_kernel<C, true> : conv3_regconv_kernel<C, false>;
    static std::atomic<bool> attr_set[2] = {};      // raise the dynamic-LDS limit once per instantiation (setting it twice is harmless)
    std::atomic<bool> &set = attr_set[a.out2 ? 1 : 0];
    if (!set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
        if (e != hipSuccess) return e;
        set.store(true, std::memory_order_release);
    }
    const int groups = (a.B + C::G - 1) / C::G;
    hipLaunchKernelGGL(kern, dim3(groups < cus ? groups : cus), dim3(512), C::LDS, stream, a);
    return hipGetLastError();
}

}  // namespace hts
