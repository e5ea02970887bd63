// conv2 forward of large bf16 batches on known grids: weights in registers, samples resident in LDS.
//
// A workgroup, one per compute unit, walks groups of two samples.  Four of its eight wavefronts keep the 512 x 32 weights of output
// channels 0-31 in registers, four those of 32-63; the samples come straight into LDS (buffer_load ... lds), up to two groups ahead, one
// barrier per group.  The tile kernel reads a conv1 activation through the L1 once per tap that touches it (24 KB per k-tile) and is
// bound by that; here each comes in once, a matrix instruction needs one LDS read, and memory bounds it: 4096 rows of 84x84 frames, 147 MB,
// 43.5 -> 38.2 us, of which each further group takes 3.8 us, 4.8 TB/s, the rate of a plain copy, and 7 us pass before the first products.
// A sample lies as two planes, its even and its odd columns, so that neighbouring outputs read neighbouring pixels, and 16-byte slot s of the
// pixel in row y, plane column x holds channel vector s ^ (x / 4 + 2 (y / 2)) % 4: the reads of sixteen neighbours fall into different banks.
// Same k order and segments as the other kernels, hence the same bits.  Not kept: weights straight from memory (32 rows of them per
// load: 20.6 us at 1024 rows, 15.0 by way of LDS).
#pragma once
#include "dmawgrad.hpp"

namespace hts {

struct RegConvArgs {
    const bf16_t *in;      // [B][HIN*WIN][32]
    const bf16_t *w;       // [64][512], k = (tap, c)
    const float *bias;
    bf16_t *out;           // [B][HO*WO][64]
    int B;
};

template <class L, int HIN_, int WIN_, int SEG_> struct RegConv {
    static constexpr int CIN = L::CIN, KSZ = L::KSZ, HIN = HIN_, WIN = WIN_, G = 2;
    static constexpr int HO = (HIN - KSZ) / 2 + 1, WO = (WIN - KSZ) / 2 + 1, POUT = HO * WO, PIN = HIN * WIN;
    static constexpr int STEPS = KSZ * KSZ * CIN / 16, SEGSTEPS = SEG_ / 16;
    static constexpr int PLANE_W = (WIN + 1) / 2, PLANE = HIN * PLANE_W;                          // pixels
    static constexpr int COPIES = (2 * PLANE * 64 + 1023) / 1024, IMG = COPIES * 1024, STAGE = G * IMG;   // of a sample; bytes
    static constexpr int PER = (G * COPIES + 7) / 8;                                              // copies of a wavefront and group
    static constexpr int ROWS = G * POUT, TILES = (ROWS + 31) / 32, STAGES = 3;
    static constexpr int LDS = 160 * 1024, WEIGHTS = LDS - 64 * 1024;      // the weights pass over the last stage and the end of the second
    static constexpr int EARLY = (WEIGHTS - STAGE) / 1024 / 8;             // copies of a wavefront that fit into the second below them
    // the swizzle and the two planes are made for conv2; PLANE_W is even: two rows down, a pixel is in the same banks
    static_assert(L::STRIDE == 2 && CIN == 32 && KSZ == 4 && L::COUT == 64 && STEPS % SEGSTEPS == 0 && PLANE_W % 2 == 0, "layer");
    static_assert(STAGES * STAGE <= LDS && STAGE <= WEIGHTS && EARLY <= PER && TILES >= 4, "shape");
};

template <class C> __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void regconv_kernel(const RegConvArgs a)
{
    constexpr int CIN = C::CIN, STEPS = C::STEPS, SS = C::SEGSTEPS, PER = C::PER;
    constexpr uint32_t NONE = 0x80000000u;
    extern __shared__ __attribute__((aligned(1024))) unsigned char rc_smem[];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = w & 1, lrow = lane & 31, kg = lane >> 5;
    const int groups = (a.B + C::G - 1) / C::G, step = gridDim.x;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)rc_smem;

    float bias[16];                            // (scalar loads)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float lo = a.bias[half * 32 + 8 * (r / 4) + r % 4], hi = a.bias[half * 32 + 8 * (r / 4) + 4 + r % 4];
        bias[r] = kg ? hi : lo;
    }
    // this lane's source of copy w + 8 i of a group (excess copies repeat the last one); its 64 slots lie one after the other in LDS
    uint32_t src[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = min(w + 8 * i, C::G * C::COPIES - 1), g = j / C::COPIES, slot = (j - g * C::COPIES) * 64 + lane, q = slot / 4;
        const int plane = q / C::PLANE, r = q - plane * C::PLANE, y = r / C::PLANE_W, xp = r - y * C::PLANE_W, x = 2 * xp + plane;
        const int c = (slot % 4) ^ ((xp / 4 + 2 * (y / 2)) % 4);
        src[i] = plane < 2 && x < C::WIN ? 2u * (uint32_t)((g * C::PIN + y * C::WIN + x) * CIN + c * 8) : NONE;      // (holes: zeros)
    }
    auto fetch = [&](int grp, int s, int from_i = 0, int to_i = C::PER) {         // beyond the batch: zeros
        const long long left = grp < groups ? (long long)(a.B - grp * C::G) * C::PIN * CIN * 2 : 0;
        const rsrc_words from = copy_source(a.in + (left ? (long long)grp * C::G * C::PIN * CIN : 0), (uint32_t)(left < (long long)NONE ? left : (long long)NONE));
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i >= from_i && i < to_i) copy16(from, src[i], 0u, lds0 + (uint32_t)(s * C::STAGE + min(w + 8 * i, C::G * C::COPIES - 1) * 1024));
    };
    fetch(blockIdx.x, 0);
    // The weights come by way of LDS: 1 KB rows, whose slot v of row r holds vector v ^ r % 16
    static_assert(STEPS == 32, "a row of weights is one copy");
    {
        const rsrc_words from = copy_source(a.w, 64 * 1024);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = w * 8 + i;
            copy16(from, 16u * (uint32_t)(lane ^ (r % 16)), (uint32_t)(r * 1024), lds0 + (uint32_t)(C::WEIGHTS + r * 1024));
        }
    }
    fetch(blockIdx.x + step, 1, 0, C::EARLY);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm<C::EARLY>());             // the first group and the weights are there
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8 wt[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k)
        wt[k] = *reinterpret_cast<const bf16x8 *>(rc_smem + C::WEIGHTS + (half * 32 + lrow) * 1024 + ((2 * k + kg) ^ (lrow % 16)) * 16);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) asm volatile("" : "+v"(wt[k]));      // in registers before anything is copied over them
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fetch(blockIdx.x + step, 1, C::EARLY);
    int s = 0, done = 0;
    for (int grp = blockIdx.x; grp < groups; grp += step, ++done) {
        // This wavefront's copies of the group have landed.  Behind them in order: the next group's copies and, of each of the last two
        // groups worked on, at least two stores.
        if (done == 0) __builtin_amdgcn_s_waitcnt(wait_imm<PER>());
        else if (done == 1) __builtin_amdgcn_s_waitcnt(wait_imm<PER + 2>());
        else __builtin_amdgcn_s_waitcnt(wait_imm<PER + 4>());
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fetch(grp + 2 * step, s == 0 ? 2 : s - 1);
        const __amdgpu_buffer_rsrc_t to = dma_source(a.out + (long long)grp * C::ROWS * 64, (uint32_t)(min(C::G, a.B - grp * C::G) * C::POUT * 128));
        for (int t = w >> 1; t < C::TILES; t += 4) {
            const int idx = t * 32 + lrow, ic = min(idx, C::ROWS - 1), g = ic / C::POUT, p = ic - g * C::POUT, oy = p / C::WO, ox = p - oy * C::WO;
            // A window's pixel (u, v) lies at a constant distance, and its swizzle differs from that of (u % 2, v / 2) by a constant: four
            // addresses, the rest is in the instructions
            const uint32_t base = (uint32_t)(s * C::STAGE + g * C::IMG + (oy * 2 * C::PLANE_W + ox) * 64);
            uint32_t at[2][2];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int e = 0; e < 2; ++e) at[x][e] = base + 64 * x + 16 * ((((ox + x) / 4 + 2 * oy) % 4) ^ kg ^ (2 * e));
            bf16x8 av[2][SS];
            auto read = [&](int k, bf16x8 &to) {
                const int u = k / 2 / C::KSZ, v = k / 2 % C::KSZ;
                to = *reinterpret_cast<const bf16x8 *>(rc_smem + at[v / 2][(k % 2) ^ (u / 2)] + ((v % 2) * C::PLANE + u * C::PLANE_W) * 64);
            };
#pragma unroll
            for (int k = 0; k < SS; ++k) read(k, av[0][k]);
            f32x16 tot;
#pragma unroll
            for (int r = 0; r < 16; ++r) tot[r] = 0.0f;
#pragma unroll
            for (int sg = 0; sg < STEPS / SS; ++sg) {
                if (sg + 1 < STEPS / SS) {
#pragma unroll
                    for (int k = 0; k < SS; ++k) read((sg + 1) * SS + k, av[(sg + 1) & 1][k]);
                }
                __builtin_amdgcn_sched_barrier(0);
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
                for (int k = 0; k < SS; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt[sg * SS + k], av[sg & 1][k], acc, 0, 0, 0);
                tot += acc;
            }
            // The two lanes of a row hold alternate groups of four channels; they trade halves, so that one has channels 0-15 and the other
            // 16-31 of the 32.  (Two stores in every case, rows that do not exist beyond the buffer's end: the waits above count them.)
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x2 pk[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Vec<bf16_t, 4> y;
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float v = tot[4 * q + e] + bias[4 * q + e]; y[e] = from_f32<bf16_t>(v > 0.0f ? v : 0.0f); }
                pk[q] = __builtin_bit_cast(u32x2, y);
            }
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
        s = s + 1 == C::STAGES ? 0 : s + 1;
    }
    __builtin_amdgcn_s_waitcnt(wait_imm<0>());       // no copy is under way when the workgroup's LDS is given back
}

// cus: compute units that the stream runs on, a workgroup for each (more than them go in rounds with as long a start each: 4096 rows of
// 84x84 frames on 192 units, 256 workgroups 59 us, 192 45)
template <class C> inline hipError_t launch_regconv(const RegConvArgs &a, int cus, hipStream_t stream)
{
    if (a.B <= 0) return hipSuccess;
    auto kern = regconv_kernel<C>;
    static std::atomic<bool> attr_set{false};       // raise the dynamic-LDS limit once per instantiation (setting it twice is harmless)
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int groups = (a.B + C::G - 1) / C::G;
    hipLaunchKernelGGL(kern, dim3(groups < cus ? groups : cus), dim3(512), C::LDS, stream, a);
    return hipGetLastError();
}

}  // namespace hts
