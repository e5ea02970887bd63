// conv1 and conv2 forward, and conv3 where it fits, of a few bf16 frames (actor) in one kernel: a workgroup forms some rows of a sample's
// conv2 output, or a row of its conv3 output, and the positions of the layers below that it needs for itself.
//
// A call of few rows is a chain of launches, each with a start, a first round trip to memory and an end of its own, and little between them;
// this takes links out.  Neighbouring workgroups form the same positions again (conv1's up to 2.8 times), which costs matrix instructions of
// which a unit has plenty.  Eight wavefronts: all convert pixels to an LDS image and form conv1's segment sums (a segment is an input channel: one
// or two channels to a wavefront, so that a weight is read by one wavefront only), which meet in LDS in binary32 and are added there in channel
// order; four of them, 16 output channels each, then form conv2, the others conv3, from weights that they requested at the start.  Same k order,
// segments and epilogues as the other kernels, hence the same bits.
// What bounds it: a rollout's step of 32 4x84x84 frames takes 19.0 us with a launch for each layer, 16.6 with conv1 and conv2 here and 13.6 with conv3
// too.  The kernel's body of these 16.6, behind a launch of 2.4: the first round trip, conv1 1.1, sums 0.5, conv2 and its store 1.5.  Weights from
// rows instead of in fragment order (16 lines an instruction, on two to four of an L2's channels): 17.4; 16x72x96 frames, 16 rows: 18.7, 17.4
// from rows, 15.6.  Not kept: one row of conv2's output a workgroup of 4x84x84 frames (16 rows 14.1 against 12.8 with conv3).
#pragma once
#include "dmagemm.hpp"

namespace hts {

struct Conv12RowsArgs {
    const uint8_t *obs;
    const int32_t *index;
    const bf16_t *w1, *w2, *w3;  // [32][64 C], [64][512], [64][576], in fragment order
    const float *b1, *b2, *b3;
    bf16_t *out;            // [B][HO*WO][64]; with conv3 [B][64][(HO-2)*(WO-2)]
    int B;
};

// NR_ rows of conv2's output, cut into XS_ pieces of a row; CONV3_: the three rows under a row of conv3's output, and that row
template <int C_, int H_, int W_, int NR_, int XS_, bool CONV3_ = false> struct Conv12Rows {
    static constexpr int C = C_, H = H_, W = W_, NR = NR_, XS = XS_;
    static constexpr bool CONV3 = CONV3_;
    static constexpr int H1 = (H - 8) / 4 + 1, W1 = (W - 8) / 4 + 1, HO = (H1 - 4) / 2 + 1, WO = (W1 - 4) / 2 + 1;
    static constexpr int XO = WO / XS, PARTS = CONV3 ? HO - 2 : HO / NR * XS;       // outputs of a row; workgroups of a sample
    static constexpr int PH = 2 * NR + 2, PW = 2 * XO + 2, POS = PH * PW;           // conv1 positions
    static constexpr int IH = 4 * PH + 4, IW = 4 * PW + 4;                          // pixels under them
    static constexpr bool WHOLE = XS == 1 && IW == W;                               // rows of pixels lie one after the other
    static constexpr int VR = (IW + 7) / 8, PITCH = WHOLE ? W : 8 * VR;             // 8-pixel vectors of a row; pixels
    static constexpr int VC = WHOLE ? IH * W / 8 : IH * VR, NV = C * VC, NP = (NV + 511) / 512;      // of a channel, in all, of a thread
    static constexpr int CH = 2 * VC * 8, TP = 36, AP = 80;                         // bytes of a channel's image; floats of a position's sums; bytes of a pixel
    static constexpr int IMG = C * CH, SUMS = C * POS * TP * 4, LDS = IMG + SUMS + POS * AP;
    static constexpr int PAIRS = C * 2 / 8;                                         // (channel, half of the outputs) of a wavefront
    static constexpr int TILES1 = POS / 16, OUTS = NR * XO, TILES2 = (OUTS + 15) / 16;
    static constexpr int STEP = CONV3 ? 1 : NR, STEPS2 = CONV3 ? 18 : 16, AP2 = 144;        // rows from workgroup to workgroup; bytes of a conv2 pixel
    static_assert(!CONV3 || (NR == 3 && XS == 1 && OUTS * AP2 <= SUMS && WO <= 18), "conv3");
    static_assert((CONV3 || HO % NR == 0) && WO % XS == 0 && POS % 16 == 0 && C % 4 == 0, "shares");
    static_assert(W % 8 == 0 || WHOLE, "rows begin at a multiple of 8 bytes");
    static_assert((H * W) % 8 == 0 && (WHOLE ? (8 * W) % 8 == 0 && IH * W % 8 == 0 : (8 * XO) % 8 == 0), "vectors");
    static_assert(WHOLE || 8 * XO * (XS - 1) + 8 * VR <= W, "the last vector of a row lies in it");
    static_assert(8 * STEP * (PARTS / XS - 1) + IH <= H && IMG % 16 == 0 && SUMS % 16 == 0 && LDS <= 160 * 1024, "shape");
};

template <class S> __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv12_rows_kernel(const Conv12RowsArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char c12r_smem[];
    constexpr int CPW = S::PAIRS > 1 ? S::PAIRS / 2 : 1, HPC = S::PAIRS > 1 ? 2 : 1;      // channels of a wavefront, halves of each
    float *sums = reinterpret_cast<float *>(c12r_smem + S::IMG);
    unsigned char *act = c12r_smem + S::IMG + S::SUMS;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, kq = lane >> 4;
    // a sample's workgroups on one XCD: they share pixels
    const int slot = (int)blockIdx.x >> 3, b = (slot / S::PARTS) * 8 + ((int)blockIdx.x & 7), part = slot % S::PARTS;
    if (b >= a.B) return;
    const int oy0 = (part / S::XS) * S::STEP, ox0 = (part % S::XS) * S::XO;
    const uint8_t *src = a.obs + (long long)(a.index ? a.index[b] : b) * (S::C * S::H * S::W) + 8 * oy0 * S::W + 8 * ox0;
    uint2 raw[S::NP];
#pragma unroll
    for (int i = 0; i < S::NP; ++i) {
        const int v = min(tid + 512 * i, S::NV - 1), ch = v / S::VC, r = v - ch * S::VC;
        raw[i] = *reinterpret_cast<const uint2 *>(src + ch * (S::H * S::W) + (S::WHOLE ? 8 * r : (r / S::VR) * S::W + 8 * (r % S::VR)));
    }
    const int ch0 = w * S::PAIRS / 2, half0 = S::PAIRS > 1 ? 0 : w & 1;
    bf16x8 w1[CPW][HPC][2];
#pragma unroll
    for (int c = 0; c < CPW; ++c)
#pragma unroll
        for (int h = 0; h < HPC; ++h)
#pragma unroll
            for (int t = 0; t < 2; ++t) w1[c][h][t] = *reinterpret_cast<const bf16x8 *>(a.w1 + (((half0 + h) * (2 * S::C) + 2 * (ch0 + c) + t) * 64 + lane) * 8);
    const f32x4 bias1 = *reinterpret_cast<const f32x4 *>(a.b1 + 4 * (tid & 7));
    // Waves 4-7 form conv2, 0-3 conv3.  (Without it these ask for bytes behind the end of an empty buffer: one count of loads under way for
    // all, so that nobody waits for conv2's weights before they are used.)
    const int oc = 16 * (w & 3);
    const __amdgpu_buffer_rsrc_t wsrc = dma_source(w < 4 && S::CONV3 ? a.w3 : a.w2, w < 4 ? (S::CONV3 ? 72u * 1024u : 0u) : 64u * 1024u);
    const int wat = (w < 4 ? 18 * 64 : 16 * 64) * oc + 16 * lane;
    bf16x8 w2[S::STEPS2];
#pragma unroll
    for (int t = 0; t < S::STEPS2; ++t) w2[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, wat, 1024 * t, 0));
    const f32x4 bias2 = *reinterpret_cast<const f32x4 *>((w < 4 && S::CONV3 ? a.b3 : a.b2) + oc + 4 * kq);
    __builtin_amdgcn_sched_barrier(0);
    // ---- pixels ----
#pragma unroll
    for (int i = 0; i < S::NP; ++i) {
        if (tid + 512 * i >= S::NV) continue;
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = from_f32<bf16_t>((float)((raw[i].x >> (8 * e)) & 0xFFu));
            v[4 + e] = from_f32<bf16_t>((float)((raw[i].y >> (8 * e)) & 0xFFu));
        }
        *reinterpret_cast<bf16x8 *>(c12r_smem + 16 * (tid + 512 * i)) = v;
    }
    __syncthreads();
    // ---- conv1: segment sums ----
    // (8 pixels, 8-byte aligned, as two single reads: merged into one two-address read they take longer)
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef const volatile u32x2 __attribute__((address_space(3))) *lds_u32x2;
    const uint32_t img0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)c12r_smem + (uint32_t)(ch0 * S::CH);
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    // unit e: tile e / CPW of 16 positions, the wavefront's channel e % CPW.  The operands of a group of them are read ahead of the products of the
    // group before: an LDS round trip a group, not a tile
    constexpr int UNITS = S::TILES1 * CPW, GR = UNITS % 5 == 0 ? 5 : 3, GROUPS = UNITS / GR;
    static_assert(UNITS % GR == 0, "whole groups");
    bf16x8 av[2][GR][2];
    auto read = [&](int g) {
#pragma unroll
        for (int i = 0; i < GR; ++i) {
            const int e = g * GR + i, p = 16 * (e / CPW) + li, py = p / S::PW, px = p - py * S::PW;
            const uint32_t at = img0 + (uint32_t)(2 * ((4 * py + kq) * S::PITCH + 4 * px));
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t o = at + (uint32_t)(e % CPW * S::CH + 2 * (4 * t * S::PITCH));
                const u32x2 lw = *(lds_u32x2)(uintptr_t)o, hw = *(lds_u32x2)(uintptr_t)(o + 8u);
                const Vec<bf16_t, 4> lo = __builtin_bit_cast(Vec<bf16_t, 4>, lw), hi = __builtin_bit_cast(Vec<bf16_t, 4>, hw);
#pragma unroll
                for (int j = 0; j < 4; ++j) { av[g & 1][i][t][j] = lo[j]; av[g & 1][i][t][4 + j] = hi[j]; }
            }
        }
    };
    read(0);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        if (g + 1 < GROUPS) read(g + 1);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 acc[GR][HPC];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < GR; ++i)
#pragma unroll
                for (int h = 0; h < HPC; ++h)
                    acc[i][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[(g * GR + i) % CPW][h][t], av[g & 1][i][t], t == 0 ? zero : acc[i][h], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < GR; ++i)
#pragma unroll
            for (int h = 0; h < HPC; ++h) {                    // register j: channel 16 half + 4 kq + j of position p
                const int e = g * GR + i, p = 16 * (e / CPW) + li;
                *reinterpret_cast<f32x4 *>(sums + ((ch0 + e % CPW) * S::POS + p) * S::TP + 16 * (half0 + h) + 4 * kq) = acc[i][h];
            }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // ---- conv1's outputs: the segments in channel order (a segment sum is never -0, so the total starts as the first) ----
    constexpr int NF = (S::POS * 8 + 511) / 512;               // (position, four channels) of a thread
    f32x4 x[NF][S::C];
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int s = 0; s < S::C; ++s)
            x[i][s] = *reinterpret_cast<const f32x4 *>(sums + (s * S::POS + min((tid >> 3) + 64 * i, S::POS - 1)) * S::TP + 4 * (tid & 7));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const int p = (tid >> 3) + 64 * i;
        f32x4 tot = x[i][0];
#pragma unroll
        for (int s = 1; s < S::C; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) tot[j] += x[i][s][j];
        Vec<bf16_t, 4> o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float y = __builtin_fmaf(tot[j], 1.0f / 255.0f, bias1[j]);
            o[j] = from_f32<bf16_t>(y > 0.0f ? y : 0.0f);
        }
        if (p < S::POS) *reinterpret_cast<Vec<bf16_t, 4> *>(act + p * S::AP + 8 * (tid & 7)) = o;
    }
    __syncthreads();
    // ---- conv2 ----
    auto conv2 = [&](unsigned char *act2) {
        uint32_t at[S::TILES2];
#pragma unroll
        for (int i = 0; i < S::TILES2; ++i) {
            const int q = min(16 * i + li, S::OUTS - 1), y = q / S::XO, x = q - y * S::XO;
            at[i] = (uint32_t)((2 * y * S::PW + 2 * x) * S::AP + 16 * kq);
        }
        f32x4 tot[S::TILES2];
#pragma unroll
        for (int i = 0; i < S::TILES2; ++i) tot[i] = zero;
        bf16x8 pv[4][S::TILES2][2];                                // four segments under way; segment sg: taps (u, v) and (u, v + 1)
        auto read2 = [&](int sg) {
            const int u = sg >> 1, v = 2 * (sg & 1);
#pragma unroll
            for (int i = 0; i < S::TILES2; ++i)
#pragma unroll
                for (int e = 0; e < 2; ++e) pv[sg & 3][i][e] = *reinterpret_cast<const bf16x8 *>(act + at[i] + (u * S::PW + v + e) * S::AP);
        };
        f32x4 acc[2][S::TILES2];
        auto add = [&](int set) {
#pragma unroll
            for (int i = 0; i < S::TILES2; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) tot[i][r] += acc[set][i][r];
        };
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) read2(sg);
#pragma unroll
        for (int sg = 0; sg < 8; ++sg) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < S::TILES2; ++i)
                    acc[sg & 1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[2 * sg + e], pv[sg & 3][i][e], e == 0 ? zero : acc[sg & 1][i], 0, 0, 0);
            if (sg < 4) read2(sg + 4);
            if (sg > 0) add((sg - 1) & 1);                         // (the segment before: this one's products are under way)
            __builtin_amdgcn_sched_barrier(0);
        }
        add(1);
#pragma unroll
        for (int i = 0; i < S::TILES2; ++i) {
            const int q = 16 * i + li, y = q / S::XO, x = q - y * S::XO;
            if (q >= S::OUTS) continue;
            Vec<bf16_t, 4> o;
#pragma unroll
            for (int r = 0; r < 4; ++r) { const float t = tot[i][r] + bias2[r]; o[r] = from_f32<bf16_t>(t > 0.0f ? t : 0.0f); }
            if constexpr (S::CONV3) *reinterpret_cast<Vec<bf16_t, 4> *>(act2 + q * S::AP2 + 2 * (oc + 4 * kq)) = o;
            else *reinterpret_cast<Vec<bf16_t, 4> *>(a.out + ((long long)b * (S::HO * S::WO) + (oy0 + y) * S::WO + ox0 + x) * 64 + oc + 4 * kq) = o;
        }
    };
    unsigned char *act2 = c12r_smem + S::IMG;                  // (over the sums)
    if (w >= 4) conv2(act2);
    if constexpr (S::CONV3) {
        __syncthreads();
        if (w >= 4) return;
        // ---- conv3: positions of one row, segments of a tap row ----
        constexpr int W3 = S::WO - 2, P3 = (S::HO - 2) * W3;
        const unsigned char *from = act2 + min(li, W3 - 1) * S::AP2 + 16 * kq;
        bf16x8 pv[18];
#pragma unroll
        for (int t = 0; t < 18; ++t) pv[t] = *reinterpret_cast<const bf16x8 *>(from + (t / 6 * S::WO + t / 2 % 3) * S::AP2 + t % 2 * 64);
        f32x4 acc[3], tot = zero;
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int u = 0; u < 3; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[6 * u + t], pv[6 * u + t], t == 0 ? zero : acc[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[r] += acc[u][r];
        if (li < W3) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float t = tot[r] + bias2[r];
                a.out[(long long)b * (64 * P3) + (oc + 4 * kq + r) * P3 + oy0 * W3 + li] = from_f32<bf16_t>(t > 0.0f ? t : 0.0f);
            }
        }
    }
}

template <class S> inline hipError_t launch_conv12_rows(const Conv12RowsArgs &a, hipStream_t stream)
{
    if (a.B <= 0) return hipSuccess;
    auto kern = conv12_rows_kernel<S>;
    static std::atomic<bool> attr_set{false};       // raise the dynamic-LDS limit once per instantiation (setting it twice is harmless)
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((a.B + 7) / 8 * 8 * S::PARTS), dim3(512), S::LDS, stream, a);
    return hipGetLastError();
}

}  // namespace hts
