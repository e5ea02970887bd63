// Streaming and per-sample kernels: conv-weight permutation, policy/value heads with seeded sampling (actor) or
// loss gradient (learner), split-K combine, returns/GAE, advantage normalisation, gradient norm, Adam.
//
// This file is compiled with floating-point contraction off: the sampler's decision rule is a fixed sequence of
// binary32 operations (see hts_act in hts.h) and must not be re-associated or fused.
#include <math.h>

#include <mutex>

#include "internal.hpp"

#pragma clang fp contract(off)

namespace hts {

// 8 consecutive floats (16-byte aligned) into registers
__device__ __forceinline__ void load_vec(const float *p, float (&v)[8])
{
    const f32x4 t0 = *reinterpret_cast<const f32x4 *>(p), t1 = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = t0[i]; v[4 + i] = t1[i]; }
}

// ------------------------------------------------------------------------------------------------------------
// The network as the kernels read it: one launch copies the caller's fp32 parameter vector into the workspace,
// converting to the operand type and re-ordering.  Workgroups are assigned to jobs by index range:
//   [0, nb_fc)            64 x 64 tiles of fc.w -> wfc (same order) and, for the learner, wfcd (transposed, rows in
//                         channel-innermost order f' = p*64 + c), through an LDS tile so both sides stay coalesced
//   [nb_fc, +nb_conv)     conv2.w / conv3.w -> wf2, wf3 (taps outermost) and, for the learner, wd2, wd3
//   [.., +nb_w1)          conv1.w -> w1s
//                         (and conv1.w, conv2.w, conv3.w in fragment order -> w1q, w2q, w3q)
//   [.., +nb_hb)          biases and heads -> hb (fp32)
// ------------------------------------------------------------------------------------------------------------
struct PrepArgs {
    const float *params;
    Geom g;
    ShadowOffsets sh;
    void *w1s, *wf2, *wf3, *wfc, *wd2, *wd3, *wfcd;
    void *w1q, *w2q, *w3q;
    float *hb;
    int nb_fc, nb_conv, nb_w1, nb_hb;
    int learn;
};

template <typename T> __global__ __launch_bounds__(256) void prep_kernel(const PrepArgs a)
{
    __shared__ float tile[64][65];
    const int t = threadIdx.x;
    int blk = blockIdx.x;
    const float *__restrict__ params = a.params;
    if (blk < a.nb_fc) {
        const int F = a.g.F, tf = F / 64;
        const int j0 = (blk / tf) * 64, f0 = (blk % tf) * 64;
        const float *src = params + a.g.fcw;
        T *wfc = (T *)a.wfc;
        const int col = t & 63, r0 = t >> 6;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = r0 + 4 * i;
            const float v = src[(long long)(j0 + r) * F + f0 + col];
            wfc[(long long)(j0 + r) * F + f0 + col] = from_f32<T>(v);
            tile[r][col] = v;
        }
        if (!a.learn) return;
        __syncthreads();
        T *wfcd = (T *)a.wfcd;
        const int P3 = a.g.P3;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int fl = r0 + 4 * i, f = f0 + fl;
            const int c = f / P3, p = f - c * P3;
            wfcd[(long long)(p * 64 + c) * 512 + j0 + col] = from_f32<T>(tile[col][fl]);
        }
        return;
    }
    blk -= a.nb_fc;
    if (blk < a.nb_conv) {
        const int i = blk * 256 + t;
        T *wf2 = (T *)a.wf2, *wf3 = (T *)a.wf3, *wd2 = (T *)a.wd2, *wd3 = (T *)a.wd3;
        if (i < 64 * 32 * 16) {               // conv2.w[n][c][u][v], 64 x 32 x 4 x 4
            const int n = i / 512, r = i % 512, c = r / 16, tap = r % 16;
            const T w = from_f32<T>(params[a.g.w2 + i]);
            wf2[n * 512 + tap * 32 + c] = w;
            ((T *)a.w2q)[frag16<T>(n, tap * 32 + c, 512)] = w;
            if (a.learn) wd2[c * 1024 + tap * 64 + n] = w;
        }
        if (i < 64 * 64 * 9) {                // conv3.w[n][c][u][v], 64 x 64 x 3 x 3
            const int n = i / 576, r = i % 576, c = r / 9, tap = r % 9;
            const T w = from_f32<T>(params[a.g.w3 + i]);
            wf3[n * 576 + tap * 64 + c] = w;
            ((T *)a.w3q)[frag16<T>(n, tap * 64 + c, 576)] = w;
            if (a.learn) wd3[c * 576 + tap * 64 + n] = w;
        }
        return;
    }
    blk -= a.nb_conv;
    if (blk < a.nb_w1) {
        const int i = blk * 256 + t;
        if (i < 32 * a.g.K1) {
            const T w = from_f32<T>(params[a.g.w1 + i]);
            ((T *)a.w1s)[i] = w;
            ((T *)a.w1q)[frag16<T>(i / a.g.K1, i % a.g.K1, a.g.K1)] = w;
        }
        return;
    }
    blk -= a.nb_w1;
    {
        const int i = blk * 256 + t;
        const int A = a.g.A;
        // hb = b1 | b2 | b3 | fc.b | pi.w | pi.b | v.w | v.b, each part starting on a 16-byte boundary
        long long src = -1;
        if (i < 32) src = a.g.b1 + i;
        else if (i >= a.sh.b2 && i < a.sh.b2 + 64) src = a.g.b2 + (i - a.sh.b2);
        else if (i >= a.sh.b3 && i < a.sh.b3 + 64) src = a.g.b3 + (i - a.sh.b3);
        else if (i >= a.sh.fcb && i < a.sh.fcb + 512) src = a.g.fcb + (i - a.sh.fcb);
        else if (i >= a.sh.piw && i < a.sh.piw + 512 * A) src = a.g.piw + (i - a.sh.piw);
        else if (i >= a.sh.pib && i < a.sh.pib + A) src = a.g.pib + (i - a.sh.pib);
        else if (i >= a.sh.vw && i < a.sh.vw + 512) src = a.g.vw + (i - a.sh.vw);
        else if (i == a.sh.vb) src = a.g.vb;
        if (src < 0) return;
        a.hb[i] = params[src];
    }
}

static PrepArgs prep_args(const Ctx &c, const float *params, bool learn)
{
    PrepArgs a;
    a.params = params; a.g = c.g; a.sh = c.sh;
    a.w1s = c.ws.w1s; a.wf2 = c.ws.wf2; a.wf3 = c.ws.wf3; a.wfc = c.ws.wfc;
    a.w1q = c.ws.w1q; a.w2q = c.ws.w2q; a.w3q = c.ws.w3q;
    a.wd2 = c.ws.wd2; a.wd3 = c.ws.wd3; a.wfcd = c.ws.wfcd; a.hb = c.ws.hb;
    a.nb_fc = (512 / 64) * (c.g.F / 64);
    a.nb_conv = (64 * 64 * 9 + 255) / 256;
    a.nb_w1 = (32 * c.g.K1 + 255) / 256;
    a.nb_hb = (int)((c.sh.count + 255) / 256);
    a.learn = learn ? 1 : 0;
    return a;
}

hipError_t launch_prep(Ctx &c, const float *params, bool learn)
{
    SiteTimer tm(c, SITE_PREP);
    const PrepArgs a = prep_args(c, params, learn);
    const int nb = a.nb_fc + a.nb_conv + a.nb_w1 + a.nb_hb;
    if (c.desc.precision == HTS_PRECISION_BF16)
        hipLaunchKernelGGL(prep_kernel<bf16_t>, dim3(nb), dim3(256), 0, c.stream, a);
    else
        hipLaunchKernelGGL(prep_kernel<float>, dim3(nb), dim3(256), 0, c.stream, a);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) { c.synced = true; c.synced_learn = learn; c.shadow_of = params; }
    return e;
}

// ------------------------------------------------------------------------------------------------------------
// counter-based uniform and the sampler's binary32 exponential
// ------------------------------------------------------------------------------------------------------------

// Philox4x32-10 (Salmon et al., SC'11), word 0 only is used by the caller.
__device__ __forceinline__ uint32_t philox_word0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                                 uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t h0 = __umulhi(0xD2511F53u, c0), l0 = 0xD2511F53u * c0;
        const uint32_t h1 = __umulhi(0xCD9E8D57u, c2), l1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
        c0 = n0; c1 = l1; c2 = n2; c3 = l0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return c0;
}

__device__ __forceinline__ float seeded_uniform(uint64_t seed, uint32_t env, uint32_t step)
{
    const uint32_t w = philox_word0(env, step, 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
    return (float)(w >> 8) * 5.9604644775390625e-08f;     // 24 random bits * 2^-24, exact
}

// exp(x), x <= 0:  0 below -87; n = rint(x*log2e); r = x - n*ln2 (two-constant reduction, fma);
// degree-6 Taylor polynomial by Horner with fma; exact scaling by 2^n.
__device__ __forceinline__ float sampler_exp(float x)
{
    if (x < -87.0f) return 0.0f;
    const float n = rintf(x * 1.44269504088896340736f);
    float r = __builtin_fmaf(n, -0.693145751953125f, x);
    r = __builtin_fmaf(n, -1.42860682030941723212e-6f, r);
    float q = 1.0f / 720.0f;
    q = __builtin_fmaf(q, r, 1.0f / 120.0f);
    q = __builtin_fmaf(q, r, 1.0f / 24.0f);
    q = __builtin_fmaf(q, r, 1.0f / 6.0f);
    q = __builtin_fmaf(q, r, 0.5f);
    q = __builtin_fmaf(q, r, 1.0f);
    q = __builtin_fmaf(q, r, 1.0f);
    const float scale = __uint_as_float((uint32_t)((int)n + 127) << 23);
    return q * scale;
}

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// max over the 64 lanes, in every lane (exact whatever the order).  Row shifts inside each row of 16 lanes, then the
// two row broadcasts: six dependent steps instead of one lane read and one comparison per lane.
__device__ __forceinline__ float wave_max(float x)
{
    auto step = [](float v, auto ctrl, auto row_mask) {
        const int moved = __builtin_amdgcn_update_dpp(__float_as_int(-INFINITY), __float_as_int(v), decltype(ctrl)::value,
                                                      decltype(row_mask)::value, 0xF, false);
        return fmaxf(v, __int_as_float(moved));
    };
    using std::integral_constant;
    x = step(x, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});     // row_shr:1
    x = step(x, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});     // row_shr:2
    x = step(x, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});     // row_shr:4
    x = step(x, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});     // row_shr:8: lane 15 of a row holds the row's max
    x = step(x, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});     // row_bcast:15 into rows 1 and 3
    x = step(x, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});     // row_bcast:31 into rows 2 and 3: lane 63 holds the max
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// value of x in lane `src`; src must be the same in every lane (it is read into a scalar register)
__device__ __forceinline__ float lane_value(float x, int src)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), __builtin_amdgcn_readfirstlane(src)));
}

// ------------------------------------------------------------------------------------------------------------
// heads: the policy and value heads of a sample, then its action (actor) or its loss gradient (learner)
// ------------------------------------------------------------------------------------------------------------
struct HeadsArgs {
    const float *fc_part;      // h = relu(fc_bias + sum_g fc_part[g][B][512]), groups added in order, is formed here ...
    const float *fc_bias;
    float *h_out;              // ... and (learner) written out for the backward pass
    int nseg;                  // number of groups
    const float *wpi, *bpi, *wv, *bv;
    int B, A;
    // actor outputs
    uint64_t seed; uint32_t step; int env_offset;
    int32_t *actions; float *logp, *values, *logits_out;
    // learner inputs / outputs
    LossArgs la;
    float *dz, *dh, *terms;
    bf16_t *dh16;              // not null: dL/dh is written here in bfloat16 (the operand type of the FC layer's backward
};                             // kernels, which then fetch half the bytes; they rounded it the same way as they loaded it)

// The last steps of one sample, by one wavefront: lane j (< A) holds logit j.
// A wavefront runs alone on its SIMD here, so every dependent instruction costs its full latency, and the steps over
// the actions are kept to one instruction each: the maximum by lane shifts (six steps), the running sums by a shift
// and an add per action; lanes >= A hold neutral values (-inf for the maximum, +0 for the sums).  (Phase stamps:
// with one lane read and two or three instructions per action 2.3 of the kernel's 9.6 thousand clock ticks were
// spent here.)
__device__ __forceinline__ void sample_action(const HeadsArgs &a, int b, int lane, float mylogit, float u01)
{
    const int A = a.A;
    const float m = wave_max(lane < A ? mylogit : -INFINITY);
    // binary32 inverse CDF: lane j evaluates e_j once; the running sums c_j are formed sequentially in index order
    // along the lanes; lane j keeps c_j, and the action is the
    // first j with c_j > u * c_{A-1} (A-1 if there is none)
    // (c_j = c_{j-1} + e_j along the lanes: every step each lane takes its left neighbour's value -- lane 0 takes
    // +0 -- and adds its own e_j.  After k steps lanes 0..k hold their c_j and keep it, so A - 1 steps of one
    // instruction give every lane its running sum in index order; lane reads into scalar registers cost three
    // instructions per action.)
    const float ej = lane < A ? sampler_exp(mylogit - m) : 0.0f;
    float mine = ej;
    for (int k = 1; k < A; ++k)
        mine = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(mine), 0x138 /* wave_shr:1 */, 0xF, 0xF, true)) + ej;
    const float total = lane_value(mine, A - 1);
    const float thr = u01 * total;
    const unsigned long long above = __ballot(lane < A && mine > thr);
    const int act = above ? __ffsll((long long)above) - 1 : A - 1;
    const float la = lane_value(mylogit, act);
    if (lane == 0) {
        a.actions[b] = act;
        a.logp[b] = (la - m) - logf(total);
    }
    if (a.logits_out && lane < A) a.logits_out[(long long)b * A + lane] = mylogit;
}

// policy terms of one sample's loss: lane j (< A) receives dL/dlogit j (other lanes 0)
__device__ __forceinline__ float policy_gradient(const HeadsArgs &a, int b, int lane, float mylogit)
{
    const int A = a.A;
    const float m = wave_max(lane < A ? mylogit : -INFINITY);
    const long long row = a.la.index ? a.la.index[b] : b;
    const float e = lane < A ? expf(mylogit - m) : 0.0f;
    const float lse = m + logf(wave_sum(e));
    const float lsm = lane < A ? mylogit - lse : 0.0f;
    const float p = lane < A ? expf(lsm) : 0.0f;
    const float ent = -wave_sum(p * lsm);
    const int act = a.la.actions[row];
    const float logp = lane_value(lsm, act);
    const float adv = a.la.adv[row];
    const float invB = 1.0f / (float)a.B;
    float dlogp, pi_term, clipped = 0.0f, kl = 0.0f;
    if (a.la.algo == HTS_ALGO_A2C) {
        pi_term = -logp * adv;
        dlogp = -adv * invB;
    } else if (a.la.algo == HTS_ALGO_A2C_TIS) {
        // truncated importance weight, a constant in the derivative
        const float old = a.la.old_logp[row];
        const float rho = expf(logp - old);
        const float w = fminf(rho, a.la.rho_bar);
        pi_term = -w * logp * adv;
        dlogp = -w * adv * invB;
        clipped = rho > a.la.rho_bar ? 1.0f : 0.0f;
        kl = old - logp;
    } else {
        const float old = a.la.old_logp[row];
        const float rho = expf(logp - old);
        const float lo = 1.0f - a.la.clip_eps, hi = 1.0f + a.la.clip_eps;
        const float rc = fminf(fmaxf(rho, lo), hi);
        pi_term = -fminf(rho * adv, rc * adv);
        const bool cut = (adv > 0.0f && rho > hi) || (adv < 0.0f && rho < lo);
        dlogp = cut ? 0.0f : -adv * rho * invB;
        clipped = (rho > hi || rho < lo) ? 1.0f : 0.0f;
        kl = old - logp;
    }
    const float dl = lane < A ? dlogp * ((lane == act ? 1.0f : 0.0f) - p) + a.la.ent_coef * invB * p * (lsm + ent)
                              : 0.0f;
    if (lane < A) a.dz[(long long)b * (A + 1) + lane] = dl;
    if (lane == 0) {
        float *t = a.terms + (long long)b * N_TERMS;
        t[0] = pi_term; t[2] = ent; t[3] = clipped; t[4] = kl;
    }
    return dl;
}

// value term of one sample's loss; returns dL/dvalue
__device__ __forceinline__ float value_gradient(const HeadsArgs &a, int b, int lane, float value)
{
    const long long row = a.la.index ? a.la.index[b] : b;
    const float R = a.la.ret[row], invB = 1.0f / (float)a.B;
    float v_term = (R - value) * (R - value), dv_row = 2.0f * (value - R);
    if (a.la.value_clip > 0.0f) {
        // clipped value loss: the larger of the plain term and the term of the value held within a radius of
        // the stored estimate; a value held at the radius does not move with the network's output
        const float ov = a.la.old_values[row];
        const float d = value - ov;
        const float dc = fminf(fmaxf(d, -a.la.value_clip), a.la.value_clip);
        const float vc = ov + dc;
        const float c_term = (vc - R) * (vc - R);
        if (c_term > v_term) {
            v_term = c_term;
            dv_row = dc == d ? 2.0f * (vc - R) : 0.0f;
        }
    }
    const float dv = a.la.vf_coef * dv_row * invB;
    if (lane == 0) {
        a.dz[(long long)b * (a.A + 1) + a.A] = dv;
        a.terms[(long long)b * N_TERMS + 1] = v_term;
    }
    return dv;
}

// One workgroup of 8 wavefronts per S samples.  Thread t owns hidden unit t: it adds the unit's FC group sums, bias and ReLU
// into LDS.  A wavefront then forms its share of the A + 1 dot products of every sample, at most HEADS_ROWS at a time (lane l:
// the 8-element partial of units 8 l .. 8 l + 7, into the sample's LDS panel [A + 1][65]); wavefront s adds the panel's rows
// of sample s in a fixed order and finishes its policy head, wavefront 4 + s its value head.  (learner) Thread t
// forms dL/d(pre-activation) of unit t.  Everything a workgroup needs from memory is requested before anything is waited for.
// What bounds it: with few samples one memory round trip and the chain of dependent steps (one wavefront per sample did all
// of it alone, a few thousand instructions at full latency each: 5.0 us at 16 rows against 3.9); with many the fetches --
// the heads are 40 KB a workgroup, whatever S (actor at 1024 / 4096 rows, with
// one wavefront per sample and a fetch of its own: 6.9 / 18 us, now 5.7 / 9.0; learner at 2048: 18.4, now 12.8).
constexpr int HEADS_WAVES = 8, HEADS_ROWS = 3;
template <bool LEARN, int S>
__global__ __launch_bounds__(64 * HEADS_WAVES) void heads_kernel(const HeadsArgs a)
{
    __shared__ __attribute__((aligned(16))) float h_lds[S][512], row_lds[S][HTS_MAX_ACTIONS + 4];
    extern __shared__ float heads_panels[];            // [S][A + 1][65]
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), A = a.A;
    const int b0 = blockIdx.x * S;
    float wrow[HEADS_ROWS][8];
    auto fetch_rows = [&](int j0) {                    // rows j0, j0 + 8, ... of the heads (row A: value head)
#pragma unroll
        for (int i = 0; i < HEADS_ROWS; ++i) {
            const int j = min(j0 + i * HEADS_WAVES, A);
            load_vec((j < A ? a.wpi + (long long)j * 512 : a.wv) + lane * 8, wrow[i]);
        }
    };
    fetch_rows(w);
    const long long gstride = (long long)a.B * 512;
    constexpr int GQ = S > 2 ? 4 : 8;                  // group sums of a unit in flight per sample
    float pv[S][GQ];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int q = 0; q < GQ; ++q) pv[s][q] = a.fc_part[(long long)min(b0 + s, a.B - 1) * 512 + tid + min(q, a.nseg - 1) * gstride];
    const float bias = a.fc_bias[tid];
    const float head_bias = lane < A ? a.bpi[lane] : 0.0f, value_bias = a.bv[0];
    constexpr int HELD = 20;                           // rows of the heads whose column `tid` is held in registers for dL/dh
    float wcol[LEARN ? HELD : 1], wvt = 0.0f;
    if constexpr (LEARN) {
        wvt = a.wv[tid];
#pragma unroll
        for (int j = 0; j < HELD; ++j) wcol[j] = a.wpi[min(j, A - 1) * 512 + tid];
    }
    float u01 = 0.0f;          // the sample's uniform: needs nothing from memory, so it is formed while the loads travel
    if constexpr (!LEARN) { if (w < S) u01 = seeded_uniform(a.seed, (uint32_t)(a.env_offset + b0 + w), a.step); }
    float h[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {                      // groups added in group order, then bias + ReLU
        const int b = min(b0 + s, a.B - 1);
        float x = 0.0f;
#pragma unroll
        for (int q = 0; q < GQ; ++q) if (q < a.nseg) x += pv[s][q];
        for (int q0 = GQ; q0 < a.nseg; q0 += GQ) {
            float more[GQ];
#pragma unroll
            for (int q = 0; q < GQ; ++q) more[q] = a.fc_part[(long long)b * 512 + tid + min(q0 + q, a.nseg - 1) * gstride];
#pragma unroll
            for (int q = 0; q < GQ; ++q) if (q0 + q < a.nseg) x += more[q];
        }
        x += bias;
        h[s] = x > 0.0f ? x : 0.0f;
        h_lds[s][tid] = h[s];
        if constexpr (LEARN) { if (b0 + s < a.B) a.h_out[(long long)b * 512 + tid] = h[s]; }
    }
    __syncthreads();
    for (int j0 = w; j0 <= A; j0 += HEADS_ROWS * HEADS_WAVES) {
        if (j0 != w) fetch_rows(j0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const f32x4 h0 = *reinterpret_cast<const f32x4 *>(&h_lds[s][lane * 8]), h1 = *reinterpret_cast<const f32x4 *>(&h_lds[s][lane * 8 + 4]);
            float d[HEADS_ROWS];
#pragma unroll
            for (int i = 0; i < HEADS_ROWS; ++i) {
                d[i] = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) d[i] = __builtin_fmaf(h0[e], wrow[i][e], d[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) d[i] = __builtin_fmaf(h1[e], wrow[i][4 + e], d[i]);
            }
#pragma unroll
            for (int i = 0; i < HEADS_ROWS; ++i)
                if (j0 + i * HEADS_WAVES <= A) heads_panels[(s * (A + 1) + j0 + i * HEADS_WAVES) * 65 + lane] = d[i];
        }
    }
    __syncthreads();
    static_assert(S <= 4 && HEADS_WAVES == 8, "wavefronts 0-3: policy heads, 4-7: value heads");
    const int ws = w & 3, b = b0 + ws;
    if (ws < S && b < a.B) {
        const float *panel = heads_panels + ws * (A + 1) * 65;
        if (w < 4) {
            // row sums: with A <= 32 (<= 16) rows, two (four) lanes share a row, each adding a contiguous half (quarter)
            // in lane order; the parts are then added in part order
            const int parts = A <= 16 ? 4 : (A <= 32 ? 2 : 1);
            const int rows_per = 64 / parts, len = 64 / parts;
            const int row = lane & (rows_per - 1), part = lane / rows_per;
            float rowsum = 0.0f;
            if (row < A) {
                const float *rp = panel + row * 65 + part * len;
                for (int t = 0; t < len; t += 16) {
                    float tv[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) tv[u] = rp[t + u];
#pragma unroll
                    for (int u = 0; u < 16; ++u) rowsum += tv[u];
                }
            }
            float tot = rowsum;
            for (int q = 1; q < parts; ++q) tot += __shfl(rowsum, row + q * rows_per, 64);
            const float logit = lane < A ? tot + head_bias : 0.0f;
            if constexpr (!LEARN) sample_action(a, b, lane, logit, u01);
            else {
                const float dl = policy_gradient(a, b, lane, logit);
                if (lane < A) row_lds[ws][lane] = dl;
            }
        } else {
            const float value = wave_sum(panel[A * 65 + lane]) + value_bias;
            if constexpr (!LEARN) { if (lane == 0) a.values[b] = value; }
            else {
                const float dv = value_gradient(a, b, lane, value);
                if (lane == 0) row_lds[ws][A] = dv;
            }
        }
    }
    if constexpr (LEARN) {
        __syncthreads();
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (b0 + s >= a.B) break;
            const float *row = row_lds[s];
            float acc = row[A] * wvt;
#pragma unroll
            for (int j = 0; j < HELD; ++j) if (j < A) acc = __builtin_fmaf(row[j], wcol[j], acc);
            for (int j = HELD; j < A; ++j) acc = __builtin_fmaf(row[j], a.wpi[j * 512 + tid], acc);
            acc = h[s] > 0.0f ? acc : 0.0f;
            if (a.dh16) a.dh16[(long long)(b0 + s) * 512 + tid] = from_f32<bf16_t>(acc); else a.dh[(long long)(b0 + s) * 512 + tid] = acc;
        }
    }
}

// sampling alone, from given logits: one wavefront per sample
__global__ __launch_bounds__(64) void sample_kernel(const HeadsArgs a, const float *__restrict__ logits)
{
    const int lane = threadIdx.x, b = blockIdx.x;
    const float logit = lane < a.A ? logits[(long long)b * a.A + lane] : 0.0f;
    sample_action(a, b, lane, logit, seeded_uniform(a.seed, (uint32_t)(a.env_offset + b), a.step));
}

template <bool LEARN> static hipError_t launch_heads(const HeadsArgs &a, hipStream_t stream)
{
    // Kernel time at S = 1 / 2 / 4, us.  Learner: one round of workgroups of a single sample ends at 768 rows (three fit a compute unit),
    // of two samples at 1024 (two fit): 512 6.3/6.4/8.9, 768 6.9/7.0/9.2, 832 9.5/7.4/8.7, 1024 10.8/7.5/9.0, 1152 11.4/11.0/10.7, 1536
    // 12.7/11.8/11.0, 2048 17.9/15.3/13.1 on 84x84 frames (seven slices of FC sums); 1152 12.4/12.8/11.3, 1536 13.7/13.4/11.6 on 72x96 (five).
    // Actor (more workgroups fit): 16 rows 3.8/4.2/5.7, 768 5.0/5.2/5.8, 1024 5.9/5.8/6.0, 1100 7.4/6.3/7.6, 1536 8.6/6.7/7.8, 2048
    // 9.4/8.4/8.4, 2560 10.6/9.9/10.0, 3072 12.1/11.3/10.7, 3584 13.9/12.8/13.4, 4096 (one slice) 14.6/12.1/8.2; 72x96: 3072 12.3/11.1/10.4,
    // 3584 14.0/12.3/13.0: two and four are level from 2048 to 4095 rows, one slice decides for four.
    const int S = a.A > 32 || a.B <= (LEARN ? 512 : 1024) ? 1 : a.B <= (LEARN ? 1024 : 3072) ? 2 : 4;
    auto kern = S == 1 ? heads_kernel<LEARN, 1> : S == 2 ? heads_kernel<LEARN, 2> : heads_kernel<LEARN, 4>;
    hipLaunchKernelGGL(kern, dim3((a.B + S - 1) / S), dim3(64 * HEADS_WAVES), (size_t)S * (a.A + 1) * 65 * sizeof(float), stream, a);
    return hipGetLastError();
}

static void heads_network(const Ctx &c, HeadsArgs &a)
{
    const float *hb = c.ws.hb;
    a.wpi = hb + c.sh.piw; a.bpi = hb + c.sh.pib; a.wv = hb + c.sh.vw; a.bv = hb + c.sh.vb;
    a.fc_part = c.ws.fc_part; a.fc_bias = hb + c.sh.fcb; a.nseg = c.fc_slices;
}

// logits_in != null: sample from these logits (no network involved); otherwise finish the forward pass first.
hipError_t launch_heads_act(Ctx &c, const float *logits_in, uint64_t seed, uint32_t step, int N, int env_offset,
                            int32_t *actions, float *logp, float *values, float *logits_out)
{
    SiteTimer tm(c, SITE_HEADS_ACT);
    HeadsArgs a = {};
    a.B = N; a.A = c.g.A;
    a.seed = seed; a.step = step; a.env_offset = env_offset;
    a.actions = actions; a.logp = logp; a.values = values; a.logits_out = logits_out;
    if (logits_in) {
        hipLaunchKernelGGL(sample_kernel, dim3(N), dim3(64), 0, c.stream, a, logits_in);
        return hipGetLastError();
    }
    heads_network(c, a);
    return launch_heads<false>(a, c.stream);
}

hipError_t launch_heads_learn(Ctx &c, const LossArgs &la, int B)
{
    SiteTimer tm(c, SITE_HEADS_LEARN);
    HeadsArgs a = {};
    heads_network(c, a);
    a.h_out = c.ws.h;
    a.B = B; a.A = c.g.A;
    a.la = la;
    a.dz = c.ws.dz; a.terms = c.ws.terms;
    if (c.desc.precision == HTS_PRECISION_BF16) a.dh16 = reinterpret_cast<bf16_t *>(c.ws.dh); else a.dh = c.ws.dh;
    return launch_heads<true>(a, c.stream);
}

// Sum over a workgroup of 256 threads, in thread 0: pairs 128, 64, ... 1 apart, one barrier (the last six steps are lane shifts of the first
// wavefront)
__device__ __forceinline__ float block_sum_256(float x, float *red)
{
    const int t = threadIdx.x;
    red[t] = x;
    __syncthreads();
    if (t < 64) {
        x = (red[t] + red[t + 128]) + (red[t + 64] + red[t + 192]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) x += __shfl_down(x, o, 64);
    }
    return x;
}

// ||g|| from the per-chunk sums, added in a fixed order by one workgroup of 256 threads (every thread gets the result)
__device__ __forceinline__ float norm_from_parts(const float *__restrict__ part, int nparts, float *red)
{
    const int t = threadIdx.x;
    float s = 0.0f;
    for (int i = t; i < nparts; i += 256) s += part[i];
    s = block_sum_256(s, red);
    __syncthreads();
    if (t == 0) red[0] = s;
    __syncthreads();
    return sqrtf(red[0]);
}

// ------------------------------------------------------------------------------------------------------------
// loss statistics: one workgroup, fixed strided sums then a fixed LDS tree
// ------------------------------------------------------------------------------------------------------------
// (the norm from its per-chunk sums, as the optimiser kernel forms it: a launch for it alone took 4.7 us)
__global__ __launch_bounds__(256) void stats_kernel(const float *__restrict__ terms, int B, const float *__restrict__ norm_part, int nparts,
                                                    hts_stats *stats)
{
    __shared__ float red[N_TERMS + 1][256];
    const int t = threadIdx.x;
    float s[N_TERMS];
#pragma unroll
    for (int i = 0; i < N_TERMS; ++i) s[i] = 0.0f;
#pragma unroll 4
    for (int b = t; b < B; b += 256)
#pragma unroll
        for (int i = 0; i < N_TERMS; ++i) s[i] += terms[(long long)b * N_TERMS + i];
#pragma unroll
    for (int i = 0; i < N_TERMS; ++i) s[i] = block_sum_256(s[i], red[i]);
    const float gn = norm_from_parts(norm_part, nparts, red[N_TERMS]);
    if (t == 0) {
        const float invB = 1.0f / (float)B;
        stats->policy_loss = s[0] * invB;
        stats->value_loss = s[1] * invB;
        stats->entropy = s[2] * invB;
        stats->clip_frac = s[3] * invB;
        stats->approx_kl = s[4] * invB;
        stats->grad_norm = gn;
        const float chk = s[0] + s[1] + s[2] + gn;
        stats->nonfinite = (chk - chk == 0.0f) ? 0 : 1;
    }
}

hipError_t launch_stats(Ctx &c, int B, hts_stats *stats)
{
    SiteTimer tm(c, SITE_STATS);
    hipLaunchKernelGGL(stats_kernel, dim3(1), dim3(256), 0, c.stream, c.ws.terms, B, c.ws.norm_part,
                       (int)((c.g.P + NORM_CHUNK - 1) / NORM_CHUNK), stats);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Combine of the split conv weight gradients, all three layers in one launch:
// g[dest(n,kcol)] = scale * sum_z part[z][n][kcol].  A workgroup owns 32 consecutive outputs; its 8 lane groups sum
// 8 contiguous ranges of z (loads in flight eight at a time, added in z order) and the 8 range sums are added in
// range order -- a fixed shape, so the result is reproducible.
// ------------------------------------------------------------------------------------------------------------
struct ReduceJob {
    const float *part;
    int nz, rows, ncol, cin, ksz, taps_outer, first_block;
    long long zstride;
    float scale;
    long long w_off, b_off;
};
struct ReduceArgs { ReduceJob job[REDUCE_JOBS]; float *g; };

__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const ReduceArgs a)
{
    __shared__ float red[8][33];
    const int blk = blockIdx.x;
    int jn = 0;
#pragma unroll
    for (int t = 1; t < REDUCE_JOBS; ++t) jn = blk >= a.job[t].first_block ? t : jn;       // first_block is non-decreasing
    const ReduceJob &jb = a.job[jn];
    const int e = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int n_el = jb.rows * jb.ncol;
    const int i = (blk - jb.first_block) * 32 + e;
    const long long zs = jb.zstride;
    const int chunk = (jb.nz + 7) / 8;
    int z = q * chunk;
    const int z1 = min(jb.nz, z + chunk);
    float s = 0.0f;
    if (i < n_el) {
        const float *src = jb.part + i;
        for (; z + 8 <= z1; z += 8) {
            float v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = src[(z + t) * zs];
#pragma unroll
            for (int t = 0; t < 8; ++t) s += v[t];
        }
        for (; z < z1; ++z) s += src[z * zs];
    }
    red[q][e] = s;
    __syncthreads();
    if (q != 0 || i >= n_el) return;
    float tot = red[0][e];
#pragma unroll
    for (int t = 1; t < 8; ++t) tot += red[t][e];
    tot *= jb.scale;
    const int n = i / jb.ncol, kcol = i - n * jb.ncol;
    const int kc = jb.ncol - 1;
    if (kcol == kc) { a.g[jb.b_off + n] = tot; return; }
    long long dst;
    if (jb.taps_outer) {              // kcol = (tap, c)  ->  w[n][c][tap]
        const int tap = kcol / jb.cin, c = kcol - tap * jb.cin;
        dst = ((long long)n * jb.cin + c) * (jb.ksz * jb.ksz) + tap;
    } else dst = (long long)n * kc + kcol;
    a.g[jb.w_off + dst] = tot;
}

hipError_t launch_wgrad_reduce(Ctx &c, const ReduceSpec (&spec)[REDUCE_JOBS], float *g)
{
    SiteTimer tm(c, SITE_WGRAD_REDUCE);
    ReduceArgs a;
    int blocks = 0;
    for (int j = 0; j < REDUCE_JOBS; ++j) {
        const ReduceSpec &sp = spec[j];
        ReduceJob &jb = a.job[j];
        jb.part = sp.part; jb.nz = sp.nz; jb.rows = sp.rows; jb.ncol = sp.ncol; jb.cin = sp.cin; jb.ksz = sp.ksz;
        jb.taps_outer = sp.taps_outer ? 1 : 0; jb.scale = sp.scale; jb.w_off = sp.w_off; jb.b_off = sp.b_off;
        jb.zstride = sp.zstride ? sp.zstride : (long long)sp.rows * sp.ncol;
        jb.first_block = blocks;
        if (sp.nz > 0) blocks += (sp.rows * sp.ncol + 31) / 32;
    }
    a.g = g;
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(blocks), dim3(256), 0, c.stream, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// returns / GAE: one lane per environment column, reverse time; neighbouring lanes read neighbouring columns
// ------------------------------------------------------------------------------------------------------------
constexpr int GAE_U = 8;
// The recurrence runs in double precision inside the lane (inputs and outputs are fp32), so a long unroll does not
// accumulate binary32 rounding: each output is the correctly rounded result of an almost exact recurrence.
// (Outputs in the place of inputs are fine: what is stored to a row depends on everything that is read of it, and no row is
// read twice.  Without __restrict__ 128x262144 takes 128 us instead of 111.)
__global__ __launch_bounds__(64) void gae_kernel(const float *__restrict__ r, const float *__restrict__ v,
                                                 const uint8_t *__restrict__ d, float gamma, float lambda, int T, int N,
                                                 float *__restrict__ adv, float *__restrict__ ret)
{
    const int n = blockIdx.x * 64 + threadIdx.x;
    if (n >= N) return;
    const double g = (double)gamma, gl = (double)gamma * (double)lambda;
    double a = 0.0;
    double vnext = (double)v[(long long)T * N + n];
    int t = T - 1;
    for (; t >= GAE_U - 1; t -= GAE_U) {
        float rr[GAE_U], vv[GAE_U];
        uint8_t dd[GAE_U];
#pragma unroll
        for (int i = 0; i < GAE_U; ++i) {
            const long long o = (long long)(t - i) * N + n;
            rr[i] = r[o]; vv[i] = v[o]; dd[i] = d[o];
        }
#pragma unroll
        for (int i = 0; i < GAE_U; ++i) {
            const long long o = (long long)(t - i) * N + n;
            const double nd = dd[i] ? 0.0 : 1.0;
            const double delta = (double)rr[i] + g * nd * vnext - (double)vv[i];
            a = delta + gl * nd * a;
            adv[o] = (float)a;
            ret[o] = (float)(a + (double)vv[i]);
            vnext = (double)vv[i];
        }
    }
    for (; t >= 0; --t) {
        const long long o = (long long)t * N + n;
        const double vt = (double)v[o];
        const double nd = d[o] ? 0.0 : 1.0;
        const double delta = (double)r[o] + g * nd * vnext - vt;
        a = delta + gl * nd * a;
        adv[o] = (float)a;
        ret[o] = (float)(a + vt);
        vnext = vt;
    }
}

// Time-chunked form: a workgroup owns COLS columns and walks time backwards in spans
// of TC chunks of GAE_L steps, one chunk per thread, 64 / COLS chunks per wavefront.  A thread holds its chunk in registers
// (one memory round trip per span).  A_t = delta_t + c_t A_{t+1} is affine in the advantage entering a chunk, so every
// chunk is first reduced to a map (S, P), A_first = S + P * A_entering; the maps are composed by lane shifts inside a
// wavefront and through LDS across wavefronts, and every chunk is then replayed from what truly enters it.  Double
// precision throughout, so the result equals the one-lane-per-column recurrence to well below binary32 rounding.
// Steps before t = 0 (a last, partial span) have S = 0 and P = 1 and write nothing.
// The outputs may take the place of inputs (no __restrict__): a span reads all of its rows before it writes any, and the value
// behind a span's last step, whose row the span after it in time has written already, comes through LDS from the thread that read it.
constexpr int GAE_L = 8, GAE_MAX_WAVES = 8;
template <int COLS> __global__ __launch_bounds__(64 * GAE_MAX_WAVES) void gae_chunked_kernel(
    const float *r, const float *v, const uint8_t *d, float gamma, float lambda, int T, int N, float *adv, float *ret)
{
    __shared__ double sS[2][GAE_MAX_WAVES][COLS], sP[2][GAE_MAX_WAVES][COLS];
    __shared__ float sV[2][COLS];                                // value of the span's first step
    const int waves = blockDim.x >> 6, TC = blockDim.x / COLS;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cx = threadIdx.x % COLS, cc = threadIdx.x / COLS;
    const int n = blockIdx.x * COLS + cx;
    const bool live = n < N;
    const long long col = live ? n : N - 1;
    const double g = (double)gamma, gl = (double)gamma * (double)lambda;
    double enter = 0.0;                                          // advantage entering the span from later times
    int buf = 0;
    for (int tend = T; tend > 0; tend -= TC * GAE_L, buf ^= 1) {
        const int t0 = tend - (TC - cc) * GAE_L;                 // this thread's chunk [t0, t0 + GAE_L); negative steps do not exist
        float rr[GAE_L], vv[GAE_L + 1];
        uint8_t dd[GAE_L];
#pragma unroll
        for (int i = 0; i < GAE_L; ++i) {
            const long long o = (long long)max(t0 + i, 0) * N + col;
            rr[i] = r[o]; vv[i] = v[o]; dd[i] = d[o];
        }
        vv[GAE_L] = v[(long long)max(t0 + GAE_L, 0) * N + col];
        if (tend != T && cc == TC - 1) vv[GAE_L] = sV[buf ^ 1][cx];
        double S = 0.0, P = 1.0;
#pragma unroll
        for (int i = GAE_L - 1; i >= 0; --i) {
            const double nd = dd[i] ? 0.0 : 1.0;
            const double delta = (double)rr[i] + g * nd * (double)vv[i + 1] - (double)vv[i], ct = gl * nd;
            if (t0 + i >= 0) { S = delta + ct * S; P = ct * P; }
        }
        // this chunk's map composed with those of the later chunks of the wavefront, then the later chunks' alone
#pragma unroll
        for (int o = COLS; o < 64; o <<= 1) {
            const double Sl = __shfl_down(S, o, 64), Pl = __shfl_down(P, o, 64);
            if (lane + o < 64) { S = S + P * Sl; P = P * Pl; }
        }
        if (lane < COLS) { sS[buf][w][lane] = S; sP[buf][w][lane] = P; }
        double Se = 0.0, Pe = 1.0;
        if constexpr (COLS < 64) {
            const double Sl = __shfl_down(S, COLS, 64), Pl = __shfl_down(P, COLS, 64);
            if (lane + COLS < 64) { Se = Sl; Pe = Pl; }
        }
        if (cc == 0) sV[buf][cx] = vv[0];
        __syncthreads();
        double a = enter, all = enter;                           // entering this wavefront's chunks; leaving the span
#pragma unroll
        for (int q = GAE_MAX_WAVES - 1; q >= 0; --q) {
            const double Sq = q < waves ? sS[buf][q][cx] : 0.0, Pq = q < waves ? sP[buf][q][cx] : 1.0;
            all = Sq + Pq * all;
            if (q > w) a = all;
        }
        enter = all;
        a = Se + Pe * a;
#pragma unroll
        for (int i = GAE_L - 1; i >= 0; --i) {
            const double nd = dd[i] ? 0.0 : 1.0;
            const double delta = (double)rr[i] + g * nd * (double)vv[i + 1] - (double)vv[i];
            a = delta + gl * nd * a;
            const long long o = (long long)(t0 + i) * N + col;
            if (live && t0 + i >= 0) { adv[o] = (float)a; ret[o] = (float)(a + (double)vv[i]); }
        }
    }
}

hipError_t launch_gae(Ctx *c, hipStream_t s, const float *r, const float *v, const uint8_t *d, float gamma, float lambda,
                      int T, int N, float *adv, float *ret)
{
    Ctx dummy;
    SiteTimer tm(c ? *c : dummy, SITE_GAE);
    // Kernel time by rocprofv3, us: plain / 4 / 16 / 64 columns a workgroup
    //   plain to 11 steps (a second chunk is mostly padding): 5x16 1.7/3.2/2.6/2.3, 9x48 2.4/4.0/3.5/2.9, 10x300 3.4/4.0/4.0/3.5, 11x70000
    //   5.8/-/-/5.6, 11x100000 5.6/-/-/6.5; 12x48 2.8/3.9/3.3/2.6, 12x300 3.7/4.0/4.0/3.7, 12x70000 5.9/-/8.0/5.6
    //   plain from 131072 columns, which hide a lane's serial walk: 128x262144 107/641/222/114, 20x140000 10.8/-/17/11.3, but 128x120000
    //   58/-/80/49, 256x100000 151/-/136/95; where a workgroup of 64 columns has five to eight wavefronts (33 to 64 steps; 65 to 96 are
    //   two such spans) few of them fit a compute unit: from 81920 columns on 40x80000 15.0/14.4, 40x90000 15.7/16.9, 80x100000 28/30
    //   64 columns, whole cache lines per load: 128x16384 29/39/13/8.0, 128x10240 18/-/8.7/7.3, 128x8192 18/-/6.6/7.2; to 40 steps at any
    //   width: 16x48 3.4/3.9/3.3/2.9, 30x4096 6.2/5.0/4.0/3.9, 40x300 7.2/-/4.2/4.0, 48x16 7.2/-/3.0/3.3
    //   4 columns beyond 256 steps, the span of 16 columns: 256x16 32/3.8/3.4/9.1, 288x16 37/4.0/5.3/11, 512x16 64/4.1/5.8/17, as long as
    //   its quarter cache lines don't count; the two meet at 900 columns for 288 steps, 700 for 384, 512 for 512, 450 for 700 and 1024,
    //   500 for 2048, 700 for 4096 (512x400 5.8/6.9, 512x640 7.9/6.9, 2048x256 18.2/19.8, 2048x900 31/28)
    //   16 else: 128x32 17/3.9/3.5/5.3, 128x4096 18/11/4.9/6.7, 512x1024 65/11/7.2/18
    // (with a chunk's rows fetched twice and one at a time, 32 columns: 512x16 12.2, 128x4096 8.0)
    if (T < 12 || N >= (T > 32 && T <= 96 ? 81920 : 131072)) {
        hipLaunchKernelGGL(gae_kernel, dim3((N + 63) / 64), dim3(64), 0, s, r, v, d, gamma, lambda, T, N, adv, ret);
    } else {
        const int cols = N > 8192 || T <= 40 ? 64 : T > 256 && N <= 512 ? 4 : 16;
        const int per_wave = 64 / cols, chunks = (T + GAE_L - 1) / GAE_L;
        int waves = (chunks + per_wave - 1) / per_wave;
        if (waves > GAE_MAX_WAVES) waves = GAE_MAX_WAVES;
        auto kern = cols == 4 ? gae_chunked_kernel<4> : cols == 16 ? gae_chunked_kernel<16> : gae_chunked_kernel<64>;
        hipLaunchKernelGGL(kern, dim3((N + cols - 1) / cols), dim3(64 * waves), 0, s, r, v, d, gamma, lambda, T, N, adv, ret);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// advantage normalisation: double-precision sums of fixed shape.  Up to NRM_ONE entries one workgroup holds the array in
// registers (one launch); beyond that up to NRM_BLOCKS workgroups each reduce a share and a second launch combines
// their sums and rescales.  Kernel times by rocprofv3: 512x16 entries 6.2 us as three strided passes of one workgroup over
// memory, 3.3 us from registers (launch, one memory round trip, two reductions across 8 wavefronts); 128x4096 entries
// 281 us with one workgroup (2 MB through one compute unit three times), 3.3 + 3.9 us (two launches; 6 MB moved).
// ------------------------------------------------------------------------------------------------------------
constexpr int NRM_ONE_THREADS = 1024, NRM_ONE_VECS = 4;                       // 4-entry vectors per thread, one workgroup
constexpr int NRM_ONE = NRM_ONE_THREADS * NRM_ONE_VECS * 4;
constexpr int NRM_THREADS = 256;

// sum over a workgroup of NT threads, returned to every thread; red: NT / 64 doubles that nobody else writes
template <int NT> __device__ __forceinline__ double block_sum_f64(double x, double *red)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) s += red[i];
    return s;
}
// entries 4 v .. 4 v + 3, zeros behind entry n - 1; VEC: adv is 16-byte aligned
template <bool VEC> __device__ __forceinline__ f32x4 load_entries(const float *adv, long long v, long long n)
{
    if (VEC && 4 * v + 4 <= n) return *reinterpret_cast<const f32x4 *>(adv + 4 * v);
    f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) if (4 * v + e < n) x[e] = adv[4 * v + e];
    return x;
}
template <bool VEC> __device__ __forceinline__ void store_entries(float *adv, long long v, long long n, const f32x4 &x)
{
    if (VEC && 4 * v + 4 <= n) { *reinterpret_cast<f32x4 *>(adv + 4 * v) = x; return; }
#pragma unroll
    for (int e = 0; e < 4; ++e) if (4 * v + e < n) adv[4 * v + e] = x[e];
}

template <bool VEC, int NT> __global__ __launch_bounds__(NT) void normalize_one_kernel(float *__restrict__ adv, int n)
{
    __shared__ double red[2][NT / 64];
    const int t = threadIdx.x;
    f32x4 x[NRM_ONE_VECS];
#pragma unroll
    for (int i = 0; i < NRM_ONE_VECS; ++i) x[i] = load_entries<VEC>(adv, t + i * NT, n);
    double s = 0.0, q = 0.0;
#pragma unroll
    for (int i = 0; i < NRM_ONE_VECS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) s += (double)x[i][e];
    const double mean = block_sum_f64<NT>(s, red[0]) / (double)n;
#pragma unroll
    for (int i = 0; i < NRM_ONE_VECS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d = 4 * (t + i * NT) + e < n ? (double)x[i][e] - mean : 0.0;
            q += d * d;
        }
    const double var = block_sum_f64<NT>(q, red[1]) / (double)(n > 1 ? n - 1 : 1);
    const double inv = 1.0 / (sqrt(var) + 1e-5);
#pragma unroll
    for (int i = 0; i < NRM_ONE_VECS; ++i) {
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (float)(((double)x[i][e] - mean) * inv);
        store_entries<VEC>(adv, t + i * NT, n, y);
    }
}

// One workgroup's share of the sums about the first entry x_0: part[1 + 2i] = sum (x - x_0), part[2 + 2i] = sum (x - x_0)^2,
// part[0] = x_0.  var = (q - s^2/n) / (n-1) then cancels little: s^2/n = n (mean - x_0)^2, and x_0's own term already
// makes the sum of squares about the mean at least (mean - x_0)^2, so at most a factor n of double precision's 2^-53.
// Calls without a context have no workspace and share one array per GPU.  All of them go to the default stream, which keeps a
// call's two launches in order; normalize_mutex keeps another thread's from coming between them.
__device__ double normalize_scratch[1 + 2 * NRM_BLOCKS];
static std::mutex normalize_mutex;
template <bool VEC> __global__ __launch_bounds__(NRM_THREADS) void normalize_sums_kernel(const float *__restrict__ adv, long long n,
                                                                                         double *part)
{
    __shared__ double red[2][NRM_THREADS / 64];
    if (!part) part = normalize_scratch;
    const double x0 = (double)adv[0];
    const long long stride = (long long)gridDim.x * NRM_THREADS, nv = (n + 3) >> 2;
    double s = 0.0, q = 0.0;
    for (long long v = (long long)blockIdx.x * NRM_THREADS + threadIdx.x; v < nv; v += 2 * stride) {
        const f32x4 x[2] = {load_entries<VEC>(adv, v, n), load_entries<VEC>(adv, v + stride < nv ? v + stride : v, n)};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double d = 4 * (v + i * stride) + e < n ? (double)x[i][e] - x0 : 0.0;
                s += d; q += d * d;
            }
    }
    const double bs = block_sum_f64<NRM_THREADS>(s, red[0]), bq = block_sum_f64<NRM_THREADS>(q, red[1]);
    if (threadIdx.x == 0) {
        part[1 + 2 * blockIdx.x] = bs; part[2 + 2 * blockIdx.x] = bq;
        if (blockIdx.x == 0) part[0] = x0;
    }
}
// launched with the grid of the kernel above: every workgroup adds all shares' sums in the same order
template <bool VEC> __global__ __launch_bounds__(NRM_THREADS) void normalize_apply_kernel(float *__restrict__ adv, long long n,
                                                                                          const double *part)
{
    static_assert(NRM_BLOCKS <= NRM_THREADS, "one share per thread");
    __shared__ double red[2][NRM_THREADS / 64];
    if (!part) part = normalize_scratch;
    const long long stride = (long long)gridDim.x * NRM_THREADS, nv = (n + 3) >> 2;
    const long long v0 = (long long)blockIdx.x * NRM_THREADS + threadIdx.x;
    f32x4 x = load_entries<VEC>(adv, v0 < nv ? v0 : 0, n);
    const int t = threadIdx.x;
    const double x0 = part[0], ps = t < (int)gridDim.x ? part[1 + 2 * t] : 0.0, pq = t < (int)gridDim.x ? part[2 + 2 * t] : 0.0;
    const double s = block_sum_f64<NRM_THREADS>(ps, red[0]), q = block_sum_f64<NRM_THREADS>(pq, red[1]);
    // (rounding may leave a sum of squares just below zero; a NaN, from an infinity or a NaN among the entries, stays one and
    // makes every result NaN, as the one-workgroup kernel's two passes do)
    const double sq = q - s * (s / (double)n), mean = x0 + s / (double)n, var = (sq < 0.0 ? 0.0 : sq) / (double)(n - 1);
    const double inv = 1.0 / (sqrt(var) + 1e-5);
    for (long long v = v0; v < nv; v += stride) {
        const f32x4 next = load_entries<VEC>(adv, v + stride < nv ? v + stride : v, n);
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (float)(((double)x[e] - mean) * inv);
        store_entries<VEC>(adv, v, n, y);
        x = next;
    }
}

hipError_t launch_normalize(Ctx *c, hipStream_t s, float *adv, long long n)
{
    Ctx dummy;
    SiteTimer tm(c ? *c : dummy, SITE_NORMALIZE);
    const bool vec = !((uintptr_t)adv & 15u);
    if (n <= NRM_ONE) {
        // as few wavefronts as hold the array, four, eight or sixteen: the launch and the two reductions take 3.0, 3.3 and 4.8 us
        const int nt = n <= NRM_ONE / 4 ? NRM_ONE_THREADS / 4 : n <= NRM_ONE / 2 ? NRM_ONE_THREADS / 2 : NRM_ONE_THREADS;
        auto kern = nt == NRM_ONE_THREADS / 4   ? (vec ? normalize_one_kernel<true, NRM_ONE_THREADS / 4> : normalize_one_kernel<false, NRM_ONE_THREADS / 4>)
                    : nt == NRM_ONE_THREADS / 2 ? (vec ? normalize_one_kernel<true, NRM_ONE_THREADS / 2> : normalize_one_kernel<false, NRM_ONE_THREADS / 2>)
                                                : (vec ? normalize_one_kernel<true, NRM_ONE_THREADS> : normalize_one_kernel<false, NRM_ONE_THREADS>);
        hipLaunchKernelGGL(kern, dim3(1), dim3(nt), 0, s, adv, (int)n);
        return hipGetLastError();
    }
    double *part = c ? c->ws.adv_part : nullptr;
    std::unique_lock<std::mutex> pair(normalize_mutex, std::defer_lock);
    if (!part) pair.lock();
    const long long need = ((n + 3) / 4 + NRM_THREADS - 1) / NRM_THREADS;
    const dim3 grid((unsigned)(need < NRM_BLOCKS ? need : NRM_BLOCKS));
    hipLaunchKernelGGL(vec ? normalize_sums_kernel<true> : normalize_sums_kernel<false>, grid, dim3(NRM_THREADS), 0, s, adv, n, part);
    hipLaunchKernelGGL(vec ? normalize_apply_kernel<true> : normalize_apply_kernel<false>, grid, dim3(NRM_THREADS), 0, s, adv, n, part);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// gradient norm: per-chunk sums of squares (fixed chunking), combined in index order where they are used
// ------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sumsq_kernel(const float *__restrict__ g, long long P, float *__restrict__ part)
{
    __shared__ float red[256];
    const int t = threadIdx.x;
    const long long base = (long long)blockIdx.x * NORM_CHUNK;
    // all of a thread's loads at once, one memory round trip (P = 1.7 M: 5.5 -> 4.6 us)
    float x[NORM_CHUNK / 256];
#pragma unroll
    for (int i = 0; i < NORM_CHUNK / 256; ++i) {
        const long long o = base + t + 256 * i;
        const float v = g[o < P ? o : P - 1];
        x[i] = o < P ? v : 0.0f;
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NORM_CHUNK / 256; ++i) s = __builtin_fmaf(x[i], x[i], s);
    s = block_sum_256(s, red);
    if (t == 0) part[blockIdx.x] = s;
}

__device__ __forceinline__ float clip_scale(float nrm, float max_norm)
{
    return max_norm > 0.0f ? fminf(1.0f, max_norm / (nrm + 1e-6f)) : 1.0f;
}

static void enqueue_sumsq(hipStream_t stream, const float *g, long long P, float *norm_part)
{
    const int nparts = (int)((P + NORM_CHUNK - 1) / NORM_CHUNK);
    hipLaunchKernelGGL(sumsq_kernel, dim3(nparts), dim3(256), 0, stream, g, P, norm_part);
}

// the statistics and the optimiser kernel form the norm and the clip factor from these sums themselves (the same additions in the same
// order, in every workgroup)
hipError_t launch_grad_norm(Ctx &c, const float *g, long long P)
{
    SiteTimer tm(c, SITE_GRAD_NORM);
    enqueue_sumsq(c.stream, g, P, c.ws.norm_part);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Adam
// ------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void adam_one(float &th, float g, float &m, float &v, float gs, float lr, float b1, float b2,
                                         float eps, float ibc1, float ibc2)
{
    g *= gs;
    m = b1 * m + (1.0f - b1) * g;
    v = b2 * v + (1.0f - b2) * g * g;
    th = th - lr * (m * ibc1) / (sqrtf(v * ibc2) + eps);
}

template <bool VEC4>
__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ theta, const float *__restrict__ g,
                                                   float *__restrict__ m, float *__restrict__ v, long long P,
                                                   const float *__restrict__ norm_part,
                                                   int nparts, float max_norm, float lr, float b1, float b2,
                                                   float eps, float ibc1, float ibc2)
{
    // the clip factor, formed here from the per-chunk sums of squares, or none
    __shared__ float red[256];
    float gs = 1.0f;
    if (norm_part) gs = clip_scale(norm_from_parts(norm_part, nparts, red), max_norm);
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if constexpr (VEC4) {
        const long long o = i * 4;
        if (o + 3 < P) {
            f32x4 th = *reinterpret_cast<f32x4 *>(theta + o);
            const f32x4 gg = *reinterpret_cast<const f32x4 *>(g + o);
            f32x4 mm = *reinterpret_cast<f32x4 *>(m + o), vv = *reinterpret_cast<f32x4 *>(v + o);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float a = th[k], b = mm[k], c2 = vv[k];
                adam_one(a, gg[k], b, c2, gs, lr, b1, b2, eps, ibc1, ibc2);
                th[k] = a; mm[k] = b; vv[k] = c2;
            }
            *reinterpret_cast<f32x4 *>(theta + o) = th;
            *reinterpret_cast<f32x4 *>(m + o) = mm;
            *reinterpret_cast<f32x4 *>(v + o) = vv;
        } else {
            for (long long k = o; k < P; ++k) adam_one(theta[k], g[k], m[k], v[k], gs, lr, b1, b2, eps, ibc1, ibc2);
        }
    } else {
        if (i < P) adam_one(theta[i], g[i], m[i], v[i], gs, lr, b1, b2, eps, ibc1, ibc2);
    }
}

// ------------------------------------------------------------------------------------------------------------
// The same update over the whole network's vector, organised like prep_kernel: a workgroup owns a piece of one
// parameter tensor, updates theta / m / v there (the element-wise arithmetic of adam_kernel, so the same bits) and
// writes the new values straight into the workspace copy of the network (converted, re-ordered, fc.w also transposed
// through the LDS tile) -- the separate pass that would otherwise re-read the whole vector before the next forward
// pass is not needed.  Every parameter belongs to exactly one job: fc.w tiles, conv2.w / conv3.w, conv1.w, and the
// fp32 block (biases, heads).
// ------------------------------------------------------------------------------------------------------------
struct AdamShadowArgs {
    PrepArgs pa;                  // destinations, geometry and job sizes (pa.params is not used)
    float *theta;
    const float *g;
    float *m, *v;
    const float *norm_part;
    int nparts;
    float max_norm, lr, b1, b2, eps, ibc1, ibc2;
};

template <typename T> __global__ __launch_bounds__(256) void adam_shadow_kernel(const AdamShadowArgs a)
{
    __shared__ float tile[64][65];
    __shared__ float red[256];
    float gs = 1.0f;
    auto find_scale = [&]() {
        if (a.norm_part) gs = clip_scale(norm_from_parts(a.norm_part, a.nparts, red), a.max_norm);
    };
    float *__restrict__ theta = a.theta;
    const float *__restrict__ g = a.g;
    float *__restrict__ m = a.m, *__restrict__ v = a.v;
    auto update = [&](long long idx) -> float {
        float th = theta[idx], mm = m[idx], vv = v[idx];
        adam_one(th, g[idx], mm, vv, gs, a.lr, a.b1, a.b2, a.eps, a.ibc1, a.ibc2);
        theta[idx] = th; m[idx] = mm; v[idx] = vv;
        return th;
    };
    const PrepArgs &p = a.pa;
    const int t = threadIdx.x;
    int blk = blockIdx.x;
    if (blk < p.nb_fc) {
        const int F = p.g.F, tf = F / 64;
        const int j0 = (blk / tf) * 64, f0 = (blk % tf) * 64;
        T *wfc = (T *)p.wfc;
        const int col = t & 63, r0 = t >> 6;
        // 16-byte accesses: a thread takes four neighbouring columns of four rows (16 lanes cover a tile row); all its
        // loads are independent and the update runs on registers.  (fc.w starts on a 16-byte boundary when the tensors
        // in front of it hold a multiple of four values; otherwise the element-wise form below is taken.)
        if (((p.g.fcw | (long long)F) & 3) == 0 && ((((uintptr_t)theta | (uintptr_t)g | (uintptr_t)m | (uintptr_t)v) & 15u) == 0)) {
            const int c4 = (t & 15) * 4, rr = t >> 4;
            f32x4 th[4], gg[4], mm[4], vv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long long idx = p.g.fcw + (long long)(j0 + rr + 16 * i) * F + f0 + c4;
                th[i] = *reinterpret_cast<const f32x4 *>(theta + idx); gg[i] = *reinterpret_cast<const f32x4 *>(g + idx);
                mm[i] = *reinterpret_cast<const f32x4 *>(m + idx); vv[i] = *reinterpret_cast<const f32x4 *>(v + idx);
            }
            find_scale();                    // while they travel
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = rr + 16 * i;
                const long long o = (long long)(j0 + r) * F + f0 + c4;
                Vec<T, 4> w4;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float a0 = th[i][k], a1 = mm[i][k], a2 = vv[i][k];
                    adam_one(a0, gg[i][k], a1, a2, gs, a.lr, a.b1, a.b2, a.eps, a.ibc1, a.ibc2);
                    th[i][k] = a0; mm[i][k] = a1; vv[i][k] = a2;
                    w4[k] = from_f32<T>(a0);
                    tile[r][c4 + k] = a0;
                }
                *reinterpret_cast<f32x4 *>(theta + p.g.fcw + o) = th[i];
                *reinterpret_cast<f32x4 *>(m + p.g.fcw + o) = mm[i];
                *reinterpret_cast<f32x4 *>(v + p.g.fcw + o) = vv[i];
                *reinterpret_cast<Vec<T, 4> *>(wfc + o) = w4;
            }
        } else {
            find_scale();
            float th[16], gg[16], mm[16], vv[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const long long idx = p.g.fcw + (long long)(j0 + r0 + 4 * i) * F + f0 + col;
                th[i] = theta[idx]; gg[i] = g[idx]; mm[i] = m[idx]; vv[i] = v[idx];
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int r = r0 + 4 * i;
                const long long o = (long long)(j0 + r) * F + f0 + col;
                adam_one(th[i], gg[i], mm[i], vv[i], gs, a.lr, a.b1, a.b2, a.eps, a.ibc1, a.ibc2);
                theta[p.g.fcw + o] = th[i]; m[p.g.fcw + o] = mm[i]; v[p.g.fcw + o] = vv[i];
                wfc[o] = from_f32<T>(th[i]);
                tile[r][col] = th[i];
            }
        }
        if (!p.learn) return;
        __syncthreads();
        T *wfcd = (T *)p.wfcd;
        const int P3 = p.g.P3;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int fl = r0 + 4 * i, f = f0 + fl;
            const int c = f / P3, q = f - c * P3;
            wfcd[(long long)(q * 64 + c) * 512 + j0 + col] = from_f32<T>(tile[col][fl]);
        }
        return;
    }
    blk -= p.nb_fc;
    find_scale();
    if (blk < p.nb_conv) {
        const int i = blk * 256 + t;
        T *wf2 = (T *)p.wf2, *wf3 = (T *)p.wf3, *wd2 = (T *)p.wd2, *wd3 = (T *)p.wd3;
        if (i < 64 * 32 * 16) {               // conv2.w[n][c][u][v], 64 x 32 x 4 x 4
            const int n = i / 512, r = i % 512, c = r / 16, tap = r % 16;
            const T w = from_f32<T>(update(p.g.w2 + i));
            wf2[n * 512 + tap * 32 + c] = w;
            ((T *)p.w2q)[frag16<T>(n, tap * 32 + c, 512)] = w;
            if (p.learn) wd2[c * 1024 + tap * 64 + n] = w;
        }
        if (i < 64 * 64 * 9) {                // conv3.w[n][c][u][v], 64 x 64 x 3 x 3
            const int n = i / 576, r = i % 576, c = r / 9, tap = r % 9;
            const T w = from_f32<T>(update(p.g.w3 + i));
            wf3[n * 576 + tap * 64 + c] = w;
            ((T *)p.w3q)[frag16<T>(n, tap * 64 + c, 576)] = w;
            if (p.learn) wd3[c * 576 + tap * 64 + n] = w;
        }
        return;
    }
    blk -= p.nb_conv;
    if (blk < p.nb_w1) {
        const int i = blk * 256 + t;
        if (i < 32 * p.g.K1) {
            const T w = from_f32<T>(update(p.g.w1 + i));
            ((T *)p.w1s)[i] = w;
            ((T *)p.w1q)[frag16<T>(i / p.g.K1, i % p.g.K1, p.g.K1)] = w;
        }
        return;
    }
    blk -= p.nb_w1;
    {
        const int i = blk * 256 + t;
        const int A = p.g.A;
        long long src = -1;
        if (i < 32) src = p.g.b1 + i;
        else if (i >= p.sh.b2 && i < p.sh.b2 + 64) src = p.g.b2 + (i - p.sh.b2);
        else if (i >= p.sh.b3 && i < p.sh.b3 + 64) src = p.g.b3 + (i - p.sh.b3);
        else if (i >= p.sh.fcb && i < p.sh.fcb + 512) src = p.g.fcb + (i - p.sh.fcb);
        else if (i >= p.sh.piw && i < p.sh.piw + 512 * A) src = p.g.piw + (i - p.sh.piw);
        else if (i >= p.sh.pib && i < p.sh.pib + A) src = p.g.pib + (i - p.sh.pib);
        else if (i >= p.sh.vw && i < p.sh.vw + 512) src = p.g.vw + (i - p.sh.vw);
        else if (i == p.sh.vb) src = p.g.vb;
        if (src < 0) return;
        p.hb[i] = update(src);
    }
}

static void enqueue_adam(hipStream_t stream, float *theta, const float *g, float *m, float *v, long long P,
                         const float *norm_part, float max_norm, float lr, float b1, float b2,
                         float eps, float bc1, float bc2)
{
    const int nparts = (int)((P + NORM_CHUNK - 1) / NORM_CHUNK);
    const bool aligned = (((uintptr_t)theta | (uintptr_t)g | (uintptr_t)m | (uintptr_t)v) & 15u) == 0;
    const float ibc1 = 1.0f / bc1, ibc2 = 1.0f / bc2;
    if (aligned) {
        const long long nthreads = (P + 3) / 4;
        hipLaunchKernelGGL(adam_kernel<true>, dim3((unsigned)((nthreads + 255) / 256)), dim3(256), 0, stream, theta, g,
                           m, v, P, norm_part, nparts, max_norm, lr, b1, b2, eps, ibc1, ibc2);
    } else {
        hipLaunchKernelGGL(adam_kernel<false>, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, stream, theta, g, m, v,
                           P, norm_part, nparts, max_norm, lr, b1, b2, eps, ibc1, ibc2);
    }
}

hipError_t launch_adam(Ctx &c, float *theta, const float *g, float *m, float *v, long long P,
                       const float *norm_part, float max_norm, float lr, float b1, float b2, float eps, float bc1, float bc2)
{
    SiteTimer tm(c, SITE_ADAM);
    enqueue_adam(c.stream, theta, g, m, v, P, norm_part, max_norm, lr, b1, b2, eps, bc1, bc2);
    return hipGetLastError();
}

hipError_t launch_adam_shadow(Ctx &c, float *theta, const float *g, float *m, float *v,
                              const float *norm_part, float max_norm, float lr, float b1, float b2, float eps, float bc1,
                              float bc2, bool learn)
{
    SiteTimer tm(c, SITE_ADAM);
    AdamShadowArgs a;
    a.pa = prep_args(c, nullptr, learn);
    a.theta = theta; a.g = g; a.m = m; a.v = v; a.norm_part = norm_part;
    a.nparts = (int)((c.g.P + NORM_CHUNK - 1) / NORM_CHUNK);
    a.max_norm = max_norm; a.lr = lr; a.b1 = b1; a.b2 = b2; a.eps = eps; a.ibc1 = 1.0f / bc1; a.ibc2 = 1.0f / bc2;
    const int nb = a.pa.nb_fc + a.pa.nb_conv + a.pa.nb_w1 + a.pa.nb_hb;
    if (c.desc.precision == HTS_PRECISION_BF16)
        hipLaunchKernelGGL(adam_shadow_kernel<bf16_t>, dim3(nb), dim3(256), 0, c.stream, a);
    else
        hipLaunchKernelGGL(adam_shadow_kernel<float>, dim3(nb), dim3(256), 0, c.stream, a);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) { c.synced = true; c.synced_learn = learn; c.shadow_of = theta; }
    return e;
}

}  // namespace hts

// ------------------------------------------------------------------------------------------------------------
// Clip + optimiser step without a context and without any allocation: the per-chunk sums of squares of the gradient
// norm live in a file-scope device array instead of a context's workspace.  For callers that cannot allocate (code
// under graph capture, tight serving loops).  Every GPU holds its own copy of the array; its device address is looked
// up once per device and only that address is handed to kernels.
// ------------------------------------------------------------------------------------------------------------
namespace {
constexpr long long STATIC_MAX_PARAMS = HTS_STATIC_MAX_PARAMS;
constexpr int STATIC_PARTS = (int)((STATIC_MAX_PARAMS + hts::NORM_CHUNK - 1) / hts::NORM_CHUNK);
static __device__ __align__(256) float scratch[STATIC_PARTS];       // 8 KiB per GPU, held until the process ends

constexpr int STATIC_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
float *g_scratch_ptr[STATIC_MAX_DEVICES] = {};                      // device address of `scratch`, per device

// Device address of the scratch array on the current device (looked up on first use, under a lock).
hipError_t scratch_on_current_device(float **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= STATIC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace

extern "C" int32_t hts_adam_apply_static(float *params, const float *grads, hts_opt_state *opt, const hts_hparams *hp,
                                         int64_t P, void *hip_stream)
{
    using namespace hts;
    if (!params || !grads || !opt || !opt->m || !opt->v || !hp) return HTS_EINVAL;
    if (P <= 0 || opt->step < 0) return HTS_EINVAL;
    if (P > STATIC_MAX_PARAMS) return HTS_ESHAPE;          // the static array holds one partial sum per 8192 parameters
    if (hp->optimizer != HTS_OPT_ADAM && hp->optimizer != HTS_OPT_RMSPROP) return HTS_EINVAL;
    float *part = nullptr;
    hipError_t e = scratch_on_current_device(&part);
    if (e != hipSuccess) { note_hip_error(e); return HTS_EHIP; }
    hipStream_t stream = (hipStream_t)hip_stream;
    const int64_t t = opt->step + 1;
    const bool rms = hp->optimizer == HTS_OPT_RMSPROP;
    const float b1 = rms ? 0.0f : hp->beta1, b2 = rms ? hp->rms_alpha : hp->beta2;
    const float bc1 = rms ? 1.0f : (float)(1.0 - pow((double)hp->beta1, (double)t));
    const float bc2 = rms ? 1.0f : (float)(1.0 - pow((double)hp->beta2, (double)t));
    const bool clip = hp->max_grad_norm > 0.0f;
    // every partial sum the optimiser kernel reads is written by the pass before it: nothing has to start at zero
    if (clip) enqueue_sumsq(stream, grads, P, part);
    enqueue_adam(stream, params, grads, opt->m, opt->v, P, clip ? part : nullptr, hp->max_grad_norm, hp->lr, b1,
                 b2, hp->adam_eps, bc1, bc2);
    e = hipGetLastError();
    if (e != hipSuccess) { note_hip_error(e); return HTS_EHIP; }
    opt->step = t;
    return HTS_OK;
}
