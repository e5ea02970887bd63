// Several independent contractions in one launch: a job is a problem with one of the tile bodies of gemm.hpp / wsgemm.hpp, and a
// workgroup finds its job by its index.  Each job keeps the grid, the tile order and the bits that it has in a launch of its own.
#pragma once
#include "dmawgrad.hpp"
#include "regwgrad.hpp"
#include "wsgemm.hpp"

namespace hts {

constexpr int GROUP_THREADS = 256;

// A job's workgroups in the order of its own launch's linear index; rounded up to a multiple of eight, so that workgroup i of every
// job runs on XCD i % 8 as the tile orders assume.
struct JobGrid {
    int blocks, total, nx, ny;
    FastDiv dx, dy;
    JobGrid() = default;
    explicit JobGrid(const dim3 &g) : blocks((int)((g.x * g.y * g.z + 7) / 8 * 8)), total((int)(g.x * g.y * g.z)), nx((int)g.x), ny((int)g.y),
                                      dx(FastDiv::make((int)g.x)), dy(FastDiv::make((int)g.y)) {}
    __device__ __forceinline__ WgAt at(int i) const
    {
        const int r = dx.div(i), z = dy.div(r);
        return {i - r * nx, r - z * ny, z, nx, ny};
    }
};

// the tile kernel's workgroups
template <class P> struct TileJob {
    P p;
    JobGrid grid;
    static constexpr size_t LDS = TileLds<P>::BYTES;
    static constexpr bool WIDE = false;
    static_assert(P::WAVES_M * P::WAVES_N * 64 == GROUP_THREADS, "workgroup");
    explicit TileJob(const P &q) : p(q), grid(gemm_grid(q)) {}
    __device__ __forceinline__ void run(int i, unsigned char *smem) const
    {
        using T = typename P::T;
        gemm_tile(p, grid.at(i), reinterpret_cast<T *>(smem), reinterpret_cast<T *>(smem + TileLds<P>::A_BYTES));
    }
};

// the wave-per-segment kernel's (PARTIAL = false), spg segments of SEG per reduction group
template <class P, int SEG> struct SegmentJob {
    P p;
    int spg;
    JobGrid grid;
    static constexpr int WAVES = GROUP_THREADS / 64;
    static constexpr size_t LDS = wsgemm_lds<P, WAVES, SEG, false>();
    static constexpr bool WIDE = false;
    SegmentJob(const P &q, int segs_per_group) : p(q)
    {
        const int nseg = (q.K + SEG - 1) / SEG;
        spg = segs_per_group < nseg ? segs_per_group : nseg;
        grid = JobGrid(wsgemm_grid<P, WAVES, SEG, false>(q, spg));
    }
    __device__ __forceinline__ void run(int i, unsigned char *smem) const { wsgemm_tile<P, WAVES, SEG, false>(p, spg, grid.at(i), smem); }
};

// register-operand weight gradient: a task per wavefront, the row tiles of a column tile next to each other.  XCD x takes the
// reduction chunks x, x + 8, ... or, where there is only one, the column tiles x, x + 8, ...  BIAS: the bias columns instead (short
// tasks: a workgroup of their own kind, or the other wavefronts' SIMDs wait).
template <class W, bool BIAS = false> struct RegJob {
    W p;
    struct { int blocks, total; } grid;
    int nz;
    FastDiv dtasks;
    static constexpr int WAVES = GROUP_THREADS / 64;
    static constexpr size_t LDS = WAVES * RW_BLOCK * 8;
    static constexpr bool WIDE = true;
    explicit RegJob(const W &q) : p(q)
    {
        nz = (q.K + q.klen - 1) / q.klen;
        const int cols = BIAS ? 1 : q.col_tiles(), tasks = W::CHUNKED ? cols * W::ROW_TILES : W::ROW_TILES, outer = W::CHUNKED ? nz : cols;
        dtasks = FastDiv::make(tasks);
        grid.blocks = grid.total = 8 * (((outer + 7) / 8 * tasks + WAVES - 1) / WAVES);
    }
    __device__ __forceinline__ void run(int i, unsigned char *smem) const
    {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = (i >> 3) * WAVES + w, o = dtasks.div(t), inner = t - o * dtasks.d, outer = o * 8 + (i & 7);
        uint32_t *table = reinterpret_cast<uint32_t *>(smem) + w * RW_BLOCK * 2;
        if (outer >= (W::CHUNKED ? nz : BIAS ? 1 : p.col_tiles())) return;
        const int rt = inner % W::ROW_TILES, c = W::CHUNKED ? inner / W::ROW_TILES : outer;
        regwgrad_task<W, BIAS>(p, rt, c, W::CHUNKED ? outer : 0, table);
    }
};

// bfloat16 weight gradient on LDS copies.  FC's shares a launch with the heads', whose 17 to 68 workgroups leave the chip idle: one
// after the other 16.2 us at 1024 rows of 84x84 frames, 24.4 at 2048 of 72x96, 10.1 at 128 of 84x84; together 13.0, 19.2 and 6.0.
// (WIDE: 13.4 and 20.1 with the accumulators in accumulation registers.)
template <class W, int HALVES, int STAGES> struct DmaJob {
    W p;
    struct { int blocks, total; } grid;
    static constexpr size_t LDS = wgrad_dma_lds<HALVES, STAGES>();
    static constexpr bool WIDE = true;
    explicit DmaJob(const W &q) : p(q) { grid.blocks = grid.total = wgrad_dma_blocks<HALVES>(q); }
    __device__ __forceinline__ void run(int i, unsigned char *smem) const { wgrad_dma_tile<W, HALVES, STAGES, GROUP_THREADS / 128>(p, i, smem); }
};

template <class... J> struct Jobs;
template <> struct Jobs<> {
    static constexpr size_t LDS = 0;
    static constexpr bool WIDE = false;
    int blocks() const { return 0; }
    __device__ __forceinline__ void run(int, unsigned char *) const {}
};
template <class H, class... R> struct Jobs<H, R...> {
    H head;
    Jobs<R...> rest;
    static constexpr size_t LDS = H::LDS > Jobs<R...>::LDS ? H::LDS : Jobs<R...>::LDS;
    static constexpr bool WIDE = H::WIDE || Jobs<R...>::WIDE;
    explicit Jobs(const H &h, const R &...r) : head(h), rest(r...) {}
    int blocks() const { return head.grid.blocks + rest.blocks(); }
    __device__ __forceinline__ void run(int i, unsigned char *smem) const
    {
        if (i >= head.grid.blocks) rest.run(i - head.grid.blocks, smem);
        else if (i < head.grid.total) head.run(i, smem);
    }
};

// (for the jobs that say WIDE four wavefronts per SIMD at most: without the bound the compiler keeps their blocks in accumulation
// registers and moves them to and fro.  Register-operand weight gradients, fewer, by asking for LDS: 183 us with four, 195 with two, 230 with one)
template <class G> __global__ __launch_bounds__(GROUP_THREADS) __attribute__((amdgpu_waves_per_eu(2, 4))) void group_wide_kernel(const G g)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    g.run((int)blockIdx.x, smem);
}
template <class G> __global__ __launch_bounds__(GROUP_THREADS) void group_kernel(const G g)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    g.run((int)blockIdx.x, smem);
}

// jobs in the order in which their workgroups should start
template <class... J> inline hipError_t launch_group(hipStream_t stream, const J &...jobs)
{
    typedef Jobs<J...> G;
    const G g(jobs...);
    static_assert(sizeof(G) <= 4096, "kernel arguments");
    void (*kern)(const G);
    if constexpr (G::WIDE) kern = group_wide_kernel<G>; else kern = group_kernel<G>;
    if constexpr (G::LDS > 65536) {
        static std::atomic<bool> attr_set{false};       // raise the dynamic-LDS limit once per instantiation (setting it twice is harmless)
        if (!attr_set.load(std::memory_order_acquire)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
            if (e != hipSuccess) return e;
            attr_set.store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL(kern, dim3(g.blocks()), dim3(GROUP_THREADS), G::LDS, stream, g);
    return hipGetLastError();
}

}  // namespace hts
