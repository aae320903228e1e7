// lbib_pool_sweep.hip -- gfx950 lattice sweep of a pool of independent simulations (one
// launch for every member's tiles).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <math.h>
#include <stdint.h>

#include "lbib_collide.hpp"
#include "lbib_device.hpp"
#include "lbib_internal.hpp"
#include "lbib_march.hpp"

namespace lbib {

// Sweep of a pool of independent simulations in one launch.  Block b sweeps up to TPB
// consecutive tiles (BX x 256/BX nodes each) of member table[b].x, starting at tile
// table[b].y; the table lists each member's tiles in order, so after the XCD remap a
// member's tiles share one XCD's L2.  ctl[member] holds the member's box of this step and,
// in pad, which buffer its particle phase just read (0: fA, 1: fB) or that it did not step
// (-1: nothing to do); it is loaded beside the member's record, so a block waits for two
// dependent loads (its table entry, then both) before its populations.  A block pays these
// lookups once for TPB tiles.  Pool buffers use the pull layout: a pool's
// working set is far larger than the MALL, where the aligned stores of the pull update
// move HBM traffic faster than the shifted stores of the push update (216 members of
// 512-2048 x 128-256 nodes, row-interleaved FP32: pull 665 us per sweep, push 764 us).
template <typename T, int BX, int TPB>
__global__ __launch_bounds__(256) void pool_sweep_kernel(const PoolSweep<T>* __restrict__ sims,
                                                         const TileDesc* __restrict__ ctl,
                                                         const int2* __restrict__ table, int nblocks)
{
    constexpr int BY = 256 / BX;
    static_assert(BX >= 64, "the sweep's addressing takes each wave's nodes from one row");
    int b = blockIdx.x;
    {
        const int q = nblocks >> 3, r = nblocks & 7, x = b & 7, k = b >> 3;
        b = (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
    }
    const int2 e = table[b];
    const TileDesc d = ctl[e.x];
    const PoolSweep<T>& ps = sims[e.x];
    if (d.pad < 0) return;
    const T* fin = d.pad ? ps.fB : ps.fA;
    T* fout = d.pad ? ps.fA : ps.fB;
    const SweepArgs a = ps.a;
    const int tx = (int)(threadIdx.x % BX), ty = (int)(threadIdx.x / BX);
    const int tend = min(e.y + TPB, ps.ntiles);
    for (int t = e.y; t < tend; ++t) {
        const int row = (int)fdiv((uint32_t)t, ps.gx);
        const int i = (t - row * (int)ps.gx.d) * BX + tx;
        const int j = row * BY + ty;
        if (i >= a.nx || j >= a.ny) continue;
        double Fx = a.gx, Fy = a.gy;
        box_force<false>(d, ps.tile, ps.ring, i, j, a.nx, Fx, Fy);
        collide_stream<T, true>(fin, fout, a, i, j, Fx, Fy);
    }
}

template <typename T>
hipError_t launch_pool_sweep(const PoolSweep<T>* sims, const TileDesc* ctl, const int2* table, int32_t n_blocks,
                             PoolSweepConfig cfg, hipStream_t stream, hipEvent_t t0, hipEvent_t t1)
{
    if (n_blocks <= 0) return hipSuccess;
#define LBIB_POOL_SWEEP(BX_, TPB_)                                                                                     \
    if (cfg.bx == BX_ && cfg.tpb == TPB_) {                                                                            \
        if (t0 || t1)                                                                                                  \
            hipExtLaunchKernelGGL(pool_sweep_kernel<T, BX_, TPB_>, dim3(n_blocks), dim3(256), 0u, stream, t0, t1, 0u,  \
                                  sims, ctl, table, n_blocks);                                                         \
        else                                                                                                           \
            hipLaunchKernelGGL((pool_sweep_kernel<T, BX_, TPB_>), dim3(n_blocks), dim3(256), 0, stream, sims, ctl,     \
                               table, n_blocks);                                                                       \
        return hipGetLastError();                                                                                      \
    }
    LBIB_POOL_SWEEP(64, 1)
    LBIB_POOL_SWEEP(64, 2)
    LBIB_POOL_SWEEP(64, 4)
    LBIB_POOL_SWEEP(64, 8)
    LBIB_POOL_SWEEP(128, 1)
    LBIB_POOL_SWEEP(128, 2)
    LBIB_POOL_SWEEP(128, 4)
    LBIB_POOL_SWEEP(128, 8)
    LBIB_POOL_SWEEP(256, 1)
    LBIB_POOL_SWEEP(256, 2)
    LBIB_POOL_SWEEP(256, 4)
    LBIB_POOL_SWEEP(256, 8)
#undef LBIB_POOL_SWEEP
    return hipErrorInvalidValue;
}

// Step n around the box of step n+1: member k's predicted box widened by a node (the sources of
// the values the second particle launch reads there), from the buffer the first launch read to
// the other one.  A wave takes 64 columns of a row; kZoneBlocks workgroups share a member's
// (a box of 90 x 35 nodes: 72 wave rows on 64 waves).
constexpr int kZoneBlocks = 16;
template <typename T>
__global__ __launch_bounds__(256) void pool_zone_kernel(const PoolSweep<T>* __restrict__ sims,
                                                        const TileDesc* __restrict__ ctl)
{
    const int k = (int)blockIdx.x / kZoneBlocks;
    const TileDesc d = ctl[k];
    const PoolSweep<T>& ps = sims[k];
    const TileDesc z = ps.zone[1];
    if (d.pad < 0 || !z.active) return;
    const T* fin = d.pad ? ps.fB : ps.fA;
    T* fout = d.pad ? ps.fA : ps.fB;
    const SweepArgs a = ps.a;
    const int j0 = max(z.j0 - 1, 0), rows = min(z.j0 + z.h, a.ny - 1) - j0 + 1;
    const int w = min(z.w + 2, a.nx), per = (w + 63) / 64;
    const int lane = (int)(threadIdx.x & 63);
    for (int e = ((int)blockIdx.x % kZoneBlocks) * 4 + (int)(threadIdx.x >> 6); e < rows * per; e += 4 * kZoneBlocks) {
        const int j = j0 + e / per, c = (e % per) * 64 + lane;
        if (c >= w) continue;
        int i = z.i0w - 1 + c;
        i = i < 0 ? i + a.nx : (i >= a.nx ? i - a.nx : i);
        double Fx = a.gx, Fy = a.gy;
        box_force<false>(d, ps.tile, ps.ring, i, j, a.nx, Fx, Fy);
        collide_stream<T, true>(fin, fout, a, i, j, Fx, Fy);
    }
}

// Both steps of a pair in one pass (march_pair); a member that made only the first: one step of
// the block's strips.
template <typename T>
__global__ __launch_bounds__(256, sizeof(typename St<T>::raw) == 8 ? 3 : 4) void pool_pair_kernel(const PoolSweep<T>* __restrict__ sims,
                                                           const TileDesc* __restrict__ ctl, int n_active,
                                                           const int2* __restrict__ table, int nblocks, int rows)
{
    int b = blockIdx.x;
    {
        const int q = nblocks >> 3, r = nblocks & 7, x = b & 7, k = b >> 3;
        b = (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
    }
    const int2 e = table[b];
    const PoolSweep<T>& ps = sims[e.x];
    const BoxForce f1{ctl[e.x], ps.tile, ps.ring}, f2{ctl[n_active + e.x], ps.tile_b, ps.ring_b};
    if (f1.d.pad < 0) return;
    const T* fin = f1.d.pad ? ps.fB : ps.fA;
    T* fout = f1.d.pad ? ps.fA : ps.fB;
    const SweepArgs a = ps.a;
    const int w = wave_row((int)(threadIdx.x >> 6));
    const int by = (int)fdiv((uint32_t)e.y, ps.px), bx = e.y - by * (int)ps.px.d;
    const int c0 = (4 * bx + w) * kStrip, r0 = by * rows;
    if (c0 >= a.nx) return;
    const int r1 = min(r0 + rows, a.ny);
    if (f2.d.pad >= 0) {
        march_pair<T, true>(fin, fout, a, c0, r0, r1, f1, f2);
        return;
    }
    const int lane = (int)(threadIdx.x & 63), i = c0 + lane;
    if (lane >= kStrip || i >= a.nx) return;
#pragma unroll 1
    for (int j = r0; j < r1; ++j) {
        double Fx = a.gx, Fy = a.gy;
        box_force<false>(f1.d, f1.tile, f1.ring, i, j, a.nx, Fx, Fy);
        collide_stream<T, true>(fin, fout, a, i, j, Fx, Fy);
    }
}

// Rows of a wave's run in the two-step sweep: the level between the steps is formed for two
// rows more, so short runs repeat work and long ones leave the GPU idle at the launch's end.
int32_t pool_pair_rows(PoolSweepConfig cfg) { return cfg.tpb == 1 ? 8 : cfg.tpb == 2 ? 12 : cfg.tpb == 4 ? 16 : 32; }

template <typename T>
hipError_t launch_pool_zone(const PoolSweep<T>* sims, const TileDesc* ctl, int32_t n_active, hipStream_t stream)
{
    if constexpr (St<T>::neq) {
        return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL(pool_zone_kernel<T>, dim3(n_active * kZoneBlocks), dim3(256), 0, stream, sims, ctl);
        return hipGetLastError();
    }
}

template <typename T>
hipError_t launch_pool_pair(const PoolSweep<T>* sims, const TileDesc* ctl, int32_t n_active, const int2* table,
                            int32_t n_blocks, PoolSweepConfig cfg, hipStream_t stream, hipEvent_t t0, hipEvent_t t1)
{
    if (n_blocks <= 0) return hipSuccess;
    if constexpr (!St<T>::neq) {
        const int rows = pool_pair_rows(cfg);
        if (t0 || t1)
            hipExtLaunchKernelGGL(pool_pair_kernel<T>, dim3(n_blocks), dim3(256), 0u, stream, t0, t1, 0u, sims, ctl,
                                  (int)n_active, table, (int)n_blocks, rows);
        else
            hipLaunchKernelGGL(pool_pair_kernel<T>, dim3(n_blocks), dim3(256), 0, stream, sims, ctl, (int)n_active,
                               table, (int)n_blocks, rows);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

#define LBIB_POOL_SWEEP_INSTANTIATE(T)                                                                      \
    template hipError_t launch_pool_sweep<T>(const PoolSweep<T>*, const TileDesc*, const int2*, int32_t,         \
                                             PoolSweepConfig, hipStream_t, hipEvent_t, hipEvent_t);              \
    template hipError_t launch_pool_zone<T>(const PoolSweep<T>*, const TileDesc*, int32_t, hipStream_t);         \
    template hipError_t launch_pool_pair<T>(const PoolSweep<T>*, const TileDesc*, int32_t, const int2*, int32_t, \
                                            PoolSweepConfig, hipStream_t, hipEvent_t, hipEvent_t);
LBIB_POOL_SWEEP_INSTANTIATE(double)
LBIB_POOL_SWEEP_INSTANTIATE(float)
LBIB_POOL_SWEEP_INSTANTIATE(half_t)
LBIB_POOL_SWEEP_INSTANTIATE(bf16_t)
LBIB_POOL_SWEEP_INSTANTIATE(half_neq_t)
LBIB_POOL_SWEEP_INSTANTIATE(bf16_neq_t)
#undef LBIB_POOL_SWEEP_INSTANTIATE

}  // namespace lbib
