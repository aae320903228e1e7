// lbib_march.hpp -- two time steps of the lattice update in one pass over memory, shared by the
// sweeps of one simulation and of a pool.
//
// A sweep of one step reads and writes every population once, so beyond the caches it is bound
// by HBM bandwidth.  Here each wave marches up a strip of 62 columns: it loads a row of level
// n, collides it (level n+1, rounded to the storage type as a store and load would), and from
// that row and the two before it, which it keeps in registers, streams and collides the row
// below (level n+2) and stores it.  The populations move sideways between lanes by one-lane
// wave shifts, so the wave's 64 lanes give 62 columns of results without LDS.  The arithmetic
// per node and step is that of the one-step sweeps in the same order on the same values, so
// results are bit-identical.
//
// What bounds it: FP64 and FP32, memory still (vector issue about 0.2 and 0.5 of the cycles), through
// the lines that neighbouring strips share and the two extra rows of a run; the 16-bit storages,
// vector issue (0.8).  No particle, us per step, one-step sweep against this one: 8192 x 4096
// FP64 867 -> 546, FP32 380 -> 273, FP16 189 -> 142; 4096 x 1024 FP64 88 -> 62, FP32 43 -> 32.6,
// FP16 23.8 -> 18.8.  Without the barrier that keeps a workgroup's
// strips on the same rows, 370 instead of 275 (FP32, 8192 x 4096); with loads past the caches
// 343; with each wave on 64 aligned columns and its neighbours' values missing (no usable
// result) 290, so the shared lines are what the barrier saves.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbib_collide.hpp"
#include "lbib_device.hpp"
#include "lbib_internal.hpp"

namespace lbib {

constexpr int kStrip = kPairStrip;

// A population as the storage holds it between two steps, in a type whose copies and lane
// shifts are cheap: the FP64 and FP32 value itself, the 16-bit one as its bits.
template <typename T>
struct Kept {
    using V = typename St<T>::raw;
};

__device__ __forceinline__ double keep_value(const double*, double v, const SweepArgs&) { return v; }
__device__ __forceinline__ float keep_value(const float*, double v, const SweepArgs&) { return (float)v; }
__device__ __forceinline__ uint16_t keep_value(const half_t*, float v, const SweepArgs& a)
{
    return __builtin_bit_cast(uint16_t, (_Float16)(v * (float)a.scale));
}
__device__ __forceinline__ uint16_t keep_value(const bf16_t*, float v, const SweepArgs&)
{
    return __builtin_bit_cast(uint16_t, (__bf16)v);
}
__device__ __forceinline__ double kept_value(const double*, double v, const SweepArgs&) { return v; }
__device__ __forceinline__ double kept_value(const float*, float v, const SweepArgs&) { return (double)v; }
__device__ __forceinline__ float kept_value(const half_t*, uint16_t v, const SweepArgs& a)
{
    return __builtin_fmaf((float)__builtin_bit_cast(_Float16, v), (float)a.inv_scale, -0.0f);
}
__device__ __forceinline__ float kept_value(const bf16_t*, uint16_t v, const SweepArgs&)
{
    return __builtin_bit_cast(float, (uint32_t)v << 16);
}

// The value of the lane to the left (column i - 1) or right (column i + 1); the wave's first or
// last lane keeps its own, which no result uses.
template <int CTRL>
__device__ __forceinline__ uint32_t lane_shift(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL, typename V>
__device__ __forceinline__ V lane_shift_v(V v)
{
    if constexpr (sizeof(V) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = lane_shift<CTRL>((uint32_t)b), hi = lane_shift<CTRL>((uint32_t)(b >> 32));
        return __builtin_bit_cast(V, ((uint64_t)hi << 32) | lo);
    } else if constexpr (sizeof(V) == 4) {
        return __builtin_bit_cast(V, lane_shift<CTRL>(__builtin_bit_cast(uint32_t, v)));
    } else {
        return __builtin_bit_cast(V, (uint16_t)lane_shift<CTRL>((uint32_t)__builtin_bit_cast(uint16_t, v)));
    }
}
template <typename V>
__device__ __forceinline__ V from_left(V v)
{
    return lane_shift_v<0x138>(v);  // DPP wave_shr:1
}
template <typename V>
__device__ __forceinline__ V from_right(V v)
{
    return lane_shift_v<0x130>(v);  // DPP wave_shl:1
}

// The spread force of one of the two steps: the particle's box and its force (PartRef; d.active
// 0: none).
struct BoxForce {
    TileDesc d;
    const int64_t* tile;
    const uint2* ring;
};

// The rows of a buffer around row j, as a buffer resource: a segment (row j - 1 + dr, population
// q) is the scalar offset dr R + q P, a column the lane's offset.  The loop then issues every
// access without a branch around it (a lane that has nothing to store gives kNoStore, which the
// resource's bound drops), so the compiler knows how many younger accesses are in flight when
// it waits for a row's loads and does not wait for those.  Row-interleaved buffers only (R = 9 P):
// the window's three pitches then hold all nine populations of its three rows.
// beyond every bound (the window's bytes are below 2^31, and so is a segment's offset, which the
// sum of the two does not carry past 32 bits)
constexpr uint32_t kNoStore = 0x80000000u;
static_assert((uint64_t)kNoStore + 0x7fffffffu <= 0xffffffffu && kNoStore > 0x7fffffffu, "dropped at every segment");

template <typename S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_window(const S* f, const SweepArgs& a, int j)
{
    const int64_t R = a.pitch;
    const S* base = sbase(f + ((int64_t)j - 1) * R);
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)(3 * R * (int64_t)sizeof(S)), 0x00027000);
}
template <typename S>
__device__ __forceinline__ S window_load(__amdgpu_buffer_rsrc_t w, uint32_t v, uint32_t s)
{
    if constexpr (sizeof(S) == 8)
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(w, v, s, 0));
    else if constexpr (sizeof(S) == 4)
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(w, v, s, 0));
    else
        return __builtin_bit_cast(S, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(w, v, s, 0));
}
// COH: visible to other XCDs without cache maintenance (sc1, as the agent-scope stores).
template <bool COH, typename V>
__device__ __forceinline__ void window_store(__amdgpu_buffer_rsrc_t w, uint32_t v, uint32_t s, V x)
{
    constexpr int aux = COH ? 16 : 0;
    if constexpr (sizeof(V) == 8) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), w, v, s, aux);
    } else if constexpr (sizeof(V) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), w, v, s, aux);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, x), w, v, s, aux);
    }
}

// Stored values of row j of level n: those update_load presents, before conversion.
template <typename T, bool PULL>
__device__ __forceinline__ void row_load(const T* __restrict__ fin, const SweepArgs& a, const Cols& c, int j,
                                         typename Kept<T>::V (&v)[9])
{
    using S = typename Kept<T>::V;
    const uint32_t P = (uint32_t)(a.plane * (int64_t)sizeof(S)), R = (uint32_t)a.pitch * (uint32_t)sizeof(S);
    const bool top = (j + 1 == a.ny), bot = (j == 0);
    const __amdgpu_buffer_rsrc_t w = row_window((const S*)fin, a, j);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint32_t s = R + q * P, o = c.o[1];
        if (PULL && kEy[q] != 0) {
            const bool wall = kEy[q] > 0 ? bot : top;
            s = wall ? R + kOpp[q] * P : (uint32_t)(1 - kEy[q]) * R + q * P;
            const uint32_t own = c.o[1], from = c.o[1 - kEx[q]];
            o = wall ? own : from;
        } else if (PULL) {
            o = c.o[1 - kEx[q]];
        }
        v[q] = window_load<S>(w, o, s);
    }
}

// The results of row j: at the node itself (pull) or scattered to the neighbours (push), as
// pull_store and push_store do.  c: the lane's columns, or kNoStore.
template <typename T, bool PULL, bool COH>
__device__ __forceinline__ void row_store(T* __restrict__ fout, const SweepArgs& a, const Cols& c, int j,
                                          const typename St<T>::C (&post)[9])
{
    using S = typename Kept<T>::V;
    const T* tag = nullptr;
    const uint32_t P = (uint32_t)(a.plane * (int64_t)sizeof(S)), R = (uint32_t)a.pitch * (uint32_t)sizeof(S);
    const bool top = (j + 1 == a.ny), bot = (j == 0);
    const __amdgpu_buffer_rsrc_t w = row_window((const S*)fout, a, j);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint32_t s = R + q * P, o = c.o[1];
        if (!PULL && kEy[q] != 0) {
            const bool wall = kEy[q] > 0 ? top : bot;
            s = wall ? R + kOpp[q] * P : (uint32_t)(1 + kEy[q]) * R + q * P;
            const uint32_t own = c.o[1], out = c.o[1 + kEx[q]];
            o = wall ? own : out;
        } else if (!PULL) {
            o = c.o[1 + kEx[q]];
        }
        window_store<COH, S>(w, o, s, keep_value(tag, post[q], a));
    }
}

// One wave: rows [r0, r1) of level n+2 of the strip of columns c0 .. c0 + 61 (those below nx),
// from level n in fin to fout.  Lane L works on column c0 - 1 + L (periodic; lanes past the
// lattice's end repeat its last); the lanes at the strip's two ends only feed their
// neighbours.  f1, f2: the spread forces of step n and n+1.  A row's loads are issued two rows
// ahead, into the registers of the row being worked on.  Every wave of the workgroup that calls
// this works on the same rows (it meets the others in a workgroup barrier every second row).
// COH: the forces come from a launch running beside this one, and such a launch reads the
// results.
template <typename T, bool PULL, bool COH = false>
__device__ __forceinline__ void march_pair(const T* __restrict__ fin, T* __restrict__ fout, const SweepArgs& a, int c0,
                                           int r0, int r1, const BoxForce& f1, const BoxForce& f2)
{
    using C = typename St<T>::C;
    using V = typename Kept<T>::V;
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int col = min(c0 - 1 + lane, a.nx);
    const int i = col < 0 ? a.nx - 1 : (col == a.nx ? 0 : col);
    const bool mine = lane >= 1 && lane <= kStrip && col < a.nx;
    const Cols c = cols<T>(i, a.nx);
    const Cols cs{{mine ? c.o[0] : kNoStore, mine ? c.o[1] : kNoStore, mine ? c.o[2] : kNoStore}};
    const T* tag = nullptr;
    // does any lane's column lie in the boxes?
    auto col_in = [&](const TileDesc& d) {
        int di = i - d.i0w;
        if (di < 0) di += a.nx;
        return __ballot(d.active && di < d.w) != 0;
    };
    const bool any1 = col_in(f1.d), any2 = col_in(f2.d);
    auto force = [&](const BoxForce& f, bool any, int j, C& Fx, C& Fy) {
        double x = a.gx, y = a.gy;
        if (any && j >= f.d.j0 && j < f.d.j0 + f.d.h) box_force<COH>(f.d, f.tile, f.ring, i, j, a.nx, x, y);
        Fx = (C)x;
        Fy = (C)y;
    };
    // level n+1: the newest row p, the row below it pm (populations 0, 1, 3 and 2, 5, 6) and the
    // row below that pn (2, 5, 6)
    V p[9], pm0{}, pm1{}, pm3{}, pm2{}, pm5{}, pm6{}, pn2{}, pn5{}, pn6{};
    const int ra = r0 > 0 ? r0 - 1 : 0, rb = min(r1, a.ny - 1);  // rows of level n+1
    // row r of level n+1, and the loads of row r + 2
    auto first = [&](int r, V(&raw)[9]) {
        C g[9], post[9], Fx, Fy;
#pragma unroll
        for (int q = 0; q < 9; ++q) g[q] = kept_value(tag, raw[q], a);
        row_load<T, PULL>(fin, a, c, min(r + 2, rb), raw);
        wall_reflect<C>(g, r, a.ny, a.uw6);
        force(f1, any1, r, Fx, Fy);
        collide_node<C>(g, a, Fx, Fy, post);
#pragma unroll
        for (int q = 0; q < 9; ++q) p[q] = keep_value(tag, post[q], a);
    };
    auto rotate = [&]() {
        pn2 = pm2;
        pn5 = pm5;
        pn6 = pm6;
        pm0 = p[0];
        pm1 = p[1];
        pm2 = p[2];
        pm3 = p[3];
        pm5 = p[5];
        pm6 = p[6];
    };
    // row j of level n+2, from rows j - 1 (pn), j (pm) and j + 1 (p) of level n+1
    auto second = [&](int j) {
        C g[9], post[9], Fx, Fy;
        g[0] = kept_value(tag, pm0, a);
        g[1] = kept_value(tag, from_left(pm1), a);
        g[2] = kept_value(tag, pn2, a);
        g[3] = kept_value(tag, from_right(pm3), a);
        g[4] = kept_value(tag, p[4], a);
        g[5] = kept_value(tag, from_left(pn5), a);
        g[6] = kept_value(tag, from_right(pn6), a);
        g[7] = kept_value(tag, from_right(p[7]), a);
        g[8] = kept_value(tag, from_left(p[8]), a);
        wall_reflect<C>(g, j, a.ny, a.uw6);
        force(f2, any2, j, Fx, Fy);
        collide_node<C>(g, a, Fx, Fy, post);
        row_store<T, PULL, COH>(fout, a, cs, j, post);
    };
    V ev[9], od[9];
    row_load<T, PULL>(fin, a, c, ra, ev);
    row_load<T, PULL>(fin, a, c, min(ra + 1, rb), od);
    int r = ra;
    first(r, ev);
    if (r0 == 0) {
        // what the bottom wall reflects into row 0, as if emitted by a row below it
        pm2 = p[4];
        pm5 = from_right(p[7]);
        pm6 = from_left(p[8]);
        rotate();
    } else {
        rotate();
        first(++r, od);
        rotate();
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const V t = ev[q];
            ev[q] = od[q];
            od[q] = t;
        }
    }
    // ev holds row r + 2, od row r + 1 (clamped to rb)
    for (++r; r <= rb; r += 2) {
        first(r, od);
        second(r - 1);
        rotate();
        if (r + 1 > rb) break;
        // the workgroup's waves, on neighbouring strips, stay on the same rows, so that a cache
        // line two strips share is fetched once (waves that have ended do not count)
        __builtin_amdgcn_s_barrier();
        first(r + 1, ev);
        second(r);
        rotate();
    }
    if (r1 == a.ny) {
        // what the top wall reflects into row ny - 1, as if emitted by a row above it
        p[4] = pm2;
        p[7] = from_left(pm5);
        p[8] = from_right(pm6);
        second(a.ny - 1);
    }
}

}  // namespace lbib
