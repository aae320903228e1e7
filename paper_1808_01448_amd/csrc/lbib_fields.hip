// lbib_fields.hip -- read-out of a population buffer as plain FP64 fields: the density, the
// velocity or the populations of every node, evaluated on the GPU from the stored values.
//
// A read-out is bound by the copy of its result to the caller's memory.  (Evaluated on the
// host from a copy of the whole buffer, the three macroscopic fields of a 2000 x 200 FP64
// lattice took 30-45 ms: one thread converting 3.6 M values and forming the moments, per
// field, with two passes over freshly allocated memory of the size of all nine populations.)
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cstring>

#include "lbib_device.hpp"
#include "lbib_host.hpp"
#include "lbib_internal.hpp"

namespace lbib {

using namespace dev;

namespace {

// The plain population f_q of node (i, j): the weight plus the stored deviation, the shifted
// equilibrium of the node that emitted it (the f - f_eq storages) and the moving wall's term.
// Each term is added on its own, in this order, and the moments below are plain sums over q.
template <typename T>
__device__ __forceinline__ double plain_population(const T* __restrict__ f, const SweepArgs& a, int q, int i, int j,
                                                   bool pull)
{
    double v;
    if constexpr (sizeof(typename St<T>::raw) == 2)
        v = (double)st_load(f, pop_index(q, i, j, a.nx, a.ny, a.pitch, a.plane, pull), 1.0, false) * a.inv_scale;
    else
        v = st_load(f, pop_index(q, i, j, a.nx, a.ny, a.pitch, a.plane, pull), 1.0, false);
    if constexpr (St<T>::neq) {
        const float* m = neq_moments(f, a.pitch, a.plane, a.ny);
        int si, sj, dir;
        pop_source(q, i, j, a.nx, a.ny, si, sj, dir);
        const int64_t c = (int64_t)sj * neq_mpitch(a.pitch, a.plane) + si;
        v += feq_shift<double>(dir, (double)m[c], (double)m[a.plane + c], (double)m[2 * a.plane + c]);
    }
    if (j == a.ny - 1) v += q == 7 ? -a.uw6 : q == 8 ? a.uw6 : 0.0;
    return kW[q] + v;
}

// One thread per value: rows v0, v0 + 1, ... of the result (row v of the populations is row
// v mod ny of population v / ny), a row of blocks for each.
template <typename T>
__global__ __launch_bounds__(256) void field_kernel(const T* __restrict__ f, SweepArgs a, int pull, int which,
                                                    int64_t v0, double* __restrict__ out)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= a.nx) return;
    const int64_t v = v0 + blockIdx.y;
    double* o = out + (int64_t)blockIdx.y * a.nx + i;
    if (which == 3) {
        const int q = (int)(v / a.ny), j = (int)(v - (int64_t)q * a.ny);
        *o = plain_population(f, a, q, i, j, pull != 0);
        return;
    }
    const int j = (int)v;
    double r = 0, jx = 0, jy = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const double p = plain_population(f, a, q, i, j, pull != 0);
        r += p;
        jx += p * kEx[q];
        jy += p * kEy[q];
    }
    *o = which == 0 ? r : which == 1 ? (jx + 0.5 * a.gx) / r : (jy + 0.5 * a.gy) / r;
}

template <typename T>
void launch_field(const void* f, const SweepArgs& a, bool pull, int which, int64_t v0, int64_t rows, double* out,
                  hipStream_t s)
{
    hipLaunchKernelGGL(field_kernel<T>, dim3((a.nx + 255) / 256, (uint32_t)rows), dim3(256), 0, s, (const T*)f, a,
                       (int)pull, which, v0, out);
}

// Largest device staging a read-out keeps: beyond it the rows go in several rounds.
constexpr size_t kStageMax = (size_t)64 << 20;

}  // namespace

void free_stage(FieldStage& st)
{
    if (st.p && st.host)
        (void)hipHostFree(st.p);
    else if (st.p)
        (void)hipFree(st.p);
    st = FieldStage{};
}

hipError_t reserve_stage(FieldStage& st, size_t want, size_t row_bytes, StageAlloc device, StageAlloc host)
{
    if (st.bytes >= want) return hipSuccess;
    free_stage(st);
    hipError_t e = hipSuccess;
    // a smaller stage where the device has no room for a large one, down to one row
    for (size_t bytes = want;; bytes = std::max(row_bytes, bytes / 2)) {
        e = device((void**)&st.p, bytes);
        if (e == hipSuccess) {
            st.bytes = bytes;
            return e;
        }
        st.p = nullptr;
        (void)hipGetLastError();
        if (e != hipErrorOutOfMemory) return e;
        if (bytes <= row_bytes) break;
    }
    if ((e = host((void**)&st.p, want)) != hipSuccess) {
        st.p = nullptr;
        (void)hipGetLastError();
        return e;
    }
    st.bytes = want;
    st.host = true;
    return hipSuccess;
}

hipError_t read_field(const void* f, const LatticeGeom& g, int which, double* out, FieldStage& st, hipStream_t s)
{
    const SweepArgs a = make_sweep_args(g);
    const int64_t rows = (which == 3 ? 9 : 1) * (int64_t)g.ny;
    const size_t row_bytes = (size_t)g.nx * sizeof(double);
    const size_t want = std::min((size_t)rows * row_bytes, std::max(kStageMax, row_bytes));
    hipError_t e = reserve_stage(
        st, want, row_bytes, [](void** p, size_t n) { return hipMalloc(p, n); },
        [](void** p, size_t n) { return hipHostMalloc(p, n, hipHostMallocDefault); });
    if (e != hipSuccess) return e;
    const int64_t most = std::min<int64_t>((int64_t)(st.bytes / row_bytes), 65535);  // rows of one launch's grid
    for (int64_t v = 0; v < rows; v += most) {
        const int64_t n = std::min(most, rows - v);
        switch (g.precision) {
            case LBIB_FP64: launch_field<double>(f, a, g.pull, which, v, n, st.p, s); break;
            case LBIB_FP32: launch_field<float>(f, a, g.pull, which, v, n, st.p, s); break;
            case LBIB_FP16: launch_field<half_t>(f, a, g.pull, which, v, n, st.p, s); break;
            case LBIB_BF16: launch_field<bf16_t>(f, a, g.pull, which, v, n, st.p, s); break;
            case LBIB_FP16_NEQ: launch_field<half_neq_t>(f, a, g.pull, which, v, n, st.p, s); break;
            default: launch_field<bf16_neq_t>(f, a, g.pull, which, v, n, st.p, s); break;
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (!st.host && (e = hipMemcpyAsync(out + (size_t)v * g.nx, st.p, (size_t)n * row_bytes, hipMemcpyDeviceToHost,
                                            s)) != hipSuccess)
            return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (st.host) std::memcpy(out + (size_t)v * g.nx, st.p, (size_t)n * row_bytes);
    }
    return hipSuccess;
}

}  // namespace lbib
