"""The host-side rules of the library, called through a small C++ shim linked with it (no GPU is
used): the shim is compiled here against the library's internal headers."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

import numpy as np

from paper_1808_01448_amd import build, lbib

SHIM = r"""
#include "lbib_host.hpp"
using namespace lbib;
extern "C" {
// interleaved, pitch, plane, element bytes, one simulation's two-step sweeps, their rows per unit
// alone and beside a particle
void plan_lattice(const lbib_lattice_desc* d, int64_t* out)
{
    const LatticeGeom g = lattice_geom(*d);
    out[0] = g.interleaved;
    out[1] = g.pitch;
    out[2] = g.plane;
    out[3] = (int64_t)g.elem;
    out[4] = pair_sweeps(g);
    out[5] = pair_rows(g, false);
    out[6] = pair_rows(g, true);
}
// helpers, marked nodes at a pose (NULL: the first) and those that LDS holds there; -1: refused
int plan_particle(const lbib_lattice_desc* d, const lbib_particle_desc* pd, const double* pose, int64_t* out)
{
    Particle p;
    std::string msg;
    if (prepare_particle(*d, *pd, p, msg) != LBIB_OK) return -1;
    const MarkedNodes m = pose ? marked_nodes(p, d->ny, pose[0], pose[1], pose[2])
                               : marked_nodes(p, d->ny, pd->xc, pd->yc, pd->theta0);
    out[0] = with_helpers(lattice_geom(*d), p);
    out[1] = m.nodes;
    out[2] = particle_lds_slots(p.box_cap, (int32_t)m.box);
    return 0;
}
// the stage that a read-out of `want` bytes in rows of `row` gets where the device can give `room`
// bytes at most and the host gives any (host_ok) or none
static int64_t room;
static int host_ok;
int plan_stage(int64_t r, int ok, int64_t want, int64_t row, int64_t* out)
{
    room = r;
    host_ok = ok;
    FieldStage st;
    const hipError_t e = reserve_stage(
        st, (size_t)want, (size_t)row,
        [](void** p, size_t n) {
            if ((int64_t)n > room) return hipErrorOutOfMemory;
            *p = (void*)0x1000;
            return hipSuccess;
        },
        [](void** p, size_t) {
            if (!host_ok) return hipErrorOutOfMemory;
            *p = (void*)0x2000;
            return hipSuccess;
        });
    out[0] = (int64_t)st.bytes;
    out[1] = st.host;
    out[2] = st.p == (double*)0x1000 ? 1 : st.p == (double*)0x2000 ? 2 : st.p == nullptr ? 0 : -1;
    return (int)e;
}
// field `which` of a lattice's initial state, through a stage in device or in host memory
int field_through(const lbib_lattice_desc* d, int which, int host, double* out)
{
    const LatticeGeom g = lattice_geom(*d);
    void* f = nullptr;
    FieldStage st;
    st.bytes = (which == 3 ? 9 : 1) * (size_t)g.nx * g.ny * sizeof(double);
    st.host = host != 0;
    hipError_t e = hipMalloc(&f, g.buf_bytes);
    if (e == hipSuccess)
        e = host ? hipHostMalloc((void**)&st.p, st.bytes, hipHostMallocDefault) : hipMalloc((void**)&st.p, st.bytes);
    if (e == hipSuccess) e = init_populations(f, g, nullptr);
    if (e == hipSuccess) e = read_field(f, g, which, out, st, nullptr);
    free_stage(st);
    (void)hipFree(f);
    return (int)e;
}
int plan_short(const lbib_lattice_desc* d, int nl, int64_t n) { return short_call(lattice_geom(*d), nl, n); }
int plan_pool(const lbib_lattice_desc* d, int64_t n)
{
    std::vector<LatticeGeom> g;
    for (int64_t k = 0; k < n; ++k) g.push_back(lattice_geom(d[k]));
    return pool_pair_sweeps(g);
}
}
"""


@functools.lru_cache(maxsize=1)
def shim():
    if not os.path.exists(lbib.LIB_PATH):
        build.build()
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(SHIM)
        libdir = os.path.dirname(lbib.LIB_PATH)
        subprocess.check_call([build.hipcc(), *build.FLAGS, "-w", "-shared", src, "-o", so, "-L", libdir,
                               "-l:" + os.path.basename(lbib.LIB_PATH), f"-Wl,-rpath,{libdir}"])
        return C.CDLL(so)


def lattice_desc(nx, ny, precision, drive=0):
    from paper_1808_01448_amd import workloads as W

    return lbib.LatticeDesc(nx, ny, 0.8, 0.5, drive, W.PRECISION[precision], 0)


def lattice(nx, ny, precision):
    out = (C.c_int64 * 7)()
    shim().plan_lattice(C.byref(lattice_desc(nx, ny, precision)), out)
    return dict(zip(("interleaved", "pitch", "plane", "elem", "pairs", "rows_alone", "rows_particle"), out))


def short_call(nx, ny, precision, nl, steps):
    return bool(shim().plan_short(C.byref(lattice_desc(nx, ny, precision)), C.c_int(nl), C.c_int64(steps)))


def stage(room, host_ok, want, row):
    out = (C.c_int64 * 3)()
    e = shim().plan_stage(C.c_int64(room), C.c_int(host_ok), C.c_int64(want), C.c_int64(row), out)
    return e, out[0], bool(out[1]), ("none", "device", "host")[out[2]]


def field_through(nx, ny, precision, which, host):
    out = np.zeros((9 if which == 3 else 1, ny, nx))
    d = lattice_desc(nx, ny, precision, drive=1)
    assert shim().field_through(C.byref(d), which, int(host), out.ctypes.data_as(C.POINTER(C.c_double))) == 0
    return out


def pool_pairs(members):
    """members: (nx, ny, precision) each."""
    d = (lbib.LatticeDesc * len(members))(*[lattice_desc(*m) for m in members])
    return bool(shim().plan_pool(d, C.c_int64(len(members))))


def particle(w, pose=None):
    """Of a workload's particle: helpers, and at the pose (x, y, theta; None: its first) the marked
    nodes and how many LDS holds."""
    lat, p = w["lattice"], w["particle"]
    d = lbib.LatticeDesc(lat["nx"], lat["ny"], lat["tau"], lat["re"], lat.get("drive", 0), lat["precision"], 0)
    pd = lbib.ParticleDesc(*[p[k] for k, _ in lbib.ParticleDesc._fields_])
    out = (C.c_int64 * 3)()
    at = None if pose is None else (C.c_double * 3)(*pose)
    assert shim().plan_particle(C.byref(d), C.byref(pd), at, out) == 0
    return dict(helpers=bool(out[0]), nodes=out[1], slots=out[2])
