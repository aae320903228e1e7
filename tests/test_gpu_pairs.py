"""GPU: simulations large enough to sweep two steps in one pass.  The default schedule must give
the serial schedule's results (one step per sweep) bit for bit: populations, trace and bonds,
over calls of odd and even lengths, in both layouts, at sizes around the strips (62 columns,
four a workgroup) and units (4 to 16 rows) of the two-step sweep."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W

pytestmark = pytest.mark.gpu

CALLS = (1, 2, 3, 4, 1, 6, 5, 2)
# (nx, ny) with at least 16 MB of traffic per step in every storage here
SIZES = [(1985, 240), (1984, 241), (2047, 256), (2233, 225)]


def workload(precision, nx, ny, *, a=8.0, b=8.0, nl=64, shape=0, xc=None, theta0=0.0, drive=0):
    w = W.channel_small_binding(precision)
    w["lattice"].update(nx=nx, ny=ny, drive=drive, re=0.5, seed=3)
    half = np.hypot(a * np.cos(theta0), b * np.sin(theta0))
    w["particle"].update(shape=shape, a_major=a, b_minor=b, n_markers=nl, theta0=theta0, xc=nx / 4 if xc is None else xc,
                         yc=-0.5 + 0.5 * W.Y_CR_HAT * ny + half)
    return w


def result(L, w, mode, layout, calls=CALLS, between=None):
    with L.Sim(w, layout=layout) as s:
        s.set_overlap(mode)
        if s.nl:
            s.trace_enable(sum(calls))
        for k, n in enumerate(calls):
            s.step(n)
            if between:
                between(s, k)
        s.sync()
        return (s.f, s.trace(sum(calls)), s.bonds()[0]) if s.nl else (s.f,)


def same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


PARTICLES = {
    "circle": dict(),
    "seam": dict(xc=1.3, shape=1, a=9.0, b=5.0, theta0=0.7),
    "wide": dict(shape=1, a=70.0, b=100.0, nl=640),  # a box wider than a workgroup's strips' third
    "top": dict(xc=700.0, a=100.0, b=100.0, nl=800),  # several units high
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("which", list(PARTICLES))
def test_particle(prec, which, layout):
    from paper_1808_01448_amd import lbib as L

    nx, ny = SIZES[list(PARTICLES).index(which)]
    w = workload(prec, nx, ny, drive=layout, **PARTICLES[which])
    same(result(L, w, 2, layout), result(L, w, 0, layout))


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("drive", [0, 1])
@pytest.mark.parametrize("prec,nx,ny", [("fp64", 1985, 61), ("fp32", 1984, 300), ("fp16", 2233, 225), ("fp32", 70000, 4),
                                        ("fp64", 28000, 5)])
def test_fluid_alone(prec, nx, ny, drive, layout):
    """A random state, against the one-step sweeps (calls of one step)."""
    from paper_1808_01448_amd import lbib as L

    w = W.without_particle(workload(prec, nx, ny, drive=drive))
    f = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None] * (1 + W.random_perturbation(5, (9, ny, nx), 1e-4))
    out = []
    for calls in (CALLS, (1,) * sum(CALLS)):
        with L.Sim(w, layout=layout) as s:
            s.write_populations(f)
            for n in calls:
                s.step(n)
            out.append(s.f)
    np.testing.assert_array_equal(*out)


def test_schedule_switches_and_state_changes():
    """Other schedules between pairs, overwritten bonds and populations, a checkpoint."""
    from paper_1808_01448_amd import lbib as L

    w = workload("fp32", 1024, 260)

    def between(s, k, switch):
        if k == 1:
            s.write_bonds(np.zeros(s.nl, np.uint8))
        if k == 3:
            s.write_populations(s.f)
        if k == 5:
            s.load(s.save())
        if switch:
            s.set_overlap((2, 1, 2, 0, 2, 1, 2, 3)[k % 8])

    got = result(L, w, 2, 0, between=lambda s, k: between(s, k, True))
    ref = result(L, w, 0, 0, between=lambda s, k: between(s, k, False))
    same(got, ref)


def test_two_resident_launches_in_a_call():
    """A call longer than one resident particle launch covers (1024 steps), odd."""
    from paper_1808_01448_amd import lbib as L

    w = workload("fp32", 1024, 260)
    same(result(L, w, 2, 0, calls=(1031,)), result(L, w, 0, 0, calls=(1031,)))


def test_interleaved_simulations():
    """Two simulations enqueued alternately, beside each other on the GPU."""
    from paper_1808_01448_amd import lbib as L

    ws = [workload("fp32", 1024, 260), workload("fp64", 1985, 240, xc=1.3)]
    sims = [L.Sim(w) for w in ws]
    for s in sims:
        s.trace_enable(sum(CALLS))
    for n in CALLS:
        for s in sims:
            s.step(n)
    for s, w in zip(sims, ws):
        s.sync()
        same((s.f, s.trace(sum(CALLS)), s.bonds()[0]), result(L, w, 0, 2))
        s.close()
