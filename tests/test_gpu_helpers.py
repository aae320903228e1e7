"""GPU: the helpers of the resident particle launch (f - f_eq storages, from 384 markers), bit for
bit against the serial schedule, which has none: the first particle that has them and the last
that has not, one and two markers a thread, more nodes than LDS holds, both storages and layouts,
a particle across the periodic edge, and runs of one step, two and many."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "below": dict(a_major=52.0, b_minor=26.0, n_markers=383, shape=1),
    "first": dict(a_major=52.0, b_minor=26.0, n_markers=384, shape=1),
    # the closest markers: the fewest nodes that the helpers share
    "dense": dict(a_major=15.5, b_minor=15.5, n_markers=384, shape=0),
    "two_a_thread": dict(a_major=98.0, b_minor=49.0, n_markers=640, shape=1),
    # about 4200 marked nodes: more than LDS holds beside the mask
    "scratch": dict(a_major=120.0, b_minor=118.0, n_markers=1024, shape=1),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("precision", ["fp16_neq", "bf16_neq"])
@pytest.mark.parametrize("which", list(SHAPES))
def test_same_as_serial(which, precision, layout):
    from paper_1808_01448_amd import lbib

    p = dict(SHAPES[which])
    ny = int(2 * p["a_major"] + 40)
    nx = int(2 * p["a_major"] + 71)
    w = W.channel_small_fp64()
    w["lattice"].update(nx=nx, ny=ny, re=1.0)
    w["lattice"]["precision"] = W.PRECISION[precision]
    w["particle"].update(p, xc=nx - 20.3, yc=p["a_major"] + 0.5 * W.Y_CR_HAT * ny - 0.5, theta0=0.0)
    calls = [1, 2, 1, 60, 33, 3]
    res = []
    for overlap in (0, 2):
        with lbib.Sim(w, layout=layout) as s:
            s.set_overlap(overlap)
            s.trace_enable(sum(calls))
            for n in calls:
                s.step(n)
            s.sync()
            res.append((s.trace(sum(calls)), s.bonds()[0], s.f))
    for a, b in zip(*res):
        assert np.array_equal(np.asarray(a), np.asarray(b))


def test_several_at_once():
    """Three simulations with helpers, their calls enqueued in turn with no wait between them."""
    from paper_1808_01448_amd import lbib

    ws = []
    for k in range(3):
        w = W.channel_small_fp64()
        w["lattice"].update(nx=600 + 37 * k, ny=300, re=1.0, precision=W.PRECISION["bf16_neq"], seed=k)
        w["particle"].update(SHAPES["two_a_thread"], xc=250.5, yc=98.0 + 0.5 * W.Y_CR_HAT * 300 - 0.5, theta0=0.0)
        ws.append(w)

    def final(overlap):
        sims = [lbib.Sim(w) for w in ws]
        for s in sims:
            s.set_overlap(overlap)
        for n in (40, 25, 60):
            for s in sims:
                s.step(n)
        out = []
        for s in sims:
            s.sync()
            out.append((s.particle(), s.bonds()[0].tobytes(), s.f.tobytes()))
            s.close()
        return out

    assert final(2) == final(0)
