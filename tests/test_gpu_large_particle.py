"""GPU: particles whose box has about a node per thread, and particles whose box has more mask
words than a round of the node map takes, with the node fields in LDS and, for the widest marker
spacing, in the global scratch; against the FP64 oracle, in both layouts and schedules."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    # boxes on both sides of a node per thread (512): taken whole, and marked and mapped
    **{f"whole_{r}": dict(a_major=r, b_minor=r, n_markers=64, shape=0) for r in (8.0, 8.4, 8.8, 9.2, 9.6)},
    # box 4100 nodes: the last that the map takes by half-waves, and the first beyond
    "words_128": dict(a_major=30.0, b_minor=30.0, n_markers=192, shape=0),
    "words_129": dict(a_major=30.5, b_minor=30.5, n_markers=192, shape=0),
    # two markers a thread, 2000 marked nodes in LDS
    "lds": dict(a_major=98.0, b_minor=49.0, n_markers=640, shape=1),
    # about 4200 marked nodes: more than LDS holds beside the mask
    "scratch": dict(a_major=120.0, b_minor=118.0, n_markers=1024, shape=1),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("overlap", [0, 2])
@pytest.mark.parametrize("which", list(SHAPES))
def test_against_the_oracle(orc, which, overlap, layout):
    from paper_1808_01448_amd import lbib

    p = dict(SHAPES[which])
    ny = int(2 * p["a_major"] + 40)
    nx = int(2 * p["a_major"] + 70)
    w = W.channel_small_fp64()
    w["lattice"].update(nx=nx, ny=ny, re=1.0)
    w["particle"].update(p, xc=nx - 20.3, yc=p["a_major"] + 0.5 * W.Y_CR_HAT * ny - 0.5, theta0=0.0)
    steps = 12
    with lbib.Sim(w, layout=layout) as s:
        s.set_overlap(overlap)
        s.trace_enable(steps)
        s.step(steps)
        s.sync()
        got, bonds, f = s.trace(steps), s.bonds()[0], s.f
    o = orc.Sim.from_workload(w)
    _, ref = o.step(steps, trace=True)
    ref = np.asarray(ref)
    col = {n: c for c, n in enumerate(lbib.STATE_FIELDS)}
    for names in (("ux", "uy"), ("fx", "fy"), ("xc", "yc")):
        a, b = (t[:, [col[n] for n in names]] for t in (got, ref))
        assert np.linalg.norm(a - b) <= 1e-10 * np.linalg.norm(b), names
    m, scale = (t[:, col["torque"]] for t in (got, ref)), np.linalg.norm(ref[:, [col["fx"], col["fy"]]])
    assert np.linalg.norm(np.subtract(*m)) <= 1e-10 * (p["a_major"] * scale + np.linalg.norm(ref[:, col["torque"]]))
    assert np.array_equal(got[:, col["n_bonds"]], ref[:, col["n_bonds"]])
    assert np.array_equal(got[:, col["n_probing"]], ref[:, col["n_probing"]])
    wq = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]
    assert np.linalg.norm(f - o.f) <= 2e-9 * np.linalg.norm(o.f - wq)
