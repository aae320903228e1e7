"""GPU: particles whose nodes are about as many as LDS holds fields of, stored as f - f_eq with
helpers: steps that are shared and steps that are the leader's alone in the same launch, bit for
bit against the serial schedule; and the host's rule for who has helpers."""
import numpy as np
import pytest

import _host_plan as H
from paper_1808_01448_amd import workloads as W


def workload(a, b, nl, precision="fp16_neq", theta0=0.0, y=None):
    ny, nx = int(2 * a + 40), int(2 * a + 71)
    w = W.channel_small_fp64()
    w["lattice"].update(nx=nx, ny=ny, re=4.0, precision=W.PRECISION[precision])
    w["particle"].update(shape=1, a_major=a, b_minor=b, n_markers=nl, theta0=theta0, xc=nx - 20.3,
                         yc=a + 0.5 * W.Y_CR_HAT * ny - 0.5 if y is None else y)
    return w


LIMIT = (122.0, 120.0, 1024)


@pytest.mark.parametrize("shape,helpers", [
    ((52.0, 26.0, 383), False), ((52.0, 26.0, 384), True), ((98.0, 49.0, 640), True),
    ((126.0, 124.0, 1024), False), ((140.0, 136.0, 1024), False)])
def test_who_has_helpers(shape, helpers):
    for prec in ("fp16_neq", "bf16_neq"):
        p = H.particle(workload(*shape, precision=prec))
        assert p["helpers"] == helpers, p
    assert not H.particle(workload(*shape, precision="fp16"))["helpers"]


def poses(w, steps, v, n):
    """Poses from which a straight motion by v a step passes the limit, found by trying."""
    rng = np.random.default_rng(7)
    found = []
    while len(found) < n:
        p = np.array([w["particle"]["xc"], w["particle"]["yc"], 0.2]) + rng.random(3) * [1.0, 1.0, 0.2]
        fit = [q["nodes"] <= q["slots"] for q in (H.particle(w, p + k * v) for k in range(0, steps, 3))]
        if any(fit[1:]) and not all(fit[1:]):
            found.append(p)
    return found


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("precision", ["fp16_neq", "bf16_neq"])
def test_steps_beyond_lds(precision, layout):
    from paper_1808_01448_amd import lbib

    w = workload(*LIMIT, precision=precision, y=141.7)
    assert H.particle(w)["helpers"]
    v = np.array([3e-3, 2e-3, 1e-5])
    starts = poses(w, 40, v, 5)
    res = []
    for overlap in (0, 2):
        with lbib.Sim(w, layout=layout) as s:
            s.set_overlap(overlap)
            s.trace_enable(40 * len(starts))
            for p in starts:
                s.write_particle(np.concatenate([p, v, p - v, v]))
                s.step(33)
                s.step(7)
            s.sync()
            res.append((s.trace(40 * len(starts)), s.bonds()[0], s.f))
    for a, b in zip(*res):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    col = [lbib.STATE_FIELDS.index(c) for c in ("xc", "yc", "theta")]
    fit = np.array([q["nodes"] <= q["slots"] for q in (H.particle(w, row[col]) for row in res[1][0])]).reshape(-1, 40)
    # (the record of a step is the pose the next one starts from)
    inside = fit[:, 1:31]
    assert sum(inside.any(1) & ~inside.all(1)) >= 3, fit
