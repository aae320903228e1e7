"""GPU: pools large enough to sweep two steps in one pass.  Every member must match its
stand-alone run (one step at a time) bit for bit, whatever its size, seam position, step count
and the calls it is stepped by; members that end or fail inside a pair make only their step."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W
from test_gpu_pool import assert_same, member, pooled

pytestmark = pytest.mark.gpu

# columns and rows around the strips (62 columns, four a workgroup) and runs (8 to 32 rows) of the
# two-step sweep; a particle across the periodic seam; a top wall in motion
EDGES = [(61, 24), (62, 25), (63, 31), (124, 32), (247, 33), (248, 40), (249, 47), (311, 48), (64, 23)]


def alone(L, w, steps):
    s = L.Sim(w)
    s.set_overlap(0)
    s.trace_enable(max(steps, 1))
    s.step(steps)
    s.sync()
    out = dict(particle=s.particle(), bonds=s.bonds()[0], f=s.f, trace=s.trace(max(steps, 1)))
    s.close()
    return out


def filler(precision):
    """A member whose lattice brings the pool past the traffic from which it sweeps pairs."""
    return member(2048, {"fp64": 400, "fp32": 720}.get(precision, 1440), a=8.0, nl=64, seed=99, precision=precision)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("tiles,graph", [(1, 0), (4, 0), (8, 5)])
def test_members_match_standalone(prec, tiles, graph):
    from paper_1808_01448_amd import lbib as L

    cases = []
    for k, (nx, ny) in enumerate(EDGES):
        w = member(nx, ny, seed=k, re=0.1 + 0.3 * k, xc=float(nx) - 0.4 if k % 2 else None, theta0=0.1 * k,
                   shape=k % 2, a=4.5, b=3.0, precision=prec)
        w["lattice"]["drive"] = 1 if k % 3 == 0 else 0
        cases.append((w, (13, 14, 1, 20, 9, 2, 17, 6, 3)[k]))
    cases.append((filler(prec), 8))
    with L.Pool(W.PRECISION[prec]) as P:
        P.set_config(256, tiles, graph)
        slots = [P.add(w, n) for w, n in cases]
        for s, (_, n) in zip(slots, cases):
            P.trace_enable(s, n)
        for n in (3, 2, 1, 4, 5, 7):
            P.step(n)
        P.poll()
        for (w, n), s in zip(cases, slots):
            assert P.status(s) == (n, L.POOL_FINISHED), w["name"]
            assert_same(pooled(P, s, n), alone(L, w, n), w["name"])


@pytest.mark.parametrize("first", [0, 1])
def test_failure_inside_a_pair(first):
    """A particle that touches the wall fails at its step, the pair's first or second."""
    from paper_1808_01448_amd import lbib as L

    bad = member(64, 32, gap=1e-6, seed=0)  # touches the wall within a few tens of steps
    ref = L.Sim(bad)
    ref.set_overlap(0)
    fail = None
    for k in range(60):
        ref.step(1)
        try:
            ref.sync()
        except L.LbibError:
            fail = k + 1
            break
    ref.close()
    assert fail is not None, "the stand-alone run did not touch the wall"
    ok = alone(L, bad, fail - 1)
    with L.Pool(L.FP64) as P:
        f = P.add(filler("fp64"), 1 << 40)
        b = P.add(bad, 10_000)
        P.trace_enable(b, 10_000)
        P.step(first)  # shifts the pairs by a step
        P.step(fail + 5)
        P.poll()
        assert P.status(b) == (fail, L.POOL_FAILED)
        tb = P.trace(b, 10_000)
        assert tb.shape[0] == fail
        np.testing.assert_array_equal(tb[: fail - 1], ok["trace"][: fail - 1])
        assert P.status(f) == (first + fail + 5, L.POOL_RUNNING)
        assert_same(dict(pooled(P, f, 1), trace=0), dict(alone(L, filler("fp64"), first + fail + 5), trace=0), "filler")


def test_field_of_a_member_mid_run():
    """The level a member has reached is read from the buffer that holds it, after odd and even
    numbers of steps, pairs and single ones."""
    from paper_1808_01448_amd import lbib as L

    w = member(200, 37, seed=2, precision="fp32")
    with L.Pool(L.FP32) as P:
        P.add(filler("fp32"), 1 << 40)
        s = P.add(w, 1 << 40)
        done = 0
        for n in (1, 2, 3, 4, 1, 2):
            P.step(n)
            done += n
            P.poll()
            np.testing.assert_array_equal(P.field(s, 3), alone(L, w, done)["f"])
