"""GPU: the fastest particle the overlapped schedules accept, whose box moves by up to two nodes in
each step: sweeps of two steps accept it as sweeps of one do, with the serial schedule's results."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W
from test_gpu_pairs import same, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("vx,vy,xc", [(1.2, 0.0, 300.0), (-1.2, 0.0, 300.0), (0.0, 1.2, 300.0),
                                      (0.0, -1.2, 300.0), (1.2, 0.0, 1019.0), (-1.2, 0.0, 6.0)])
def test_two_nodes_a_step(vx, vy, xc, layout):
    from paper_1808_01448_amd import lbib as L

    w = workload("fp32", 1024, 260)
    w["particle"].update(xc=xc, yc=130.0)
    out = []
    for mode in (0, 1, 2):
        with L.Sim(w, layout=layout) as s:
            s.set_overlap(mode)
            s.trace_enable(7)
            s.step(2)
            s.write_particle([xc, 130.0, 0.0, vx, vy, 0.0, xc - vx, 130.0 - vy, 0.0, vx, vy, 0.0])
            s.step(5)
            s.sync()
            out.append((s.f, s.trace(7), s.bonds()[0]))
    same(out[1], out[0])
    same(out[2], out[0])
    # more than two nodes in two steps
    col = [L.STATE_FIELDS.index(c) for c in ("xc", "yc")]
    x = out[0][1][2:, col]
    assert (np.abs(x[2:] - x[:-2]).max(1) > 2.0).all()
