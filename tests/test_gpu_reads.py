"""GPU: the record and the bond flags read after steps, after writes of the state and after a
checkpoint is restored, against the trace and the values written."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("particles", [1, 3])
def test_reads_follow_the_state(particles):
    from paper_1808_01448_amd import lbib as L

    if particles == 1:
        w = W.channel_small_binding("fp64")
    else:
        w = W.multi_particle_channel(256, 96, particles, seed=1, precision="fp64", area_frac=0.02)
        for e in w["particles"]:  # bonds from the first steps
            e["ligand"].update(y_cr_hat=0.9, k_f=0.5)
    with L.Sim(w) as s:
        for k in range(particles):
            assert s.particle(k)["step"] == -1 and not s.bonds(k)[0].any()
            s.trace_enable(40, k)
        done = 0
        for n in (1, 1, 7, 2, 9):
            s.step(n)
            done += n
            for k in range(particles):
                last = s.trace(40, k)[done - 1]
                rec, (b, lig) = s.particle(k), s.bonds(k)
                assert [rec[f] for f in L.STATE_FIELDS] == list(last)
                assert int(b.sum()) == rec["n_bonds"] and not np.any(b & ~lig & 1)
        assert s.bonds(0)[0].any()
        blob, rec, b = s.save(), s.particle(0), s.bonds(0)[0]
        s.write_bonds(np.zeros(s.nls[0], np.uint8))
        assert not s.bonds(0)[0].any()
        s.step(3)
        assert s.particle(0)["step"] == done + 2
        s.load(blob)
        assert s.particle(0) == rec
        np.testing.assert_array_equal(s.bonds(0)[0], b)
