"""GPU: the field read-outs against numpy on the values the storage holds, including results
larger than one staging round (64 MiB) and rows that are no multiple of the launch width."""
import numpy as np
import pytest

from paper_1808_01448_amd import workloads as W

pytestmark = pytest.mark.gpu

WQ = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
EX = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1])
EY = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("drive", [0, 1])
@pytest.mark.parametrize("precision,nx,ny", [("fp64", 4, 4), ("fp32", 257, 5), ("fp32", 1201, 801), ("fp64", 300, 31)])
def test_fields_are_the_stored_values(precision, nx, ny, drive, layout):
    from paper_1808_01448_amd import lbib

    w = W.without_particle(W.with_precision(W.channel_small_fp64(), precision))
    w["lattice"].update(nx=nx, ny=ny, drive=drive)
    lat = w["lattice"]
    f = WQ[:, None, None] * (1.0 + W.random_perturbation(7, (9, ny, nx), 1e-3))
    with lbib.Sim(w, layout=layout) as s:
        s.write_populations(f)
        got, (rho, ux, uy) = s.f, s.fields()
    # the stored deviation, the moving wall's term kept out of the two values it reaches
    nu = (lat["tau"] - 0.5) / 3.0
    um = lat["re"] * nu / ny
    term = np.zeros((9, ny, 1))
    if drive == 1:
        term[7, -1], term[8, -1] = -um / 6.0, um / 6.0
    g = f - WQ[:, None, None] - term
    if precision == "fp32":
        g = g.astype(np.float32).astype(np.float64)
    ref = WQ[:, None, None] + (g + term)
    assert np.array_equal(got, ref)
    # the moments: each of the nine additions rounds at most to 2^-53 of the running sum
    gx = 0.0 if drive == 1 else 8.0 * nu * um / (ny * ny)
    r = ref.sum(0)
    assert np.max(np.abs(rho - r)) <= 16 * 2.0**-53
    assert np.max(np.abs(ux - ((ref * EX[:, None, None]).sum(0) + 0.5 * gx) / r)) <= 16 * 2.0**-53
    assert np.max(np.abs(uy - (ref * EY[:, None, None]).sum(0) / r)) <= 16 * 2.0**-53
