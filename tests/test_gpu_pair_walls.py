"""GPU: sweeps of two steps beside a particle, with the moving wall in the push layout and the
resting walls in the pull layout: bit for bit the serial schedule's results."""
import pytest

from test_gpu_pairs import PARTICLES, SIZES, result, same, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("which", ["seam", "top"])
def test_particle(prec, which, layout):
    from paper_1808_01448_amd import lbib as L

    nx, ny = SIZES[list(PARTICLES).index(which)]
    w = workload(prec, nx, ny, drive=1 - layout, **PARTICLES[which])
    same(result(L, w, 2, layout), result(L, w, 0, layout))


def test_default_layout_is_push():
    """... where a shear flow is swept in pairs by default."""
    from paper_1808_01448_amd import lbib as L

    w = workload("fp64", *SIZES[0], drive=1)
    with L.Sim(w) as s:
        assert not s.pull
    same(result(L, w, 2, 2), result(L, w, 0, 2))
