"""The rules that choose a sweep, evaluated on the host.  CPU only."""
import itertools

import pytest

import _host_plan as H

INT32_MAX = 2**31 - 1
ELEM = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}


def columns(prec):
    """Around the row length at which lattice_geom turns from rows of nine segments to population
    planes, and around those whose window reaches a buffer resource's bound."""
    align = 256 // ELEM[prec]
    edge = INT32_MAX // 9 // align * align
    bound = {"rows": 2**31 // (27 * ELEM[prec]), "planes": 2**31 // (3 * ELEM[prec])}
    near = [edge + d for d in (-align, 0, 1, align, 2 * align)]
    near += [b // align * align + d for b in bound.values() for d in (-align, 0, 1, align)]
    return sorted({n for n in near + [4, 61, 4096, 8192, 300_000_000, 357_000_000] if n * 4 <= 2**31})


@pytest.mark.parametrize("prec", list(ELEM))
def test_two_step_windows_hold_every_population(prec):
    """Where one simulation or a pool sweeps two steps in one pass, the window of three pitches
    that starts a row below a node's holds all nine populations of the three rows, and its
    offsets fit 32 bits."""
    chosen = 0
    for nx, ny in itertools.product(columns(prec), (4, 7, 9)):
        if nx * ny > 2**31:
            continue
        g = H.lattice(nx, ny, prec)
        if not (g["pairs"] or H.pool_pairs([(nx, ny, prec)])):
            continue
        chosen += 1
        window = 3 * g["pitch"] * g["elem"]
        # the last access: row 2 of the window, population 8, the last column
        last = (2 * g["pitch"] + 8 * g["plane"] + nx) * g["elem"]
        assert last <= window < 2**31, (nx, ny, g)
    assert chosen > 0


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_population_planes_are_swept_step_by_step(prec):
    """238 609 408 columns: nine rows exceed a 32-bit pitch, three planes' rows do not."""
    g = H.lattice(238_609_408, 4, prec)
    assert not g["interleaved"] and 3 * g["pitch"] * g["elem"] < 2**31
    assert not g["pairs"]
    assert not H.pool_pairs([(2048, 4096, prec), (238_609_408, 4, prec)])


@pytest.mark.parametrize("nx,ny,prec,nl,serial,overlapped", [
    # steps of a call that run faster one way, by 4 us or more
    (256, 64, "fp64", 64, (1, 2, 3), (6, 7, 8, 100)),
    (512, 128, "fp32", 128, (1, 2, 3), (6, 8)),
    (1024, 256, "fp32", 192, (1, 2), (6, 8)),
    (1024, 400, "fp16", 384, (1, 2), (4, 6, 8)),
    (2000, 200, "fp64", 320, (1,), (3, 4, 6, 8)),
    (2048, 600, "fp32", 576, (1,), (3, 4, 6, 8)),
    (4096, 1024, "fp32", 64, (1,), (2, 3, 4, 6)),
    (4096, 1024, "fp32", 256, (1,), (2, 3, 4, 6)),
    (4096, 1024, "fp32", 960, (1,), (2, 3, 4, 6)),
    (4096, 1024, "fp64", 576, (), (1, 2, 3, 4)),
    (4096, 1024, "fp64", 960, (), (1, 2, 3, 4)),
    (8192, 4096, "fp16", 960, (), (2, 3, 4)),
    (2999, 777, "bf16_neq", 384, (1,), (2, 3, 4)),
    (2999, 777, "bf16_neq", 640, (1,), (3, 4)),
])
def test_short_calls(nx, ny, prec, nl, serial, overlapped):
    """The calls that mode 2 runs serially, by lattice, markers and steps."""
    assert [H.short_call(nx, ny, prec, nl, n) for n in serial] == [True] * len(serial)
    assert [H.short_call(nx, ny, prec, nl, n) for n in overlapped] == [False] * len(overlapped)


def test_the_pair_tests_sweep_pairs():
    """The lattices and calls of the GPU tests of the two-step sweeps take that path."""
    import test_gpu_pairs as P
    import test_gpu_pool_pairs as Q

    for (nx, ny), prec in itertools.product(P.SIZES + [(1024, 260)], ("fp64", "fp32", "fp16", "bf16")):
        if (nx, ny) == (1024, 260) and prec in ("fp16", "bf16"):
            continue  # used with the wider storages
        assert H.lattice(nx, ny, prec)["pairs"], (nx, ny, prec)
        for q in P.PARTICLES.values():
            long = [n for n in P.CALLS if not H.short_call(nx, ny, prec, q.get("nl", 64), n)]
            assert any(n % 2 for n in long) and any(n % 2 == 0 for n in long), (nx, ny, prec, long)
    for prec, nx, ny in next(m for m in P.test_fluid_alone.pytestmark if m.args[:1] == ("prec,nx,ny",)).args[1]:
        assert H.lattice(nx, ny, prec)["pairs"], (nx, ny, prec)
    for prec in ("fp64", "fp32", "fp16", "bf16"):
        f = Q.filler(prec)["lattice"]
        assert H.pool_pairs([(nx, ny, prec) for nx, ny in Q.EDGES] + [(f["nx"], f["ny"], prec)])
        assert H.pool_pairs([(64, 32, prec), (f["nx"], f["ny"], prec)])
    assert not H.lattice(256, 64, "fp64")["pairs"] and not H.pool_pairs([(256, 64, "fp64")] * 12)
