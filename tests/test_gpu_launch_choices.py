"""GPU tests of choices between kernels that give the same results: each
compares the time of the choice taken with a form of the same work that
cannot take the other one, with room for the spread of short timings."""

import time

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, need_gpu

pytestmark = pytest.mark.gpu

HAM_SQ = si.WORKLOADS["square32_fp64"].hamiltonian
HAM_TRI = si.WORKLOADS["triangular512_sllg"].hamiltonian


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _best(call, repeats=9, inner=1):
    call()
    times = []
    for _ in range(repeats):
        t0 = time.perf_counter()
        for _ in range(inner):
            call()
        times.append((time.perf_counter() - t0) / inner)
    return min(times)


def _batch_time(geos):
    import torch

    import paper_1901_11350_amd as pk

    b = pk.Batch(0)
    for r, geo in enumerate(geos):
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        e.set_spins(si.uniform_sphere(e.N, r))
        b.add(e, 0.3, 0.001, T=0.0, seed=5, replica=r)
        e.close()

    def run():
        b.run(256)
        torch.cuda.synchronize()

    t = _best(run)
    b.close()
    return t


def test_mixed_batch_steps_in_one_launch():
    """Three small replicas of different boundary forms (power-of-two sides,
    periodic, open) step in about the time of three open ones: launches one
    after another took 2.6 times as long."""
    announce("mixed batch launches")
    mixed = [si.square(128, 128), si.square(96, 80), si.square(75, 70, periodic=(0, 1, 0))]
    alike = [si.square(128, 128, periodic=(0, 1, 0)), si.square(96, 80, periodic=(0, 1, 0)), mixed[2]]
    assert _batch_time(mixed) < 1.6 * _batch_time(alike)


def test_replicas_of_a_mixed_batch_equal_single_engines():
    """Tiled replicas of all three boundary forms, bit for bit their
    single-engine runs on the batch's tile configuration."""
    import paper_1901_11350_amd as pk

    announce("mixed batch bits")
    geos = [si.square(128, 64), si.square(96, 80), si.square(75, 70, periodic=(0, 1, 0)), si.square(256, 128)]
    b = pk.Batch(0)
    b.set_chunk(4)
    inits = []
    for r, geo in enumerate(geos):
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        inits.append(si.uniform_sphere(e.N, 70 + r))
        e.set_spins(inits[r])
        b.add(e, 0.3, 0.001, T=20.0, seed=5, replica=r)
        e.close()
    b.run(9)
    for r, geo in enumerate(geos):
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        e.step_path = "shape2d/32x16x512"
        e.set_spins(inits[r])
        e.run(0.3, 0.001, 9, T=20.0, seed=5, replica=r)
        assert np.array_equal(b.get_spins(r), e.get_spins()), f"replica {r}"
        e.close()
    b.close()


@pytest.mark.parametrize("case", ["square45x45", "tri64x32", "tri32x32"])
def test_single_steps_of_small_lattices_cost_no_more_than_a_tile_launch(case):
    """One call of llg_step on the path the engine chose itself against the
    tile kernel chosen by name (one workgroup for all sites took 1.2 to 1.4
    times as long on the larger two)."""
    import paper_1901_11350_amd as pk

    announce(f"single steps {case}")
    geo, ham = {"square45x45": (si.square(45, 45), HAM_TRI), "tri64x32": (si.triangular(64, 32), HAM_TRI),
                "tri32x32": (si.triangular(32, 32), HAM_TRI)}[case]
    e = pk.Engine(0, "f32")
    e.set_geometry(geo)
    e.set_hamiltonian(ham)
    e.set_spins(si.uniform_sphere(e.N, 1))

    def step():
        e.llg_step(0.1, 0.0005)
        e.synchronize()

    own = _best(step, inner=30)
    e.step_path = e.step_path
    tile = _best(step, inner=30)
    assert own < 1.12 * tile


def test_few_bonds_are_not_summed_on_tiles():
    """Six bonds of two cells' length per site (100^3, FP32), where staging the
    halo costs more than the loop over the bonds, against the same table with
    one pair too far for any frame, which only the loop takes: the smaller
    table is the faster one (on tiles it took 1.25 times as long)."""
    import paper_1901_11350_amd as pk

    announce("few bonds")
    pairs = [(0, 0, d, 0.5, (0.0, 0.0, 0.0)) for d in ((2, 0, 0), (0, 2, 0), (0, 0, 2))]
    times = []
    for extra in ([], [(0, 0, (40, 40, 40), 0.5, (0.0, 0.0, 0.0))]):
        e = pk.Engine(0, "f32")
        e.set_geometry(si.simple_cubic(100, 100, 100))
        e.set_hamiltonian(si.Hamiltonian(mu=(2.0,), B=(0, 0, 0.3), K=(0.1,), K_axis=((0, 0, 1),)))
        e.set_pairs(pairs + extra)
        e.set_spins(si.uniform_sphere(e.N, 1))
        e.step_path = "twopass"
        times.append(_best(lambda: e.run(0.3, 0.001, 50), repeats=5))
        e.close()
    assert times[0] < 1.05 * times[1]


def test_pair_tiles_add_little_to_an_engine_s_setup():
    """Creating an engine, its Hamiltonian and destroying it: a honeycomb
    lattice, whose gradients take pair tiles, against a triangular one, which
    has none (an allocation and a copy for the tiles' records made the first
    1.4 times the second)."""
    import torch

    import paper_1901_11350_amd as pk

    announce("pair tile setup")
    honey = si.honeycomb(86, 47)
    ham = {"honeycomb": si.Hamiltonian(mu=(2.0, 2.0), B=(0, 0, 0.3), K=(0.1, 0.1), K_axis=((0, 0, 1),) * 2,
                                       J=(1.0, -0.2, -0.1), D=(0.2,)),
           "triangular": si.Hamiltonian(mu=(2.0,), B=(0, 0, 0.3), K=(0.1,), K_axis=((0, 0, 1),),
                                        J=(1.0, -0.2, -0.1), D=(0.2,))}
    geo = {"honeycomb": honey, "triangular": si.triangular(94, 86)}
    times = {}
    for name in ("triangular", "honeycomb"):

        def cycle():
            e = pk.Engine(0, "f32")
            e.set_geometry(geo[name])
            e.set_hamiltonian(ham[name])
            torch.cuda.synchronize()
            e.close()

        times[name] = _best(cycle, repeats=30)
    assert times["honeycomb"] < 1.2 * times["triangular"]


@pytest.mark.parametrize("shells", [1, 3])
def test_steps_at_zero_temperature_draw_no_field(shells):
    """Steps of a periodic lattice with power-of-two sides at T = 0 against the
    same steps at T > 0: cheaper, as no thermal field is drawn (0.99 times as
    long when it was drawn and not used)."""
    import paper_1901_11350_amd as pk

    announce(f"zero temperature {shells}")
    e = pk.Engine(0, "f32")
    e.set_geometry(si.square(256, 256))
    e.set_hamiltonian(si.Hamiltonian(mu=(2.0,), B=(0, 0, 0.3), K=(0.1,), K_axis=((0, 0, 1),),
                                     J=(1.0, 0.4, -0.2)[:shells]))
    e.set_spins(si.uniform_sphere(e.N, 1))
    times = [_best(lambda: e.run(0.3, 0.001, 1000, T=T, seed=3), repeats=7) for T in (0.0, 20.0)]
    e.close()
    assert times[0] < 0.96 * times[1]


@pytest.mark.parametrize("dmi", [False, True], ids=["exchange", "dmi"])
def test_thermal_steps_of_open_26_bond_lattices(dmi):
    """Three shells of an open cubic lattice at T > 0 against the same steps at
    T = 0 (1.25 to 1.28 times as long with the generator that holds more
    registers, 1.16 to 1.18 with the other one)."""
    import paper_1901_11350_amd as pk

    announce(f"open 26 bonds {dmi}")
    e = pk.Engine(0, "f32")
    e.set_geometry(si.simple_cubic(64, 64, 64, periodic=(0, 0, 0)))
    e.set_hamiltonian(si.Hamiltonian(mu=(2.0,), B=(0, 0.1, 0.3), K=(0.1,), K_axis=((0, 0, 1),), J=(1.0, 0.4, -0.2),
                                     D=(0.2,) if dmi else ()))
    e.set_spins(si.uniform_sphere(e.N, 1))
    times = [_best(lambda: e.run(0.3, 0.001, 300, T=T, seed=1), repeats=7) for T in (0.0, 20.0)]
    e.close()
    assert times[1] < 1.22 * times[0]
