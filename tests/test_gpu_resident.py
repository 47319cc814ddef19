"""GPU tests of the resident launches of small 2D lattices (one workgroup,
many steps) against the tile kernel of the same path, chosen by name, and the
oracle: one and two sites per thread, ragged and one-row lattices, open
edges, every solver, chunks of any length and the step counter."""

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, make_pair, need_gpu

pytestmark = pytest.mark.gpu

HAM_SQ = si.WORKLOADS["square32_fp64"].hamiltonian
HAM_TRI = si.WORKLOADS["triangular512_sllg"].hamiltonian

CASES = {
    "square8x8": (si.square(8, 8), HAM_SQ),
    "square32x32": (si.square(32, 32), HAM_SQ),
    "square33x31_open": (si.square(33, 31, periodic=(0, 1, 0)), HAM_SQ),
    "square1025": (si.square(41, 25), HAM_SQ),            # FP32: the first size with two sites per thread
    "tri64x32": (si.triangular(64, 32), HAM_TRI),         # FP32: the last resident size
    "tri65x32": (si.triangular(65, 32), HAM_TRI),         # the first beyond it
    "tri7x9_open": (si.triangular(7, 9, periodic=(0, 0, 0)), HAM_TRI),
}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("solver", ["depondt", "heun", "sib"])
@pytest.mark.parametrize("case", list(CASES))
def test_resident_run_matches_oracle_and_tile_kernel(ora, case, solver, precision):
    """The repository's parity bounds against the oracle (FP64 1e-12, FP32
    1e-5) after 21 stochastic steps in chunks of 5; against the tile kernel,
    which evaluates the same expressions, the FP32 bound of its own instances
    (1e-6) and 1e-13 in FP64."""
    announce(f"resident {case} {solver} {precision}")
    geo, ham = CASES[case]
    e, s = make_pair(ora, geo, ham, precision)
    n0 = si.uniform_sphere(geo.n_sites, 5)
    kw = dict(T=10.0, seed=99, solver=solver)
    e.set_spins(n0)
    e.step = (1 << 32) - 10                     # the counter's low word overflows on the way
    obs = e.run(0.1, 0.0005, 21, observe_every=5, **kw)
    assert e.step == (1 << 32) + 11 and len(obs) == 4
    got = e.get_spins()
    label = e.step_path
    e.step_path = label                         # chosen by name: the tile kernel
    e.set_spins(n0)
    e.step = (1 << 32) - 10
    tile_obs = e.run(0.1, 0.0005, 21, observe_every=5, **kw)
    bound = 1e-13 if precision == "f64" else 1e-6
    assert np.abs(got - e.get_spins()).max() <= bound
    for a, b in zip(obs, tile_obs):
        assert a["step"] == b["step"] and abs(a["E"] - b["E"]) <= 10 * bound * abs(b["E"])
    # single steps from the same start
    e.set_hamiltonian(ham)                      # the engine's own choice again
    e.set_spins(n0)
    e.step = 3
    for _ in range(4):
        e.llg_step(0.1, 0.0005, **kw)
    one = e.get_spins()
    e.set_spins(n0)
    e.step = 3
    e.run(0.1, 0.0005, 4, **kw)
    assert np.array_equal(one, e.get_spins())
    e.set_spins(n0)
    e.step = 0
    e.run(0.1, 0.0005, 21, **kw)
    ref, _ = s.run(n0, 0.1, 0.0005, 21, **kw)
    assert_close(e.get_spins(), ref, precision, what=f"resident {case}")


def test_resident_convergence_stop():
    """The run stops at the observation that passes and leaves its state."""
    import paper_1901_11350_amd as pk

    announce("resident convergence")
    e = pk.Engine(0, "f64")
    geo = si.square(16, 16)
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    e.set_spins(si.skyrmion_ansatz(geo, radius=3.0, noise_rad=0.1, seed=2))
    obs, done = e.run_tol(0.5, 0.002, 40000, 50, 1e-3)
    assert 0 < done < 40000 and done % 50 == 0 and e.step == done
    assert obs[-1]["max_torque"] < 1e-3 <= obs[-2]["max_torque"]
    assert abs(e.observe()["E"] - obs[-1]["E"]) <= 1e-12 * abs(obs[-1]["E"])
