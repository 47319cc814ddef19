"""GPU tests of LLG steps with the FFT dipole field (row kernel with the local
field, spectra carried from step to step) against the FP64 oracle: rows of
several 64-site segments, periodic axes with wraps and own images, cells of
two and three atoms, one to four planes, odd numbers of channels, tables of
more than 64 bonds, observations that break the chain of spectra, every
solver, and the convergence stop."""

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import TOL, announce, assert_close, make_pair, need_gpu

pytestmark = pytest.mark.gpu

SP_DDI_FFT = 3


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _ham(k=1, J=(1.0,), D=()):
    return si.Hamiltonian(mu=(2.0, 1.5, 0.7)[:k], B=(0.1, 0.0, 0.3), K=(0.2, 0.1, 0.3)[:k],
                          K_axis=((0, 0, 1), (1, 0, 0), (0, 1, 0))[:k], J=J, D=D, ddi=SP_DDI_FFT)


def _box(r):
    """Every pair within a box once; every fourth with a DMI vector."""
    out = []
    for a in range(-r[0], r[0] + 1):
        for b in range(-r[1], r[1] + 1):
            for c in range(-r[2], r[2] + 1):
                if (a, b, c) > (0, 0, 0):
                    k = len(out)
                    out.append((0, 0, (a, b, c), 0.5 * (-1) ** k / (a * a + b * b + c * c),
                                (0.02, -0.01, 0.03) if k % 4 == 0 else (0.0, 0.0, 0.0)))
    return out


# lattice, Hamiltonian, pairs (None: shells)
CASES = {
    "film140x6x4": (si.simple_cubic(140, 6, 4, periodic=(0, 0, 0)), _ham(), None),     # 12 segments of a row
    "film33x18x1": (si.simple_cubic(33, 18, 1, periodic=(0, 0, 0)), _ham(J=(1.0, -0.2)), None),
    "film20x12x3": (si.simple_cubic(20, 12, 3, periodic=(0, 0, 0)), _ham(D=(0.2,)), None),
    "film20x12x5": (si.simple_cubic(20, 12, 5, periodic=(0, 0, 0)), _ham(), None),     # the separate kernels
    "periodic24x20x2": (si.simple_cubic(24, 20, 2, periodic=(1, 1, 0)), _ham(J=(1.0, 0.3), D=(0.2, 0.1)), None),
    # offsets of a whole axis (the site itself), beyond it, and beyond an open one
    "images3x20x2": (si.simple_cubic(3, 20, 2, periodic=(1, 1, 1)), _ham(),
                     [(0, 0, (3, 0, 0), 0.3, (0.0, 0.1, 0.0)), (0, 0, (4, 1, 0), 0.4, (0.1, 0.0, 0.0)),
                      (0, 0, (0, 0, 1), 0.5, (0.0, 0.0, 0.1)), (0, 0, (-2, 21, 0), 0.2, (0.0, 0.0, 0.0))]),
    "open6x9x2": (si.simple_cubic(6, 9, 2, periodic=(0, 1, 0)), _ham(),
                  [(0, 0, (7, 0, 0), 3.0, (1.0, 0.0, 0.0)), (0, 0, (1, 2, 1), 0.4, (0.1, 0.0, 0.0)),
                   (0, 0, (-5, 1, 0), 0.5, (0.0, 0.2, 0.0))]),
    "honeycomb18x11": (si.honeycomb(18, 11), _ham(2, J=(1.0, 0.2), D=(0.1,)), None),
    "kagome17x9": (si.kagome(17, 9), _ham(3, J=(1.0, 0.2)), None),
    "bonds74_12x10x4": (si.simple_cubic(12, 10, 4, periodic=(1, 0, 0)), _ham(), _box((2, 2, 1))),
    "bonds124_70x6x2": (si.simple_cubic(70, 6, 2, periodic=(1, 1, 0)), _ham(), _box((2, 2, 2))),
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", list(CASES))
def test_observed_steps_match_oracle(ora, case, precision):
    """Seven stochastic steps, observed after the third and the sixth: spins
    and observations within the parity bounds (FP64 1e-12, FP32 1e-5; energies
    relative to the sum of the terms' magnitudes)."""
    announce(f"fft steps {case} {precision}")
    geo, ham, pairs = CASES[case]
    e, s = make_pair(ora, geo, ham, precision)
    if pairs:
        e.set_pairs(pairs)
        s.set_pairs(pairs)
    n0 = si.uniform_sphere(geo.n_sites, 41)
    e.set_spins(n0)
    e.step = 5
    obs = e.run(0.2, 0.001, 7, T=15.0, seed=12, observe_every=3)
    ref, ref_obs = s.run(n0, 0.2, 0.001, 7, T=15.0, seed=12, step0=5, observe_every=3)
    assert_close(e.get_spins(), ref, precision, what=f"spins {case}")
    assert [o["step"] for o in obs] == [o["step"] for o in ref_obs] == [8, 11]
    for o, r in zip(obs, ref_obs):
        scale = sum(abs(x) for x in r["per_term"])
        assert abs(o["E"] - r["E"]) <= 10 * TOL[precision] * scale


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("solver", ["heun", "sib"])
@pytest.mark.parametrize("case", ["film33x18x1", "kagome17x9", "periodic24x20x2"])
def test_other_solvers_match_oracle(ora, case, solver, precision):
    announce(f"fft steps {case} {solver} {precision}")
    geo, ham, _ = CASES[case]
    e, s = make_pair(ora, geo, ham, precision)
    n0 = si.uniform_sphere(geo.n_sites, 42)
    e.set_spins(n0)
    e.run(0.2, 0.001, 5, T=15.0, seed=12, solver=solver)
    ref, _ = s.run(n0, 0.2, 0.001, 5, T=15.0, seed=12, solver=solver)
    assert_close(e.get_spins(), ref, precision, what=f"spins {case} {solver}")


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_chained_steps_equal_single_ones(precision):
    """Steps of one run, of two runs and one by one, and a field evaluated in
    between: the same spins, bit for bit."""
    import paper_1901_11350_amd as pk

    announce(f"fft chained steps {precision}")
    geo, ham, _ = CASES["film20x12x3"]
    n0 = si.uniform_sphere(geo.n_sites, 43)
    out = []
    for way in ("run", "runs", "steps", "fields"):
        e = pk.Engine(0, precision)
        e.set_geometry(geo)
        e.set_hamiltonian(ham)
        e.set_spins(n0)
        if way == "run":
            e.run(0.2, 0.001, 6, T=15.0, seed=12)
        elif way == "runs":
            e.run(0.2, 0.001, 2, T=15.0, seed=12)
            e.run(0.2, 0.001, 4, T=15.0, seed=12, observe_every=1)
        else:
            for _ in range(6):
                e.llg_step(0.2, 0.001, T=15.0, seed=12)
                if way == "fields":
                    e.dipole_gradient()
                    e.observe()
        out.append(e.get_spins())
        e.close()
    for other in out[1:]:
        assert np.array_equal(out[0], other)


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_convergence_stop_leaves_the_observed_state(precision):
    """A damped run stops at the observation that passes; its spins are those
    of a run of as many steps, and further steps go on from them."""
    import paper_1901_11350_amd as pk

    announce(f"fft convergence {precision}")
    geo, ham, _ = CASES["film20x12x3"]
    n0 = si.skyrmion_ansatz(geo, radius=3.0, noise_rad=0.1, seed=2)
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(ham)
    e.set_spins(n0)
    obs, done = e.run_tol(0.5, 0.002, 700, 7, 1.2)
    assert 0 < done < 700 and done % 7 == 0 and e.step == done
    assert obs[-1]["max_torque"] < 1.2 <= obs[-2]["max_torque"]
    stopped = e.get_spins()
    e.set_spins(n0)
    e.step = 0
    e.run(0.5, 0.002, done, observe_every=7)
    assert np.array_equal(e.get_spins(), stopped)
    e.run(0.5, 0.002, 3)
    e2 = pk.Engine(0, precision)
    e2.set_geometry(geo)
    e2.set_hamiltonian(ham)
    e2.set_spins(stopped)
    e2.run(0.5, 0.002, 3)
    assert np.allclose(e.get_spins(), e2.get_spins(), rtol=0, atol=1e-12 if precision == "f64" else 1e-6)
