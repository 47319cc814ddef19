"""GPU tests of the direct dipole sum against the oracle's pair sums at the
sizes where the matrix-core form changes shape: 16-site tiles and 64-site
source chunks with and without a remainder along a, sixteen-row blocks along
b, one to four wavefronts per workgroup, several planes and atoms per cell,
and lattices whose padding leaves them to the vector form."""

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, need_gpu

pytestmark = pytest.mark.gpu

CASES = {
    "16x16x1": si.simple_cubic(16, 16, 1, periodic=(0, 0, 0)),
    "17x15x2": si.simple_cubic(17, 15, 2, periodic=(0, 0, 0)),
    "33x32x3": si.simple_cubic(33, 32, 3, periodic=(0, 0, 0)),
    "64x17x1": si.simple_cubic(64, 17, 1, periodic=(0, 0, 0)),
    "65x16x1": si.simple_cubic(65, 16, 1, periodic=(0, 0, 0)),
    "130x31x2": si.simple_cubic(130, 31, 2, periodic=(1, 0, 0)),
    "triangular48x33": si.triangular(48, 33),
    "honeycomb20x18": si.honeycomb(20, 18),
    "kagome33x16": si.kagome(33, 16),
    "chain300": si.simple_cubic(300, 1, 1, periodic=(0, 0, 0)),
    "column5x3x90": si.simple_cubic(5, 3, 90, periodic=(0, 0, 0)),
}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", list(CASES))
def test_direct_sum_matches_oracle(ora, case, precision):
    """The repository's parity bounds (FP64 1e-12, FP32 1e-5 normwise): a sum
    of a few thousand rounded products with two-level accumulation errs by
    some hundred roundings at most."""
    import paper_1901_11350_amd as pk

    announce(f"direct dipole {case} {precision}")
    geo = CASES[case]
    k = geo.n_basis
    ham = si.Hamiltonian(mu=(2.0, 1.5, 0.7)[:k], B=(0, 0, 0), K=(0.0,) * k, K_axis=((0, 0, 1),) * k, ddi=True)
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(ham)
    n = si.uniform_sphere(geo.n_sites, 31)
    e.set_spins(n)
    got = e.dipole_gradient()
    s = ora.System(geo, ham)
    sites = np.unique(np.concatenate([np.random.default_rng(9).choice(geo.n_sites, min(250, geo.n_sites), replace=False),
                                      [0, geo.n_sites - 1]]))
    assert_close(got[:, sites], s.dipole_gradient_sites(n, sites), precision, what=f"direct dipole {case}")
