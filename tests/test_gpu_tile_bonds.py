"""GPU tests of the basis-lattice tile kernels' two bond loops: DMI on no bond,
on the first, a middle or the last one, on one atom's own bonds only and on
all of them, against the FP64 oracle."""

import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, make_pair, need_gpu

pytestmark = pytest.mark.gpu

HAM = si.Hamiltonian(mu=(2.0, 1.5), B=(0.1, -0.3, 0.8), K=(0.2, 0.1), K_axis=((0, 0, 1), (1, 0, 0)))
BONDS = [(0, 1, (0, 0, 0), 1.0), (0, 1, (-1, 0, 0), 0.9), (0, 1, (0, -1, 0), 0.8), (0, 0, (1, 0, 0), -0.3),
         (0, 0, (0, 1, 0), -0.25), (0, 0, (1, -1, 0), 0.2), (1, 1, (1, 0, 0), 0.15), (1, 1, (0, 1, 0), -0.1)]
WHERE = {"none": (), "first": (0,), "middle": (4,), "last": (7,), "atom1": (6, 7), "all": tuple(range(8))}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("where", sorted(WHERE))
def test_dmi_anywhere_in_the_bond_table(ora, where, precision):
    announce(f"tile bonds {where} {precision}")
    pairs = [b + ((0.1 * k - 0.3, 0.2, 0.05 * k) if k in WHERE[where] else (0.0, 0.0, 0.0),)
             for k, b in enumerate(BONDS)]
    e, s = make_pair(ora, si.honeycomb(37, 24, periodic=(1, 0, 0)), HAM, precision)
    e.set_pairs(pairs)
    s.set_pairs(pairs)
    assert e.step_path == "fusedtile"
    n = si.uniform_sphere(s.N, 23)
    e.set_spins(n)
    assert_close(e.gradient(), s.gradient(n), precision, what="gradient")
    e.run(0.3, 0.001, 6, T=12.0, seed=4)
    m, _ = s.run(n, 0.3, 0.001, 6, T=12.0, seed=4)
    assert_close(e.get_spins(), m, precision, what="six steps")
