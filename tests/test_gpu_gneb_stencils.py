"""GPU tests of the GNEB gradient tiles on the stencils of reach two and three
(two and three shells of the square and triangular lattices, with and without
DMI), on ragged lattices with open and periodic sides and on both tile sides,
against the oracle."""

import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _ham(J, D=()):
    return si.Hamiltonian(mu=(2.0,), B=(0.0, 0.1, 0.5), K=(0.1,), K_axis=((0, 0, 1),), J=J, D=D)


# lattice, Hamiltonian, images (32 x 32 tiles from 256 workgroups on, else 16 x 16)
CASES = {
    "square2_16": (si.square(21, 18), _ham((1.0, -0.2), (0.3,)), 7),
    "square2_32": (si.square(37, 33, periodic=(0, 1, 0)), _ham((1.0, -0.2)), 70),
    "square3_16": (si.square(17, 35, periodic=(0, 0, 0)), _ham((1.0, -0.2, 0.1), (0.3,)), 6),
    "square3_32": (si.square(33, 40), _ham((1.0, -0.2, 0.1), (0.3,)), 70),
    "tri1_16": (si.triangular(19, 33, periodic=(1, 0, 0)), _ham((1.0,), (0.2,)), 5),
    "tri2_16": (si.triangular(18, 20), _ham((1.0, 0.3)), 9),
    "tri2_32": (si.triangular(34, 38), _ham((1.0, 0.3), (0.2,)), 70),
    "tri3_16": (si.triangular(23, 17, periodic=(0, 1, 0)), si.WORKLOADS["triangular512_sllg"].hamiltonian, 6),
    "tri3_32": (si.triangular(40, 35, periodic=(1, 0, 0)), si.WORKLOADS["triangular512_sllg"].hamiltonian, 70),
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", list(CASES))
def test_gneb_stencils_match_oracle(ora, case, precision):
    """Forces at the start and the chain after three iterations within the
    parity bounds (FP64 1e-12, FP32 1e-5)."""
    import paper_1901_11350_amd as pk

    announce(f"gneb stencils {case} {precision}")
    geo, ham, M = CASES[case]
    a = si.skyrmion_ansatz(geo, radius=5.0, width=1.5)
    chain = si.geodesic_chain(a, si.ferromagnet(geo.n_sites, (0, 0, 1)), M, fallback_axis=(1, 0, 0))
    kw = dict(k_spring=1.0, vp_dt=0.1, vp_mass=1.0)
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(ham)
    assert e.step_path.startswith("shape2d")
    g = pk.Gneb(e, chain, **kw)
    o = ora.Gneb(ora.System(geo, ham), chain, **kw)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert_close(g.forces()["F"], o.forces()["F"], precision, tol, what=f"forces {case}")
    g.iterate(3)
    o.iterate(3)
    assert_close(g.chain(), o.chain, precision, tol, what=f"chain {case}")
    g.close()
