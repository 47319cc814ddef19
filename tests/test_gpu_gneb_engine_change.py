"""GPU tests of a GNEB chain whose engine gets another Hamiltonian while the
chain lives: every image, the fixed ones too, is evaluated with the engine's
present Hamiltonian from the next iteration on, whatever kernels and tiles
that Hamiltonian takes (oracle: the same switch between iterations)."""

import dataclasses

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, need_gpu

pytestmark = pytest.mark.gpu

HAM_SQ = si.WORKLOADS["square32_fp64"].hamiltonian
FIELD = dataclasses.replace(HAM_SQ, B=(0.0, 0.4, 1.5), K=(0.3,))
GAUSS = dataclasses.replace(HAM_SQ, gauss=((0.4, 0.5, (0.0, 0.6, 0.8)),))
PAIRS = [(0, 0, (1, 0, 0), 0.8, (0.0, 0.2, 0.0)), (0, 0, (0, 1, 0), 0.9, (-0.2, 0.0, 0.0)),
         (0, 0, (2, 1, 0), 0.1, (0.0, 0.0, 0.0))]

# lattice, images, first and second Hamiltonian, second as explicit pairs
CASES = {
    "field": (si.square(45, 37), 8, HAM_SQ, FIELD, False),
    "tiles_to_sites": (si.square(128, 128), 20, HAM_SQ, GAUSS, False),      # 16 tiles, then 64 blocks per image
    "tiles_to_pairs": (si.square(45, 37), 12, HAM_SQ, HAM_SQ, True),
    "sites_to_tiles": (si.square(17, 33, periodic=(0, 1, 0)), 5, GAUSS, FIELD, False),   # 3 blocks, then 6 tiles
}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _chain(geo, M):
    a = si.skyrmion_ansatz(geo, radius=5.0, width=1.5)
    return si.geodesic_chain(a, si.ferromagnet(geo.n_sites, (0, 0, 1)), M, fallback_axis=(1, 0, 0))


@pytest.mark.parametrize("how", ["iterate", "tol", "batch"])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_chain_follows_the_engine(ora, case, precision, how):
    """One iteration before the switch and two after it (a batch, which
    captures its chunk of two: two and two), within the parity bounds of the
    chains (FP64 1e-12, FP32 1e-5); the energies of all images, relative to
    the largest."""
    import paper_1901_11350_amd as pk

    announce(f"gneb engine change {case} {precision} {how}")
    if how == "batch" and precision == "f64":
        pytest.skip("batches are FP32")
    geo, M, first, second, as_pairs = CASES[case]
    chain = _chain(geo, M)
    kw = dict(k_spring=1.0, vp_dt=0.1, vp_mass=1.0)
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(first)
    g = pk.Gneb(e, chain, **kw)
    o = ora.Gneb(ora.System(geo, first), chain, **kw)
    b = None
    if how == "batch":
        r = pk.Engine(0, "f32")
        r.set_geometry(si.square(32, 32))
        r.set_hamiltonian(HAM_SQ)
        r.set_spins(si.uniform_sphere(r.N, 1))
        b = pk.Batch(0)
        b.set_chunk(2)
        b.add(r, 0.3, 0.001)
        b.add_gneb(g)

    def go(n):
        if how == "iterate":
            g.iterate(n)
        elif how == "tol":
            assert g.iterate_tol(n, 1e-30) == n
        else:
            b.run(n)

    n_before = 2 if how == "batch" else 1
    go(n_before)
    o.iterate(n_before)
    e.set_hamiltonian(second)
    s = ora.System(geo, second)
    if as_pairs:
        e.set_pairs(PAIRS)
        s.set_pairs(PAIRS)
    o.s = s
    go(2)
    o.iterate(2)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert_close(g.chain(), o.chain, precision, tol, what=f"chain {case}")
    f = g.forces()
    E = o.forces()["E"]
    assert np.abs(f["E"] - E).max() <= tol * np.abs(E).max()
    g.close()


def test_chain_refuses_an_engine_without_its_lattice():
    """Another number of sites, or no Hamiltonian: SP_E_ORDER, nothing runs."""
    import paper_1901_11350_amd as pk
    from paper_1901_11350_amd.engine import SpError

    announce("gneb engine without its lattice")
    geo = si.square(20, 18)
    e = pk.Engine(0, "f64")
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    g = pk.Gneb(e, _chain(geo, 5))
    g.iterate(2)
    before = g.chain()
    e.set_geometry(geo)                             # drops the Hamiltonian
    for call in (lambda: g.iterate(1), lambda: g.iterate_tol(1, 1e-3)):
        with pytest.raises(SpError) as err:
            call()
        assert err.value.code == pk.SP_E_ORDER
    e.set_geometry(si.square(24, 24))
    e.set_hamiltonian(HAM_SQ)
    with pytest.raises(SpError) as err:
        g.iterate(1)
    assert err.value.code == pk.SP_E_ORDER
    assert np.array_equal(g.chain(), before)
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    g.iterate(1)
    assert np.abs(g.chain() - before).max() > 0
    g.close()
