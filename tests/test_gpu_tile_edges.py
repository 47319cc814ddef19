"""GPU tests at the edges of the tiled kernels' ranges: frames of the pair
tiles (ragged tiles, sides below the reach, offsets of half a lattice, open
axes, frames too large for LDS), the GNEB kernels' tile sides and images per
workgroup, replica batches of mixed boundary forms, and the forms of the
Monte Carlo pair sums."""

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import TOL, announce, assert_close, make_pair, need_gpu

pytestmark = pytest.mark.gpu

HAM = si.Hamiltonian(mu=(2.0,), B=(0.1, -0.3, 0.8), K=(0.2,), K_axis=((0, 0, 1),))
HAM2 = si.Hamiltonian(mu=(2.0, 1.5), B=(0.2, 0.1, 0.5), K=(0.1, 0.3), K_axis=((0, 0, 1), (1, 0, 0)))
HAM_SQ = si.WORKLOADS["square32_fp64"].hamiltonian


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _box(reach, axes=3):
    """Every direction once within a box of the given reach (the reverse of a
    pair is implied), DMI on every third pair."""
    out = []
    r = list(reach) + [0] * (3 - axes)
    for a in range(-r[0], r[0] + 1):
        for b in range(-r[1], r[1] + 1):
            for c in range(-r[2], r[2] + 1):
                if (a, b, c) <= (0, 0, 0):
                    continue
                k = len(out)
                out.append((0, 0, (a, b, c), 0.5 * (-1) ** k / (a * a + b * b + c * c),
                            (0.02, -0.01 * k / 60, 0.03) if k % 3 == 0 else (0.0, 0.0, 0.0)))
    return out


BASIS2_GEO = si.Geometry(((1.0, 0, 0), (0, 1.0, 0), (0, 0, 1.0)), ((0, 0, 0), (0.3, 0.4, 0.5)), (19, 5, 9), (1, 0, 1))
PAIRS = {
    # every bond list a multiple of eight or not, sites of the last tile outside
    "cubic17x9x7": (si.simple_cubic(17, 9, 7), HAM, _box((2, 2, 1))),
    "cubic16x16x8_open": (si.simple_cubic(16, 16, 8, periodic=(0, 0, 0)), HAM, _box((2, 1, 2))),
    # sides below the reach: offsets fold onto nearer images and the site itself
    "cubic3x40x2": (si.simple_cubic(3, 40, 2), HAM, [(0, 0, (3, 0, 0), 0.3, (0.0, 0.1, 0.0)),
                                                    (0, 0, (2, 1, 0), 0.4, (0.1, 0.0, 0.0)),
                                                    (0, 0, (1, 5, 1), -0.2, (0.0, 0.0, 0.1)),
                                                    (0, 0, (0, 20, 0), 0.25, (0.0, 0.2, 0.0)),   # half the side
                                                    (0, 0, (0, 21, 1), 0.15, (0.0, 0.0, 0.0))]),
    # open axis shorter than an offset: the bond has no partner anywhere
    "cubic24x6x4_open": (si.simple_cubic(24, 6, 4, periodic=(1, 0, 0)), HAM,
                         _box((1, 1, 1)) + [(0, 0, (0, 7, 0), 5.0, (1.0, 1.0, 1.0))]),
    "basis19x5x9": (BASIS2_GEO, HAM2, [(0, 1, (0, 0, 0), 0.8, (0.1, 0.0, -0.2)), (1, 0, (2, 1, 0), 0.3, (0.0, 0.2, 0.0)),
                                       (0, 0, (3, 1, 4), -0.2, (0.05, 0.05, 0.05)), (1, 1, (0, 2, -5), 0.5, (0, 0, 0))]),
    # the fused tile path, DMI in the last group of four bonds of one atom only
    "basis21x10_late_dmi": (si.Geometry(((1.0, 0, 0), (0, 1.0, 0), (0, 0, 1.0)), ((0, 0, 0), (0.3, 0.4, 0)),
                                        (21, 10, 1), (1, 0, 0)), HAM2,
                            [(0, 0, (1, 0, 0), 0.8, (0, 0, 0)), (0, 0, (0, 1, 0), 0.3, (0, 0, 0)),
                             (0, 1, (0, 0, 0), -0.2, (0, 0, 0)), (0, 1, (1, 0, 0), 0.4, (0, 0, 0)),
                             (0, 0, (2, 1, 0), 0.1, (0.2, 0.1, -0.3)), (1, 1, (1, 1, 0), 0.5, (0, 0, 0))]),
    # a frame past LDS: the site loop
    "square140x130_far": (si.square(140, 130), HAM, _box((1, 1), 2) + [(0, 0, (62, 1, 0), 0.3, (0.0, 0.1, 0.0)),
                                                                       (0, 0, (3, 61, 0), -0.2, (0.1, 0.0, 0.0))]),
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", sorted(PAIRS))
def test_pair_tiles_match_oracle(ora, case, precision):
    """Gradient, observables and three stochastic steps within the parity
    bounds (FP64 1e-12, FP32 1e-5)."""
    announce(f"pair tiles {case} {precision}")
    geo, ham, pairs = PAIRS[case]
    e, s = make_pair(ora, geo, ham, precision)
    e.set_pairs(pairs)
    s.set_pairs(pairs)
    n = si.uniform_sphere(s.N, 23)
    e.set_spins(n)
    assert_close(e.gradient(), s.gradient(n), precision, what=f"gradient {case}")
    o = e.observe()
    assert o["E"] == pytest.approx(s.energy(n), rel=10 * TOL[precision], abs=10 * TOL[precision] * s.N)
    ref, _ = s.run(n, 0.3, 0.001, 3, T=20.0, seed=5, step0=3)
    for path in ["twopass"] + ([e.step_path] if e.step_path != "twopass" else []):
        e.step_path = path
        e.set_spins(n)
        e.step = 3
        e.run(0.3, 0.001, 3, T=20.0, seed=5)
        assert_close(e.get_spins(), ref, precision, what=f"steps {path} {case}")


def _chain(geo, M):
    a = si.skyrmion_ansatz(geo, radius=5.0, width=1.5)
    return si.geodesic_chain(a, si.ferromagnet(geo.n_sites, (0, 0, 1)), M, fallback_axis=(1, 0, 0))


GNEB = {
    "tile16_1image": (si.square(45, 37), 12),
    "tile16_open": (si.square(17, 33, periodic=(0, 1, 0)), 3),
    "tile32_2images": (si.square(45, 37), 101),               # an odd number of interior images
    "tile32_4images": (si.square(45, 37, periodic=(1, 0, 0)), 300),
    "partials_summed_apart": (si.square(72, 64), 460),        # 115 x 18 partials
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", sorted(GNEB))
def test_gneb_tiles_match_oracle(ora, case, precision):
    """Forces and the chain after three iterations (an odd count leaves the
    chain in its other buffer) within the parity bounds."""
    import paper_1901_11350_amd as pk

    announce(f"gneb tiles {case} {precision}")
    geo, M = GNEB[case]
    chain = _chain(geo, M)
    kw = dict(k_spring=1.0, vp_dt=0.1, vp_mass=1.0)
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    g = pk.Gneb(e, chain, **kw)
    o = ora.Gneb(ora.System(geo, HAM_SQ), chain, **kw)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert_close(g.forces()["F"], o.forces()["F"], precision, tol, what=f"forces {case}")
    g.iterate(3)
    o.iterate(3)
    assert_close(g.chain(), o.chain, precision, tol, what=f"chain {case}")


def test_batch_of_mixed_boundary_forms_equals_single_engines():
    """Tiled replicas with power-of-two, other periodic and open sides and
    resident ones in one batch: each within the FP32 bound between instances
    (1e-6) of its single-engine run."""
    import paper_1901_11350_amd as pk

    announce("batch of mixed boundary forms")
    geos = [si.square(128, 128), si.square(96, 80), si.square(75, 70, periodic=(0, 1, 0)), si.square(32, 32),
            si.square(64, 256), si.square(90, 66, periodic=(0, 0, 0)), si.square(64, 64)]
    b = pk.Batch(0)
    b.set_chunk(4)
    inits = []
    for r, geo in enumerate(geos):
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        n0 = si.uniform_sphere(e.N, 300 + r)
        e.set_spins(n0)
        assert b.add(e, 0.3, 0.001, T=20.0, seed=5, replica=r) == r
        inits.append(n0)
        e.close()
    b.run(6)
    b.run(5)
    for r, geo in enumerate(geos):
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        e.step_path = "shape2d/32x16x512"
        e.set_spins(inits[r])
        e.run(0.3, 0.001, 11, T=20.0, seed=5, replica=r)
        assert np.abs(b.get_spins(r) - e.get_spins()).max() <= 1e-6, f"replica {r}"
        e.close()


MC_FAR = {   # lattice, pairs within it, and the same pairs written one lattice length further
    "square12x8": (si.square(12, 8), [((1, 0, 0), 1.0), ((0, 1, 0), 0.7)], (12, 8, 0)),
    "tri12x6": (si.triangular(12, 6), [((1, 0, 0), 1.0), ((0, 1, 0), 1.0), ((-1, 1, 0), 0.8)], (12, 6, 0)),
    "cubic6x8x10": (si.simple_cubic(6, 8, 10), [((1, 0, 0), 1.0), ((0, 1, 0), 0.7), ((0, 0, 1), -0.4)], (6, 8, 10)),
}


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", sorted(MC_FAR))
def test_mc_pair_forms_agree(case, precision):
    """The same bonds as nearest images without DMI, with a DMI vector too
    small to reach any sum's last bit, and written one lattice length further
    (wrapped by the general division): three instances of the pair sums, one
    chain, bit for bit."""
    import paper_1901_11350_amd as pk

    announce(f"mc pair forms {case} {precision}")
    geo, pairs, length = MC_FAR[case]
    n0 = si.uniform_sphere(geo.n_sites, 4)
    out = []
    for form in ("near", "dmi", "far"):
        D = (0.0, 0.0, 1e-300) if form == "dmi" else (0.0, 0.0, 0.0)
        off = [tuple(x + (n if form == "far" and x else 0) for x, n in zip(d, length)) for d, _ in pairs]
        e = pk.Engine(0, precision)
        e.set_geometry(geo)
        e.set_hamiltonian(HAM)
        e.set_pairs([(0, 0, o, J, D) for o, (_, J) in zip(off, pairs)])
        e.set_spins(n0)
        _, acc = e.mc_run(8.0, 40.0, 5, seed=3)[:2]
        out.append((acc, e.get_spins()))
        e.close()
    assert 0 < out[0][0] < 5 * geo.n_sites
    for acc, n in out[1:]:
        assert acc == out[0][0] and np.array_equal(n, out[0][1])


@pytest.mark.parametrize("n", [(43, 41), (591, 591), (592, 592), (803, 700)])
def test_readbacks_in_chunks(n):
    """FP32 spins read back below and above the 2^20 values from which chunks of
    65,536 are used (591^2 x 3 = 1,047,843, 592^2 x 3 = 1,051,392; the last
    chunk ragged) and small ones after large ones: every value the one
    stored."""
    import paper_1901_11350_amd as pk

    announce(f"readback {n}")
    geo = si.square(*n)
    e = pk.Engine(0, "f32")
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    for seed in (1, 2):
        n0 = si.uniform_sphere(geo.n_sites, seed)
        e.set_spins(n0)
        assert np.array_equal(e.get_spins(), n0.astype(np.float32).astype(np.float64))
    g0 = e.gradient()
    assert np.array_equal(g0, e.gradient())
    b = pk.Batch(0)
    small = si.square(40, 24)
    s = pk.Engine(0, "f32")
    s.set_geometry(small)
    s.set_hamiltonian(HAM_SQ)
    m0 = si.uniform_sphere(small.n_sites, 3)
    s.set_spins(m0)
    for x in (e, s):
        b.add(x, 0.3, 0.001, T=0.0, seed=5)
    assert np.array_equal(b.get_spins(1), s.get_spins())     # before the first run
    b.run(2)
    big = b.get_spins(0)
    got = b.get_spins(1)
    s.step_path = "shape2d/32x16x512"
    s.run(0.3, 0.001, 2, T=0.0, seed=5)
    assert np.abs(got - s.get_spins()).max() <= 1e-6
    assert np.array_equal(big, b.get_spins(0)) and np.isfinite(big).all()
