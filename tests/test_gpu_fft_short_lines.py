"""GPU tests of the FFT dipole field on lattices with short axes: lines of 4, 8
and 16 points, axes of one cell, which are not transformed (along a they
change places with b), in the separate kernels (more than four planes, and
FP64 with few rows or columns) and beside them the fused ones."""

import dataclasses
import time

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, need_gpu

pytestmark = pytest.mark.gpu

SP_DDI_FFT = 3

CASES = {
    "1x1x9": si.simple_cubic(1, 1, 9, periodic=(0, 0, 0)),
    "1x2x7": si.simple_cubic(1, 2, 7, periodic=(0, 0, 0)),
    "2x1x7": si.simple_cubic(2, 1, 7, periodic=(0, 0, 0)),
    "2x3x6": si.simple_cubic(2, 3, 6, periodic=(0, 0, 0)),
    "4x5x6": si.simple_cubic(4, 5, 6, periodic=(0, 0, 0)),
    "8x9x5": si.simple_cubic(8, 9, 5, periodic=(0, 0, 0)),
    "40x1x20": si.simple_cubic(40, 1, 20, periodic=(0, 0, 0)),
    "1x33x20": si.simple_cubic(1, 33, 20, periodic=(0, 0, 0)),
    "300x1x2": si.simple_cubic(300, 1, 2, periodic=(0, 0, 0)),
    "1x300x2": si.simple_cubic(1, 300, 2, periodic=(0, 0, 0)),
    "257x16x1": si.simple_cubic(257, 16, 1, periodic=(0, 0, 0)),
    "257x17x1": si.simple_cubic(257, 17, 1, periodic=(0, 0, 0)),
    "9x65x3": si.simple_cubic(9, 65, 3, periodic=(0, 0, 0)),
    "triangular1x30": si.triangular(1, 30),               # the axes that change places are not at right angles
    "kagome1x18": si.kagome(1, 18),
    "kagome19x1": si.kagome(19, 1),
}


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _ham(k):
    return si.Hamiltonian(mu=(2.0, 1.5, 0.7)[:k], B=(0, 0, 0), K=(0.0,) * k, K_axis=((0, 0, 1),) * k, ddi=SP_DDI_FFT)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", list(CASES))
def test_short_lines_match_the_direct_sum(ora, case, precision):
    """Field within the parity bounds (FP64 1e-12, FP32 1e-5), and two steps."""
    import paper_1901_11350_amd as pk

    announce(f"fft short lines {case} {precision}")
    geo = CASES[case]
    ham = dataclasses.replace(_ham(geo.n_basis), B=(0.1, 0.0, 0.4))
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(ham)
    n = si.uniform_sphere(geo.n_sites, 29)
    e.set_spins(n)
    s = ora.System(geo, ham)
    assert_close(e.dipole_gradient(), s.dipole_gradient_sites(n, np.arange(geo.n_sites)), precision,
                 what=f"FFT dipole {case}")
    e.run(0.3, 0.001, 2, T=10.0, seed=3)
    ref, _ = s.run(n, 0.3, 0.001, 2, T=10.0, seed=3)
    assert_close(e.get_spins(), ref, precision, what=f"steps {case}")


@pytest.mark.parametrize("flat", [(512, 1, 64), (1, 512, 64)])
def test_an_axis_of_one_cell_costs_no_padded_lines(flat):
    """A film that lies in the plane of a (or b) and c: its field takes a small
    part of the time of one sixteen cells deep, whose lines are 32 points."""
    import torch

    import paper_1901_11350_amd as pk

    announce(f"fft flat film {flat}")

    def field_time(cells):
        e = pk.Engine(0, "f32")
        e.set_geometry(si.simple_cubic(*cells, periodic=(0, 0, 0)))
        e.set_hamiltonian(_ham(1))
        n = torch.tensor(si.uniform_sphere(e.N, 1), dtype=torch.float32, device="cuda").contiguous()
        g = torch.empty_like(n)
        torch.cuda.synchronize()
        best = 1e9
        for _ in range(6):
            t0 = time.perf_counter()
            for _ in range(5):
                e.dipole_gradient_dev(n, g)
            e.synchronize()
            best = min(best, time.perf_counter() - t0)
        e.close()
        return best

    deep = tuple(16 if x == 1 else x for x in flat)
    assert 4.0 * field_time(flat) < field_time(deep)
