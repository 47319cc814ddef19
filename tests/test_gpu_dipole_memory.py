"""GPU test of the memory that a Hamiltonian with the FFT dipole field holds:
the arrays that its fields and steps read, and no interaction table of the
direct sum."""

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, need_gpu

pytestmark = pytest.mark.gpu

HAM = si.Hamiltonian(mu=(2.0,), B=(0, 0, 0.2), K=(0.2,), K_axis=((0, 0, 1),), J=(1.0,), ddi=3)


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def test_fft_mode_holds_no_table_of_the_direct_sum():
    """512 x 512 x 4 sites, FP32: kernel spectra 513 x 24 x 1024 and half
    spectra 513 x 12 x 512 complex values (126 MB), eight vectors, the
    positions and the direct sum's partials in one slice (126 MB); the table
    would be 7 x 1023 x 6 x 1028 values (177 MB).  Bound: half a table above
    what is read."""
    import torch

    import paper_1901_11350_amd as pk

    announce("fft dipole memory")
    geo = si.simple_cubic(512, 512, 4, periodic=(0, 0, 0))
    e = pk.Engine(0, "f32")
    e.set_geometry(geo)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    e.set_hamiltonian(HAM)
    torch.cuda.synchronize()
    held = free - torch.cuda.mem_get_info()[0]
    read = 8 * 513 * (24 * 1024 + 12 * 512) + 10 * 12 * geo.n_sites
    assert held <= read + 4 * 7 * 1023 * 6 * 1028 // 2, f"{held / 1e6:.0f} MB held, {read / 1e6:.0f} MB read"


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_noalloc_form_of_an_fft_engine(ora, precision):
    """The allocation-free entry point of an engine in FFT mode, where the
    direct sum runs without a table: parity bounds against the oracle's sum."""
    import ctypes

    import torch

    import paper_1901_11350_amd as pk
    from gpu_util import assert_close

    announce(f"noalloc of an fft engine {precision}")
    geo = si.simple_cubic(24, 20, 4, periodic=(0, 0, 0))
    e = pk.Engine(0, precision)
    e.set_geometry(geo)
    e.set_hamiltonian(HAM)
    dt = torch.float64 if precision == "f64" else torch.float32
    n = torch.tensor(si.uniform_sphere(e.N, 41), dtype=dt, device="cuda").contiguous()
    g = torch.full((3, e.N), float("nan"), dtype=dt, device="cuda")
    torch.cuda.synchronize()
    assert pk.lib().sp_dipole_gradient_dev_noalloc(e._h, ctypes.c_void_p(n.data_ptr()),
                                                   ctypes.c_void_p(g.data_ptr()), e.N) == 0
    e.synchronize()
    s = ora.System(geo, HAM)
    ref = s.dipole_gradient_sites(n.double().cpu().numpy(), np.arange(s.N))
    assert_close(g.double().cpu().numpy(), ref, precision, what="noalloc of an fft engine")
