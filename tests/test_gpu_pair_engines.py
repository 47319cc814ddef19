"""GPU test of several engines on the pair tiles at once: the LDS a tile
takes differs between them and belongs to each launch, not to the engine that
was set up last."""

import pytest

import spin_inputs as si
from gpu_util import announce, assert_close, make_pair, need_gpu

pytestmark = pytest.mark.gpu

HAM = si.Hamiltonian(mu=(2.0,), B=(0.1, -0.3, 0.8), K=(0.2,), K_axis=((0, 0, 1),))


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _reach(r):
    """Thirteen pairs, the farthest r cells away along a and along b."""
    return [(0, 0, (k, 0, 0), 0.5 / k, (0.0, 0.02, 0.0)) for k in (1, 2, 3, 4, 5, r)] + \
           [(0, 0, (0, k, 0), 0.4 / k, (0.0, 0.0, 0.0)) for k in (1, 2, 3, 4, 5, r)] + [(0, 0, (1, 1, 0), 0.1, (0, 0, 0))]


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_engines_of_different_frames_in_turn(ora, precision):
    """Frames of 66, 56 and 18 cells a side (FP32 70, 50 and 5 KB; FP64 twice
    that), the largest set up first; gradient and steps of each after all are
    set up, within the parity bounds."""
    announce(f"pair engines {precision}")
    geo = si.square(70, 66)
    pairs = [_reach(25), _reach(20), _reach(1)[:1]]
    made = []
    for k, p in enumerate(pairs):
        e, s = make_pair(ora, geo, HAM, precision)
        e.set_pairs(p)
        s.set_pairs(p)
        n = si.uniform_sphere(s.N, 60 + k)
        e.set_spins(n)
        e.step_path = "twopass"
        made.append((e, s, n))
    for k, (e, s, n) in enumerate(made):
        assert_close(e.gradient(), s.gradient(n), precision, what=f"gradient {k}")
    for k, (e, s, n) in enumerate(made):
        e.run(0.3, 0.001, 2, T=20.0, seed=5)
        ref, _ = s.run(n, 0.3, 0.001, 2, T=20.0, seed=5)
        assert_close(e.get_spins(), ref, precision, what=f"steps {k}")
