"""GPU tests of readbacks of one object from several threads at once: each
thread gets the values stored, whichever of them holds the pinned chunks."""

import threading

import numpy as np
import pytest

import spin_inputs as si
from gpu_util import announce, need_gpu

pytestmark = pytest.mark.gpu

HAM_SQ = si.WORKLOADS["square32_fp64"].hamiltonian


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _in_threads(read, ref, n_threads=4, n_reads=12):
    bad, gate = [], threading.Barrier(n_threads)

    def work(k):
        gate.wait()
        for r in range(n_reads):
            if not np.array_equal(read(k), ref(k)):
                bad.append((k, r))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(n_threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, f"(thread, read) with other values: {bad}"


def test_one_engine_read_by_several_threads():
    """1,051,392 values: the smallest size that takes the chunks; the first
    reads are among the concurrent ones."""
    import paper_1901_11350_amd as pk

    announce("engine readback threads")
    geo = si.square(592, 592)
    e = pk.Engine(0, "f32")
    e.set_geometry(geo)
    e.set_hamiltonian(HAM_SQ)
    n0 = si.uniform_sphere(geo.n_sites, 7)
    e.set_spins(n0)
    want = n0.astype(np.float32).astype(np.float64)
    _in_threads(lambda k: e.get_spins(), lambda k: want)


def test_replicas_of_a_batch_read_by_several_threads():
    """A replica above the chunks' threshold and small ones, which take the
    chunks once they are there, each read by a thread of its own."""
    import paper_1901_11350_amd as pk

    announce("batch readback threads")
    b = pk.Batch(0)
    want = []
    for k, n in enumerate([(592, 592), (300, 200), (592, 600), (64, 64)]):
        geo = si.square(*n)
        e = pk.Engine(0, "f32")
        e.set_geometry(geo)
        e.set_hamiltonian(HAM_SQ)
        e.set_spins(si.uniform_sphere(geo.n_sites, k))
        b.add(e, 0.3, 0.001, T=0.0, seed=5)
        e.close()
    b.run(2)
    want = [b.get_spins(k) for k in range(4)]
    assert all(np.isfinite(w).all() for w in want)
    _in_threads(b.get_spins, lambda k: want[k])
