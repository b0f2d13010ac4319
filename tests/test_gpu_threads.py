"""Lattices of several threads: a call on one does not wait for another's."""
import threading
import time

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def I():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1007_3726_amd import ising
    ising.lib()
    return ising


def test_lone_sweeps_beside_a_running_batch(I):
    """While one thread is inside a batched call of about a second (replayed
    from captured sweeps), another one's sweeps are enqueued at once."""
    import torch
    T = 2.3
    batch = [I.Lattice(1024, seed=1, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
             for i in range(16)]
    side = torch.cuda.Stream()
    lats = [I.Lattice(L, seed=4, init=workloads.INIT_HOT, beta=1 / T, stream=side)
            for L in (1000, 1002, 2048)]
    torch.cuda.synchronize()
    began, done = threading.Event(), threading.Event()

    def run():
        began.set()
        I.multi_sweep(batch, 80000, form="fused")
        done.set()

    th = threading.Thread(target=run)
    th.start()
    assert began.wait(10)
    time.sleep(0.2)  # the batch's tables and capture
    for lat in lats:
        for n in (2, 3, 5):
            lat.sweep(n)
    assert not done.is_set()
    th.join()
    for lat in lats:
        s, _ = oracle.run(lat.L, 1 / T, 4, 0, workloads.INIT_HOT, 10)
        assert np.array_equal(lat.get_spins(), s), lat.L
