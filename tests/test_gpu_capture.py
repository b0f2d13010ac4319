"""Sweeps recorded into a graph of the caller's: nothing but launches is
enqueued, the same number in every replay, and the lattice's own planes, series
and generators hold the result after each."""
import numpy as np
import pytest

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


def _lattice(I, L, kind, stream=None):
    lat = I.Lattice(L, seed=5, stream_id=2, init=workloads.INIT_HOT, beta=1 / 2.3, stream=stream)
    if kind == "lcg":
        lat.use_lcg()
    elif kind != "plain":
        lat.use_pool(12, linear=kind == "linear")
    return lat


# one strip, strips (even and odd numbers of sweeps), tiles
@pytest.mark.parametrize("kind", ["plain", "lcg", "pool", "linear"])
@pytest.mark.parametrize("L,n", [(64, 7), (512, 9), (1000, 5), (8192, 2)])
def test_replays_equal_eager_sweeps(I, kind, L, n):
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        lat = _lattice(I, L, kind, side)
        EM = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        lat.sweep(n, EM)
    eager = _lattice(I, L, kind)
    for k in range(3):
        with torch.cuda.stream(side):
            graph.replay()
        side.synchronize()
        eager.sweep_count = 0  # a recorded sweep keeps its counter
        want = eager.sweep_em(n).cpu().numpy()
        assert np.array_equal(EM.cpu().numpy(), want), k
        assert np.array_equal(lat.get_spins(), eager.get_spins()), k
        if kind == "lcg":
            assert np.array_equal(lat.lcg_states(), eager.lcg_states()), k
        torch.ones(1 << 16, device="cuda").sum().item()  # the program's own work between
