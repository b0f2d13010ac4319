"""Tiles of lattices whose rows start inside a Philox block (L % 8 != 0),
against the oracle, bit for bit: rows of one word, partial last words, every
offset of a row's first site in its block (L / 2 odd and even), the cut and
the plain compares, one and several words per lane.  (Block indices beyond
2^32: the 185368^2 lattice of test_gpu_huge.py.)"""
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
    yield ising
    ising.tuning_clear()


@pytest.mark.parametrize("T", [1.45, 2.25])
@pytest.mark.parametrize("L", [4, 6, 66, 126, 130, 132, 254, 258, 700, 1002, 1022, 4098, 8194])
def test_one_sweep_at_a_time(I, L, T):
    I.tuning_set([{"L_min": L, "L_max": L, "form": I.ISING_FORM_TILE, "rpw": 1,
                   "max_blocks": 2048, "small_lds_bytes": 0, "updates_per_ns": 0.0}])
    try:
        lat = I.Lattice(L, seed=21, stream_id=4, init=workloads.INIT_HOT, beta=1 / T)
    finally:
        I.tuning_clear()
    n = 2 if L > 1100 else 5
    s = oracle.init(L, 21, 4, workloads.INIT_HOT)
    for t in range(n):
        em = lat.sweep_em(1).cpu().numpy()
        assert np.array_equal(em, oracle.sweeps(s, 1 / T, 21, 4, t, 1)), t
        assert np.array_equal(lat.get_spins(), s), t
    lat.sweep(1)  # no series
    oracle.sweeps(s, 1 / T, 21, 4, n, 1)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("L", [12002, 16386, 23174])
def test_larger_sides_by_windows(I, L):
    # 1, 2 and 4 words per lane
    n, T = 3, 2.25
    lat = I.Lattice(L, seed=8, stream_id=1, init=workloads.INIT_HOT, beta=1 / T)
    em = lat.sweep_em(n).cpu().numpy()
    assert tuple(em[-1]) == lat.measure()
    for (x0, y0) in [(0, 0), (L - 20, L - 5), (L - 7, 1000), (L // 2, L // 2 + 1)]:
        want = oracle.window(L, 1 / T, 8, 1, workloads.INIT_HOT, 0, n, x0, y0, 40, 12)
        ys, xs = (y0 + np.arange(12)) % L, (x0 + np.arange(40)) % L
        got = np.stack([lat.get_window(0, int(y), L, 1)[0][xs] for y in ys])
        assert np.array_equal(got, want), (x0, y0)
