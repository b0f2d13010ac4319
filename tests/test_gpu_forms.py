"""The form that a call runs in (ising_sweep_plan) is the one a test means:
blocks at the largest sides that take them, and the tiled sweep of narrow and
wide rows and of the flat mapping without a second copy of the planes, over
several sweeps, at temperatures on both sides of the cut's range; against the
oracle, bit for bit."""
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


def _no_copy(I, lat):
    I.check(I.lib().ising_set_spare(lat.h, None, 0))


# 130, 264: rows of 2 and 3 words; 520: 5 words, 4 sites in the last; 1024:
# narrow rows; 4098: any row start; 8072: wide rows
@pytest.mark.parametrize("T", [1.45, 2.0, 5.8])
@pytest.mark.parametrize("L", [130, 264, 520, 1024, 4098, 8072])
def test_tiles(I, L, T):
    n = 3
    lat = I.Lattice(L, seed=11, stream_id=2, init=workloads.INIT_HOT, beta=1 / T)
    _no_copy(I, lat)
    assert lat.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    em = lat.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, 11, 2, workloads.INIT_HOT, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("T", [1.5, 2.0, 5.8])
@pytest.mark.parametrize("L", [136, 520, 1024])
def test_generators_in_tiles(I, L, T):
    n = 3
    lat = I.Lattice(L, seed=77, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_lcg()
    _no_copy(I, lat)
    assert lat.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    em = lat.sweep_em(n).cpu().numpy()
    s = oracle.init(L, 77, 0, workloads.INIT_HOT)
    st = oracle.lcg_seed(L, 77)
    assert np.array_equal(em, oracle.lcg_sweeps(s, 1 / T, st, n))
    assert np.array_equal(lat.get_spins(), s)
    assert np.array_equal(lat.lcg_states(), st)


@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("L", [136, 520, 1024])
def test_pools_in_tiles(I, L, linear):
    n, m, T = 3, 11, 2.2
    lat = I.Lattice(L, seed=5, stream_id=3, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_pool(m, linear=linear)
    _no_copy(I, lat)
    assert lat.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    em = lat.sweep_em(n).cpu().numpy()
    s = oracle.init(L, 5, 3, workloads.INIT_HOT)
    assert np.array_equal(em, oracle.pool_sweeps(s, 1 / T, 5, 3, 0, n, m, linear))
    assert np.array_equal(lat.get_spins(), s)


# one strip; strips of uneven sides; the largest sides that take blocks
@pytest.mark.parametrize("T", [1.45, 2.25])
@pytest.mark.parametrize("L,n", [(64, 5), (130, 5), (520, 7), (1002, 9), (4096, 8), (5000, 24),
                                 (7680, 24)])
def test_blocks(I, L, n, T):
    lat = I.Lattice(L, seed=9, stream_id=3, init=workloads.INIT_COLD_UP, beta=1 / T)
    form, launches = lat.sweep_plan(n)
    assert form == I.ISING_FORM_BLOCK and launches < 2 * n
    em = lat.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, 9, 3, workloads.INIT_COLD_UP, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("kind,L,n", [("lcg", 9216, 24), ("pool", 9152, 24), ("linear", 9000, 9),
                                      ("linear", 12008, 7)])
def test_largest_blocks_of_the_alternative_dynamics(I, kind, L, n):
    T, m = 2.3, 12
    lat = I.Lattice(L, seed=7, init=workloads.INIT_COLD_UP, beta=1 / T)
    lat.use_lcg() if kind == "lcg" else lat.use_pool(m, linear=kind == "linear")
    assert lat.sweep_plan(n)[0] == I.ISING_FORM_BLOCK
    em = lat.sweep_em(n).cpu().numpy()
    s = oracle.init(L, 7, 0, workloads.INIT_COLD_UP)
    if kind == "lcg":
        st = oracle.lcg_seed(L, 7)
        assert np.array_equal(em, oracle.lcg_sweeps(s, 1 / T, st, n))
        assert np.array_equal(lat.lcg_states(), st)
    else:
        assert np.array_equal(em, oracle.pool_sweeps(s, 1 / T, 7, 0, 0, n, m, kind == "linear"))
    assert np.array_equal(lat.get_spins(), s)


def test_arguments(I):
    import ctypes
    lat = I.Lattice(64, seed=1, beta=0.4)
    form, launches = ctypes.c_int32(), ctypes.c_int64()
    f, k = ctypes.byref(form), ctypes.byref(launches)
    for args in ((None, 1, f, k), (lat.h, 0, f, k), (lat.h, 1, None, k), (lat.h, 1, f, None)):
        assert I.lib().ising_sweep_plan(*args) == I.ISING_EINVAL
    assert lat.sweep_plan(1)[1] == 1 and lat.sweep_plan(10 ** 6) == (I.ISING_FORM_BLOCK, 1)


def test_sweeps_beyond_what_launches_count(I):
    """Strips take up to 2^30 sweeps in a call (32-bit launch numbers; planned
    only, nothing runs), a single strip any number."""
    lat = I.Lattice(4096, seed=1, beta=0.4)
    assert lat.sweep_plan(2 ** 30)[0] == I.ISING_FORM_BLOCK
    for n in (2 ** 30 + 1, 2 ** 32 - 1):
        assert lat.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    small = I.Lattice(64, seed=1, beta=0.4)
    assert small.sweep_plan(2 ** 32) == (I.ISING_FORM_BLOCK, 2 ** 12)


def test_second_copy_is_allocated_for_dynamics_that_use_it(I):
    """Plain lattices above 8000^2 hold one copy of the planes; linear pools
    bring the second one with them."""
    L = 12008
    lat = I.Lattice(L, seed=1, beta=0.4)
    assert lat.buf.numel() == I.ising_lattice_bytes(L)
    assert lat.sweep_plan(24)[0] == I.ISING_FORM_TILE
    lat.use_lcg()
    assert lat.sweep_plan(24)[0] == I.ISING_FORM_TILE
    lat.use_pool(10, linear=True)
    assert lat.sweep_plan(24)[0] == I.ISING_FORM_BLOCK
    assert lat.buf.numel() == I.ising_lattice_bytes(L)


def test_buffer_holds_the_lattice_alone(I):
    """A lattice's tensor is ising_lattice_bytes long, with and without a
    second copy, so that one saved on the device fits wherever it is put."""
    import torch
    n, T = 8, 2.3
    for L in (64, 130, 1024):
        lat = I.Lattice(L, seed=4, init=workloads.INIT_HOT, beta=1 / T)
        assert lat.sweep_plan(n)[0] == I.ISING_FORM_BLOCK
        saved = torch.empty(I.ising_lattice_bytes(L), dtype=torch.uint8, device="cuda")
        lat.sweep(n)
        saved.copy_(lat.buf)
        lat.sweep(n)
        back = I.Lattice(L, seed=4, beta=1 / T)
        back.buf.copy_(saved)
        back.sweep_count = n
        back.sweep(n)
        assert np.array_equal(back.get_spins(), lat.get_spins()), L


def test_installed_tile_shapes_bind_plain_sweeps_only(I):
    """A shape timed for plain sweeps leaves generators and pools their
    blocks; the autotuner keeps the size rule where blocks are ahead."""
    L, n, T = 1024, 9, 2.3
    for form in (I.ISING_FORM_TILE, I.ISING_FORM_STRIP):
        I.tuning_set([{"L_min": L, "L_max": L, "form": form, "rpw": 1, "max_blocks": 2048,
                       "small_lds_bytes": 0, "updates_per_ns": 0.0}])
        lats = [I.Lattice(L, seed=7, init=workloads.INIT_HOT, beta=1 / T) for _ in range(4)]
        I.tuning_clear()
        lats[1].use_lcg()
        lats[2].use_pool(11)
        lats[3].use_pool(11, linear=True)
        forms = [lat.sweep_plan(n)[0] for lat in lats]
        assert forms == [I.ISING_FORM_TILE] + 3 * [I.ISING_FORM_BLOCK]
        ems = [lat.sweep_em(n).cpu().numpy() for lat in lats]
        want = oracle.run(L, 1 / T, 7, 0, workloads.INIT_HOT, n)[1]
        assert np.array_equal(ems[0], want)
        st = oracle.lcg_seed(L, 7)
        assert np.array_equal(ems[1], oracle.lcg_sweeps(oracle.init(L, 7, 0, workloads.INIT_HOT),
                                                        1 / T, st, n))
        assert np.array_equal(lats[1].lcg_states(), st)
        for k, linear in ((2, False), (3, True)):
            s = oracle.init(L, 7, 0, workloads.INIT_HOT)
            assert np.array_equal(ems[k], oracle.pool_sweeps(s, 1 / T, 7, 0, 0, n, 11, linear))
    try:
        e = I.autotune(2048, trial_sweeps=20)
        assert e["rpw"] == 0 and e["form"] == I.ISING_FORM_TILE
        assert I.Lattice(2048, seed=1, beta=0.4).sweep_plan(24)[0] == I.ISING_FORM_BLOCK
    finally:
        I.tuning_clear()


@pytest.mark.parametrize("kind", ["lcg", "pool", "linear"])
def test_installed_workgroup_sizes_bind_plain_sweeps_only(I, kind):
    """640^2 with 64 KiB of planes installed for one workgroup: plain sweeps
    take one, generators and pools strips, or tiles without a second copy."""
    L, n, T, m = 640, 6, 2.3, 11
    I.tuning_set([{"L_min": L, "L_max": L, "form": I.ISING_FORM_TILE, "rpw": 0,
                   "max_blocks": 2048, "small_lds_bytes": 65536, "updates_per_ns": 0.0}])
    plain, strips, tiles = [I.Lattice(L, seed=7, init=workloads.INIT_HOT, beta=1 / T)
                            for _ in range(3)]
    I.tuning_clear()
    assert plain.sweep_plan(n) == (I.ISING_FORM_BLOCK, 1)
    for lat in (strips, tiles):
        lat.use_lcg() if kind == "lcg" else lat.use_pool(m, linear=kind == "linear")
    _no_copy(I, tiles)
    form, launches = strips.sweep_plan(n)
    assert form == I.ISING_FORM_BLOCK and launches > 1
    assert tiles.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    s = oracle.init(L, 7, 0, workloads.INIT_HOT)
    if kind == "lcg":
        want = oracle.lcg_sweeps(s, 1 / T, oracle.lcg_seed(L, 7), n)
    else:
        want = oracle.pool_sweeps(s, 1 / T, 7, 0, 0, n, m, kind == "linear")
    for lat in (strips, tiles):
        assert np.array_equal(lat.sweep_em(n).cpu().numpy(), want)
        assert np.array_equal(lat.get_spins(), s)


# 1.2, 1.8 and 1.9 rounds of tiles: dealt in runs of 64 and in one run per XCD,
# by the size of the pool and the last round's fill
@pytest.mark.parametrize("L,m,linear", [(18000, 12, False), (22016, 12, False), (22016, 19, False),
                                        (22528, 12, True), (23000, 12, True)])
def test_pools_in_uneven_rounds_of_tiles(I, L, m, linear):
    n, T = 2, 2.25
    lat = I.Lattice(L, seed=8, stream_id=1, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_pool(m, linear=linear)
    assert lat.sweep_plan(n) == (I.ISING_FORM_TILE, 2 * n)
    em = lat.sweep_em(n).cpu().numpy()
    assert tuple(em[-1]) == lat.measure()
    pool = oracle.pool_fill(1 / T, 8, 1, m)
    for (x0, y0) in [(0, 0), (L - 20, L - 5), (L - 7, 1000), (L // 2, L // 2 + 1)]:
        want = oracle.pool_window(L, 1 / T, 8, 1, workloads.INIT_HOT, 0, n, m, linear, x0, y0, 40,
                                  12, pool)
        rows = [lat.get_window(0, (y0 + i) % L, L, 1)[0] for i in range(12)]
        xs = (x0 + np.arange(40)) % L
        assert np.array_equal(np.stack([r[xs] for r in rows]), want), (x0, y0)
