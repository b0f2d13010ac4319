"""Several sweeps per launch on rows held in LDS (csrc/ising_block.hip)
against the oracle, bit for bit: strips at sides where rows, halves, lanes per
half and the last strip come out uneven, sweep counts that the launches share
unevenly, temperatures with and without the cut, lattices with and without the
spare copy of the planes, and batches whose lattices run different numbers of
strips, sweeps and launches."""
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


def _check(I, L, T, n, seed=9, sid=3, init=workloads.INIT_HOT):
    print("case L=%d T=%g n=%d" % (L, T, n), flush=True)
    lat = I.Lattice(L, seed=seed, stream_id=sid, init=init, beta=1 / T)
    em = lat.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, seed, sid, init, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)
    # without a series, and from a counter that is not 0: the same lattice
    again = I.Lattice(L, seed=seed, stream_id=sid, init=init, beta=1 / T)
    again.sweep(1)
    again.sweep(n - 1)
    assert np.array_equal(again.get_spins(), s)
    assert again.measure() == tuple(oem[-1])


@pytest.mark.parametrize("n", [2, 3, 25, 61])
@pytest.mark.parametrize("T", [1.4, 2.25])
@pytest.mark.parametrize("L", [4, 10, 64, 66, 100, 128, 130, 136, 200, 258, 264, 384, 520])
def test_small_sides(I, L, T, n):
    _check(I, L, T, n)


@pytest.mark.parametrize("n", [2, 9, 26])
@pytest.mark.parametrize("T", [1.4, 2.25, 6.5])
@pytest.mark.parametrize("L", [1000, 1002, 1022, 1024, 1538, 2048, 2050])
def test_middle_sides(I, L, T, n):
    _check(I, L, T, n, init=workloads.INIT_COLD_DOWN)


@pytest.mark.parametrize("T", [1.4, 2.25])
@pytest.mark.parametrize("L", [3000, 4094, 4096, 4098, 5000, 8200, 8702, 8704])
def test_largest_sides(I, L, T):
    _check(I, L, T, 7)


@pytest.mark.parametrize("L", [300, 640, 682])
def test_one_workgroup_up_to_its_lds(I, L):
    """682^2: 65472 bytes of planes, the most that one workgroup takes."""
    I.tuning_set([{"L_min": L, "L_max": L, "form": I.ISING_FORM_TILE, "rpw": 0,
                   "max_blocks": 2048, "small_lds_bytes": 65536, "updates_per_ns": 0.0}])
    try:
        for T in (1.4, 2.25):
            _check(I, L, T, 35)
    finally:
        I.tuning_clear()


@pytest.mark.parametrize("L", [136, 514, 1024, 3000])
def test_spare_copy_changes_nothing(I, L):
    n = 11
    a = I.Lattice(L, seed=2, init=workloads.INIT_HOT, beta=1 / 2.3)
    b = I.Lattice(L, seed=2, init=workloads.INIT_HOT, beta=1 / 2.3)
    I.check(I.lib().ising_set_spare(b.h, None, 0))
    for k in (n, 1, 4):
        assert np.array_equal(a.sweep_em(k).cpu().numpy(), b.sweep_em(k).cpu().numpy()), k
        assert np.array_equal(a.get_spins(), b.get_spins()), k
    # taken away between calls, and a buffer that is too small or misaligned
    I.check(I.lib().ising_set_spare(a.h, None, 0))
    assert np.array_equal(a.sweep_em(3).cpu().numpy(), b.sweep_em(3).cpu().numpy())
    need = int(I.lib().ising_spare_bytes(L))
    assert I.lib().ising_set_spare(a.h, a.buf.data_ptr(), need - 1) == I.ISING_ENOMEM
    assert I.lib().ising_set_spare(a.h, a.buf.data_ptr() + 4, need) == I.ISING_EINVAL


@pytest.mark.parametrize("spec", [
    [(8, 2.2), (30, 1.4), (64, 2.3), (66, 2.1), (128, 5.0)],         # one workgroup each
    [(64, 2.2), (512, 1.4), (258, 2.3), (100, 2.1), (32, 9.0)],      # strips beside singles
    [(1024, 2.2), (34, 1.4), (2048, 2.3), (130, 2.1), (1000, 2.4)],
])
def test_batches(I, spec):
    import torch
    n = 27
    lats = [I.Lattice(L, seed=6, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, (L, T) in enumerate(spec)]
    # one lattice without a series
    EMs = [torch.empty((n, 2), dtype=torch.int64, device="cuda") for _ in spec]
    EMs[1] = None
    I.multi_sweep(lats, n, EMs)
    for i, (L, T) in enumerate(spec):
        s, oem = oracle.run(L, 1 / T, 6, i, workloads.INIT_HOT, n)
        if EMs[i] is not None:
            assert np.array_equal(EMs[i].cpu().numpy(), oem), (L, T)
        assert np.array_equal(lats[i].get_spins(), s), (L, T)


# more strips than compute units, two workgroups share one; more lattices than
# compute units
@pytest.mark.parametrize("spec", [
    [(L, T) for T in (1.4, 2.25, 6.5) for L in (4, 8, 10, 32, 64, 66, 100, 128, 130, 136, 200)] * 8,
    [(2048, 2.25), (2050, 2.25), (2048, 1.4), (2050, 1.4), (512, 2.25), (1002, 2.0), (64, 2.0)],
    # no side a multiple of 8: together all the same
    [(1002, 2.2), (10, 2.3), (66, 1.4), (258, 6.5), (1002, 1.4), (514, 2.0)]])
def test_batches_of_many_strips(I, spec):
    test_batches(I, spec)


def test_served_requests_of_uneven_length(I):
    reqs = [{"L": L, "beta": 1 / T, "seed": 40 + i, "stream_id": i, "init": workloads.INIT_HOT,
             "n_sweeps": n, "record_series": True, "return_spins": True}
            for i, (L, T, n) in enumerate([(32, 2.0, 70), (256, 2.2, 9), (512, 1.45, 41),
                                           (1024, 2.3, 1), (96, 3.0, 33), (34, 2.5, 17),
                                           (1002, 2.2, 12)])]
    for arena in (4 << 20, 64 << 20):  # without and with room for spare copies
        srv = I.Server(arena, quantum_sweeps=16)
        tickets = srv.submit(reqs)
        srv.run_until_idle()
        for r, t in zip(reqs, tickets):
            got = srv.poll(t)
            s, oem = oracle.run(r["L"], r["beta"], r["seed"], r["stream_id"], r["init"],
                                r["n_sweeps"])
            assert np.array_equal(got["series"], oem), (arena, r["L"])
            assert np.array_equal(got["spins"], s), (arena, r["L"])
        srv.close()


@pytest.mark.parametrize("seed", [5, 0xABCDE])
@pytest.mark.parametrize("L", [200, 512, 1002])
def test_shuffled_barriers(I, L, seed):
    n = 6
    I.debug_perturb(seed)
    try:
        lat = I.Lattice(L, seed=3, init=workloads.INIT_HOT, beta=1 / 2.269185)
        em = lat.sweep_em(n).cpu().numpy()
    finally:
        I.debug_perturb(0)
    s, oem = oracle.run(L, 1 / 2.269185, 3, 0, workloads.INIT_HOT, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("n", [2, 7, 26])
@pytest.mark.parametrize("L", [8, 64, 72, 128, 136, 200, 264, 520, 1000, 2056])
def test_generators(I, L, n):
    """The paper's generators: lattice, series and generator states, over two
    calls (the second from advanced states)."""
    T = 2.3
    print("case lcg L=%d n=%d" % (L, n), flush=True)
    lat = I.Lattice(L, seed=7, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_lcg()
    s = oracle.init(L, 7, 0, workloads.INIT_HOT)
    st = oracle.lcg_seed(L, 7)
    for k in (n, 3):
        em = lat.sweep_em(k).cpu().numpy()
        assert np.array_equal(em, oracle.lcg_sweeps(s, 1 / T, st, k))
        assert np.array_equal(lat.get_spins(), s)
        assert np.array_equal(lat.lcg_states(), st)


@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("L,m,n", [(8, 10, 5), (64, 10, 40), (72, 11, 9), (128, 12, 26),
                                   (136, 10, 26), (264, 10, 9), (1000, 12, 9), (1024, 10, 26),
                                   (4096, 14, 5), (9000, 16, 5)])
def test_pools(I, L, m, n, linear):
    T = 2.2
    print("case pool L=%d m=%d n=%d linear=%d" % (L, m, n, linear), flush=True)
    lat = I.Lattice(L, seed=5, stream_id=3, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_pool(m, linear=linear)
    s = oracle.init(L, 5, 3, workloads.INIT_HOT)
    t = 0
    for k in (n, 3):
        em = lat.sweep_em(k).cpu().numpy()
        assert np.array_equal(em, oracle.pool_sweeps(s, 1 / T, 5, 3, t, k, m, linear))
        assert np.array_equal(lat.get_spins(), s)
        t += k


# a word per lane: last words of 4, 44 and 64 sites, rows of odd and even words
@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("L,n", [(1032, 27), (2056, 9), (2136, 8), (2048, 11), (3072, 5)])
def test_pools_of_whole_words(I, L, n, linear):
    test_pools(I, L, 12, n, linear)


def test_largest_pool_block(I):
    """16384^2, linear reads: strips of 64 rows that fill a compute unit's LDS."""
    L, m, n, T = 16384, 12, 4, 2.2
    lat = I.Lattice(L, seed=5, stream_id=3, init=workloads.INIT_COLD_UP, beta=1 / T)
    lat.use_pool(m, linear=True)
    em = lat.sweep_em(n).cpu().numpy()
    s = oracle.init(L, 5, 3, workloads.INIT_COLD_UP)
    assert np.array_equal(em, oracle.pool_sweeps(s, 1 / T, 5, 3, 0, n, m, True))
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("kind", ["lcg", "pool", "linear"])
def test_shuffled_barriers_of_the_alternative_dynamics(I, kind):
    L, n, T = 520, 9, 2.25
    ems = []
    for seed in (0, 77):
        I.debug_perturb(seed)
        try:
            lat = I.Lattice(L, seed=3, init=workloads.INIT_HOT, beta=1 / T)
            lat.use_lcg() if kind == "lcg" else lat.use_pool(12, linear=kind == "linear")
            ems.append(lat.sweep_em(n).cpu().numpy())
        finally:
            I.debug_perturb(0)
    assert np.array_equal(ems[0], ems[1])


# a batch of odd sides runs, to the same result, in a work buffer of any size
@pytest.mark.parametrize("share", [0.0, 0.5, 1.0])
def test_odd_batch_with_less_than_its_tables(I, share):
    import ctypes

    import torch
    spec = [(258, 2.2), (66, 1.4), (10, 2.3), (1002, 2.2)]
    lats = [I.Lattice(L, seed=6, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, (L, T) in enumerate(spec)]
    hs = (ctypes.c_void_p * len(lats))(*[lat.h.value for lat in lats])
    need = ctypes.c_size_t()
    I.check(I.lib().ising_multi_sweep_work_bytes(hs, len(lats), ctypes.byref(need)))
    assert need.value > 0
    size = int(need.value * share)
    buf = torch.empty(max(size, 1), dtype=torch.uint8, device="cuda")
    I.check(I.lib().ising_multi_sweep(hs, len(lats), 12, None, buf.data_ptr() if size else None,
                                      size))
    I.check(I.lib().ising_multi_sweep_static(hs, len(lats), 5, None))
    for i, (L, T) in enumerate(spec):
        s, _ = oracle.run(L, 1 / T, 6, i, workloads.INIT_HOT, 17)
        assert np.array_equal(lats[i].get_spins(), s), (L, T)


def test_pool_block_that_fills_the_lds(I):
    """16064^2, linear reads, 9 sweeps: the plan nearest to a compute unit's
    LDS (rows and the kernel's own part together)."""
    L, m, n, T = 16064, 12, 9, 2.2
    lat = I.Lattice(L, seed=5, stream_id=3, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_pool(m, linear=True)
    em = lat.sweep_em(n).cpu().numpy()
    assert tuple(em[-1]) == lat.measure()
    pool = oracle.pool_fill(1 / T, 5, 3, m)
    for (x0, y0) in [(0, 0), (L - 20, L - 5), (L // 2, 8037)]:
        want = oracle.pool_window(L, 1 / T, 5, 3, workloads.INIT_HOT, 0, n, m, True, x0, y0, 40,
                                  12, pool)
        rows = [lat.get_window(0, (y0 + i) % L, L, 1)[0] for i in range(12)]
        xs = (x0 + np.arange(40)) % L
        assert np.array_equal(np.stack([r[xs] for r in rows]), want), (x0, y0)


# one copy for all, and copies that overlap in part
@pytest.mark.parametrize("shift", [0, 4096])
def test_batch_of_lattices_that_share_a_spare_copy(I, shift):
    import torch
    n, spec = 14, [(1024, 2.2), (512, 1.4), (1002, 2.3), (1024, 2.0)]
    lats = [I.Lattice(L, seed=6, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, (L, T) in enumerate(spec)]
    need = int(I.lib().ising_spare_bytes(1024))
    buf = torch.empty(need + 8 * shift, dtype=torch.uint8, device="cuda")
    for i, lat in enumerate(lats):
        I.check(I.lib().ising_set_spare(lat.h, buf.data_ptr() + i * shift, need))
    I.multi_sweep(lats, n)
    for lat in lats:  # one after another
        lat.sweep(5)
    for i, (L, T) in enumerate(spec):
        s, _ = oracle.run(L, 1 / T, 6, i, workloads.INIT_HOT, n + 5)
        assert np.array_equal(lats[i].get_spins(), s), (L, T)


def test_spare_copy_may_not_overlap_its_lattice(I):
    L = 512
    lat = I.Lattice(L, seed=2, init=workloads.INIT_HOT, beta=1 / 2.3)
    need, size = int(I.lib().ising_spare_bytes(L)), I.ising_lattice_bytes(L)
    for off in (0, 4096, size - 8):
        assert I.lib().ising_set_spare(lat.h, lat.buf.data_ptr() + off, need) == I.ISING_EINVAL
    lat.sweep(9)  # the copy is still the one behind the lattice
    s, _ = oracle.run(L, 1 / 2.3, 2, 0, workloads.INIT_HOT, 9)
    assert np.array_equal(lat.get_spins(), s)
