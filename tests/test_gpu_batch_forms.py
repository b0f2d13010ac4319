"""Which form a batch takes: lattices that do not fit one workgroup stay
together where the others are packed, and many large ones are not swept one
after another."""
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


def test_packed_beside_lattices_of_several_workgroups(I):
    import torch
    n = 5
    spec = [(64, 2.2), (1024, 1.4), (704, 2.3), (256, 6.5), (1032, 2.1), (680, 2.0)]
    lats = [I.Lattice(L, seed=6, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, (L, T) in enumerate(spec)]
    EMs = [torch.empty((n, 2), dtype=torch.int64, device="cuda") for _ in spec]
    I.multi_sweep(lats, n, EMs, form="packed")
    for i, (L, T) in enumerate(spec):
        s, oem = oracle.run(L, 1 / T, 6, i, workloads.INIT_HOT, n)
        assert np.array_equal(EMs[i].cpu().numpy(), oem), (L, T)
        assert np.array_equal(lats[i].get_spins(), s), (L, T)


@pytest.mark.parametrize("L,count", [(1024, 1024), (512, 300), (128, 4000)])
def test_batches_beyond_the_sites_of_blocks(I, L, count):
    """More sites than are cut into strips: as fast as the fused form at
    least (1024 lattices of 1024^2 one after another took five times as
    long)."""
    import torch
    n, T = 10, 2.25
    lats = [I.Lattice(L, seed=3, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i in range(count)]
    EM = torch.empty((count, n, 2), dtype=torch.int64, device="cuda")
    best = {}
    t = 0
    for form in ("fused", None, "fused", None):
        t0 = time.perf_counter()
        I.multi_sweep(lats, n, list(EM), form=form)
        dt = time.perf_counter() - t0
        best[form] = min(best.get(form, dt), dt)
        t += n
    print("fused %.2f ms, chosen %.2f ms" % (1e3 * best["fused"], 1e3 * best[None]), flush=True)
    assert best[None] < 1.5 * best["fused"]
    for i in (0, count - 1):
        s, oem = oracle.run(L, 1 / T, 3, i, workloads.INIT_HOT, t)
        assert np.array_equal(EM[i].cpu().numpy(), oem[-n:])
        assert np.array_equal(lats[i].get_spins(), s)


# (with tables for fewer strips than the best cut has)
@pytest.mark.parametrize("Ls", [[336] * 3, [512, 336], [200] * 4 + [640]])
def test_few_lattices_take_strips_within_their_tables(I, Ls):
    import torch
    n, T = 60, 2.25
    lats = [I.Lattice(L, seed=3, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, L in enumerate(Ls)]
    EMs = [torch.empty((n, 2), dtype=torch.int64, device="cuda") for _ in Ls]
    best, t = {}, 0
    for form in ("fused", None) * 3:
        t0 = time.perf_counter()
        I.multi_sweep(lats, n, EMs, form=form)
        dt = time.perf_counter() - t0
        best[form] = min(best.get(form, dt), dt)
        t += n
    print("fused %.3f ms, chosen %.3f ms" % (1e3 * best["fused"], 1e3 * best[None]), flush=True)
    assert best[None] < 0.7 * best["fused"]
    for i, L in enumerate(Ls):
        s, oem = oracle.run(L, 1 / T, 3, i, workloads.INIT_HOT, t)
        assert np.array_equal(EMs[i].cpu().numpy(), oem[-n:])
        assert np.array_equal(lats[i].get_spins(), s)


def test_static_tables_of_many_small_lattices(I):
    """13400 lattices of 8^2 by the entry point that allocates nothing: within
    its 4 MiB by the record of 240 bytes that its limit was set with."""
    import ctypes

    import torch
    count, n, T = 13400, 3, 2.2
    size = (I.ising_lattice_bytes(8) + 255) // 256 * 256
    buf = torch.empty(count * size, dtype=torch.uint8, device="cuda")
    stream = int(torch.cuda.current_stream().cuda_stream)
    hs = (ctypes.c_void_p * (count + 200))()
    for i in range(count + 200):  # the last ones share a place and are never swept
        h = ctypes.c_void_p()
        I.check(I.lib().ising_create(8, 5, i, workloads.INIT_HOT,
                                     buf.data_ptr() + min(i, count - 1) * size, size, stream,
                                     ctypes.byref(h)))
        I.check(I.lib().ising_set_beta(h, 1 / T))
        hs[i] = h.value
    assert I.lib().ising_multi_sweep_static(hs, count + 200, n, None) == I.ISING_ENOMEM
    # (the lattices that shared the place left it hot with another stream id)
    h = ctypes.c_void_p(hs[count - 1])
    host = oracle.init(8, 5, count - 1, workloads.INIT_HOT)
    I.check(I.lib().ising_set_spins(h, host.ctypes.data))
    I.check(I.lib().ising_multi_sweep_static(hs, count, n, None))
    got = np.empty((8, 8), dtype=np.int8)
    for i in (0, 1, 777, 11914, 11915, count - 1):
        I.check(I.lib().ising_get_spins(ctypes.c_void_p(hs[i]), got.ctypes.data))
        s, _ = oracle.run(8, 1 / T, 5, i, workloads.INIT_HOT, n)
        assert np.array_equal(got, s), i
    for v in hs:
        I.lib().ising_destroy(ctypes.c_void_p(v))
