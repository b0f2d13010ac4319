"""Served mode: continuous batching with HBM-budget admission.

Each request's result (per-sweep E/M series and final spins) must be
bit-identical whether it runs alone or in a mix admitted as memory frees,
with or without an injected (host-forced) quantum failure; admission never
exceeds the arena; oversized or invalid requests are rejected.
"""
import sys

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


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _requests():
    rng = np.random.default_rng(5)
    reqs = []
    for i, L in enumerate([32, 64, 96, 128, 160, 256, 320, 512, 34, 1024, 64, 2048]):
        reqs.append({"L": L, "beta": 1.0 / float(rng.uniform(1.5, 3.5)), "seed": 1000 + i,
                     "stream_id": 0, "init": workloads.INIT_HOT,
                     "n_sweeps": int(rng.integers(5, 40)), "n_discard": 2,
                     "record_series": True, "return_spins": True})
    return reqs


def _run(I, reqs, arena_bytes, quantum, fault_at=None):
    srv = I.Server(arena_bytes, quantum_sweeps=quantum)
    if fault_at is not None:
        srv.inject_fault(fault_at)
    tickets = srv.submit(reqs)
    srv.run_until_idle()
    results = [srv.poll(t) for t in tickets]
    stats = srv.stats()
    srv.close()
    return results, stats


def test_alone_equals_mix(I):
    reqs = _requests()
    need = max(I.ising_lattice_bytes(r["L"]) for r in reqs) + (4 << 20)
    _say("case alone")
    alone = [_run(I, [r], need, 6)[0][0] for r in reqs]
    _say("case mix (small arena forces queueing)")
    mix, stats = _run(I, reqs, 3 * need // 2, 6)
    assert stats["done"] == len(reqs) and stats["admitted"] == len(reqs)
    assert stats["peak_bytes"] <= 3 * need // 2
    for r, a, m in zip(reqs, alone, mix):
        assert np.array_equal(a["series"], m["series"]), r
        assert np.array_equal(a["spins"], m["spins"]), r
        assert (a["E_final"], a["M_final"]) == (m["E_final"], m["M_final"])
        assert m["sweeps_done"] == r["n_sweeps"]


def test_requests_match_plain_path_and_oracle(I):
    reqs = _requests()
    res, _ = _run(I, reqs, 64 << 20, 9)
    for r, got in zip(reqs, res):
        lat = I.Lattice(r["L"], seed=r["seed"], stream_id=r["stream_id"], init=r["init"],
                        beta=r["beta"])
        em = lat.sweep_em(r["n_sweeps"]).cpu().numpy()
        assert np.array_equal(got["series"], em), r
        assert np.array_equal(got["spins"], lat.get_spins())
        if r["L"] <= 128:
            s, oEM = oracle.run(r["L"], r["beta"], r["seed"], r["stream_id"], r["init"],
                                r["n_sweeps"])
            assert np.array_equal(got["series"], oEM)
            assert np.array_equal(got["spins"], s)
        M = [int(v) for v in em[r["n_discard"]:, 1]]
        assert got["n_kept"] == len(M)
        assert got["sum_M2"] == float(sum(v * v for v in M))
        assert got["sum_M4"] == float(sum(v ** 4 for v in M))


def test_fault_injection_recovers_bit_identically(I):
    reqs = _requests()[:8]
    clean, _ = _run(I, reqs, 64 << 20, 5)
    faulty, stats = _run(I, reqs, 64 << 20, 5, fault_at=2)
    assert stats["faults_recovered"] == 1
    for a, b in zip(clean, faulty):
        assert np.array_equal(a["series"], b["series"])
        assert np.array_equal(a["spins"], b["spins"])


def test_fifo_admission_and_budget(I):
    reqs = [{"L": 256, "beta": 0.4, "seed": i, "n_sweeps": 10 + i} for i in range(6)]
    one = I.ising_lattice_bytes(256) + 16 * 20 + 512
    srv = I.Server(2 * one, quantum_sweeps=4)
    tickets = srv.submit(reqs)
    seen_peak = 0
    while srv.step():
        seen_peak = max(seen_peak, srv.stats()["bytes_in_use"])
    res = [srv.poll(t) for t in tickets]
    st = srv.stats()
    assert st["peak_bytes"] <= 2 * one and seen_peak <= 2 * one
    admits = [r["t_admit"] for r in res]
    assert admits == sorted(admits), "admission is not FIFO"
    srv.close()


def test_rejections(I):
    srv = I.Server(1 << 20, quantum_sweeps=4)
    with pytest.raises(I.IsingError) as e:
        srv.submit([{"L": 4096, "beta": 0.4, "n_sweeps": 10}])  # larger than the arena
    assert e.value.code == I.ISING_ENOMEM
    with pytest.raises(I.IsingError):
        srv.submit([{"L": 64, "beta": 0.4, "n_sweeps": 5},
                    {"L": 63, "beta": 0.4, "n_sweeps": 5}])  # odd L: nothing queued
    with pytest.raises(I.IsingError):
        srv.submit([{"L": 64, "beta": -1.0, "n_sweeps": 5}])
    assert srv.stats()["admitted"] == 0
    assert not srv.step()
    with pytest.raises(I.IsingError) as e:
        srv.poll(12345)
    assert e.value.code == I.ISING_ENOTFOUND
    srv.close()


@pytest.mark.parametrize("quantum", [12, 400])
def test_served_stream_requests_against_the_oracle(I, quantum):
    """The first 24 requests of the served stream (L from 32 to 8032, hot and
    cold starts, their own temperatures, seeds and stream ids), sweeps capped
    at 30, served together; quantum 12 makes them cross quanta, 400 is the
    benchmark's.  L <= 256: the whole series and lattice equal the oracle's;
    larger L: oracle light-cone windows of the returned spins, the series'
    invariants, and the last E/M recounted from the returned spins."""
    stream = workloads.served_stream()[:24]
    reqs = [{"L": q.L, "beta": 1.0 / q.T, "seed": q.seed, "stream_id": q.stream_id,
             "init": q.init, "n_sweeps": min(q.sweeps, 30), "n_discard": 0,
             "record_series": True, "return_spins": True} for q in stream]
    _say("case served stream prefix, quantum %d" % quantum)
    res, stats = _run(I, reqs, 256 << 20, quantum)
    assert stats["done"] == len(reqs)
    for r, got in zip(reqs, res):
        L, n = r["L"], r["n_sweeps"]
        assert got["sweeps_done"] == n
        if L <= 256:
            s, oEM = oracle.run(L, r["beta"], r["seed"], r["stream_id"], r["init"], n)
            assert np.array_equal(got["series"], oEM), r
            assert np.array_equal(got["spins"], s), r
            continue
        sp = got["spins"].astype(np.int64)
        E = -int(np.sum(sp * (np.roll(sp, -1, axis=1) + np.roll(sp, -1, axis=0))))
        assert (got["E_final"], got["M_final"]) == (E, int(sp.sum())), r
        assert tuple(got["series"][-1]) == (E, int(sp.sum())), r
        assert np.all(got["series"][:, 0] % 4 == 0), r
        for (x0, y0) in [(L - 20, L - 6), (L // 3, L // 2 + 1)]:
            ys = (y0 + np.arange(12)) % L
            xs = (x0 + np.arange(40)) % L
            want = oracle.window(L, r["beta"], r["seed"], r["stream_id"], r["init"], 0, n, x0, y0,
                                 40, 12)
            assert np.array_equal(got["spins"][np.ix_(ys, xs)], want), (r, x0, y0)


def test_schedule_never_changes_results(I):
    """Five 8192^2 lattices with different sweep counts in quanta of 8
    sweeps (they leave the fused launches at different quanta, and the
    lattices left take the plain path or fused launches by the cost model),
    beside small lattices: every result equals the same request alone on
    the plain path."""
    reqs = []
    for i, (L, n) in enumerate([(8192, 30), (8192, 11), (8192, 47), (8192, 20), (8192, 36),
                                (64, 900), (256, 300), (32, 5000), (128, 70)]):
        reqs.append({"L": L, "beta": 1.0 / (2.0 + 0.1 * i), "seed": 77 + i, "stream_id": i,
                     "init": workloads.INIT_HOT, "n_sweeps": n, "n_discard": 0,
                     "record_series": True, "return_spins": L <= 256})
    _say("case schedule: five 8192^2 and four small lattices, quantum 8")
    res, stats = _run(I, reqs, 1 << 30, 8)
    assert stats["done"] == len(reqs)
    for r, got in zip(reqs, res):
        lat = I.Lattice(r["L"], seed=r["seed"], stream_id=r["stream_id"], init=r["init"],
                        beta=r["beta"])
        em = lat.sweep_em(r["n_sweeps"]).cpu().numpy()
        assert np.array_equal(got["series"], em), r
        if r["L"] <= 256:
            assert np.array_equal(got["spins"], lat.get_spins()), r
        del lat


def test_second_copies_never_hold_a_request_back(I):
    """Two lattices whose second copies fill the arena to less than half, then
    a request that fits beside the lattices but not beside the copies: it is
    admitted in the next step, and everything's results are the plain path's.
    Memory in use counts requests only."""
    def req(L, n, i):
        return {"L": L, "beta": 1 / 2.3, "seed": 60 + i, "stream_id": i,
                "init": workloads.INIT_HOT, "n_sweeps": n, "record_series": True,
                "return_spins": True}

    reqs = [req(1024, 60, 0), req(1024, 45, 1), req(4608, 12, 2), req(1024, 20, 3)]
    size = [(I.ising_lattice_bytes(r["L"]) + 255) // 256 * 256 +
            (16 * r["n_sweeps"] + 255) // 256 * 256 for r in reqs]
    arena = (sum(size[:3]) + (32 << 10)) * 32 // 31  # 1/32 holds the task tables
    assert sum(size[:3]) + 2 * int(I.lib().ising_spare_bytes(1024)) > arena
    srv = I.Server(arena, quantum_sweeps=10)
    tickets = srv.submit(reqs[:2])
    srv.step()
    assert srv.stats()["admitted"] == 2 and srv.stats()["bytes_in_use"] == sum(size[:2])
    tickets += srv.submit(reqs[2:])
    srv.step()
    assert srv.stats()["admitted"] >= 3
    srv.run_until_idle()
    assert srv.stats()["peak_bytes"] <= sum(size)
    for r, t in zip(reqs, tickets):
        got = srv.poll(t)
        lat = I.Lattice(r["L"], seed=r["seed"], stream_id=r["stream_id"], init=r["init"],
                        beta=r["beta"])
        assert np.array_equal(got["series"], lat.sweep_em(r["n_sweeps"]).cpu().numpy()), r["L"]
        assert np.array_equal(got["spins"], lat.get_spins()), r["L"]
    srv.close()


def test_requests_come_and_go_around_second_copies(I):
    """Uneven sides and lengths in arenas where copies are given, moved over
    and taken away: every result is the plain path's."""
    rng = np.random.default_rng(17)
    reqs = [{"L": int(L), "beta": 1 / float(rng.uniform(1.6, 3.0)), "seed": 90 + i,
             "stream_id": i, "init": workloads.INIT_HOT, "n_sweeps": int(rng.integers(3, 60)),
             "record_series": True, "return_spins": True}
            for i, L in enumerate(8 * rng.integers(8, 200, 40))]
    alone = []
    for r in reqs:
        lat = I.Lattice(r["L"], seed=r["seed"], stream_id=r["stream_id"], init=r["init"],
                        beta=r["beta"])
        alone.append((lat.sweep_em(r["n_sweeps"]).cpu().numpy(), lat.get_spins()))
    for arena in (1 << 20, 3 << 20, 12 << 20):
        srv = I.Server(arena, quantum_sweeps=7)
        srv.inject_fault(3)
        tickets = []
        for at in range(0, len(reqs), 5):  # five more every other step
            tickets += srv.submit(reqs[at:at + 5])
            srv.step()
            srv.step()
        srv.run_until_idle()
        for r, t, (em, s) in zip(reqs, tickets, alone):
            got = srv.poll(t)
            assert np.array_equal(got["series"], em), (arena, r["L"])
            assert np.array_equal(got["spins"], s), (arena, r["L"])
        srv.close()
