"""Sweeps at temperatures on both sides of the cut's range (1.516 to 5.77,
csrc/ising_cut.hpp) against the oracle, bit for bit, in every kernel that
chooses between the cut and the plain compares: the tiled sweep (full rows,
partial last words, flat mapping), strips, the fused batch with lattices of
both kinds in one launch, and row-strip shares."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

TEMPS = [1.45, 1.51, 1.52, 2.0, 3.5, 5.7, 5.8, 9.0]


@pytest.fixture(scope="module")
def I():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1007_3726_amd import ising
    ising.lib()
    yield ising
    ising.tuning_clear()


@pytest.mark.parametrize("T", TEMPS)
@pytest.mark.parametrize("L", [520, 1024, 8072])
def test_tiles(I, L, T):
    # 520: flat mapping, 4-bit last word; 1024: narrow rows; 8072: wide rows
    print("case L=%d T=%g" % (L, T), flush=True)
    n = 2
    lat = I.Lattice(L, seed=11, stream_id=2, init=workloads.INIT_HOT, beta=1 / T)
    em = lat.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, 11, 2, workloads.INIT_HOT, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("T", [1.51, 2.0, 5.8])
def test_strips(I, T):
    L, n = 8072, 2
    I.tuning_set([{"L_min": L, "L_max": L, "form": I.ISING_FORM_STRIP, "rpw": 8,
                   "max_blocks": 2048, "small_lds_bytes": 0, "updates_per_ns": 0.0}])
    lat = I.Lattice(L, seed=11, stream_id=2, init=workloads.INIT_HOT, beta=1 / T)
    I.tuning_clear()
    em = lat.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, 11, 2, workloads.INIT_HOT, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)


@pytest.mark.parametrize("form", ["fused", "packed"])
def test_batch_of_both_kinds(I, form):
    import torch
    n = 3
    spec = [(L, T) for L in (8, 64, 136, 256) for T in TEMPS]
    lats = [I.Lattice(L, seed=4, stream_id=i, init=workloads.INIT_HOT, beta=1 / T)
            for i, (L, T) in enumerate(spec)]
    EMs = [torch.empty((n, 2), dtype=torch.int64, device="cuda") for _ in spec]
    I.multi_sweep(lats, n, EMs, form=form)
    for i, (L, T) in enumerate(spec):
        s, oem = oracle.run(L, 1 / T, 4, i, workloads.INIT_HOT, n)
        assert np.array_equal(EMs[i].cpu().numpy(), oem), (L, T)
        assert np.array_equal(lats[i].get_spins(), s), (L, T)


@pytest.mark.parametrize("T", [1.51, 2.0, 5.8])
def test_shares(I, T):
    L, n = 256, 3
    st = I.StripSet(L, 3, seed=5, beta=1 / T)
    em = st.sweep_em(n).cpu().numpy()
    s, oem = oracle.run(L, 1 / T, 5, 0, workloads.INIT_HOT, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(st.get_spins(), s)


@pytest.mark.parametrize("T", [1.5, 2.07, 2.09, 3.5, 5.7, 5.8, 9.0])
@pytest.mark.parametrize("L", [24, 520, 1024, 8072])
def test_lcg(I, L, T):
    # the generators' cut reaches from 2.08 to 5.77
    n = 3
    lat = I.Lattice(L, seed=77, init=workloads.INIT_HOT, beta=1 / T)
    lat.use_lcg()
    em = lat.sweep_em(n).cpu().numpy()
    s = oracle.init(L, 77, 0, workloads.INIT_HOT)
    st = oracle.lcg_seed(L, 77)
    oem = oracle.lcg_sweeps(s, 1 / T, st, n)
    assert np.array_equal(em, oem)
    assert np.array_equal(lat.get_spins(), s)
    assert np.array_equal(lat.lcg_states(), st)
