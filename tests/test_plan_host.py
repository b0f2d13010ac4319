"""Plans of the block form (csrc/ising_plan.cpp, host only): what every plan
has to keep to, whatever the sides, dynamics, sweeps per call and compute
units."""
import os
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PHILOX, LCG, POOL, POOL_LINEAR = range(4)
COMPARE = -1  # Philox at thresholds without a cut
# 160 KiB of LDS per compute unit; the kernels' own: 32 sweeps' counts of 16
# waves, and where generators or pools are compiled in the starts of 64 groups
CU_LDS = 160 * 1024
STATIC_LDS = {PHILOX: 32 * 16 * 8, LCG: 32 * 16 * 8 + 2 * 64 * 4}
STATIC_LDS[COMPARE] = STATIC_LDS[PHILOX]
STATIC_LDS[POOL] = STATIC_LDS[POOL_LINEAR] = STATIC_LDS[LCG]
# calls of fewer sweeps are planned each by itself, of 24 and more alike
SWEEPS = range(2, 25)


@pytest.fixture(scope="module")
def plans():
    src = os.path.join(HERE, "xref", "plan_probe.cpp")
    csrc = os.path.join(os.path.dirname(HERE), "paper_1007_3726_amd", "csrc")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "plan_probe")
        subprocess.run(["g++", "-O2", "-std=c++17", "-I" + csrc, "-o", out, src,
                        os.path.join(csrc, "ising_plan.cpp")], check=True)

        def run(cases):
            """cases: (kind, n, cus, Ls); (microseconds per sweep, strips, shapes,
            microseconds of planning, whether cheaper than a launch per colour step) of
            each."""
            text = "".join("%d %d %d %d %s\n" % (k, n, c, len(Ls), " ".join(map(str, Ls)))
                           for k, n, c, Ls in cases)
            r = subprocess.run([out], input=text, capture_output=True, text=True, check=True)
            res = []
            for ln in r.stdout.splitlines():
                f = ln.split()
                v = [int(x) for x in f[4:-1]]
                shapes = [dict(zip(("rows", "strips", "ls", "pass", "threads", "sweeps", "lds"),
                                   v[7 * i:7 * i + 7])) for i in range(int(f[3]))]
                res.append((float(f[1]), int(f[2]), shapes, float(f[0]), f[-1] == "1"))
            assert len(res) == len(cases)
            return res
        yield run


def _sides(kind):
    # generators and pools need sides that are multiples of 8
    return range(4, 16385, 2) if kind <= PHILOX else range(8, 16385, 8)


@pytest.mark.parametrize("kind", [COMPARE, PHILOX, LCG, POOL, POOL_LINEAR])
def test_every_lone_plan_can_be_launched(plans, kind):
    """Side by side over all sides: the strips fit a compute unit's LDS with
    the kernel's own part of it, and the halos stay inside the lattice."""
    for cus in (256, 64):
        cases = [(kind, n, cus, [L]) for n in SWEEPS for L in _sides(kind)]
        for (_, n, _, Ls), (_, _, shapes, _, _) in zip(cases, plans(cases)):
            L, W = Ls[0], (Ls[0] // 2 + 63) // 64
            for s in shapes:
                where = (L, n, cus, s)
                R = L if s["strips"] == 1 else s["rows"] + 4 * s["sweeps"]
                assert s["lds"] == R * W * (24 if kind == LCG else 16), where
                assert s["lds"] + STATIC_LDS[kind] <= CU_LDS, where
                assert s["threads"] <= 1024 and s["threads"] % 64 == 0, where
                assert R <= L and s["strips"] <= 256 and s["sweeps"] <= 12, where
                if s["strips"] > 1:  # the first strips reduce a launch's sweeps, one each
                    assert s["sweeps"] <= s["strips"] and (s["strips"] - 1) * s["rows"] < L, where
                if kind == POOL_LINEAR:  # groups of 256 words, the lattice's first ones again
                    assert R * W // 256 + 3 <= 64, where


SETS = [[64 + 16 * k for k in range(24)], [64 + 8 * k for k in range(87)],
        [64 + 8 * k for k in range(279)], [8 + 2 * (k % 120) for k in range(600)],
        [8 * (k + 1) for k in range(60)], [256] * 200, [6 + 2 * (k % 9) for k in range(900)]]


@pytest.mark.parametrize("Ls", SETS)
def test_planning_is_short_beside_the_sweeps(plans, Ls):
    """Batches of many sides, 24 sweeps: planning is a fraction of the time
    that the sweeps take (every cut of 279 sides took 21 ms, of 120 sides
    10.5), and the cut nearly as good as that of a long call, for which every
    side is searched."""
    (short, _, shapes, us, _), (long_, _, best, _, _) = plans([(PHILOX, 24, 256, Ls),
                                                        (PHILOX, 10 ** 6, 256, Ls)])
    assert us < 1000
    assert bool(shapes) == bool(best)
    assert short <= 1.25 * long_


def test_second_copies_are_for_sides_that_use_them(plans):
    """The binding's limits: beyond them no lone lattice of the MI355X's 256
    compute units takes strips, and each is within a twentieth of the last
    side that does."""
    from paper_1007_3726_amd import ising
    limits = [ising._SPARE_SIDES[k] for k in (ising.ISING_RNG_PHILOX, ising.ISING_RNG_LCG,
                                              ising.ISING_RNG_POOL,
                                              ising.ISING_RNG_POOL_LINEAR)]
    for kind, limit in enumerate(limits):
        cases = [(kind, 24, 256, [L]) for L in _sides(kind) if L > 0.95 * limit]
        used = [Ls[0] for (_, _, _, Ls), r in zip(cases, plans(cases)) if r[4]]
        assert used and max(used) <= limit, kind
    # no batch with a larger side is cut into strips
    assert limits[0] ** 2 <= 6.4e7 < (limits[0] + 2) ** 2


def test_blocks_end_earlier_without_a_cut(plans):
    """Without the cut a block's instructions grow by more than a tile's: at
    6144^2 tiles are ahead then (16 sweeps at T = 1.5 22.5 us each in tiles and
    23.4 in blocks, at T = 2.3 as long in both), at 5120^2 and 7680^2 blocks."""
    sides = (1024, 4096, 5120, 6144, 7680)
    chosen = [r[4] for r in plans([(COMPARE, 24, 256, [L]) for L in sides])]
    assert chosen == [True, True, True, False, True]
    assert all(r[4] for r in plans([(PHILOX, 24, 256, [L]) for L in sides]))
