"""The one-multiply cut of a uniform at both Metropolis thresholds
(csrc/ising_cut.hpp, host part) against the two plain compares: code 0 iff
u < t8, code 1 iff t8 <= u < t4, else 2 or more, at the uniforms beside each
threshold, at the ends of the range, at the code steps' own spacing and at
random ones, for temperatures over and beyond the cut's range and for
threshold pairs at its limits."""
import math
import os
import subprocess
import tempfile

import numpy as np
import pytest

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
TOP = 2 ** 32 - 1


@pytest.fixture(scope="module")
def probe():
    src = os.path.join(HERE, "xref", "cut_probe.cpp")
    inc = os.path.join(os.path.dirname(HERE), "paper_1007_3726_amd", "csrc")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "cut_probe")
        subprocess.run(["g++", "-O1", "-std=c++17", "-I" + inc, "-o", out, src], check=True)

        def run(cases):
            r = subprocess.run([out], input="\n".join("%d %d %d %d" % c for c in cases) + "\n",
                               capture_output=True, text=True, check=True)
            return [tuple(int(v) for v in ln.split()) for ln in r.stdout.splitlines()]
        yield run


def _uniforms(t4, t8, top, rng):
    u = {0, top, t4, t8}
    u |= {int(v) for v in rng.integers(0, top, 60)}
    d = max(t4 - t8, 1)
    for k in range(-2, 18):  # every place where the code steps
        u |= {t8 + k * d + e for e in (-2, -1, 0, 1, 2)}
    for t in (t4, t8):
        u |= {t + e for e in (-2, -1, 0, 1, 2)}
    return sorted(v for v in u if 0 <= v <= top)


def _check(probe, pairs, top=TOP):
    """Compares all pairs on the uniforms 0 .. top; says which have a cut."""
    rng = np.random.default_rng(8)
    cases = [(t4, t8, top, u) for t4, t8 in pairs for u in _uniforms(t4, t8, top, rng)]
    has = {}
    for (t4, t8, _, u), (x, code) in zip(cases, probe(cases)):
        has[(t4, t8)] = x != 0
        if x:
            assert min(code, 2) == (0 if u < t8 else 1 if u < t4 else 2), (t4, t8, u, code)
    return has


def test_code_equals_the_two_compares_over_temperature(probe):
    Ts = [float(v) for v in np.linspace(0.3, 8.0, 700)] + [2.0, 2.269185, 3.0, 1e9]
    pairs = {T: tuple(oracle.thresholds(1.0 / T)) for T in Ts}
    has = _check(probe, sorted(set(pairs.values())))
    for T, p in pairs.items():
        if 1.53 <= T <= 5.7:  # the range that the served and grid workloads use
            assert has[p], T
        if T < 1.5 or T > 5.8:
            assert not has[p], T


def test_code_at_the_limits_of_the_thresholds(probe):
    pairs = [(0, 0), (TOP, TOP), (TOP, 0), (1, 0), (TOP, TOP - 1)]
    pairs += [tuple(oracle.thresholds(b)) for b in (0.0, math.inf)]
    # differences around the powers of two where the multiplier changes size,
    # each with the smallest and the largest t8 that a cut may have
    for d in (2 ** 28 - 1, 2 ** 28, 2 ** 28 + 1, 2 ** 29 + 3, 2 ** 30 - 1, 2 ** 30, 2 ** 30 + 1,
              2 ** 31):
        for t8 in (0, 1, d // 2, d - 1, d, d + 1):
            if t8 + d <= TOP:
                pairs.append((t8 + d, t8))
    _check(probe, pairs)


def test_code_of_the_lcg_range(probe):
    """|int32| + 1, 1 .. 2^31 + 1, against thresholds of that scale plus one."""
    def t(T, dE):
        return min(int(math.floor(math.ldexp(math.exp(-dE / T), 31))), 2 ** 31) + 1
    Ts = [float(v) for v in np.linspace(0.3, 8.0, 400)] + [2.269185, 1e9]
    pairs = {T: (t(T, 4), t(T, 8)) for T in Ts}
    has = _check(probe, sorted(set(pairs.values())), 2 ** 31 + 1)
    for T, p in pairs.items():
        if 2.1 <= T <= 5.7:
            assert has[p], T
        if T < 2.05 or T > 5.8:
            assert not has[p], T
    d = 2 ** 28
    _check(probe, [(0, 0), (2 ** 31, 0), (2 ** 31, 2 ** 31), (d, 0), (d + 1, 0), (2 * d + 1, d),
                   (2 * d + 3, d + 1)], 2 ** 31 + 1)
