"""Accuracy of the unit phasors exp(-i q x) of the sum kernels' tables (half-turn reduction
with q / pi = hi + lo, polynomials in r^2 on |r| <= 1/2).

The same source is compiled for the host with hipcc and compared with exp(-i q x) of the
exact product q x, reduced by a 200-bit pi: over the phases of the sums, next to integer and
half-integer half turns of either parity, for negative arguments, and up to the range limit of
2^30 half turns, beyond which the library's sine and cosine take over.

Bound of an absolute error, in units of 2^-52: the two fused products of the reduction round
r <= 1/2 by 2^-55 each, pi times that in the phase (0.8); Horner's rule, the square r^2 and the
last product or sum add at most 2.
"""
import math
import os
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_18444_amd", "csrc")
HIPCC = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
TOL = 3.0 * 2.0 ** -52


def _arctan_inverse(n, bits=220):
    """arctan(1 / n) in units of 2^-bits."""
    term = (1 << bits) // n
    total, k = term, 1
    while term:
        term //= n * n
        total += (-1) ** k * (term // (2 * k + 1))
        k += 1
    return total


PI = Fraction(4 * (4 * _arctan_inverse(5) - _arctan_inverse(239)), 1 << 220)  # Machin


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if HIPCC is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("phasor") / "phasor_check")
    src = os.path.join(ROOT, "tests", "native", "phasor_check.cpp")
    res = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC, src, "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


def _run(exe, pairs):
    inp = "".join(f"{float(q).hex()} {float(x).hex()}\n" for q, x in pairs)
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout.split("\n")
    return np.array([[float.fromhex(v) for v in l.split()] for l in out if l])


def _exact(q, x):
    """(cos, -sin) of the exact product."""
    phase = Fraction(float(q)) * Fraction(float(x))
    quarter = round(phase / (PI / 2))
    r = float(phase - quarter * (PI / 2))
    s, c = math.sin(r), math.cos(r)
    s, c = [(s, c), (c, -s), (-s, -c), (-c, s)][quarter % 4]
    return c, -s


def _check_fast(exe, pairs):
    got = _run(exe, pairs)
    assert all(abs(x) < r for (_, x), r in zip(pairs, got[:, 4])), "arguments inside the range"
    ref = np.array([_exact(q, x) for q, x in pairs])
    err = np.abs(got[:, :2] - ref)
    worst = int(err.max(axis=1).argmax())
    assert err.max() <= TOL, (pairs[worst], err[worst] / 2.0 ** -52)


def test_random_phases(checker):
    rng = np.random.default_rng(41)
    pairs = [(q, x) for q, x in zip(rng.uniform(-4.0, 4.0, 4000), rng.uniform(-60.0, 60.0, 4000))]
    pairs += [(q, x) for q, x in zip(10.0 ** rng.uniform(-6, 3, 3000), 10.0 ** rng.uniform(-6, 3, 3000))]
    pairs += [(0.0, 1.0), (1.0, 0.0), (-0.0, 5.0), (1e-300, 1e-300)]
    _check_fast(checker, pairs)


def test_next_to_whole_and_half_turns(checker):
    """q x / pi near every multiple of 1/2: the rounding of k, its parity and the poles of the
    polynomials' interval."""
    rng = np.random.default_rng(42)
    pairs = []
    for m in list(range(-41, 42)) + [int(v) for v in rng.integers(-10 ** 6, 10 ** 6, 200)]:
        q = float(rng.uniform(0.01, 3.0))
        x = float(Fraction(m) / 2 * PI / Fraction(q))
        for v in (x, np.nextafter(x, np.inf), np.nextafter(x, -np.inf)):
            pairs.append((q, float(v)))
            pairs.append((-q, float(v)))
    _check_fast(checker, pairs)


def test_up_to_the_range_limit(checker):
    rng = np.random.default_rng(43)
    qs = [float(v) for v in 10.0 ** rng.uniform(-3, 3, 300)]
    limits = _run(checker, [(q, 0.0) for q in qs])[:, 4]
    pairs = []
    for q, r in zip(qs, limits):
        assert abs(q * r / math.pi) <= 2.0 ** 30 * (1 + 1e-12)
        for f in (1.0 - 2.0 ** -50, 0.5, float(rng.uniform(0.1, 1.0 - 1e-9))):
            pairs += [(q, f * float(r)), (q, -f * float(r))]
    _check_fast(checker, pairs)


def test_library_beyond_the_range(checker):
    """The library's form rounds the phase itself: q, pi and two products."""
    rng = np.random.default_rng(44)
    pairs = [(float(q), float(x)) for q, x in zip(rng.uniform(-3, 3, 200), 10.0 ** rng.uniform(0, 11, 200))]
    got = _run(checker, pairs)
    for (q, x), g in zip(pairs, got):
        ref = _exact(q, x)
        bound = 4.0 * 2.0 ** -53 * abs(q * x) + TOL
        assert abs(g[2] - ref[0]) <= bound and abs(g[3] - ref[1]) <= bound, (q, x)
    special = _run(checker, [(1.0, math.inf), (1.0, -math.inf), (1.0, math.nan)])
    assert np.isnan(special[:, 2:4]).all()
