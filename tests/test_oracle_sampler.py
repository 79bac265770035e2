"""Pins for oracle/philox.py and oracle/sampler.py."""
import math
import os
import struct
from fractions import Fraction

import numpy as np
import pytest

from oracle import philox, sampler

GOLD = os.path.join(os.path.dirname(__file__), "golden", "philox4x32_10_kat.txt")


def test_philox_known_answers():
    """Published known-answer vectors (Salmon et al., SC'11)."""
    rows = 0
    for line in open(GOLD):
        if line.startswith("#") or not line.strip():
            continue
        w = [int(x, 16) for x in line.split()]
        assert philox.philox4x32_10(w[0:4], w[4:6]) == tuple(w[6:10])
        rows += 1
    assert rows == 3


def test_philox_counter_layout_and_uniformity():
    # distinct (seq, step) -> distinct 64-bit draws; roughly uniform
    seen = set()
    n = 20000
    acc = np.zeros(16, np.int64)
    for s in range(100):
        for t in range(200):
            u = philox.uniform_u64(7, s, t)
            seen.add(u)
            acc[u >> 60] += 1
    assert len(seen) == n
    chi2 = float(((acc - n / 16) ** 2 / (n / 16)).sum())
    assert chi2 < 45.0                                   # 15 dof, p ~ 1e-4
    assert philox.uniform_u64(7, 1, 2) != philox.uniform_u64(7, 2, 1)
    assert philox.uniform_u64(7, 1, 2) != philox.uniform_u64(8, 1, 2)
    assert philox.uniform_u64(7, 1 << 40, 2) != philox.uniform_u64(7, 0, 2)
    assert philox.uniform_u64(1 << 40, 1, 2) != philox.uniform_u64(0, 1, 2)


def test_exp2_fixed_accuracy_and_anchors():
    x = np.linspace(-41, 0, 200001).astype(np.float32)
    q = sampler.exp2_fixed(x).astype(np.float64)
    ref = np.exp2(x.astype(np.float64)) * 2.0 ** 40
    # polynomial + fp32 rounding: < 2e-7 relative; the floor: < 1 absolute
    assert np.all(np.abs(q - ref) <= ref * 2e-7 + 1.0)
    assert np.all(q <= ref * (1 + 2e-7))
    assert int(sampler.exp2_fixed(np.float32(0.0))) == 1 << 40
    assert int(sampler.exp2_fixed(np.float32(-1.0))) == 1 << 39
    assert int(sampler.exp2_fixed(np.float32(-40.0))) == 1
    assert int(sampler.exp2_fixed(np.float32(-41.5))) == 0
    assert int(sampler.exp2_fixed(np.float32(-1e30))) == 0
    assert int(sampler.exp2_fixed(np.float32(-np.inf))) == 0
    # monotone on a fine grid (a wrong coefficient order breaks this)
    assert np.all(np.diff(q) >= 0)


def test_pick_exhaustive_small_vocab():
    """Brute force: for tiny integer weight vectors, sweep u so that t takes every
    value in [0, S) and check that token k is chosen for exactly q_k thresholds."""
    rng = np.random.default_rng(0)
    for _ in range(20):
        v = int(rng.integers(2, 9))
        q = rng.integers(0, 6, size=v).astype(np.uint64)
        q[int(rng.integers(0, v))] += np.uint64(1)
        total = int(q.sum())
        counts = np.zeros(v, np.int64)
        for t in range(total):
            u = -((-t << 64) // total)                   # smallest u with floor(u*S/2^64) == t
            assert (u * total) >> 64 == t
            k = sampler.pick(q, u)
            counts[k] += 1
            assert int(q[:k].sum()) <= t < int(q[:k + 1].sum())
        np.testing.assert_array_equal(counts, q.astype(np.int64))
    assert sampler.pick(np.array([0, 0, 5, 0], np.uint64), (1 << 64) - 1) == 2
    assert sampler.pick(np.array([0, 0, 5, 0], np.uint64), 0) == 2


def test_one_hot_and_low_temperature_pick_argmax():
    rng = np.random.default_rng(1)
    z = rng.normal(size=1000).astype(np.float32)
    am = int(np.argmax(z))
    for step in range(50):
        tok, lp = sampler.sample_row(z, 1e-4, 5, 9, step)
        assert tok == am and abs(lp) < 1e-6
    onehot = np.full(300, -1e9, np.float32)
    onehot[123] = 4.0
    for step in range(20):
        assert sampler.sample_row(onehot, 1.0, 5, 9, step)[0] == 123


@pytest.mark.parametrize("temperature", [1.0, 0.7])
def test_sampled_distribution_matches_fp64_softmax(temperature):
    rng = np.random.default_rng(2)
    v = 24
    z = (rng.normal(size=v) * 1.5).astype(np.float32)
    inv_t = sampler.inv_temperature(temperature)
    q = sampler.weights_u64(z, inv_t)
    # the integer weights themselves are the softmax to ~1e-7
    p_ref = np.exp(z.astype(np.float64) / temperature)
    p_ref /= p_ref.sum()
    p_q = q.astype(np.float64) / float(q.sum())
    assert np.max(np.abs(p_q - p_ref) / p_ref) < 1e-6
    # and the Philox-driven draws follow it (chi-square, 23 dof)
    n = 60000
    counts = np.zeros(v, np.int64)
    for s in range(n):
        counts[sampler.pick(q, __import__("oracle.philox", fromlist=["x"]).uniform_u64(11, s, 3))] += 1
    chi2 = float(((counts - n * p_ref) ** 2 / (n * p_ref)).sum())
    assert chi2 < 60.0                                   # p ~ 4e-5 at 23 dof


def test_logprob_output_and_row_map():
    rng = np.random.default_rng(3)
    z = rng.normal(size=(3, 50)).astype(np.float32)
    toks, lps = sampler.sample(z, 0.9, 1, np.arange(6, dtype=np.uint64), 0,
                               row_map=np.array([0, 0, 1, 1, 2, 2]))
    from scipy.special import log_softmax
    ref = log_softmax(z.astype(np.float64) * float(sampler.inv_temperature(0.9)), axis=-1)
    for r in range(6):
        assert abs(lps[r] - ref[r // 2, toks[r]]) < 1e-12
    # same row, different seq_id -> an independent draw, same (seq, step) -> same draw
    t2, _ = sampler.sample(z, 0.9, 1, np.arange(6, dtype=np.uint64), 0,
                           row_map=np.array([0, 0, 1, 1, 2, 2]))
    np.testing.assert_array_equal(toks, t2)


def _sweep_weights(x):
    """p 2^n of the kernel's sweep as doubles: x + 1.5 * 2^23 rounds x and holds n in its low bits, and p 2^n is an
    integer addition to p's bits."""
    c = np.fmax(x, np.float32(-60.0))
    t = c + np.float32(1.5 * 2 ** 23)
    f = c - (t - np.float32(1.5 * 2 ** 23))
    p = np.full_like(f, sampler.COEF[7])
    for k in sampler.COEF[6::-1]:
        p = p * f
        p = p + k
    return (p.view(np.uint32) + (t.view(np.uint32) << np.uint32(23))).view(np.float32).astype(np.float64)


def _edge_exponents():
    edges = np.array([0.0, -0.0, -0.5, -1.5, -2.5, -39.5, -40.0, -40.5, -41.0, -59.9, -60.0, -1e30, -np.inf], np.float32)
    return np.concatenate([edges, np.nextafter(edges[:11], np.float32(-1e3)), np.nextafter(edges[2:11], np.float32(0))])


def test_weights_of_the_sweep():
    rng = np.random.default_rng(0)
    x = np.concatenate([_edge_exponents(), (-62.0 * rng.random(200000)).astype(np.float32)])
    w = _sweep_weights(x)
    np.testing.assert_array_equal(np.floor(w * 2.0 ** 40).astype(np.uint64), sampler.exp2_fixed(x))


def _add_f64(acc, w, toward_zero=True):
    """acc + w in double precision, rounded toward zero (or to nearest, ties to even), from the exact sum."""
    exact = Fraction(acc) + Fraction(w)
    last = Fraction(2) ** (math.frexp(float(exact))[1] - 53)
    if exact < last * 2 ** 52:                       # float() has rounded up to the next power of two
        last /= 2
    n = exact / last
    return float((math.floor(n) if toward_zero else round(n)) * last)


def _bits(v):
    return struct.unpack("<q", struct.pack("<d", v))[0]


def test_weights_as_a_truncating_double_sum():
    """The kernel's sum of 16 weights: doubles added to 2^12 with rounding toward zero, the integer sum read off the
    mantissa (a double in [2^12, 2^13) has a last place of 2^-40)."""
    rng = np.random.default_rng(1)
    below = np.float32(-41.0) + rng.uniform(-1e-3, 1.0, size=(20, 16)).astype(np.float32)   # around 2^-40 and below
    spread = (-62.0 * rng.random((100, 16))).astype(np.float32)
    peaked = (-3.0 * rng.random((60, 16))).astype(np.float32)
    e = _edge_exponents()
    edges = rng.choice(e, size=(40, 16))
    x = np.concatenate([np.zeros((1, 16), np.float32), np.full((1, 16), -41.0, np.float32),
                        np.full((1, 16), -np.inf, np.float32), below, spread, peaked, edges])
    differ = 0
    for row in x:
        want = int(np.sum(sampler.exp2_fixed(row), dtype=np.uint64))
        acc = nearest = 4096.0
        for w in _sweep_weights(row):
            acc, nearest = _add_f64(acc, float(w)), _add_f64(nearest, float(w), toward_zero=False)
        assert 4096.0 <= acc < 8192.0 and _bits(acc) - _bits(4096.0) == want
        differ += _bits(nearest) - _bits(4096.0) != want
    assert differ > 50                               # the rounding mode is what makes the sums exact


def test_double_addition_of_this_test():
    rng = np.random.default_rng(2)
    for a, b in zip(4096.0 + 3000.0 * rng.random(500), np.ldexp(rng.random(500), rng.integers(-60, 3, size=500))):
        assert _add_f64(a, b, toward_zero=False) == a + b
        assert _add_f64(a, b) in (a + b, math.nextafter(a + b, 0.0)) and Fraction(_add_f64(a, b)) <= Fraction(a) + Fraction(b)
