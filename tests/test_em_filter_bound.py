"""The E-step's filter takes its scores from fp16 halves added up on the matrix cores; how far a score can be off is a
constant of the kernel.  Here the arithmetic is modelled in numpy with the least favourable addition (truncated, one
product after the other, the largest first) on inputs whose terms all have one sign, and the constant has to hold."""
import os
import re

import numpy as np
import pytest

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_15319_amd", "csrc", "vq_em.hip")


def score_error(d):
    """What the kernel allows a score of dimension d to be off by, in 2^-20 of the sum of its terms' magnitudes."""
    m = re.search(r"kScoreError = ([\d.]+)f \+ ([\d.]+)f \* D;", open(SOURCE).read())
    assert m, "the constant is not where this test looks for it"
    return float(m[1]) + float(m[2]) * d


def truncate(v, bits=24):
    """v towards zero to a significand of that many bits."""
    m, e = np.frexp(v)
    return np.ldexp(np.trunc(np.ldexp(m, bits)), e - bits)


def halves_toward_zero(v):
    hi = truncate(v, 11)
    return hi, truncate(v - hi, 11)


def halves_nearest(v):
    hi = v.astype(np.float16).astype(np.float64)
    return hi, (v - hi).astype(np.float16).astype(np.float64)


@pytest.mark.parametrize("d", [2, 4])
def test_a_score_is_off_by_no_more_than_the_kernel_allows(d):
    rng = np.random.default_rng(d)
    n = 200_000
    f32 = lambda v: v.astype(np.float32).astype(np.float64)
    h = f32(rng.uniform(32, 64, (n, d)) * 2.0 ** rng.integers(-3, 1, (n, 1)))     # scaled as the kernel scales them
    c = f32(rng.uniform(1, 64, (n, d)))
    x = -f32(np.exp(rng.uniform(np.log(0.01), np.log(60), (n, d))))               # the opposite sign: nothing cancels
    hx = f32(h * x)
    exact = (h * c * c - 2 * h * x * c).sum(1)
    size = (h * c * c + 2 * np.abs(h * x * c)).sum(1)
    terms = []
    for t in range(d):
        sq, mul = halves_nearest(f32(c[:, t] ** 2)), halves_nearest(-2 * c[:, t])
        terms += [a * b for a in halves_toward_zero(h[:, t]) for b in sq]
        terms += [a * b for a in halves_toward_zero(hx[:, t]) for b in mul]
    terms = np.stack(terms, 1)
    terms = np.take_along_axis(terms, np.argsort(-np.abs(terms), axis=1), axis=1)
    total = np.zeros(n)
    for i in range(terms.shape[1]):
        total = truncate(total + terms[:, i])
    off = np.abs(total - exact) / size * 2.0 ** 20
    print(f"d = {d}: worst {off.max():.2f}, allowed {score_error(d)}")
    assert off.max() <= score_error(d)
    assert off.max() > 0.2 * score_error(d)      # the inputs do reach for it
