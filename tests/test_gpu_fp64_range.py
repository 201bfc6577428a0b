"""The device's FP64 square root, quotient and reciprocal against the host's correctly rounded ones
(numpy), over the magnitudes that the step meets and at the ends of the doubles' range.

Magnitudes of the step: no difference is allowed. The step's operations are Newton's iterations with
a last correction by the exact remainder, correctly rounded there; the observables and the reverse
step divide with the compiler's operator and rely on equal bits. Outside, the probe answers with the
compiler's IEEE operations: zeros, infinities and NaN exactly; a subnormal quotient may be rounded
twice (scaled, then into the subnormal range), one unit in the last place."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _probe(a, b):
    import torch
    from paper_1410_2569_amd.lbm import fp64_probe

    sq, qt = fp64_probe(torch.from_numpy(np.ascontiguousarray(a)).cuda(),
                        torch.from_numpy(np.ascontiguousarray(b)).cuda())
    return sq.cpu().numpy(), qt.cpu().numpy()


def _operands(rng, n):
    """Magnitudes from 1e-15 to 1e6: random ones, those next to powers of two, and mantissas of few
    or nearly all ones."""
    v = 10.0 ** rng.uniform(-15, 6, n)
    p = 2.0 ** rng.integers(-45, 20, n // 8)
    k = rng.integers(1, 6, n // 8)
    return np.concatenate([v, p * (1 + k * 2.0 ** -52), p * (1 - k * 2.0 ** -53),
                           p * (1 + 2.0 ** -rng.integers(1, 52, n // 8).astype(float)),
                           p * (2 - 2.0 ** -rng.integers(1, 52, n // 8).astype(float)), p])


@pytest.mark.parametrize("seed", [1, 2])
def test_no_rounding_differs_at_the_steps_magnitudes(gpu, seed):
    rng = np.random.default_rng(seed)
    a, b = _operands(rng, 2_000_000), _operands(rng, 2_000_000)
    rng.shuffle(b)
    b *= rng.choice([-1.0, 1.0], b.size)
    sq, qt = _probe(a, b)
    assert np.array_equal(sq, np.sqrt(a)) and np.array_equal(qt, a / b)
    assert np.array_equal(_probe(np.ones_like(b), b)[1], 1.0 / b)
    # next to exact quotients and squares, where a remainder decides
    near = np.nextafter(a * b, np.where(rng.random(a.size) < 0.5, -np.inf, np.inf))
    assert np.array_equal(_probe(near, b)[1], near / b)
    x = np.nextafter(a * a, np.where(rng.random(a.size) < 0.5, 0.0, np.inf))
    assert np.array_equal(_probe(x, b)[0], np.sqrt(x))


def test_ends_of_the_range(gpu):
    v = [0.0, 5e-324, 1e-310, 2.2250738585072014e-308, 1e-300, 1e-160, 1.0, 3.0, 1e160, 1e300,
         1.7976931348623157e308, np.inf, np.nan]
    v += [-x for x in v]
    a, b = (np.array(x) for x in zip(*itertools.product(v, v)))
    with np.errstate(all="ignore"):
        want_sq, want_qt = np.sqrt(a), a / b
    sq, qt = _probe(a, b)
    for got, want, ops in ((sq, want_sq, "sqrt"), (qt, want_qt, "quotient")):
        nan = np.isnan(want)
        assert np.array_equal(np.isnan(got), nan), (ops, a[np.isnan(got) != nan], b[np.isnan(got) != nan])
        assert np.array_equal(np.signbit(got[~nan]), np.signbit(want[~nan])), ops
        off = np.abs(got[~nan].view(np.int64) - want[~nan].view(np.int64))
        tiny = (np.abs(want[~nan]) < 2.2250738585072014e-308) & (want[~nan] != 0)
        assert off[~tiny].max() == 0 and off[tiny].max(initial=0) <= 1, ops
