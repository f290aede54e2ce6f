"""BOOST's triggered sum through a clamp (csrc/mmlike_boost_impl.h), its steps carried out in fp32 on the CPU: a term at the
clamp is found whatever the plain sums beside it do (CPU only)."""
import numpy as np
import pytest

F = np.float32


def found(terms, plain, limit, starts=True):
    """One lane's partial sums over `terms` (folds x 64 of t = clamp(..), per draw) beside the scaled plain sums of each fold:
    whether the tile is formed again."""
    part = np.zeros(terms.shape[2], F)
    main, most = part.copy(), part.copy()
    for t, s in zip(terms, plain):
        for k in range(64):
            part = part + t[k]
        v = part + s
        m = main + v
        most = np.maximum(most, part)
        part, main = v - (m - main), m
        if starts:
            most = np.maximum(most, np.abs(part))
    return ~(most < F(limit))


@pytest.mark.parametrize("size", [2.0 ** -8, 1.0, 2.0 ** 10, 2.0 ** 19, 2.0 ** 24])
def test_a_term_at_the_clamp_is_found(size):
    """Random sums of both signs that grow to `size` and fall back, one term at the clamp in a random place; and the same steps
    with neither bound let such terms pass, as this arithmetic once did."""
    rng = np.random.default_rng(7)
    folds, draws = 6, 4000
    plain = (rng.uniform(-1, 1, (folds, draws)) * size).astype(F)
    plain[3] = -(plain[0] + plain[1] + plain[2]) * F(0.999)     # (what cancels leaves sums far below what they rounded)
    terms = (rng.uniform(0, 1, (folds, 64, draws)) ** 8 * rng.choice([0.0, 2.0 ** -20, 2.0 ** -9], draws)).astype(F)
    at = rng.integers(0, folds, draws), rng.integers(0, 64, draws), np.arange(draws)
    terms[at] = 1.0
    assert found(terms, plain, 0.5).all()
    terms[at] = 0.0
    if size <= 1.0:      # small terms and sums stay where they are
        assert not found(terms, plain, 0.5).any()
    terms[at] = 1.0
    if size >= 1.0:
        assert not found(terms, plain, 1.0, False).all()
