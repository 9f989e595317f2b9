"""Pauli-sum expectations over tile sets and windows, against the oracle.

Sizes around the tile (11 and 12 bits) and the smallest window, X masks inside
one window, across tile sets and of more than four bits, every Y parity, Z-only
sums, more terms than one set takes."""
import numpy as np
import pytest

import workloads as W
from oracle import statevec as sv

pytestmark = pytest.mark.gpu


def _terms(n, seed):
    rng = np.random.default_rng(seed)
    t = W.xxz_terms(n) + W.x_terms(n) + W.z_terms(n) + [(0.7, 0, 0)]
    for _ in range(40):  # strings of 1 to 6 factors anywhere
        k = int(rng.integers(1, min(6, n) + 1))
        ops = {int(q): "XYZ"[int(rng.integers(0, 3))] for q in rng.choice(n, size=k, replace=False)}
        t.append(W.pauli(float(rng.standard_normal()), ops))
    return t


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 6, 9, 11, 12, 13, 17])
def test_terms_against_oracle(n, dtype):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    psi = W.gaussian_state(n, 100 + n)
    if dtype == "c64":
        psi = psi.astype(np.complex64).astype(np.complex128)
    terms = _terms(n, n) if n > 1 else [(0.5, 1, 0), (1.5, 1, 1), (2.0, 0, 1), (1.0, 0, 0)]
    st = qs.State(n, dtype, init=None).upload(psi)
    tot, got = qs.expect(st, terms, per_term=True)
    ref = np.array([sv.expect(psi, n, [t]) for t in terms])
    # FP64 sums of 2^n products of a unit vector: a few rounding steps of each
    # term's absolute sum, at most |coeff|
    tol = 64 * np.finfo(np.float64).eps * np.maximum(1.0, np.abs([t[0] for t in terms]))
    assert np.all(np.abs(got - ref) <= tol)
    assert abs(tot - ref.sum()) <= tol.sum()


@pytest.mark.parametrize("n,count", [(10, 700), (14, 300)])
def test_more_terms_than_a_set_holds(n, count):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(count)
    psi = W.gaussian_state(n, 5)
    terms = []
    for k in range(count):
        x = int(rng.integers(0, 4)) << int(rng.integers(0, n - 1)) if k % 3 else 0
        terms.append((float(rng.standard_normal()), x, int(rng.integers(0, 1 << n))))
    st = qs.State(n, "c128", init=None).upload(psi)
    got = qs.expect(st, terms, per_term=True)[1]
    ref = np.array([sv.expect(psi, n, [t]) for t in terms])
    assert np.all(np.abs(got - ref) <= 64 * np.finfo(np.float64).eps * np.maximum(1.0, np.abs([t[0] for t in terms])))
