"""Dense complex64 windows applied again and again to the same wires, as Trotter
steps apply them: the error must not grow faster than that of FP32 products.

The yardstick is those products on the CPU, each multiply-add rounded once to
float in the order of the FP32 matrix cores' forms.  Both sides start from the
same float amplitudes and the same float matrix, and the exact result is that
matrix in complex128.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _window(k, eps, seed):
    """A unitary within eps of the identity, its entries rounded to float."""
    rng = np.random.default_rng(seed)
    h = rng.normal(size=(1 << k, 1 << k)) + 1j * rng.normal(size=(1 << k, 1 << k))
    w, v = np.linalg.eigh((h + h.conj().T) / 2 / np.sqrt(2 << k))
    return ((v * np.exp(1j * eps * w)) @ v.conj().T).astype(np.complex64).astype(np.complex128)


def _fp32(u, x):
    """u @ x, four depths at a time: real and imaginary part by two chains of four
    multiply-adds each (exact products, one rounding to float per addition)."""
    yr, yi = np.zeros(x.shape, np.float32), np.zeros(x.shape, np.float32)

    def chain(y, a, b):
        for j in range(a.shape[1]):
            y = (y.astype(np.float64) + a[:, j:j + 1] * b[j:j + 1]).astype(np.float32)
        return y

    for j in range(0, u.shape[1], 4):
        a, b = u[:, j:j + 4], x[j:j + 4]
        yr = chain(chain(yr, a.real, b.real), a.imag, -b.imag)
        yi = chain(chain(yi, a.real, b.imag), a.imag, b.real)
    return yr + 1j * yi.astype(np.float64)


@pytest.mark.parametrize("eps", [1e-3, 0.02])
@pytest.mark.parametrize("k", [5, 6])
def test_repeated_window_error_is_no_larger_than_fp32(k, eps):
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    n = k + 4
    u = _window(k, eps, k)
    psi = W.gaussian_state(n, 3).astype(np.complex64)
    st = qs.State(n, "c64", init=None)
    st.upload(psi)
    plan = qs.Plan(n, [W.G("UNITARY", *range(k), mat=u)])  # the rows are the leading qubits
    assert [L["kind"] for L in plan.describe()["layers"]] == ["dense"]
    x = psi.astype(np.complex128).reshape(1 << k, -1)
    exact, model = x, x
    for rep in range(1, 401):
        qs.apply(st, plan)
        exact, model = u @ exact, _fp32(u, model)
        if rep in (1, 40, 400):
            err = np.linalg.norm(st.download().astype(np.complex128) - exact.ravel())
            ref = np.linalg.norm(model - exact)
            assert err <= ref, (rep, err, ref)


@pytest.mark.parametrize("power", [-100, -105, -110, -115])
@pytest.mark.parametrize("k", [5, 6])
def test_tiny_states_keep_their_bits(k, power):
    """A power of two in front of the state changes no significant bit: the error
    stays within the FP32 chain's, one rounding (half a unit at most, uniform) per
    product of a complex entry, all at the size of the result."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    n = k + 5
    u = W.random_unitary(1 << k, np.random.default_rng(k)).astype(np.complex64).astype(np.complex128)
    psi = W.gaussian_state(n, 3).astype(np.complex64) * np.float32(2.0 ** power)
    st = qs.State(n, "c64", init=None)
    st.upload(psi)
    qs.apply(st, qs.Plan(n, [W.G("UNITARY", *range(k), mat=u)]))
    exact = (u @ psi.astype(np.complex128).reshape(1 << k, -1)).ravel()
    err = np.linalg.norm(st.download().astype(np.complex128) - exact) / np.linalg.norm(exact)
    assert err <= np.sqrt(4 * (1 << k) / 2 / 3) * 2.0 ** -24, err


@pytest.mark.parametrize("k", [5, 6])
def test_tiny_columns_next_to_ordinary_ones(k):
    """Some columns of a tile far below the split's range, one empty: every column
    keeps the accuracy that it has by itself."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    n = k + 6
    u = W.random_unitary(1 << k, np.random.default_rng(k)).astype(np.complex64).astype(np.complex128)
    psi = W.gaussian_state(n, 5).astype(np.complex64).reshape(1 << k, -1)
    psi[:, 3] *= np.float32(2.0 ** -110)
    psi[:, 17] *= np.float32(2.0 ** -113)
    psi[:, 40] = 0
    st = qs.State(n, "c64", init=None)
    st.upload(psi.ravel())
    qs.apply(st, qs.Plan(n, [W.G("UNITARY", *range(k), mat=u)]))
    exact = u @ psi.astype(np.complex128)
    got = st.download().astype(np.complex128).reshape(exact.shape)
    assert not got[:, 40].any()
    size = np.linalg.norm(exact, axis=0)
    size[40] = 1.0
    err = np.linalg.norm(got - exact, axis=0) / size
    # twice the rms bound: a column's 2^(k+1) numbers against the mean
    assert err.max() <= 2 * np.sqrt(4 * (1 << k) / 2 / 3) * 2.0 ** -24, err.max()


@pytest.mark.parametrize("head", [0.0, 2.0 ** -80])
@pytest.mark.parametrize("big", [1.0, 2.0 ** 70, 2.0 ** 100])
@pytest.mark.parametrize("k", [5, 6])
def test_columns_that_start_tiny(k, big, head):
    """Columns whose leading rows are empty or tiny, the others ordinary or large."""
    import torch  # noqa: F401  (its HIP runtime first)
    import paper_2609_19147_amd as qs
    n = k + 6
    u = W.random_unitary(1 << k, np.random.default_rng(k)).astype(np.complex64).astype(np.complex128)
    psi = W.gaussian_state(n, 5).astype(np.complex64).reshape(1 << k, -1)
    psi[: 1 << (k - 1), ::3] *= np.float32(head)
    psi[1 << (k - 1):, ::3] *= np.float32(big)
    st = qs.State(n, "c64", init=None)
    st.upload(psi.ravel())
    qs.apply(st, qs.Plan(n, [W.G("UNITARY", *range(k), mat=u)]))
    exact = u @ psi.astype(np.complex128)
    got = st.download().astype(np.complex128).reshape(exact.shape)
    err = np.linalg.norm(got - exact, axis=0) / np.linalg.norm(exact, axis=0)
    assert err.max() <= 2 * np.sqrt(4 * (1 << k) / 2 / 3) * 2.0 ** -24, err.max()
