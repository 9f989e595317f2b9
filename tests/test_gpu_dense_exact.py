"""Dense blocks whose results are known to the last bit, and the error of the
complex64 five- and six-qubit blocks, whose products run on the bf16 matrix
cores as sums of exact three-part splits.

Sizes: the smallest tiles (n = k + 4, k + 5), one full tile, and the first sizes
at which a workgroup takes several tiles."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = [(dt, k, n) for dt in ("c64", "c128") for k in (4, 5, 6)
         for n in (k + 4, k + 5, k + 6, 14, 21 if dt == "c64" else 20)]
CASES += [("c64", 6, 23), ("c64", 4, 22), ("c128", 6, 21)]


def _wires(n, k, rng):
    return [int(w) for w in rng.permutation(n)[:k]]


def _state(qs, n, dtype, seed):
    st = qs.State(n, dtype, init=None)
    W.gaussian_state_torch(n, seed, dtype, out=st.tensor())
    return st


def _columns(n, wires):
    """Indices of the state as (columns, 2^k rows), row bits most significant first."""
    import torch
    rest = [q for q in range(n) if q not in wires]
    idx = torch.arange(1 << n, device="cuda").reshape([2] * n)
    return idx.permute(*rest, *wires).reshape(-1, 1 << len(wires))


@pytest.mark.parametrize("dtype,k,n", CASES)
def test_signed_permutations_are_exact(dtype, k, n):
    import torch
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(n * 10 + k)
    wires = _wires(n, k, rng)
    perm, ph = rng.permutation(1 << k), rng.integers(0, 4, 1 << k)
    m = np.zeros((1 << k, 1 << k), np.complex128)
    m[np.arange(1 << k), perm] = np.array([1, 1j, -1, -1j])[ph]  # row r: phase * x[perm[r]]
    st = _state(qs, n, dtype, n)
    cols = _columns(n, wires)
    ref = st.tensor().clone()
    f = torch.tensor(np.array([1, 1j, -1, -1j])[ph], dtype=ref.dtype, device="cuda")
    ref[cols] = f * st.tensor()[cols[:, torch.tensor(perm, device="cuda")]]
    plan = qs.Plan(n, [W.G("UNITARY", *wires, mat=m)])
    assert [L["kind"] for L in plan.describe()["layers"]] == ["dense"]
    qs.apply(st, plan)
    assert torch.equal(st.tensor(), ref)


@pytest.mark.parametrize("k,n", [(5, 9), (5, 13), (6, 10), (6, 14), (5, 21), (6, 21)])
def test_complex64_error_against_complex128(k, n):
    import torch
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(n * 10 + k)
    wires = _wires(n, k, rng)
    m = W.random_unitary(1 << k, rng)
    a = _state(qs, n, "c64", n)
    b = qs.State(n, "c128", init=None)
    b.tensor().copy_(a.tensor())
    cols = _columns(n, wires)
    # |y - y64| <= gamma sum |u| |x| over the 2^k products of a row: U's rounding to
    # float, at most one rounding per partial product and accumulator entry, and
    # the products left out
    x = b.tensor()[cols].abs() @ torch.tensor(np.abs(m).T, device="cuda")
    bound = (2 * (1 << k) + 4) * 2.0 ** -24 * 2 * x
    plan = qs.Plan(n, [W.G("UNITARY", *wires, mat=m)])
    qs.apply(a, plan)
    qs.apply(b, plan)
    err = (a.tensor().to(torch.complex128) - b.tensor())[cols].abs()
    assert bool((err <= bound).all()), (err / bound).max().item()
    # rms: the 4 2^k products of a complex entry, each rounded once at the size of
    # the partial sum (uniform in half a unit), is the FP32 chain's error
    rms = err.pow(2).mean().sqrt().item() * 2.0 ** (n / 2)
    assert rms <= np.sqrt(4 * (1 << k) / 2 / 3) * 2.0 ** -24, rms


@pytest.mark.parametrize("k", [5, 6])
def test_complex64_errors_have_no_common_direction(k):
    import torch
    import paper_2609_19147_amd as qs
    n = 22
    rng = np.random.default_rng(k)
    h = W.random_unitary(1 << k, rng)
    m, _ = np.linalg.qr(np.eye(1 << k) + 0.02 * (h - h.conj().T))
    a = _state(qs, n, "c64", n)
    b = qs.State(n, "c128", init=None)
    b.tensor().copy_(a.tensor())
    plan = qs.Plan(n, [W.G("UNITARY", *_wires(n, k, rng), mat=m)])
    qs.apply(a, plan)
    qs.apply(b, plan)
    err = a.tensor().to(torch.complex128) - b.tensor()
    # the 16 2^k amplitudes of a column block may share a direction, the blocks
    # are independent: six standard deviations of their sum
    bound = 6 * np.sqrt((1 << n) * 16 * (1 << k)) * err.abs().pow(2).mean().sqrt().item()
    assert abs(err.sum().item()) <= bound


@pytest.mark.parametrize("big", [np.float32(3.4e38), np.float32(np.inf)])
@pytest.mark.parametrize("k,n", [(5, 9), (5, 14), (6, 10), (6, 14)])
def test_values_beyond_bf16(k, n, big):
    import torch
    import paper_2609_19147_amd as qs
    rng = np.random.default_rng(n * 10 + k)
    wires = _wires(n, k, rng)
    perm = rng.permutation(1 << k)
    m = np.zeros((1 << k, 1 << k), np.complex128)
    m[np.arange(1 << k), perm] = 1
    st = _state(qs, n, "c64", n)
    cols = _columns(n, wires)
    hit = cols[cols.shape[0] // 3]
    st.tensor()[hit[3]] = complex(big, 0)
    ref = st.tensor().clone()
    ref[cols] = st.tensor()[cols[:, torch.tensor(perm, device="cuda")]]
    qs.apply(st, qs.Plan(n, [W.G("UNITARY", *wires, mat=m)]))
    got = st.tensor()
    row = hit[int(np.nonzero(perm == 3)[0][0])]
    assert got[row].real.item() == float(big)
    if np.isinf(big):  # 0 * inf: the rest of that column is no number, as in any product
        ref[hit] = 0
        got[hit] = 0
    assert torch.equal(got, ref)
