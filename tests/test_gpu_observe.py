"""Sums over a state (csrc/reduce.hip) against numpy's on the same amplitudes:
states smaller than a row of 64 items, one row, and many rows with a remainder;
measured qubits low, high, mixed, all and in any order; and Pauli strings whose
pairs share an item, lie in one row, or lie far apart."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# sums in float64 of numbers that add up to 1 in magnitude: no more than 2^n
# roundings of 1.1e-16, and far fewer in a tree of partial sums
TOL = 1e-13


@pytest.fixture(scope="module")
def Q():
    from paper_1604_06460_amd import qs
    return qs


def _state(Q, n, dtype, seed):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    v = v.astype(np.complex128 if dtype else np.complex64)
    st = Q.State(n, dtype)
    st.set(v)
    return st, v.astype(np.complex128), rng


def _marginal(v, qubits):
    i = np.arange(v.size)
    o = np.zeros(v.size, dtype=np.int64)
    for r, q in enumerate(qubits):
        o |= ((i >> q) & 1) << r
    return np.bincount(o, weights=np.abs(v) ** 2, minlength=1 << len(qubits))


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 5, 6, 7, 8, 13, 18])
def test_marginals_and_collapse(Q, n, dtype):
    st, v, rng = _state(Q, n, dtype, 7 * n + dtype)
    sets = [[0], [n - 1], list(range(min(n, 7))), list(range(n - 1, max(-1, n - 18), -1))]
    sets += [[int(q) for q in rng.permutation(n)[:rng.integers(1, min(n, 16) + 1)]] for _ in range(4)]
    for qubits in sets:
        _, p = st.measure(qubits)
        assert np.abs(p - _marginal(v, qubits)).max() <= TOL, qubits
    qubits = sets[-1]
    out, p = st.measure(qubits, [0.37], collapse=True)
    i = np.arange(v.size)
    keep = np.ones(v.size, dtype=bool)
    for r, q in enumerate(qubits):
        keep &= ((i >> q) & 1) == ((int(out[0]) >> r) & 1)
    got = st.get()
    assert not got[~keep].any()
    want = v[keep] / np.sqrt(p[int(out[0])])
    assert np.abs(got[keep] - want).max() <= (1e-13 if dtype else 1e-7)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 9, 17, 21])
def test_pauli_and_norm(Q, n, dtype):
    st, v, rng = _state(Q, n, dtype, 90 + 7 * n + dtype)
    assert abs(st.norm2() - np.vdot(v, v).real) <= TOL
    i = np.arange(v.size, dtype=np.uint64)
    strings = [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1 << (n - 1), 0, 0), (0, 0, (1 << n) - 1)]
    for _ in range(5):
        k = rng.integers(0, 4, n)
        strings.append(tuple(int(sum(1 << q for q in range(n) if k[q] == a)) for a in (1, 2, 3)))
    for x, y, z in strings:
        sign = 1.0 - 2.0 * (np.bitwise_count(i & np.uint64(y | z)) & 1)
        want = np.vdot(v[i ^ np.uint64(x | y)], sign * v) * 1j ** bin(y).count("1")
        assert abs(st.expectation(x, y, z) - want) <= TOL, (x, y, z)
