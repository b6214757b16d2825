"""Dense unitaries and the controlled powers of phase estimation on the GPU
(Sec. III-C) against the oracle: the dense matrix of a gate list, its
square, a controlled application at every kind of control position, and
the emulated powers against the gate-level ones (2^j runs of U)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 1e-10}


@pytest.fixture(scope="module")
def Q():
    from paper_1604_06460_amd import qs
    return qs


def _circuit(S, m, seed):
    rng = np.random.default_rng(seed)
    g = [S.Gate((q,), S.haar_2x2(rng)) for q in range(m)]
    g += [S.cnot(q, (q + 1) % m) for q in range(m)] if m > 1 else []
    g += [S.Gate((q,), S.haar_2x2(rng)) for q in range(m)]
    return g


@pytest.mark.parametrize("m", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("max_k", [1, 4])
def test_dense_unitary_and_square_vs_oracle(Q, O, S, m, max_k):
    gates = _circuit(S, m, 10 + m)
    ref = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m, max_k)
    assert np.abs(u.get() - ref).max() < 1e-12
    u.square()
    assert np.abs(u.get() - ref @ ref).max() < 1e-11
    u.free()


@pytest.mark.parametrize("m", [8, 9, 10])
def test_matrix_core_square_vs_oracle_product(Q, O, S, m):
    """U^2 from the library's matrix-core complex GEMM (several 128 x 128
    tiles, and one partial tile at m = 8) against the oracle's dense U
    multiplied by itself in FP64, and against the rocBLAS baseline."""
    gates = S.tfim_trotter_step(m, dt=0.37)
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    u.square()
    got = u.get()
    ref = U @ U
    assert np.abs(got - ref).max() < 1e-14 * (1 << m)
    Q.tune_set(Q.QS_TUNE_GEMM_LIB, 1)
    try:
        v = Q.Unitary(gates, m)
        v.square()
        lib = v.get()
        v.free()
    finally:
        Q.tune_set(Q.QS_TUNE_GEMM_LIB, 0)
    assert np.abs(got - lib).max() < 1e-14 * (1 << m)
    u.free()


@pytest.mark.parametrize("dtype", [1, 0])
def test_controlled_unitary_many_batches_matrix_core(Q, O, S, dtype):
    """m = 7 controlled by qubits 7, 9 and 12 of a 14-qubit state: the
    column lists of the matrix-core GEMM (runs of 2^(c-m) columns in
    2^(n-c-1) batches) against the oracle's controlled gate list."""
    m, n = 7, 14
    gates = S.tfim_trotter_step(m, dt=0.21)
    u = Q.Unitary(gates, m)
    psi0 = S.normal_state(n, 44)
    for ctrl in (7, 9, 12):
        st = Q.State(n, dtype)
        st.set(psi0)
        u.apply_controlled(st, ctrl)
        ref = O.apply_circuit(psi0, [S.Gate(g.targets, g.matrix, g.ctrl_mask | (1 << ctrl),
                                            g.ctrl_vals | (1 << ctrl)) for g in gates])
        assert np.abs(st.get() - ref).max() < TOL[dtype], ctrl
        st.free()
    u.free()


@pytest.mark.parametrize("dtype", [1, 0])
@pytest.mark.parametrize("m,n", [(5, 13), (6, 21), (6, 22), (7, 21), (7, 22), (7, 24), (9, 18)])
def test_controlled_unitary_every_tile_size(Q, S, dtype, m, n):
    """Registers of 2^m and columns on both sides of every tile size's rule,
    against the product in FP64 on the device."""
    torch = pytest.importorskip("torch")
    u = Q.Unitary(_circuit(S, m, 5 + m), m)
    U = torch.from_numpy(u.get()).cuda()
    g = torch.Generator(device="cuda").manual_seed(n)
    ctype, eps = (torch.complex128, 1.2e-16) if dtype else (torch.complex64, 6e-8)
    psi = torch.randn(1 << n, dtype=ctype, device="cuda", generator=g) / 2.0 ** (n / 2)
    want = psi.to(torch.complex128).reshape(2, -1, 1 << m)
    want = torch.stack([want[0], want[1] @ U.T.contiguous()]).reshape(-1)
    buf = psi.clone()
    torch.cuda.synchronize()
    st = Q.State(n, dtype, device_buf=buf.data_ptr())
    u.apply_controlled(st, n - 1)
    st.sync()
    # an entry is a sum of 4 * 2^m real products of numbers below max |psi|
    assert (buf - want).abs().max().item() <= 4 * 2 ** m * eps * psi.abs().max().item()
    st.free()
    u.free()


@pytest.mark.parametrize("dtype", [1, 0])
def test_controlled_unitary_every_control_position(Q, O, S, dtype):
    m, n = 3, 11
    gates = _circuit(S, m, 3)
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    psi0 = S.normal_state(n, 6)
    for ctrl in (m, m + 1, 6, n - 1):
        st = Q.State(n, dtype)
        st.set(psi0)
        u.apply_controlled(st, ctrl)
        ref = O.full_matrix(n, list(range(m)), U, 1 << ctrl, 1 << ctrl) @ psi0
        assert np.abs(st.get() - ref).max() < TOL[dtype], ctrl
        st.free()
    with pytest.raises(Q.QSError):
        u.apply_controlled(Q.State(n, dtype), m - 1)      # control inside the register
    u.free()


@pytest.mark.parametrize("dtype", [1, 0])
@pytest.mark.parametrize("m,b,n", [(4, 4, 9), (2, 5, 8), (6, 3, 10)])
def test_emulated_powers_equal_gate_level(Q, O, S, dtype, m, b, n):
    gates = S.tfim_trotter_step(m, dt=0.3)
    psi0 = S.normal_state(n, 7 + m)
    ref = O.qpe_powers(psi0, gates, m, b)
    st = Q.State(n, dtype)
    st.set(psi0)
    Q.emulate_qpe_powers(st, gates, m, m, b)
    assert np.abs(st.get() - ref).max() < TOL[dtype]
    st.free()


def test_phase_estimation_end_to_end(Q, S):
    """Eigen qubit |1> of diag(1, e^{2 pi i k / 2^b}): Hadamards, emulated
    powers, emulated inverse QFT -> the control register reads k exactly."""
    b, k = 6, 45
    gates = [S.Gate((0,), np.diag([1.0, np.exp(2j * np.pi * k / 2 ** b)]))]
    st = Q.State(1 + b, Q.QS_C128)
    st.apply_gates([S.g1(S.MAT_X, 0)] + [S.g1(S.MAT_H, 1 + j) for j in range(b)])
    Q.emulate_qpe_powers(st, gates, 1, 1, b)
    st.emulate_qft(1, b, inverse=True)
    psi = st.get()
    assert abs(abs(psi[(k << 1) | 1]) - 1) < 1e-12
    st.free()


def test_unitary_rejects_gates_outside_the_register(Q, S):
    with pytest.raises(Q.QSError):
        Q.Unitary([S.g1(S.MAT_H, 3)], 3)
    with pytest.raises(Q.QSError):
        Q.Unitary([S.mcx([4], 0)], 3)


# ---------------------------------------------------------------------------
# The eigensolver route
# ---------------------------------------------------------------------------
BETA = 0.4011269376164746        # the Hermitian blend's beta (qs_unitary_eig)


def _check_eig(u, U, tol=1e-10):
    th, V = u.eig_get()
    d = U.shape[0]
    assert np.abs(V.conj().T @ V - np.eye(d)).max() < tol
    assert np.abs((V * np.exp(1j * th)) @ V.conj().T - U).max() < tol
    w = np.linalg.eigvals(U)
    assert max(np.abs(np.exp(1j * th) - x).min() for x in w) < tol
    assert np.all(th > -np.pi - 1e-12) and np.all(th <= np.pi + 1e-12)


@pytest.mark.parametrize("m", [1, 2, 4, 6, 8])
def test_eig_reconstructs_the_unitary(Q, O, S, m):
    gates = S.tfim_trotter_step(m, dt=0.4) if m > 1 else _circuit(S, 1, 5)
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    u.eig()
    _check_eig(u, U)
    u.free()


@pytest.mark.parametrize("m", [8, 10, 12])
def test_eig_residual_of_the_ising_step(Q, O, S, m):
    """The checked residual of the Table 2 example: V^dagger U V is diagonal
    to within the 1e-10 the entry point demands."""
    u = Q.Unitary(S.tfim_trotter_step(m), m)
    u.eig()
    r = u.eig_residual()
    print("m=%d eig residual %.3e" % (m, r))
    assert 0 <= r <= 1e-10
    u.free()


@pytest.mark.parametrize("m,mult", [(4, (2, 1)), (4, (1, 2)), (4, (3, 1)), (4, (2, 2)), (5, (5, 3)), (6, (20, 12))])
def test_eig_mirror_clusters_are_resolved(Q, O, S, m, mult):
    """A phase with a multiplicity plus its mirror image about atan(beta):
    three or more eigenvectors share one eigenvalue of the Hermitian blend.
    The cluster's K = (B - B^dagger)/(2i) separates the two phases, so the
    decomposition must succeed with the residual under the bar and
    reproduce U."""
    d = 1 << m
    phi = np.arctan(BETA)
    rng = np.random.default_rng(40 + 3 * mult[0] + mult[1] + m)
    t1 = 1.1
    th = rng.uniform(-np.pi, np.pi, d)
    th[:mult[0]] = t1
    th[mult[0]:mult[0] + mult[1]] = 2 * phi - t1
    q, _ = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    M = (q * np.exp(1j * th)) @ q.conj().T
    gates = [S.Gate(tuple(range(m)), M)]
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    u.eig()
    r = u.eig_residual()
    print("m %d mult %s: residual %.3e" % (m, mult, r))
    assert r <= 1e-10
    _check_eig(u, U, 1e-9)
    u.free()


def test_eig_cluster_of_seventy_is_resolved(Q, O, S):
    """A cluster of 70 coinciding blend eigenvalues (K alone fills 78 KB of
    LDS): a 6-qubit gate with 20 copies of one phase and 15 of its mirror
    image, in a 7-qubit register (each eigenphase doubles)."""
    m, d6 = 7, 64
    phi = np.arctan(BETA)
    rng = np.random.default_rng(77)
    th = rng.uniform(-np.pi, np.pi, d6)
    th[:20] = 0.7
    th[20:35] = 2 * phi - 0.7
    q, _ = np.linalg.qr(rng.standard_normal((d6, d6)) + 1j * rng.standard_normal((d6, d6)))
    M = (q * np.exp(1j * th)) @ q.conj().T
    gates = [S.Gate(tuple(range(6)), M)]
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    u.eig()
    r = u.eig_residual()
    print("cluster of 70: residual %.3e" % r)
    assert r <= 1e-10
    _check_eig(u, U, 1e-9)
    u.free()


def test_eig_separates_phases_the_hermitian_blend_confuses(Q, O, S):
    """Eigenphases in pairs mirrored about atan(beta): the blend's eigenvalues
    cos + beta sin coincide within each pair (and two exact degeneracies of U
    itself), so only the pair rotations recover U's eigenvectors."""
    m, d = 4, 16
    phi = np.arctan(BETA)
    rng = np.random.default_rng(12)
    delta = rng.uniform(0.1, 1.4, d // 2 - 1)
    th = np.concatenate([phi + delta, phi - delta, [0.3, 0.3]])
    q, r = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    M = (q * np.exp(1j * th)) @ q.conj().T
    gates = [S.Gate(tuple(range(m)), M)]
    U = O.block_matrix(m, gates)
    u = Q.Unitary(gates, m)
    u.eig()
    _check_eig(u, U, 1e-9)
    psi0 = S.normal_state(m + 3, 2)
    st = Q.State(m + 3, Q.QS_C128)
    st.set(psi0)
    u.apply_qpe_eig(st, m, 3)
    assert np.abs(st.get() - O.qpe_powers(psi0, gates, m, 3)).max() < 1e-9
    st.free()
    u.free()


@pytest.mark.parametrize("dtype", [1, 0])
@pytest.mark.parametrize("m,b,n", [(4, 4, 9), (2, 5, 8), (6, 3, 10), (3, 2, 8)])
def test_qpe_eig_equals_gate_level(Q, O, S, dtype, m, b, n):
    """Every controlled power from the eigendecomposition against the oracle's
    2^j runs of the gate list per control qubit (spectators above the
    control register in the last two cases)."""
    gates = S.tfim_trotter_step(m, dt=0.3) if m > 1 else _circuit(S, 1, 8)
    psi0 = S.normal_state(n, 17 + m)
    ref = O.qpe_powers(psi0, gates, m, b)
    u = Q.Unitary(gates, m)
    u.eig()
    st = Q.State(n, dtype)
    st.set(psi0)
    u.apply_qpe_eig(st, m, b)
    assert np.abs(st.get() - ref).max() < TOL[dtype]
    st.free()
    u.free()


def test_qpe_eig_equals_squaring_route_at_10_qubits(Q, S):
    """m = 10, b = 10 on a 22-qubit state: the two emulation routes agree."""
    m, b, n = 10, 10, 22
    gates = S.tfim_trotter_step(m)
    psi0 = S.normal_state(n, 3)
    a = Q.State(n, Q.QS_C128)
    a.set(psi0)
    Q.emulate_qpe_powers(a, gates, m, m, b)
    u = Q.Unitary(gates, m)
    u.eig()
    e = Q.State(n, Q.QS_C128)
    e.set(psi0)
    u.apply_qpe_eig(e, m, b)
    assert np.abs(a.get() - e.get()).max() < 1e-9
    for s in (a, e):
        s.free()
    u.free()


def test_qpe_eig_end_to_end_and_errors(Q, S):
    b, k = 7, 99
    gates = [S.Gate((0,), np.diag([1.0, np.exp(2j * np.pi * k / 2 ** b)]))]
    u = Q.Unitary(gates, 1)
    st = Q.State(1 + b, Q.QS_C128)
    with pytest.raises(Q.QSError):
        u.apply_qpe_eig(st, 1, b)                  # no eigendecomposition yet
    u.eig()
    with pytest.raises(Q.QSError):
        u.apply_qpe_eig(st, 0, b)                  # control register inside U's register
    st.apply_gates([S.g1(S.MAT_X, 0)] + [S.g1(S.MAT_H, 1 + j) for j in range(b)])
    u.apply_qpe_eig(st, 1, b)
    st.emulate_qft(1, b, inverse=True)
    assert abs(abs(st.get()[(k << 1) | 1]) - 1) < 1e-12
    st.free()
    u.free()
