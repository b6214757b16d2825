"""CPU-only checks of the planner of the tile passes (csrc/passes.cpp) through
qs_plan_passes: what becomes an operation of a pass, what is left alone, what
the choice between passes and blocks rests on."""
import numpy as np
import pytest

# places in PassPlan.ops
GENERAL, CONTROLLED, MOVE_X, TWO, REAL, DIAGONAL = range(6)


@pytest.fixture(scope="module")
def Q():
    from paper_1604_06460_amd import qs
    return qs


def _unitary(rng, k):
    d = 1 << k
    q, r = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def test_plan_counts_what_a_run_does(Q, S):
    """A layered circuit moves the state once per pass, far less often than
    block by block; no plan is made for states smaller than a tile."""
    gates = S.random_layer_circuit(17, 8, seed=3)
    for dtype in (Q.QS_C64, Q.QS_C128):
        p = Q.plan_passes(gates, 17, dtype, 4)
        assert 0 < p.n_passes < len(Q.plan_fusion(gates, 17, 4)[1]) and p.cost < p.block_cost
        assert p.n_alone == 0 and p.n_stages >= p.n_passes
        assert p.ops[REAL] + p.ops[GENERAL] == 17 * 8 and p.ops[DIAGONAL] > 0
        assert p.program == 1 and p.circuit == 1
    small = Q.plan_passes(S.random_layer_circuit(9, 8, seed=3), 9, Q.QS_C128, 4)
    assert (small.n_passes, small.n_stages, small.cost, small.program, small.circuit) == (0, 0, 0.0, 0, 0)
    assert small.block_cost > 0


def test_plan_of_each_gate(Q, S):
    rng = np.random.default_rng(1)
    mixed = _unitary(rng, 2)
    wide = S.Gate((1, 5, 7), _unitary(rng, 3))
    cases = [(S.g1(S.MAT_X, 5), MOVE_X, 1), (S.mcx((0, 11), 5), MOVE_X, 1), (S.cnot(3, 9), MOVE_X, 1),
             (S.swap(2, 9), MOVE_X, 3), (S.g1(S.MAT_H, 5), REAL, 1), (S.cz(4, 9), DIAGONAL, 1),
             (S.Gate((5,), np.array([[0, -1j], [1j, 0]])), GENERAL, 1), (S.Gate((4, 9), mixed), TWO, 1),
             (S.Gate((4,), _unitary(rng, 1), 8, 8), CONTROLLED, 1)]
    for g, op, count in cases:
        p = Q.plan_passes([g], 12, Q.QS_C128, 4)
        assert p.n_passes == 1 and p.n_alone == 0 and p.ops[op] == count, (g.name, list(p.ops))
    p = Q.plan_passes([S.g1(S.MAT_H, 5), wide, S.g1(S.MAT_H, 5)], 15, Q.QS_C128, 4)
    assert (p.n_passes, p.n_alone) == (2, 1)
    assert p.circuit == p.program


def test_plan_rejects_bad_input(Q, S):
    g = [S.g1(S.MAT_H, 3)]
    for args in ((g, 3, Q.QS_C128, 4), (g, 0, Q.QS_C128, 4), (g, 35, Q.QS_C128, 4), (g, 5, 2, 4), (g, 5, Q.QS_C64, 7)):
        with pytest.raises(Q.QSError):
            Q.plan_passes(*args)


@pytest.mark.parametrize("scale", [1e-200, 1e-16, 1e-15, 1e-8, 1.0, 1e8, 1e200])
def test_matrices_that_are_no_rotation_stay_general(Q, S, scale):
    """Any 2 x 2 matrix is a gate; only one that is a real matrix between
    phases, to rounding of each of its entries, may be replaced by these."""
    rng = np.random.default_rng(4)
    z = scale * (rng.standard_normal((40, 2, 2)) + 1j * rng.standard_normal((40, 2, 2)))
    z[0] = scale * np.array([[1, 1e-10 * np.exp(0.3j)], [3e-10, 1]])     # weak: each entry counts
    p = Q.plan_passes([S.Gate((q % 12,), m) for q, m in enumerate(z)], 12, Q.QS_C128, 4)
    assert (p.ops[GENERAL], p.ops[REAL]) == (40, 0)


def test_scaled_unitaries_are_planned_alike(Q, S):
    rng = np.random.default_rng(5)
    us = [_unitary(rng, 1) for _ in range(60)] + [S.MAT_H]

    def ops(scale):
        return list(Q.plan_passes([S.Gate((q % 12,), scale * u) for q, u in enumerate(us)], 12, Q.QS_C128, 4).ops)

    assert ops(1.0)[REAL] > 50
    assert ops(2.0 ** -40) == ops(1.0) == ops(2.0 ** 40)
    # entries that are off by 1e-16 are rounding next to one, not next to 1e-8
    off = [1e-8 * u + 1e-16 * (rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2))) for u in us]
    p = Q.plan_passes([S.Gate((q % 12,), m) for q, m in enumerate(off)], 12, Q.QS_C128, 4)
    assert p.ops[REAL] == 0


def _layers(S, rng, n, qubits, count):
    gates = []
    while len(gates) < count:
        gates += S.random_layer_on(qubits, rng)
    return gates[:count]


def _long_circuit(S, name, count):
    rng = np.random.default_rng(8)
    if name == "layers":
        return 25, _layers(S, rng, 25, list(range(25)), count)
    if name == "idle qubits":                # some idle, one only under phases
        gates = _layers(S, rng, 25, list(range(20)), count)
        return 25, [S.cz(g.targets[0], 22) if i % 11 == 0 else g for i, g in enumerate(gates)]
    if name == "one tile":
        return 12, _layers(S, rng, 12, list(range(12)), count)
    if name == "four qubits":
        return 14, _layers(S, rng, 14, [3, 6, 9, 11], count)
    if name == "phases":
        return 25, [S.cr(int(a), int(b), 0.1) for a, b in (rng.permutation(25)[:2] for _ in range(count))]
    assert name == "alone"
    wide = S.Gate((1, 5, 7), _unitary(rng, 3))
    return 16, [wide if i % 2 else S.g1(S.MAT_H, i % 16) for i in range(count)]


@pytest.mark.parametrize("name", ["layers", "idle qubits", "one tile", "four qubits", "phases", "alone"])
def test_planning_time_grows_with_the_gates(Q, S, name):
    """Eight times the gates take eight times the planning, give or take; a
    planner that looks at the whole circuit for each pass takes 64 times."""
    import ctypes
    import time
    times = []
    for count in (5000, 40000):
        n, gates = _long_circuit(S, name, count)
        pc, plan, best = Q.PackedCircuit(gates), Q.PassPlan(), float("inf")
        for _ in range(3):
            t0 = time.process_time()
            assert Q.lib().qs_plan_passes(ctypes.byref(pc.c), n, Q.QS_C128, 4, ctypes.byref(plan)) == Q.QS_OK
            best = min(best, time.process_time() - t0)
        times.append(best)
    print("%s: %.1f ms, %.1f ms" % (name, times[0] * 1e3, times[1] * 1e3))
    assert times[1] < 20 * times[0]


@pytest.mark.parametrize("n", [14, 26])
def test_gates_alone_are_priced_by_all_their_qubits(Q, S, n):
    """A gate left alone runs as a block over targets and controls."""
    rng = np.random.default_rng(2)
    for dtype in (Q.QS_C64, Q.QS_C128):
        def cost(gate):
            return Q.plan_passes([S.g1(S.MAT_H, 5), gate], n, dtype, 4).cost

        controlled = cost(S.Gate((0, 1), _unitary(rng, 2), 0xf00, 0xf00))
        assert controlled == cost(S.Gate((0, 1, 8, 9, 10, 11), _unitary(rng, 6)))
        assert controlled > cost(S.Gate((0, 1), _unitary(rng, 2), 0x100, 0x100))


def test_price_of_moves(Q, S):
    """An X costs the kernel as many instructions as a general gate (a real
    rotation half of them), a SWAP one and a half times that."""
    n = 30
    base = Q.plan_passes([S.g1(S.MAT_H, 5)], n, Q.QS_C128, 4).cost
    y = np.array([[0, -1j], [1j, 0]])

    def extra(gate):
        return Q.plan_passes([S.g1(S.MAT_H, 5), gate], n, Q.QS_C128, 4).cost - base

    assert extra(S.g1(S.MAT_X, 9)) == pytest.approx(extra(S.Gate((9,), y)), rel=0.01)
    assert extra(S.swap(9, 11)) == pytest.approx(1.5 * extra(S.Gate((9,), y)), rel=0.01)


def test_no_exception_leaves_the_library():
    """Host memory that runs out while planning is QS_ENOMEM, not an abort."""
    import subprocess
    import sys
    code = """
import ctypes, resource
from paper_1604_06460_amd import qs as Q
from synth import circuits as S
pc, plan, nb = Q.PackedCircuit([S.g1(S.MAT_H, 5)] * 600000), Q.PassPlan(), ctypes.c_int()
out = [Q._ptr(__import__('numpy').zeros(600000 * k, dtype='int32')) for k in (1, 1, 6)]
size = int(open('/proc/self/statm').read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + (1 << 19), size + (1 << 19)))
print(Q.lib().qs_plan_passes(ctypes.byref(pc.c), 20, Q.QS_C128, 4, ctypes.byref(plan)),
      Q.lib().qs_plan_fusion(ctypes.byref(pc.c), 20, 4, ctypes.byref(nb), *out), flush=True)
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.split() == ["2", "2"], (r.returncode, r.stdout, r.stderr[-400:])


def test_one_call_counts_what_compiling_takes(Q, S):
    """An Ising step on 10 to 14 qubits: its blocks would run sooner than its
    passes, were they there; composing them takes longer than both."""
    for n in (10, 12, 14):
        for k in (4, 6):
            p = Q.plan_passes(S.tfim_trotter_step(n), n, Q.QS_C64, k)
            assert p.circuit == 1 and p.program == 0, (n, k, p.cost, p.block_cost)
