"""A 4x4 superoperator on a qubit is applied together with the last one on it
when nothing in between touches the qubit.  Circuits in which every kind of op
stands between two of them, on the qubit and beside it, through the generic
tiles and the compiled passes, against the oracle.

Tolerance: entries are at most 1; each op multiplies by matrices of norm at
most 2 (a channel of strength below 0.3) with at most 33 roundings of e =
2^-53 (2^-24 in complex64) per entry, and the channels and unitaries do not
grow the sum of errors, so ops x 64 e."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = {'C128': 2.0 ** -53, 'C64': 2.0 ** -24}


@pytest.fixture(scope='module')
def q():
    import paper_1802_08032_amd as m
    return m


@pytest.fixture(scope='module')
def env(q):
    e = q.Env(0)
    yield e
    e.close()


def between(kind, a, b, c, rng):
    """An op of `kind` on the given qubits."""
    from workloads import Op, haar_unitary, haar_unitary_k
    return {'u': lambda: Op('u', target=a, u=haar_unitary(rng)),
            'cu': lambda: Op('u', target=a, controls=(b,), u=haar_unitary(rng)),
            'cx': lambda: Op('x', target=a, controls=(b,)),
            'ccx': lambda: Op('x', target=a, controls=(b, c)),
            'phase': lambda: Op('phase', qubits=(a,), angle=0.7),
            'cphase': lambda: Op('phase', qubits=(a, b), angle=-1.1),
            'u2': lambda: Op('unitary', targets=(a, b), u=haar_unitary_k(rng, 2))}[kind]()


def circuit(N, rng):
    from workloads import Op, haar_unitary
    ops = []
    for kind in ('u', 'cu', 'cx', 'ccx', 'phase', 'cphase', 'u2'):
        t = int(rng.integers(0, N))
        o = [int(v) for v in rng.permutation([k for k in range(N) if k != t])]
        for qubits in ((t, o[0], o[1]), (o[0], t, o[1]), (o[1], o[0], t), (o[0], o[1], o[2])):
            ops.append(Op('u', target=t, u=haar_unitary(rng)))
            ops.append(Op('damping', target=t, p=0.2))
            ops.append(between(kind, *qubits, rng))
            ops.append(Op('depolarising', target=t, p=0.1))
            ops.append(Op('dephasing', target=o[0], p=0.15))
    return ops


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('N,tile,tb', [(5, 9, 6), (5, 10, 7), (6, 12, 8)])
def test_merged_superoperators(q, env, oracle_lib, prec, N, tile, tb):
    from workloads import random_state
    rng = np.random.default_rng(10 * N + tile)
    ops = circuit(N, rng)
    rho = sum(w * oracle_lib.dm_pure(N, random_state(N, s)) for w, s in ((0.7, 3), (0.3, 4)))
    if prec == 'C64':
        rho = rho.astype(np.complex64).astype(np.complex128)
    want = rho.copy()
    for op in ops:
        oracle_lib.apply_dm(want, N, op)
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    circ = q.Circuit(ops)
    for run in (lambda: circ.run_tiled(reg, tile, tb), lambda: circ.run(reg, 0)):
        reg.set_amps(rho)
        run()
        err = float(np.max(np.abs(reg.get_amps() - want)))
        assert err <= 64 * len(ops) * EPS[prec], err
    circ.close()
    reg.close()
