"""Density-matrix gates, phases and channels on qubits within a 128-byte line
(complex128: qubits 0..2, complex64: 0..3), above it and on both sides,
against the oracle, in registers smaller than a wave up to the large-register
step.

Tolerances: an output is a sum of at most four products with coefficients of
magnitude at most 1 and entries of at most 1, with a handful of roundings of
half a unit in the last place (e) each: 16 e bounds it."""
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


def ops_on(N, qubits, rng):
    from workloads import Op, haar_unitary
    ops = []
    for t in qubits:
        others = [c for c in range(N) if c != t]
        ctrl_sets = [()] + [tuple(int(c) for c in rng.permutation(others)[:k]) for k in (1, 1, 2) if k <= len(others)]
        if 0 in others:
            ctrl_sets.append((0,))
        for cs in ctrl_sets:
            ops.append(Op('u', target=t, controls=cs, u=haar_unitary(rng)))
            ops.append(Op('x', target=t, controls=cs))
            ops.append(Op('phase', qubits=(t,) + cs, angle=float(rng.uniform(-3, 3))))
        ops += [Op('dephasing', target=t, p=0.3), Op('depolarising', target=t, p=0.4),
                Op('damping', target=t, p=0.2)]
    return ops


def check(q, env, oracle, prec, N, ops, seed):
    from workloads import random_state
    rho0 = sum(w * oracle.dm_pure(N, random_state(N, seed + i)) for i, w in enumerate((0.7, 0.3)))
    if prec == 'C64':
        rho0 = rho0.astype(np.complex64).astype(np.complex128)
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    for op in ops:
        want = rho0.copy()
        oracle.apply_dm(want, N, op)
        reg.set_amps(rho0)
        reg.apply(op)
        err = float(np.max(np.abs(reg.get_amps() - want)))
        assert err <= 16 * EPS[prec], (N, op, err)
    reg.close()


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('N', [1, 2, 3, 4, 5, 6, 7])
def test_every_target(q, env, oracle_lib, prec, N):
    rng = np.random.default_rng(N)
    check(q, env, oracle_lib, prec, N, ops_on(N, range(N), rng), 20 * N)


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('t', [0, 2, 3, 4, 10])
def test_large_register_steps(q, env, oracle_lib, prec, t):
    rng = np.random.default_rng(100 + t)
    check(q, env, oracle_lib, prec, 11, ops_on(11, [t], rng), 5)
