"""Phases of pi in the generic fused kernel, against long double.

exp(i pi) of the double next to pi is -1 + 1.2e-16 i.  Taken as -1, every CZ of
a circuit is off the same way, and the error grows with their number.

Tolerance: an op computed with unit round-off e adds at most 4 e to the 2-norm
error of a normalised state (8 multiply-adds per component pair, two roundings
each); the roundings of different ops are independent, so m ops add up to
4 e sqrt(m).  Left out, 1.2e-16 = 1.1 e of half the CZs' amplitudes add up to
about 0.25 e m, which is more from m = 256 on."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

E = 2.0 ** -53


@pytest.fixture(scope='module')
def q():
    import paper_1802_08032_amd as m
    return m


@pytest.fixture(scope='module')
def env(q):
    e = q.Env(0)
    yield e
    e.close()


def sign_ops(n, count, seed, angles):
    """`count` phases of pi on two or three qubits, a one-qubit gate after
    every tenth, and some of them twice in a row."""
    from workloads import Op, haar_unitary
    rng = np.random.default_rng(seed)
    ops = []
    while len(ops) < count:
        qubits = tuple(int(v) for v in rng.permutation(n)[:2 if rng.random() < 0.9 else 3])
        ops += [Op('phase', qubits=qubits, angle=float(rng.choice(angles)))] * (2 if rng.random() < 0.1 else 1)
        if rng.random() < 0.1:
            ops.append(Op('u', target=int(rng.integers(n)), u=haar_unitary(rng)))
    return ops


def exact(n, ops, psi):
    x = psi.astype(np.clongdouble)
    i = np.arange(1 << n)
    for op in ops:
        if op.kind == 'u':
            y = x.reshape(-1, 2, 1 << op.target)
            u = op.u.astype(np.clongdouble)
            x = np.stack([u[0, 0] * y[:, 0] + u[0, 1] * y[:, 1],
                          u[1, 0] * y[:, 0] + u[1, 1] * y[:, 1]], 1).reshape(-1)
            continue
        mask = sum(1 << b for b in op.qubits)
        a = np.longdouble(op.angle)
        x = np.where((i & mask) == mask, x * (np.cos(a) + 1j * np.sin(a)), x)
    return x


def off(got, want):
    return float(np.sqrt((np.abs(got - want) ** 2).sum() / (np.abs(want) ** 2).sum()))


@pytest.mark.parametrize('angles', [(math.pi,), (-math.pi,), (math.pi, math.pi, math.pi, -math.pi)])
@pytest.mark.parametrize('n,tile,tb', [(9, 9, 6), (12, 10, 7), (13, 12, 8)])
def test_state_vectors(q, env, n, tile, tb, angles):
    from workloads import random_state
    psi = random_state(n, tile)
    ops = sign_ops(n, 1500, tile, angles)
    reg = q.Register(env, n)
    reg.set_amps(psi)
    c = q.Circuit(ops)
    c.run_tiled(reg, tile, tb)
    err = off(reg.get_amps(), exact(n, ops, psi))
    c.close()
    reg.close()
    assert err <= 4 * E * math.sqrt(len(ops)), err


def test_batch(q, env):
    sizes = [9, 10, 12, 13]
    circuits = [sign_ops(n, 1500, 40 + n, (math.pi,)) for n in sizes]
    regs = [q.Register(env, n) for n in sizes]
    circs = [q.Circuit(o) for o in circuits]
    b = q.Batch(regs, circs, 10)
    b.run(init_zero=True)
    for n, ops, reg in zip(sizes, circuits, regs):
        zero = np.zeros(1 << n, dtype=complex)
        zero[0] = 1.0
        err = off(reg.get_amps(), exact(n, ops, zero))
        assert err <= 4 * E * math.sqrt(len(ops)), (n, err)
    b.close()
    for h in circs + regs:
        h.close()


def test_density_matrix(q, env):
    """The columns' phases are of -pi."""
    from workloads import random_state
    N = 6
    psi = random_state(N, 1)
    ops = sign_ops(N, 700, 3, (math.pi,))
    pure, rho = q.Register(env, N), q.Register(env, N, q.DENSITY)
    pure.set_amps(psi)
    rho.init_pure_state(pure)
    start = off(rho.get_amps(), np.multiply.outer(psi.conj(), psi.astype(np.clongdouble)).reshape(-1))
    c = q.Circuit(ops)
    c.run_tiled(rho, 10, 7)
    x = exact(N, ops, psi)
    err = off(rho.get_amps(), np.multiply.outer(x.conj(), x).reshape(-1))
    c.close()
    rho.close()
    pure.close()
    assert err <= start + 4 * E * math.sqrt(2 * len(ops)), err
