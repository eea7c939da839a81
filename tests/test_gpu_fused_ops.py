"""Passes of the generic fused kernel that run op by op: 4x4s on a register that
fills the chip, with every other kind of op among them, at every tile shape,
against the oracle.

Tolerance: an op computed with unit round-off e adds at most about 8 e to the
2-norm error of a normalised state (a 4x4 sums 8 products per component), so
the largest amplitude is off by at most 8 e per op."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = {'C128': 2.0 ** -53, 'C64': 2.0 ** -24}
N = 22  # four waves for each SIMD at 16 amplitudes a thread
SHAPES = [('C128', s) for s in ((6, 3), (7, 3), (8, 3), (8, 4), (9, 3), (9, 4), (10, 3))]
SHAPES += [('C64', s) for s in ((6, 3), (7, 3), (8, 3), (8, 4), (9, 3), (9, 4), (10, 3), (10, 4), (8, 5))]


@pytest.fixture(scope='module')
def q():
    import paper_1802_08032_amd as m
    return m


@pytest.fixture(scope='module')
def env(q):
    e = q.Env(0)
    yield e
    e.close()


def ops_of(n):
    """Between one 4x4 and the next: a core, a NOT behind it with and without
    controls, controlled general and diagonal gates, a phase and a sign, and a
    gate off from unitary by 1e-12, on random qubits."""
    from workloads import Op, haar_unitary, haar_unitary_k, rz
    rng = np.random.default_rng(n)
    ops = []
    for k in range(9):
        for _ in range(4):
            a, b = (int(v) for v in rng.permutation(n)[:2])
            ops.append(Op('unitary', targets=(a, b), u=haar_unitary_k(rng, 2)))
        p = [int(v) for v in rng.permutation(n)]
        ops += [Op('u', target=p[0], u=haar_unitary(rng)), Op('x', target=p[0], controls=(p[1],))]
        ops.append([Op('x', target=p[2]), Op('x', target=p[2], controls=(p[3], p[4])),
                    Op('u', target=p[2], controls=(p[3],), u=haar_unitary(rng))][k % 3])
        ops.append([Op('u', target=p[5], controls=(p[6], p[7]), u=haar_unitary(rng)),
                    Op('u', target=p[5], controls=(p[6],), u=rz(0.3 + k)),
                    Op('u', target=p[5], u=haar_unitary(rng) + 1e-12 * rng.standard_normal((2, 2)))][k % 3])
        ops.append(Op('phase', qubits=tuple(p[8:8 + 1 + k % 4]), angle=[0.7, math.pi, -math.pi][k % 3]))
    return ops


@pytest.fixture(scope='module')
def reference(oracle_lib):
    ops = ops_of(N)
    return ops, oracle_lib.run_sv(N, ops)


@pytest.mark.parametrize('prec,shape', SHAPES)
def test_state_vectors_of_every_shape(q, env, reference, prec, shape):
    ops, want = reference
    reg = q.Register(env, N, q.STATEVEC, getattr(q, prec))
    reg.init_zero()
    c = q.Circuit(ops)
    c.run_tiled(reg, sum(shape), shape[0])
    err = float(np.max(np.abs(reg.get_amps() - want)))
    c.close()
    reg.close()
    assert err <= 8 * EPS[prec] * len(ops), err


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('tile,tb', [(9, 6), (12, 8)])
def test_density_matrix(q, env, oracle_lib, tile, tb, prec):
    from workloads import Op
    M = N // 2
    ops = [Op('u', target=t, u=np.array([[0.6, 0.8], [0.8, -0.6]])) for t in (0, 5, M - 1)]
    for a in (0, 4, 5, 9):
        ops.append(Op('x', target=a + 1, controls=(a,)))
        for t in (a, a + 1):
            ops += [Op('depolarising', target=t, p=0.05), Op('damping', target=t, p=0.02)]
    want = oracle_lib.run_dm(M, ops)
    reg = q.Register(env, M, q.DENSITY, getattr(q, prec))
    reg.init_zero()
    c = q.Circuit(ops)
    c.run_tiled(reg, tile, tb)
    err = float(np.max(np.abs(reg.get_amps() - want)))
    c.close()
    reg.close()
    assert err <= 8 * EPS[prec] * 2 * len(ops), err


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('tile', [9, 10, 11, 12, 13, 14])
def test_batches(q, env, oracle_lib, prec, tile):
    """Registers run op by op and by records in one batch, before and after an
    update of the parameters."""
    from workloads import haar_unitary, param_circuit
    rng = np.random.default_rng(tile)
    sizes = [9, 10, 12, 13, 15]
    circuits = [ops_of(n) for n in sizes] + [param_circuit(n, 2, n) for n in sizes]
    sizes = sizes + sizes
    regs = [q.Register(env, n, q.STATEVEC, getattr(q, prec)) for n in sizes]
    circs = [q.Circuit(o) for o in circuits]
    b = q.Batch(regs, circs, tile)
    b.capture(init_zero=True)
    for update in (False, True):
        if update:
            for ops, c in zip(circuits, circs):
                for k, o in enumerate(ops):
                    if o.kind == 'u':  # gates off from unitary stay so
                        near = np.abs(o.u.conj().T @ o.u - np.eye(2)).max() > 1e-14
                        o.u = haar_unitary(rng) + near * 1e-12 * rng.standard_normal((2, 2))
                        c.set_unitary(k, o.u)
                    elif o.kind == 'phase':
                        o.angle = 0.1 * k
                        c.set_phase(k, o.angle)
            b.update()
        b.replay()
        for n, ops, reg in zip(sizes, circuits, regs):
            err = float(np.max(np.abs(reg.get_amps() - oracle_lib.run_sv(n, ops))))
            assert err <= 8 * EPS[prec] * len(ops), (update, n, err)
    b.close()
    for h in circs + regs:
        h.close()
