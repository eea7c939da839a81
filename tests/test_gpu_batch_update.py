"""Parameters of a captured batch: updates that change the form of gates.

A gate that is unitary to 1e-10 but not to 1e-14 is applied as a full matrix
instead of a core.  What follows it has the same ops all the same: two such
gates in different phases may trade forms, and any gate may change its own.

Tolerance: a gate computed with unit round-off e adds at most about 4 e to the
2-norm error of a normalised state, and a gate off by d from unitary changes
the core form by at most 1e-14."""
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


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('extra', [0, 2])
@pytest.mark.parametrize('tile', [9, 10, 12])
def test_gates_of_two_phases_trade_forms(q, env, oracle_lib, tile, extra, prec):
    from workloads import Op, haar_unitary
    rng = np.random.default_rng(tile)
    n = tile + extra
    exact = [haar_unitary(rng), haar_unitary(rng)]
    near = [u + 1e-12 * (rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2))) for u in exact]
    # the swapped gates on the highest qubit and on a low one, each followed by
    # a controlled gate on it; the qubits between fill the phases' registers
    ops, at = [], []
    for j, target in enumerate((n - 1, 3)):
        at.append(len(ops))
        ops.append(Op('u', target=target, u=exact[j]))
        ops.append(Op('u', target=target, controls=(target - 1,), u=haar_unitary(rng)))
        ops += [Op('u', target=t, u=haar_unitary(rng)) for t in (range(n - 2, 3, -1) if j == 0 else range(4))]
    want_of = []
    for forms in ((near, exact), (exact, near)):
        ops[at[0]].u, ops[at[1]].u = forms[0][0], forms[1][1]
        want_of.append(oracle_lib.run_sv(n, ops))
    for first in (0, 1):  # core -> full in the first phase, and full -> core
        ops[at[0]].u, ops[at[1]].u = (near, exact)[first][0], (exact, near)[first][1]
        reg = q.Register(env, n, q.STATEVEC, getattr(q, prec))
        circ = q.Circuit(ops)
        b = q.Batch([reg], [circ], tile)
        b.capture(init_zero=True)
        for step in (0, 1, 0):
            now = (first + step) % 2
            circ.set_unitary(at[0], (near, exact)[now][0])
            circ.set_unitary(at[1], (exact, near)[now][1])
            b.update()
            b.replay()
            err = float(np.max(np.abs(reg.get_amps() - want_of[now])))
            assert err <= 4 * EPS[prec] * len(ops) + 1e-13, (first, step, err)
        b.close()
        circ.close()
        reg.close()


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('tile', [9, 10, 12])
def test_one_gate_changes_its_form(q, env, oracle_lib, tile, prec):
    from workloads import Op, haar_unitary
    rng = np.random.default_rng(100 + tile)
    n = tile + 1
    ops = [Op('u', target=t, u=haar_unitary(rng)) for t in range(n)]
    ops += [Op('x', target=t, controls=(t - 1,)) for t in range(1, n)]
    ops += [Op('u', target=t, controls=(t - 1, 0) if t > 1 else (t - 1,), u=haar_unitary(rng)) for t in range(1, n)]
    reg = q.Register(env, n, q.STATEVEC, getattr(q, prec))
    circ = q.Circuit(ops)
    b = q.Batch([reg], [circ], tile)
    b.capture(init_zero=True)
    for k, off in ((n - 1, 1e-12), (0, 1e-11), (n - 1, 0.0), (n // 2, 1e-12), (0, 0.0)):
        ops[k].u = haar_unitary(rng) + off * (rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2)))
        circ.set_unitary(k, ops[k].u)
        b.update()
        b.replay()
        err = float(np.max(np.abs(reg.get_amps() - oracle_lib.run_sv(n, ops))))
        assert err <= 4 * EPS[prec] * len(ops) + 1e-13, (k, off, err)
    b.close()
    circ.close()
    reg.close()
