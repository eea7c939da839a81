"""Gates on several qubits and Kraus maps against the oracle, at the places
where their kernels divide: targets within a 128-byte line, above it and both,
controls on either side, registers of fewer amplitudes than a wave, and the
large-register step.

Tolerances: an output is a sum of D products of normalised data, each multiply
and add off by at most half a unit in the last place (e): the largest
amplitude is off by at most 2 (D + 1) e times the norm of the group, which is
at most 1; a density matrix goes through two such sums."""
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


def rounded(a, prec):
    return a if prec == 'C128' else a.astype(np.complex64).astype(np.complex128)


def sv_case(q, env, oracle, prec, n, targets, controls, seed):
    from workloads import Op, haar_unitary_k, random_state
    rng = np.random.default_rng(seed)
    u = haar_unitary_k(rng, len(targets))
    psi = rounded(random_state(n, seed), prec)
    want = psi.copy()
    oracle.apply_sv(want, n, Op('unitary', targets=tuple(targets), controls=tuple(controls), u=u))
    reg = q.Register(env, n, q.STATEVEC, getattr(q, prec))
    reg.set_amps(psi)
    reg.multi_qubit_unitary(targets, u, controls)
    got = reg.get_amps()
    reg.close()
    d = 1 << len(targets)
    err = float(np.max(np.abs(got - want)))
    assert err <= 2 * (d + 1) * EPS[prec], (n, targets, controls, err)
    outside = np.ones(1 << n, dtype=bool)
    for c in controls:
        outside &= ((np.arange(1 << n) >> c) & 1) == 1
    assert np.array_equal(got[~outside], psi[~outside])  # unselected amplitudes keep their bits


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('k', [1, 2, 3, 4, 5])
def test_targets_and_controls_on_both_sides_of_a_line(q, env, oracle_lib, prec, k):
    rng = np.random.default_rng(10 * k)
    cases = []
    for n in (k, k + 1, 6, 7, 10, 12):
        if n < k:
            continue
        cases.append((n, list(range(k)), []))                       # as low as they go
        cases.append((n, list(range(n - k, n))[::-1], []))          # as high, order reversed
        for _ in range(4):
            c = int(rng.integers(0, min(3, n - k) + 1))
            qs = [int(v) for v in rng.permutation(n)[:k + c]]
            cases.append((n, qs[:k], qs[k:]))
        if n >= k + 1:
            cases.append((n, list(range(1, k + 1)), [0]))
        if n == 12:
            for low in range(min(k, 4) + 1):                        # `low` targets within a line
                cases.append((n, list(range(low))[::-1] + [5 + j for j in range(k - low)], [11, 4]))
    for i, (n, t, c) in enumerate(cases):
        sv_case(q, env, oracle_lib, prec, n, t, c, 1000 * k + i)


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('targets,controls', [((0, 1), ()), ((20, 7), (2,)), ((2, 0, 1), ()), ((1, 9, 20), (4,)),
                                              ((0, 1, 2, 3), ()), ((5, 20, 9, 0), (1, 6)), ((4, 3, 2, 1, 0), ()),
                                              ((20, 8, 11, 14, 17), (0,))])
def test_large_register_steps(q, env, oracle_lib, prec, targets, controls):
    sv_case(q, env, oracle_lib, prec, 21, list(targets), list(controls), 77)


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('N', [1, 2, 3, 4, 5, 6])
def test_density_matrices(q, env, oracle_lib, prec, N):
    """Unitaries on 1..3 qubits (with and without controls), and Kraus maps on
    one and two, on every target of a random density matrix."""
    from workloads import Op, haar_unitary_k, random_kraus, random_state
    rng = np.random.default_rng(N)
    rho0 = rounded(sum(w * oracle_lib.dm_pure(N, random_state(N, 7 + i)) for i, w in enumerate((0.6, 0.4))), prec)
    ops = []
    for t in range(N):
        ops.append(Op('unitary', targets=(t,), u=haar_unitary_k(rng, 1)))
        ops.append(Op('kraus', targets=(t,), kraus=random_kraus(rng, 1, 3)))
        if N > 1:
            s = (t + 1) % N
            ops.append(Op('unitary', targets=(t, s), u=haar_unitary_k(rng, 2)))
            ops.append(Op('unitary', targets=(t,), controls=(s,), u=haar_unitary_k(rng, 1)))
            ops.append(Op('kraus', targets=(s, t), kraus=random_kraus(rng, 2, 4)))
        if N > 2:
            ops.append(Op('unitary', targets=(t, (t + 2) % N), controls=((t + 1) % N,), u=haar_unitary_k(rng, 2)))
            ops.append(Op('unitary', targets=(t, (t + 1) % N, (t + 2) % N), u=haar_unitary_k(rng, 3)))
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    for op in ops:
        want = rho0.copy()
        oracle_lib.apply_dm(want, N, op)
        reg.set_amps(rho0)
        reg.apply(op)
        err = float(np.max(np.abs(reg.get_amps() - want)))
        d = 1 << len(op.targets)
        assert err <= 4 * (d * d + 1) * EPS[prec], (op.kind, op.targets, op.controls, err)
    reg.close()
