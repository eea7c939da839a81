"""Sums, overlaps, copies and measurements at the sizes where their kernels
divide: one block and several, one and several rows of bin sums, one and
several groups of ten qubits.

Tolerances: sums are compensated in double over values read exactly, so a few
units in the last place of a total of at most 1 (1e-14); probabilities of later
qubits are quotients of such sums (1e-12); a collapsed complex64 entry is
rounded to it once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope='module')
def q():
    import paper_1802_08032_amd as m
    return m


@pytest.fixture(scope='module')
def env(q):
    e = q.Env(0)
    yield e
    e.close()


def state(n, seed, prec):
    from workloads import random_state
    psi = random_state(n, seed)
    return psi if prec == 'C128' else psi.astype(np.complex64).astype(np.complex128)


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('n', [1, 4, 5, 12, 13, 14, 15, 20, 22])
def test_sums_overlaps_and_copies(q, env, prec, n):
    a, b = state(n, n, prec), state(n, n + 50, prec)
    ra, rb = (q.Register(env, n, q.STATEVEC, getattr(q, prec)) for _ in range(2))
    ra.set_amps(a)
    rb.set_amps(b)
    p = np.abs(a) ** 2
    assert abs(ra.calc_total_prob() - p.sum()) <= 1e-14
    for t in {0, n // 2, n - 1}:
        one = ((np.arange(1 << n) >> t) & 1) == 1
        for o in (0, 1):
            assert abs(ra.calc_prob_of_outcome(t, o) - p[one == bool(o)].sum()) <= 1e-14
    assert abs(ra.calc_inner_product(rb) - np.vdot(a, b)) <= 1e-14
    rb.clone_from(ra)
    assert np.array_equal(rb.get_amps(), a)
    ra.close()
    rb.close()


def measured(diag, n, draws):
    """Outcomes and probabilities of qubits 0..n-1 in turn."""
    w, outs, probs = np.asarray(diag, dtype=np.float64).copy(), [], []
    idx, g = np.arange(1 << n), 1.0
    for k in range(n):
        zero = ((idx >> k) & 1) == 0
        p = [w[zero].sum() * g, w[~zero].sum() * g]
        o = 0 if draws[k] < p[0] else 1
        w[zero if o else ~zero] = 0.0
        outs.append(o)
        probs.append(p[o])
        g /= p[o]
    return outs, probs, g


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('n', [1, 2, 9, 10, 11, 13, 14, 15, 20, 21])
def test_measure_all(q, env, prec, n):
    from workloads import measurement_draws
    a = state(n, 3 * n, prec)
    draws = measurement_draws(9, n, n)
    reg = q.Register(env, n, q.STATEVEC, getattr(q, prec))
    reg.set_amps(a)
    o, p = reg.measure_all(draws)
    wo, wp, g = measured(np.abs(a) ** 2, n, draws)
    assert list(o) == wo
    assert np.max(np.abs(np.array(p) - wp)) <= 1e-12
    pos = sum(b << k for k, b in enumerate(wo))
    got = reg.get_amps()
    assert abs(got[pos] - a[pos] * np.sqrt(g)) <= (1e-11 if prec == 'C128' else 1e-6)
    got[pos] = 0
    assert not got.any()
    reg.close()


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('N', [1, 4, 10, 11])
def test_measure_all_of_a_density_matrix(q, env, prec, N):
    from workloads import measurement_draws
    rho = sum(w * np.outer(v, v.conj()) for w, v in ((0.6, state(N, 5, prec)), (0.4, state(N, 6, prec))))
    if prec == 'C64':
        rho = rho.astype(np.complex64).astype(np.complex128)
    draws = measurement_draws(4, N, N)
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    reg.set_amps(rho.T.reshape(-1))  # entry j + 2^N k is rho[j][k]
    o, p = reg.measure_all(draws)
    wo, wp, _ = measured(np.real(np.diag(rho)), N, draws)
    assert list(o) == wo
    assert np.max(np.abs(np.array(p) - wp)) <= 1e-12
    pos = sum(b << k for k, b in enumerate(wo))
    got = reg.get_amps()
    assert abs(got[pos + (pos << N)] - 1.0) <= (1e-11 if prec == 'C128' else 1e-6)
    got[pos + (pos << N)] = 0
    assert not got.any()
    reg.close()


@pytest.mark.parametrize('n', [3, 12])
def test_measuring_a_null_state_is_an_error_and_leaves_it(q, env, n):
    reg = q.Register(env, n, q.STATEVEC, q.C128)
    reg.set_amps(np.zeros(1 << n, dtype=np.complex128))
    with pytest.raises(q.QStateError):
        reg.measure_all([0.5] * n)
    assert not reg.get_amps().any()
    reg.init_basis(1)
    o, p = reg.measure_all([0.5] * n)
    assert list(o) == [1] + [0] * (n - 1) and list(p) == [1.0] * n
    reg.close()
