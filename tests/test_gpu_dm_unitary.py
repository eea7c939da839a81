"""Uncontrolled unitaries on one and two qubits of a density matrix: parity at
the places where their kernels divide, and an error no larger than that of the
two passes of Eq. 2 done one after the other (U on the rows, conj(U) on the
columns, every multiply-add rounded once)."""
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


def mixed(N, seed):
    """A random full-rank rho as a matrix."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((1 << N, 1 << N)) + 1j * rng.standard_normal((1 << N, 1 << N))
    r = a @ a.conj().T
    return r / np.trace(r)


def rounded(a, prec):
    return a if prec == 'C128' else a.astype(np.complex64).astype(np.complex128)


def on_rows(u, x, N, targets, work=None):
    """u on the row index of x; with `work` (a real type), every multiply-add
    rounded to it."""
    k = len(targets)
    axes = [N - 1 - t for t in reversed(targets)]
    y = np.moveaxis(x.reshape([2] * N + [x.shape[1]]), axes, range(k))
    shape = y.shape
    y = y.reshape(1 << k, -1)
    if work is None:
        out = (u[:, :, None] * y[None]).sum(1)
    else:
        wide = np.longdouble
        yr, yi = y.real.astype(work), y.imag.astype(work)
        out = np.empty_like(y)
        for i in range(1 << k):
            re, im = np.zeros(y.shape[1], work), np.zeros(y.shape[1], work)
            for j in range(1 << k):
                a, b = wide(work(u[i, j].real)), wide(work(u[i, j].imag))
                re = (a * yr[j] + re).astype(work)
                re = (-b * yi[j] + re).astype(work)
                im = (a * yi[j] + im).astype(work)
                im = (b * yr[j] + im).astype(work)
            out[i] = re.astype(float) + 1j * im.astype(float)
    return np.moveaxis(out.reshape(shape), range(k), axes).reshape(x.shape)


def both_sides(u, x, N, targets, work=None):
    y = on_rows(u, x, N, targets, work)
    return on_rows(u.conj(), np.ascontiguousarray(y.T), N, targets, work).T


def run(q, env, prec, N, targets, u, x):
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    reg.set_amps(np.ascontiguousarray(x.T).reshape(-1))  # entry (row, column) at row + 2^N column
    reg.multi_qubit_unitary(targets, u)
    got = reg.get_amps()
    reg.close()
    return got.reshape(1 << N, 1 << N).T


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('N,targets', [(1, (0,)), (2, (0, 1)), (2, (1, 0)), (3, (2, 0)), (4, (3, 2)), (5, (0, 4)),
                                       (6, (1, 2)), (9, (0, 1)), (9, (8, 3)), (10, (2, 5)), (10, (9,)), (11, (4, 10))])
def test_parity(q, env, prec, N, targets):
    """Each entry is two sums of D products of entries of size 1 at most, each
    multiply and add off by at most half a unit in the last place."""
    from workloads import haar_unitary_k
    u = haar_unitary_k(np.random.default_rng(N), len(targets))
    x = rounded(mixed(N, N), prec)
    err = float(np.max(np.abs(run(q, env, prec, N, targets, u, x) - both_sides(u, x, N, targets))))
    assert err <= 4 * (2 ** len(targets) + 1) * EPS[prec], err


@pytest.mark.parametrize('prec', ['C128', 'C64'])
@pytest.mark.parametrize('k', [1, 2])
def test_no_further_off_than_two_passes(q, env, k, prec):
    """Mean relative error of 12 random cases of 4096 entries each against long
    double; those means differ by about a percent from one draw to another, so
    5% above the two passes is further off."""
    from workloads import haar_unitary_k
    N, work = 6, np.float64 if prec == 'C128' else np.float32
    ours, two = [], []
    for seed in range(12):
        rng = np.random.default_rng(seed)
        u = haar_unitary_k(rng, k)
        targets = [int(t) for t in rng.permutation(N)[:k]]
        x = rounded(mixed(N, seed), prec)
        want = both_sides(u.astype(np.clongdouble), x.astype(np.clongdouble), N, targets)
        norm = np.sqrt((np.abs(want) ** 2).sum())
        off = lambda y: float(np.sqrt((np.abs(y - want) ** 2).sum()) / norm)
        ours.append(off(run(q, env, prec, N, targets, u, x)))
        two.append(off(both_sides(u, x, N, targets, work)))
    assert np.mean(ours) <= 1.05 * np.mean(two), (np.mean(ours), np.mean(two))
