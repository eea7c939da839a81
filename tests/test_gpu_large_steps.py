"""Calls on registers that touch 512 MiB or more, where the streaming kernels
take another grid and an LDS reserve: one-qubit gates, NOTs, phases, groups of
two and three qubits, copies and collapses of state vectors, and gates, phases,
channels and collapses of density matrices, low and high qubits and controls.
Every amplitude is compared, on the device, with torch's complex128.

Tolerances: an entry is a sum of D products (two such sums for a density
matrix), each multiply and add off by at most half a unit in the last place of
values up to sqrt(D) times the largest entry."""
import math

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


def part(x, bits):
    """View of the entries of x whose index has the given values at some bits."""
    shape, index, high = [], [], x.numel().bit_length() - 1
    for b in sorted(bits, reverse=True):
        shape += [1 << (high - 1 - b), 2]
        index += [slice(None), bits[b]]
        high = b
    return x.view(*shape, 1 << high)[tuple(index)]


def group(x, u, targets, ones=()):
    """u on the targets' bits of x (matrix index bit j <-> targets[j]) where the
    bits of `ones` are 1."""
    d = 1 << len(targets)
    member = [part(x, {**{c: 1 for c in ones}, **{t: (r >> j) & 1 for j, t in enumerate(targets)}}) for r in range(d)]
    old = [m.clone() for m in member]
    for i in range(d):
        member[i].copy_(sum(complex(u[i, j]) * old[j] for j in range(d)))


def register(q, env, prec, n, kind, seed, scale=1.0):
    """A register of random entries, and the same entries in complex128."""
    import torch
    reg = q.Register(env, n, kind, getattr(q, prec))
    g = torch.Generator(device=reg.tensor.device).manual_seed(seed)
    torch.view_as_real(reg.tensor).normal_(std=scale, generator=g)
    return reg, reg.tensor.to(torch.complex128, copy=True)


def compare(reg, want, tol):
    """Largest error, in slices (the whole difference would be another copy)."""
    import torch
    torch.cuda.synchronize()
    err = max(float((a.to(torch.complex128) - b).abs().max()) for a, b in
              zip(reg.tensor.split(1 << 24), want.split(1 << 24)))
    assert err <= tol, (err, tol)


# one control halves what is touched: 1 GiB of state
SV = [('C128', 26), ('C64', 27)]


@pytest.mark.parametrize('prec,n', SV)
@pytest.mark.parametrize('targets,controls', [
    ((0,), ()), ((3,), (2,)), ((5,), (25,)), ((6,), ()), ((25,), (0,)), ((17,), (9,)),           # one qubit
    ((20, 7), ()), ((25, 8), (1,)), ((0, 11), ()), ((1, 0), (13,)), ((2, 9), (0,)),              # two
    ((8, 24, 15), ()), ((9, 4, 25), (0,)), ((0, 10, 20), (5,)), ((1, 2, 12), ()), ((2, 0, 1), (25,))])
def test_unitaries(q, env, prec, n, targets, controls):
    from workloads import haar_unitary_k
    u = haar_unitary_k(np.random.default_rng(len(targets)), len(targets))
    reg, want = register(q, env, prec, n, q.STATEVEC, 1)
    d = 1 << len(targets)
    tol = 2 * (d + 1) * EPS[prec] * math.sqrt(d) * float(want.abs().max())
    reg.multi_qubit_unitary(targets, u, controls)
    group(want, u, targets, controls)
    compare(reg, want, tol)
    reg.close()


@pytest.mark.parametrize('prec,n', SV)
def test_nots_and_phases(q, env, prec, n):
    reg, want = register(q, env, prec, n, q.STATEVEC, 2)
    big = float(want.abs().max())
    for controls, target in (((), 25), ((1,), 12), ((24,), 7), ((4,), 3)):
        reg.multi_controlled_not(controls, target)
        group(want, np.array([[0, 1], [1, 0]]), (target,), controls)
    compare(reg, want, 0.0)
    for qubits in ((0,), (25,), (2, 14), (1, 3), (3,)):
        reg.multi_controlled_phase(qubits, 0.7)
        part(want, {b: 1 for b in qubits}).mul_(complex(math.cos(0.7), math.sin(0.7)))
    compare(reg, want, 5 * 4 * EPS[prec] * big)
    reg.close()


@pytest.mark.parametrize('prec,n', SV)
def test_copies_and_collapses(q, env, prec, n):
    import torch
    scale = 2.0 ** (-(n + 1) / 2)  # norm 1 or nearly
    reg, want = register(q, env, prec, n, q.STATEVEC, 3, scale)
    other = q.Register(env, n, q.STATEVEC, getattr(q, prec))
    other.tensor.fill_(7.0)
    other.clone_from(reg)
    assert torch.equal(other.tensor, reg.tensor)
    reg.tensor.zero_()
    reg.init_pure_state(other)
    assert torch.equal(other.tensor, reg.tensor)
    other.close()
    for qubit, draw in ((1, 0.1), (25, 0.9)):
        outcome, p = reg.measure(qubit, draw)
        assert outcome == (0 if draw < 0.5 else 1)
        part(want, {qubit: 1 - outcome}).zero_()
        kept = float((part(want, {qubit: outcome}).abs() ** 2).sum())
        assert abs(kept - p) <= 1e-6 * p
        want *= 1.0 / math.sqrt(p)
    compare(reg, want, 6 * EPS[prec] * float(want.abs().max()))
    reg.close()


@pytest.mark.parametrize('prec,N', [('C128', 13), ('C64', 14)])
def test_density_matrices(q, env, prec, N):
    import torch
    from workloads import haar_unitary_k
    rng = np.random.default_rng(N)
    reg, want = register(q, env, prec, N, q.DENSITY, 4)

    def both(u, targets, controls=()):
        group(want, u, targets, controls)
        group(want, u.conj(), [t + N for t in targets], [c + N for c in controls])

    def check(sums, d):
        compare(reg, want, 2 * sums * (d + 1) * EPS[prec] * d * float(want.abs().max()))
        reg.tensor.copy_(want)  # the next call starts from equal entries
        want.copy_(reg.tensor)

    for t, controls in ((0, ()), (N - 1, (1,)), (2, (7,)), (5, ())):
        u = haar_unitary_k(rng, 1)
        reg.multi_controlled_unitary(controls, t, u)
        both(u, (t,), controls)
        check(2, 2)
    for targets in ((N - 1,), (1, 0), (8, 3)):
        u = haar_unitary_k(rng, len(targets))
        reg.multi_qubit_unitary(targets, u)
        both(u, targets)
        check(2, 1 << len(targets))
    for qubits in ((0, 1), (2, N - 1), (6,)):
        reg.multi_controlled_phase(qubits, 0.3)
        f = complex(math.cos(0.3), math.sin(0.3))
        part(want, {b: 1 for b in qubits}).mul_(f)
        part(want, {b + N: 1 for b in qubits}).mul_(f.conjugate())
        check(2, 2)
    for t in (1, N - 1):
        for name, p in (('dephasing', 0.2), ('depolarising', 0.3), ('damping', 0.4)):
            getattr(reg, 'mix_' + name)(t, p)
            r = [[part(want, {t: a, t + N: b}) for b in (0, 1)] for a in (0, 1)]
            d0, d1 = r[0][0].clone(), r[1][1].clone()
            f = {'dephasing': 1 - 2 * p, 'depolarising': 1 - 4 * p / 3, 'damping': math.sqrt(1 - p)}[name]
            r[0][1].mul_(f)
            r[1][0].mul_(f)
            if name == 'depolarising':
                r[0][0].copy_((1 - 2 * p / 3) * d0 + 2 * p / 3 * d1)
                r[1][1].copy_((1 - 2 * p / 3) * d1 + 2 * p / 3 * d0)
            elif name == 'damping':
                r[0][0].copy_(d0 + p * d1)
                r[1][1].copy_((1 - p) * d1)
            check(1, 2)
    # P(0) of a diagonal of positive entries, then the collapse
    diag = reg.tensor[:: (1 << N) + 1]
    diag.copy_(torch.full_like(diag, 2.0 ** -N))
    want.copy_(reg.tensor)
    outcome, p = reg.measure(2, 0.7)
    assert outcome == 1 and abs(p - 0.5) <= 1e-12
    part(want, {2: 0}).zero_()
    part(want, {2 + N: 0}).zero_()
    want *= 2.0
    check(1, 1)
    reg.close()
    torch.cuda.empty_cache()
