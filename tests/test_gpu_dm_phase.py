"""Phases of a density matrix on qubits within a 128-byte line and above it:
one pass over everything or one for the rows and one for the columns, at the
sizes and qubit sets where the choice turns.  Entries that keep their value are
the same bits; a turned one is one complex product with (cos, sin) rounded to
the register's type, so both parts are within 4 roundings of |factor| |entry|."""
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
# 5: everything in one pass; 11 and 12: on both sides of 32 MiB in either type
@pytest.mark.parametrize('N', [5, 11, 12])
def test_phase_qubit_sets(q, env, prec, N):
    import torch
    top = N - 1
    sets = [(0,), (0, 1, 2), (0, top), (2, top), (0, 1, top), (0, 1, 2, top), (3, top), (2, 3, 4), (0, 2, 3, 4),
            (1, 2, 3, 4), (top,), (3, 4)]
    reg = q.Register(env, N, q.DENSITY, getattr(q, prec))
    g = torch.Generator(device='cuda').manual_seed(N)
    index = torch.arange(1 << 2 * N, device='cuda')
    for k, qs in enumerate(sets):
        angle = 0.3 + 0.7 * k
        x = torch.randn(1 << 2 * N, dtype=torch.complex64 if prec == 'C64' else torch.complex128, device='cuda',
                        generator=g)
        reg.tensor.copy_(x)
        reg.multi_controlled_phase(list(qs), angle)
        env.sync()
        m = sum(1 << t for t in set(qs))
        row, col = (index & m) == m, (index >> N & m) == m
        got, x = reg.tensor, x.to(torch.complex128)
        turn = torch.complex(torch.tensor(np.cos(angle)), torch.tensor(np.sin(angle))).to(x)
        want = torch.where(row & ~col, x * turn, torch.where(col & ~row, x * turn.conj(), x))
        err = (torch.view_as_real(got.to(torch.complex128)) - torch.view_as_real(want)).abs().amax(1)
        assert bool((err <= 4 * EPS[prec] * x.abs()).all()), (qs, float(err.max()))
        same = row == col
        assert bool((got[same] == x[same]).all()), qs
    reg.close()
