"""Performance cases of the engine: what a program that simulates circuits has
it do, through the public calls of ``paper_1802_08032_amd``.

Seven families, each over register sizes from the smallest calls (launches and
latency count) to registers of many GiB (memory bandwidth or arithmetic
counts), in complex128 and complex64:

* ``gates``    -- a state vector driven gate by gate (an interactive program,
  or one whose next gate depends on a result): named gates, controlled and
  multi-controlled unitaries, NOTs and phases;
* ``blocks``   -- dense unitaries on 1..5 qubits with 0..2 controls;
* ``noise``    -- a density matrix driven call by call: gates, phases, the
  three named channels and general Kraus maps on one and two qubits;
* ``fused``    -- a recorded circuit run by the generic fused kernel from
  |0..0> (what the serving loop does with each request), then one read;
* ``compiled`` -- a recorded circuit run as run-time compiled passes from a
  basis state, with the fused readouts on state vectors (the benchmark's
  step);
* ``batch``    -- many small registers replayed from one captured graph, then
  a read of each (a variational sweep);
* ``readout``  -- probabilities, overlaps and measurements of a prepared
  state, as a sampling program does between shots.

States are random normalised vectors and random mixed density matrices; a
case's circuit is fixed by its ``circuit`` number, its inputs by the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1802_08032_amd as q
from workloads import (SQRT_X, SQRT_Y, H, haar_unitary, haar_unitary_k, layered_circuit, measurement_draws,
                       noisy_circuit, param_circuit, random_kraus, ry, rz)

DEVICE = 'cuda:0'
# tile shapes of compiled passes as the benchmark runs them: tile qubits,
# thread bits, contiguous qubits
TILES = {'c128': (12, 8, 4), 'c64': (14, 10, 5)}
FUSION = 12          # tile qubits of the generic fused kernel (the serving loop's)
BATCH_TILE = 10      # tile qubits of a batch (what the batch autotuner picks)


def listed():
    return [
        # one small register driven gate by gate: all launch latency
        {'name': 'gates_11q_c128', 'family': 'gates', 'n': 11, 'prec': 'c128', 'ops': 24, 'circuit': 1},
        # a register of the size of the on-chip caches
        {'name': 'gates_22q_c64', 'family': 'gates', 'n': 22, 'prec': 'c64', 'ops': 24, 'circuit': 2},
        # a register far beyond the caches: 8 GiB
        {'name': 'gates_29q_c128', 'family': 'gates', 'n': 29, 'prec': 'c128', 'ops': 24, 'circuit': 3},
        # dense blocks, two of each width
        {'name': 'blocks_25q_c128', 'family': 'blocks', 'n': 25, 'prec': 'c128', 'ops': 10, 'circuit': 4},
        # noise on a small and on a large density matrix (512 MiB)
        {'name': 'noise_6q_c128', 'family': 'noise', 'n': 6, 'prec': 'c128', 'ops': 18, 'circuit': 5},
        {'name': 'noise_13q_c64', 'family': 'noise', 'n': 13, 'prec': 'c64', 'ops': 18, 'circuit': 6},
        # served requests: a state vector and a noisy density matrix
        {'name': 'fused_17q_c128', 'family': 'fused', 'n': 17, 'prec': 'c128', 'dm': False, 'depth': 10, 'circuit': 7},
        {'name': 'fused_9q_dm_c64', 'family': 'fused', 'n': 9, 'prec': 'c64', 'dm': True, 'depth': 6, 'circuit': 8},
        # the benchmark's step at 16 GiB
        {'name': 'compiled_30q_c128', 'family': 'compiled', 'n': 30, 'prec': 'c128', 'dm': False, 'depth': 10,
         'circuit': 9},
        # the benchmark's batch of 10..20 qubit registers, as many as a state returns whole
        {'name': 'batch_60_c64', 'family': 'batch', 'count': 60, 'lo': 10, 'hi': 20, 'prec': 'c64', 'depth': 16,
         'circuit': 10},
        # reads of a small state (latency) and of a 4 GiB one
        {'name': 'readout_13q_c64', 'family': 'readout', 'n': 13, 'prec': 'c64', 'dm': False, 'circuit': 11},
        {'name': 'readout_28q_c128', 'family': 'readout', 'n': 28, 'prec': 'c128', 'dm': False, 'circuit': 12},
    ]


def draw(rng: random.Random):
    family = rng.choice(['gates', 'gates', 'blocks', 'blocks', 'noise', 'noise', 'fused', 'fused', 'compiled', 'batch',
                         'readout', 'readout'])
    c = {'family': family, 'prec': rng.choice(['c128', 'c64']), 'circuit': rng.randrange(1000, 1 << 20)}
    # sizes are exponents: uniform qubit counts spread work over its logarithm
    if family == 'gates':
        c.update(n=rng.randint(8, 29), ops=rng.randint(8, 24))
    elif family == 'blocks':
        c.update(n=rng.randint(10, 26), ops=rng.randint(5, 10))
    elif family == 'noise':
        c.update(n=rng.randint(4, 13), ops=rng.randint(9, 18))
    elif family == 'fused':
        dm = rng.random() < 0.4
        c.update(dm=dm, n=rng.randint(6, 11) if dm else rng.randint(12, 25), depth=rng.randint(5, 16))
    elif family == 'compiled':
        dm = rng.random() < 0.25
        c.update(dm=dm, n=rng.randint(8, 13) if dm else rng.randint(16, 29), depth=rng.randint(4, 10))
    elif family == 'batch':
        lo = rng.randint(9, 14)
        c.update(count=rng.randint(8, 60), lo=lo, hi=rng.randint(lo + 1, 20), depth=rng.randint(4, 16))
    else:
        dm = rng.random() < 0.3
        c.update(dm=dm, n=rng.randint(4, 13) if dm else rng.randint(8, 29))
    return c


# --- the calls of a case ------------------------------------------------------


def _gate_calls(case):
    """Register calls of a `gates` case: (method, arguments)."""
    rng = np.random.default_rng(case['circuit'])
    n, calls = case['n'], []
    kinds = ['hadamard', 'rotate_x', 'rotate_y', 'rotate_z', 't_gate', 'sqrt_x', 'sqrt_y', 'cnot', 'cnot', 'cz',
             'unitary', 'unitary', 'controlled_unitary', 'multi_controlled_unitary', 'multi_controlled_not',
             'multi_controlled_phase']
    order = [kinds[i % len(kinds)] for i in range(case['ops'])]
    rng.shuffle(order)
    for kind in order:
        a, b, c, d = (int(v) for v in rng.choice(n, size=4, replace=False))
        theta = float(rng.uniform(0.0, 2.0 * math.pi))
        calls.append((kind, {
            'hadamard': (a,), 'rotate_x': (a, theta), 'rotate_y': (a, theta), 'rotate_z': (a, theta), 't_gate': (a,),
            'sqrt_x': (a,), 'sqrt_y': (a,), 'cnot': (a, b), 'cz': (a, b), 'unitary': (a, haar_unitary(rng)),
            'controlled_unitary': (a, b, haar_unitary(rng)),
            'multi_controlled_unitary': ([a, b], c, haar_unitary(rng)), 'multi_controlled_not': ([a, b], c),
            'multi_controlled_phase': ([a, b, c, d], theta)}[kind]))
    return calls


def _block_calls(case):
    """(targets, matrix, controls) of a `blocks` case."""
    rng = np.random.default_rng(case['circuit'])
    calls = []
    for i in range(case['ops']):
        k, nc = i % 5 + 1, int(rng.integers(0, 3))
        qs = [int(v) for v in rng.choice(case['n'], size=k + nc, replace=False)]
        calls.append((qs[:k], haar_unitary_k(rng, k), qs[k:]))
    return calls


def _noise_calls(case):
    """Register calls of a `noise` case: (method, arguments)."""
    rng = np.random.default_rng(case['circuit'])
    calls = []
    kinds = ['unitary', 'mix_depolarising', 'cnot', 'mix_dephasing', 'mix_damping', 'cz', 'mix_kraus', 'two_qubit_unitary',
             'mix_two_qubit_kraus']
    for i in range(case['ops']):
        a, b = (int(v) for v in rng.choice(case['n'], size=2, replace=False))
        p = float(rng.uniform(1e-3, 0.1))
        kind = kinds[i % len(kinds)]
        calls.append((kind, {
            'unitary': (a, haar_unitary(rng)), 'mix_depolarising': (a, p), 'mix_dephasing': (a, p),
            'mix_damping': (a, p), 'cnot': (a, b), 'cz': (a, b),
            'mix_kraus': (a, np.stack(random_kraus(rng, 1, 3))), 'two_qubit_unitary': (a, b, haar_unitary_k(rng, 2)),
            'mix_two_qubit_kraus': (a, b, np.stack(random_kraus(rng, 2, 4)))}[kind]))
    return calls


def _circuit(case, seed=None):
    """Gate list of a recorded circuit; `seed` gives other values of the same structure."""
    s = case['circuit'] if seed is None else seed
    if case['dm']:
        return noisy_circuit(case['n'], case['depth'], s)
    return layered_circuit(case['n'], case['depth'], s, mcphase=case['family'] == 'compiled')


def _batch_circuits(case, seed):
    rng = np.random.default_rng(case['circuit'])
    sizes = [int(v) for v in rng.integers(case['lo'], case['hi'] + 1, case['count'])]
    return sizes, [param_circuit(n, case['depth'], 1000 * seed + i) for i, n in enumerate(sizes)]


def _basis(case, seed):
    return random.Random(seed).randrange(1 << case['n'])


def _draws(case, seed):
    return measurement_draws(seed, case['circuit'], case['n'] + 1)


# --- inputs -------------------------------------------------------------------


def _random_vector(n, prec, seed, device=DEVICE):
    """A normalised Gaussian vector of 2^n amplitudes."""
    g = torch.Generator(device=device).manual_seed(seed)
    v = torch.empty(1 << n, dtype=torch.complex128 if prec == 'c128' else torch.complex64, device=device)
    r = torch.view_as_real(v)
    r.normal_(generator=g)
    r.mul_(1.0 / torch.linalg.vector_norm(r).item())
    return v


def _random_density(N, prec, seed, device=DEVICE):
    """A mixed state of rank 4, entry rho[j][k] at j + 2^N k."""
    p = torch.stack([_random_vector(N, 'c128', 4 * seed + i, device) for i in range(4)])
    w = torch.tensor([[0.4], [0.3], [0.2], [0.1]], dtype=torch.complex128, device=device)
    m = (w * p.conj()).T.contiguous() @ p  # [k][j]
    return m.reshape(-1).to(torch.complex128 if prec == 'c128' else torch.complex64)


def _input(case, seed):
    dm = case['family'] == 'noise' or case.get('dm', False)
    return (_random_density if dm else _random_vector)(case['n'], case['prec'], seed)


_env = None


def _environment():
    global _env
    if _env is None:
        _env = q.Env(0)
    return _env


class _State(dict):
    """What the program holds; its registers and handles are closed with it."""

    def own(self, *handles):
        self.setdefault('_handles', []).extend(handles)
        return handles[0] if len(handles) == 1 else handles

    def __del__(self):
        for h in reversed(self.get('_handles', [])):
            h.close()


def prepare(case, seed):
    env = _environment()
    prec = q.C128 if case['prec'] == 'c128' else q.C64
    s = _State(family=case['family'], case=case)

    def register(n, dm=False):
        return s.own(q.Register(env, n, q.DENSITY if dm else q.STATEVEC, prec))

    family = case['family']
    if family in ('gates', 'blocks', 'noise'):
        s['reg'] = register(case['n'], family == 'noise')
        s['reg'].tensor.copy_(_input(case, seed))
        s['calls'] = {'gates': _gate_calls, 'blocks': _block_calls, 'noise': _noise_calls}[family](case)
    elif family == 'fused':
        s['reg'] = register(case['n'], case['dm'])
        s['circuit'] = s.own(q.Circuit(_circuit(case, seed)))
    elif family == 'compiled':
        s['reg'] = register(case['n'], case['dm'])
        s['circuit'] = s.own(q.Circuit(_circuit(case)))
        s['basis'] = _basis(case, seed)
    elif family == 'batch':
        sizes, ops = _batch_circuits(case, seed)
        s['regs'] = [register(n) for n in sizes]
        circuits = [s.own(q.Circuit(o)) for o in ops]
        s['batch'] = s.own(q.Batch(s['regs'], circuits, BATCH_TILE))
        s['batch'].capture(init_zero=True)
    else:
        s['reg'], s['work'] = register(case['n'], case['dm']), register(case['n'], case['dm'])
        s['reg'].tensor.copy_(_input(case, seed))
        s['pure'] = register(case['n'])
        s['pure'].tensor.copy_(_random_vector(case['n'], case['prec'], seed + 500))
        s['draws'] = _draws(case, seed)
    return s


def run(s):
    family, case = s['family'], s['case']
    if family in ('gates', 'noise'):
        reg = s['reg']
        for name, args in s['calls']:
            getattr(reg, name)(*args)
        return {'state': reg.tensor}
    if family == 'blocks':
        reg = s['reg']
        for targets, u, controls in s['calls']:
            reg.multi_qubit_unitary(targets, u, controls)
        return {'state': reg.tensor}
    if family == 'fused':
        reg = s['reg']
        reg.init_zero()
        if case['dm']:
            s['circuit'].run_tiled(reg, FUSION, 8)
        else:
            s['circuit'].run(reg, FUSION)
        return {'state': reg.tensor, 'p': reg.calc_prob_of_outcome(case['n'] - 1, 0)}
    if family == 'compiled':
        reg, (tile, threads, contig) = s['reg'], TILES[case['prec']]
        if case['dm']:
            s['circuit'].run_compiled(reg, tile, threads, 0, contig, init_basis=s['basis'])
            return {'state': reg.tensor}
        _, probs = s['circuit'].run_compiled_probs(reg, tile, threads, 0, contig, init_basis=s['basis'])
        return {'state': reg.tensor, 'probs': probs}
    if family == 'batch':
        s['batch'].replay()
        p0, total = s['batch'].probs(0)
        return {'states': [r.tensor for r in s['regs']], 'p0': p0, 'total': total}
    reg, work, n = s['reg'], s['work'], case['n']
    out = {'total': reg.calc_total_prob(), 'p_high': reg.calc_prob_of_outcome(n - 1, 1),
           'p_low': reg.calc_prob_of_outcome(0, 0), 'fidelity': reg.calc_fidelity(s['pure'])}
    if case['dm']:
        out['purity'] = reg.calc_purity()
    else:
        z = s['pure'].calc_inner_product(reg)
        out['overlap'] = np.array([z.real, z.imag])
    work.clone_from(reg)
    o, p = work.measure(n // 2, s['draws'][n])
    outcomes, probs = work.measure_all(s['draws'][:n])
    out.update(first=np.array([o]), first_p=p, outcomes=np.array(outcomes), probs=np.array(probs), state=work.tensor)
    return out


# --- what a pass cannot do without --------------------------------------------


def _elem(case):
    return 16 if case['prec'] == 'c128' else 8


def _named(kind, args):
    """(targets, matrix, controls) of a named gate call; a phase is a 2x2 diagonal with controls."""
    def phase(a):
        return np.diag([1.0, np.exp(1j * a)])

    def rx(a):
        c, s = math.cos(a / 2), math.sin(a / 2)
        return np.array([[c, -1j * s], [-1j * s, c]])

    x = np.array([[0, 1], [1, 0]], dtype=complex)
    return {
        'hadamard': lambda t: ([t], H, []), 'rotate_x': lambda t, a: ([t], rx(a), []),
        'rotate_y': lambda t, a: ([t], ry(a), []), 'rotate_z': lambda t, a: ([t], rz(a), []),
        't_gate': lambda t: ([t], phase(math.pi / 4), []), 'sqrt_x': lambda t: ([t], SQRT_X, []),
        'sqrt_y': lambda t: ([t], SQRT_Y, []), 'cnot': lambda c, t: ([t], x, [c]),
        'cz': lambda a, b: ([b], phase(math.pi), [a]), 'unitary': lambda t, u: ([t], u, []),
        'controlled_unitary': lambda c, t, u: ([t], u, [c]),
        'multi_controlled_unitary': lambda c, t, u: ([t], u, list(c)),
        'multi_controlled_not': lambda c, t: ([t], x, list(c)),
        'multi_controlled_phase': lambda qs, a: ([qs[-1]], phase(a), list(qs[:-1])),
        'two_qubit_unitary': lambda a, b, u: ([a, b], u, []),
    }[kind](*args)


_PHASES = {'t_gate': 1, 'cz': 2, 'multi_controlled_phase': 4}


def _op_flops(o, nbits):
    """14 real operations per amplitude of a dense 2x2 gate, 6 of a phase, none of a NOT."""
    if o.kind == 'u':
        return 14.0 * 2.0 ** (nbits - len(o.controls))
    return 6.0 * 2.0 ** (nbits - len(o.qubits)) if o.kind == 'phase' else 0.0


def work(case):
    family, e = case['family'], _elem(case)
    if family == 'batch':
        sizes, circuits = _batch_circuits(case, 0)
        return {'bytes': float(sum(2 * e * 2 ** n for n in sizes)),
                'flops': sum(_op_flops(o, n) for n, ops in zip(sizes, circuits) for o in ops)}
    dm = family == 'noise' or case.get('dm', False)
    nbits = case['n'] * (2 if dm else 1)
    amps = float(2 ** nbits)
    if family == 'gates':
        b = f = 0.0
        for kind, args in _gate_calls(case):
            _, u, controls = _named(kind, args)
            part = amps / 2 ** (_PHASES[kind] if kind in _PHASES else len(controls))
            b += 2 * e * part
            f += part * (6 if kind in _PHASES else 0 if kind in ('cnot', 'multi_controlled_not') else 14)
        return {'bytes': b, 'flops': f}
    if family == 'blocks':
        parts = [(amps / 2 ** len(c), 2 ** len(t)) for t, _, c in _block_calls(case)]
        return {'bytes': sum(2 * e * p for p, _ in parts), 'flops': sum(8.0 * d * p for p, d in parts)}
    if family == 'noise':
        # share of the entries a call changes, and its operations per changed entry
        cost = {'unitary': (1, 28), 'cnot': (0.75, 0), 'cz': (0.375, 1), 'mix_depolarising': (1, 4),
                'mix_dephasing': (0.5, 2), 'mix_damping': (1, 3), 'mix_kraus': (1, 32), 'two_qubit_unitary': (1, 64),
                'mix_two_qubit_kraus': (1, 128)}
        calls = [cost[kind] for kind, _ in _noise_calls(case)]
        return {'bytes': sum(2 * e * amps * s for s, _ in calls), 'flops': sum(f * amps * s for s, f in calls)}
    if family in ('fused', 'compiled'):
        flops = 0.0
        for o in _circuit(case):
            # on a density matrix a gate acts on rows and columns; a channel costs about 4 per entry
            flops += _op_flops(o, nbits) * (2 if dm else 1) if o.kind in ('u', 'x', 'phase') else 4 * amps
        reads = e * (2 ** case['n'] if dm else amps / 2) if family == 'fused' else 0.0  # the one probability
        return {'bytes': e * amps + reads, 'flops': flops}
    # readout, in registers read and written: total, two outcomes, overlaps, clone, measurement (sums, then
    # the kept part read and everything written), measure-all (sums, then everything written)
    diag = float(2 ** case['n']) if dm else amps
    sums = (5 if dm else 4.5) * diag
    overlaps = 2 if dm else 4
    moved = sums + (overlaps + 2 + (1.25 if dm else 1.5) + 1) * amps
    return {'bytes': e * moved, 'flops': 4.0 * (sums + overlaps * amps)}


# --- the same in 64 bits --------------------------------------------------------


def _apply(v, nbits, targets, m, controls=()):
    """v (complex128, in place) <- m on `targets` (matrix index bit j is targets[j]) where the controls are 1."""
    k, pos = len(targets), sorted(list(targets) + list(controls), reverse=True)
    shape, top = [], nbits
    for p in pos:
        shape += [1 << (top - 1 - p), 2]
        top = p
    x = v.view(shape + [1 << top])
    axis = {p: 2 * i + 1 for i, p in enumerate(pos)}
    index = [slice(None)] * x.dim()
    for c in controls:
        index[axis[c]] = slice(1, 2)
    x = x[tuple(index)]
    x = x.movedim([axis[t] for t in reversed(targets)], list(range(k)))  # leading axes spell the matrix index
    d = 1 << k
    m = torch.as_tensor(np.asarray(m, dtype=np.complex128)).to(v.device)
    if k == 1:
        a, b = x[0], x[1]
        mh = m.cpu().numpy()
        if mh[0, 1] == 0 and mh[1, 0] == 0:
            for i in range(2):
                if mh[i, i] != 1:
                    x[i] *= complex(mh[i, i])
            return
        na = a * complex(mh[0, 0]) + b * complex(mh[0, 1])
        x[1] = a * complex(mh[1, 0]) + b * complex(mh[1, 1])
        x[0] = na
        return
    y = m @ x.reshape(d, -1)
    x.copy_(y.view(x.shape))


def _channel_kraus(kind, p):
    i2, z = np.eye(2, dtype=complex), np.diag([1, -1]).astype(complex)
    x, y = np.array([[0, 1], [1, 0]], dtype=complex), np.array([[0, -1j], [1j, 0]])
    if kind == 'dephasing':
        return [math.sqrt(1 - p) * i2, math.sqrt(p) * z]
    if kind == 'depolarising':
        return [math.sqrt(1 - p) * i2] + [math.sqrt(p / 3) * g for g in (x, y, z)]
    return [np.diag([1, math.sqrt(1 - p)]).astype(complex), np.array([[0, math.sqrt(p)], [0, 0]], dtype=complex)]


def _apply_dm(v, N, targets, m, controls=()):
    """Rows by m, columns by conj(m)."""
    _apply(v, 2 * N, targets, m, controls)
    _apply(v, 2 * N, [t + N for t in targets], np.conj(m), [c + N for c in controls])


def _apply_kraus(v, N, targets, ops):
    s = sum(np.kron(np.conj(k), k) for k in ops)  # columns are the high index bits
    _apply(v, 2 * N, list(targets) + [t + N for t in targets], s)


def _op_matrix(o):
    """(targets, matrix, controls) of a recorded gate."""
    if o.kind == 'u':
        return [o.target], o.u, list(o.controls)
    if o.kind == 'x':
        return [o.target], np.array([[0, 1], [1, 0]]), list(o.controls)
    return [o.qubits[-1]], np.diag([1.0, np.exp(1j * o.angle)]), list(o.qubits[:-1])


def _run_exact(v, n, ops, dm):
    for o in ops:
        if o.kind in ('u', 'x', 'phase'):
            (_apply_dm if dm else _apply)(v, n, *_op_matrix(o))
        else:
            _apply_kraus(v, n, [o.target], _channel_kraus(o.kind, o.p))


def _weights(v, n, dm):
    return v.view(1 << n, 1 << n).diagonal().real.clone() if dm else torch.view_as_real(v).square().sum(-1)


def _p(w, qubit, outcome):
    return w.view(-1, 2, 1 << qubit)[:, outcome].sum().item()


def exact(case, seed):
    family, n = case['family'], case.get('n')
    if family == 'batch':
        states, p0, total = [], [], []
        for size, ops in zip(*_batch_circuits(case, seed)):
            v = torch.zeros(1 << size, dtype=torch.complex128, device=DEVICE)
            v[0] = 1
            _run_exact(v, size, ops, False)
            w = _weights(v, size, False)
            states.append(v)
            p0.append(_p(w, 0, 0))
            total.append(w.sum().item())
        return {'states': states, 'p0': np.array(p0), 'total': np.array(total)}
    dm = family == 'noise' or case.get('dm', False)
    nbits = 2 * n if dm else n
    if family in ('gates', 'blocks', 'noise'):
        v = _input(case, seed).to(torch.complex128)
        if family == 'gates':
            for kind, args in _gate_calls(case):
                _apply(v, n, *_named(kind, args))
        elif family == 'blocks':
            for targets, u, controls in _block_calls(case):
                _apply(v, n, targets, u, controls)
        else:
            for kind, args in _noise_calls(case):
                if kind == 'mix_kraus':
                    _apply_kraus(v, n, [args[0]], args[1])
                elif kind == 'mix_two_qubit_kraus':
                    _apply_kraus(v, n, list(args[:2]), args[2])
                elif kind.startswith('mix_'):
                    _apply_kraus(v, n, [args[0]], _channel_kraus(kind[4:], args[1]))
                else:
                    _apply_dm(v, n, *_named(kind, args))
        return {'state': v}
    if family in ('fused', 'compiled'):
        basis = _basis(case, seed) if family == 'compiled' else 0
        v = torch.zeros(1 << nbits, dtype=torch.complex128, device=DEVICE)
        v[basis + (basis << n) if dm else basis] = 1
        _run_exact(v, n, _circuit(case, None if family == 'compiled' else seed), dm)
        w = _weights(v, n, dm)
        if family == 'fused':
            return {'state': v, 'p': _p(w, n - 1, 0)}
        if dm:
            return {'state': v}
        return {'state': v, 'probs': np.array([w.sum().item()] + [_p(w, k, 0) for k in range(n)])}
    # readout
    v = _input(case, seed).to(torch.complex128)
    pure = _random_vector(n, case['prec'], seed + 500).to(torch.complex128)
    w = _weights(v, n, dm)
    out = {'total': w.sum().item(), 'p_high': _p(w, n - 1, 1), 'p_low': _p(w, 0, 0)}
    if dm:
        rho = v.view(1 << n, 1 << n)  # [k][j]
        out['fidelity'] = torch.dot(pure, rho @ pure.conj()).real.item()
        out['purity'] = torch.view_as_real(v).square().sum().item()
    else:
        z = torch.sum(pure.conj() * v)
        out['fidelity'] = z.real.item() ** 2 + z.imag.item() ** 2
        out['overlap'] = np.array([z.real.item(), z.imag.item()])
    draws = _draws(case, seed)
    p0 = _p(w, n // 2, 0)
    o = 0 if draws[n] < min(max(p0, 0.0), 1.0) else 1
    p = _p(w, n // 2, o)
    w = w.view(-1, 2, 1 << (n // 2)).clone()
    w[:, 1 - o] = 0
    w = w.reshape(-1) / p
    g, index, outcomes, probs = 1.0 / p, 0, [], []
    for k in range(n):
        pair = w.view(-1, 2)
        p0 = pair[:, 0].sum().item()
        b = 0 if draws[k] < min(max(p0, 0.0), 1.0) else 1
        pb = p0 if b == 0 else pair[:, 1].sum().item()
        w = pair[:, b] / pb
        outcomes.append(b)
        probs.append(pb)
        index |= b << k
        g /= pb
    state = torch.zeros_like(v)
    at = index + (index << n) if dm else index
    state[at] = v[at] * (g if dm else math.sqrt(g))
    out.update(first=np.array([o]), first_p=p, outcomes=np.array(outcomes), probs=np.array(probs), state=state)
    return out
