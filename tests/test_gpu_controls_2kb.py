"""Controls and phases whose qubit is the address bit of 2 KB or 4 KB, at the
sizes where these set the grid and the number of workgroups on a CU (512 MiB and
128 MiB touched).  Every amplitude is compared, on the device, with torch's
complex128; tolerances as in test_gpu_large_steps."""
import math

import numpy as np
import pytest

from .test_gpu_large_steps import EPS, compare, env, group, part, q, register  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('prec,bit', [('C128', 7), ('C64', 8)])
@pytest.mark.parametrize('n', [24, 26, 27])
def test_control(q, env, prec, bit, n):  # noqa: F811
    from workloads import haar_unitary_k
    reg, want = register(q, env, prec, n, q.STATEVEC, n)
    for c in (bit, bit + 1):
        for targets in ((0,), (4,), (14,), (n - 1,), (14, 15), (0, 14), (4, 5), (14, 15, 17), (0, 5, 14)):
            want.copy_(reg.tensor)  # the next call starts from equal entries
            d = 1 << len(targets)
            tol = 2 * (d + 1) * EPS[prec] * math.sqrt(d) * float(want.abs().max())
            u = haar_unitary_k(np.random.default_rng(c), len(targets))
            reg.multi_qubit_unitary(targets, u, [c])
            group(want, u, targets, [c])
            compare(reg, want, tol)
        want.copy_(reg.tensor)
        reg.cnot(c, 14)
        group(want, np.array([[0, 1], [1, 0]]), (14,), [c])
        compare(reg, want, 0.0)
        for qubits in ((c,), (c, 16)):
            want.copy_(reg.tensor)
            reg.multi_controlled_phase(qubits, 0.7)
            part(want, {b: 1 for b in qubits}).mul_(complex(math.cos(0.7), math.sin(0.7)))
            compare(reg, want, 4 * EPS[prec] * float(want.abs().max()))
    reg.close()
