"""Passes of compiled density-matrix circuits (CPU): 4x4s of a qubit that lie
apart in the circuit are not joined before planning."""
import pytest

from workloads import noisy_circuit


@pytest.mark.parametrize('N,depth,seed,prec,tile,passes', [(14, 10, 0, 'C64', (14, 10, 5), 10),
                                                           (13, 5, 1, 'C128', (12, 8, 4), 5)])
def test_passes_of_noisy_circuits(N, depth, seed, prec, tile, passes):
    import paper_1802_08032_amd as q
    c = q.Circuit(noisy_circuit(N, depth, seed))
    _, n = c.source(N, getattr(q, prec), tile[0], tile[1], 0, 0, tile[2], q.DENSITY)
    c.close()
    assert n <= passes
