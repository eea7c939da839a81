"""Copies of a state on both sides of 256 MiB, where the kernel takes over from
the runtime's copy: every bit is the source's, and the source stays as it is."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('prec,n', [('C128', 1), ('C128', 23), ('C128', 24), ('C64', 2), ('C64', 24), ('C64', 25)])
def test_clone_and_pure_state(prec, n):
    import torch
    import paper_1802_08032_amd as q
    env = q.Env(0)
    a, b = (q.Register(env, n, q.STATEVEC, getattr(q, prec)) for _ in range(2))
    g = torch.Generator(device=a.tensor.device).manual_seed(n)
    torch.view_as_real(a.tensor).normal_(generator=g)
    want = a.tensor.clone()
    b.tensor.fill_(7.0)
    b.clone_from(a)
    env.sync()
    assert torch.equal(b.tensor, want) and torch.equal(a.tensor, want)
    b.tensor.fill_(7.0)
    b.init_pure_state(a)
    env.sync()
    assert torch.equal(b.tensor, want) and torch.equal(a.tensor, want)
    a.close()
    b.close()
    env.close()
