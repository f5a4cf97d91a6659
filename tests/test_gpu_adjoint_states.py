"""The states that the two-level adjoint keeps (adjoint.forward_states)."""
import pytest
import torch

from paper_1111_1129_amd import adjoint as AD
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import dev_flags

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k", [(1, 1), (1, 5), (2, 1), (5, 2), (7, 3), (6, 6), (9, 4)])
def test_two_level_states_are_those_of_a_plain_run(T, k):
    """forward_states keeps the arrays that hold the states instead of copies:
    every checkpoint and the final state are those of one plain run, also after
    the returned state has been stepped on, and checkpoints kept elsewhere
    (host memory, a strided view) give the same gradient."""
    g = I.pbb_box(4, 12)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    n = lat.n_fluid
    ns = torch.zeros(lat.stride, dtype=torch.float64, device="cuda")
    ns[:n] = torch.from_numpy(g.ns).cuda().view(-1)[lat.cell_of.long()]
    prm = L.params(0.8, 3 / 16, (1e-4, 0, 0), "f64s")
    J, ckpts, st = AD.forward_states(lat, prm, ns, T, k)
    plain = L.init(lat, prm, ns=ns)
    want = []
    for t in range(T):
        if t % k == 0:
            want.append(plain.f[:, :n].clone())
        L.step(plain, 1)
    assert len(ckpts) == len(want) and st.steps == T
    assert J.item() == L.objective(plain)[0].item()
    assert torch.equal(st.f[:, :n], plain.f[:, :n])
    grad = AD.adjoint_gradient(lat, prm, ns, T, k, ckpts)
    L.step(st, 3)
    for c, w in zip(ckpts, want):
        assert torch.equal(c[:, :n], w)
    wide = [torch.empty((19, 2 * lat.stride), dtype=torch.float64, device="cuda")[:, ::2].copy_(c)
            for c in ckpts]
    for other in ([c.cpu() for c in ckpts], wide):
        assert torch.equal(AD.adjoint_gradient(lat, prm, ns, T, k, other)[:n], grad[:n])
