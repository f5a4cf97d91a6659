"""adjoint_gradient from checkpoints of a run longer than T: those at T and later
do not enter the gradient of the first T steps."""
import pytest
import torch

from paper_1111_1129_amd import adjoint as AD
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,longer", [(5, 2, 9), (4, 2, 9), (3, 4, 12), (1, 1, 4), (0, 2, 3)])
def test_checkpoints_past_the_last_step_are_not_used(T, k, longer):
    print_case("checkpoints of a longer run", T, k, longer)
    g = I.pbb_box(4, 12)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    n = lat.n_fluid
    ns = torch.zeros(lat.stride, dtype=torch.float64, device="cuda")
    ns[:n] = torch.from_numpy(g.ns).cuda().view(-1)[lat.cell_of.long()]
    prm = L.params(0.8, 3 / 16, (1e-4, 0, 0), "f64s")
    _, ckpts, _ = AD.forward_states(lat, prm, ns, longer, k)
    want = AD.adjoint_gradient(lat, prm, ns, T, k)
    assert torch.equal(AD.adjoint_gradient(lat, prm, ns, T, k, ckpts)[:n], want[:n])
