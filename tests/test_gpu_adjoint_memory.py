"""What a PermeabilityFn holds between its passes: one state per segment of k
steps and the adjacency codes; after the backward pass neither."""
import pytest
import torch

from paper_1111_1129_amd import adjoint as AD
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu

SLACK = 4 << 20  # a quarter of a state; what the allocator leaves unsplit is below 1 MiB


@pytest.mark.parametrize("T,k", [(1, 1), (4, 4), (5, 5), (9, 3), (10, 3), (12, 4), (3, 1)])
def test_states_held_between_the_passes(T, k):
    print_case("held states", T, k)
    g = I.pbb_box(4, 56)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    n = lat.n_fluid
    state = 19 * 8 * lat.stride
    assert state > 4 * SLACK
    x = torch.zeros(lat.stride, dtype=torch.float64, device="cuda")
    x[:n] = torch.from_numpy(g.ns).cuda().view(-1)[lat.cell_of.long()]
    x.requires_grad_(True)
    prm = L.params(0.8, 3 / 16, (1e-4, 0, 0), "f64s")
    comp = AD.codes_of(lat, None)
    codes = sum(t.numel() * t.element_size() for t in (comp.codes, comp.codes8, comp.tile_records))
    before = torch.cuda.memory_allocated()
    J = AD.PermeabilityFn.apply(x, lat, prm, T, k)
    held = torch.cuda.memory_allocated() - before
    assert held <= -(-T // k) * state + codes + SLACK
    J.backward()
    assert torch.cuda.memory_allocated() - before <= SLACK
    assert torch.isfinite(x.grad[:n]).all()
