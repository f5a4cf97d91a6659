"""The two-array sweep of states somewhat larger than the last-level cache:
plain stores, one run of the list per XCD and alternating directions whatever the
launch hints, up to a size that depends on the form (8-bit codes 256 MiB,
16-bit codes 384 MiB, full list 512 MiB).  On both sides of each limit every
form is bitwise the in-place sweep in hardware order, which follows the hints."""
import pytest
import torch

from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L
from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu

# scaled FP16, bytes per cell 94 / 112 / 148: below and above 256 MiB over 8-bit
# codes, 384 MiB over 16-bit codes, 512 MiB over the list
BOXES = [(142, 142, 141), (142, 142, 142), (153, 153, 153), (154, 154, 152), (154, 154, 153)]


@pytest.mark.parametrize("dims", BOXES)
@pytest.mark.parametrize("nt,chunk", [(False, 0), (True, 2)])
def test_forms_agree_on_both_sides_of_the_limits(dims, nt, chunk):
    print_case("between cache sizes", dims, nt, chunk)
    g = I.all_fluid(*dims)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    comp = L.narrow(L.compress(lat))
    n = lat.n_fluid
    gen = torch.Generator(device="cuda").manual_seed(7)
    f0 = 1e-2 * torch.randn((19, n), generator=gen, device="cuda")

    def state(init, prm):
        st = init(lat, prm)
        st.f[:, :n] = f0
        return st

    one = state(L.init_inplace, L.params(0.8, 3 / 16, (1e-5, 0, 0), "f16s12", xcd_chunk=1))
    L.step_inplace(one, 4)
    prm = L.params(0.8, 3 / 16, (1e-5, 0, 0), "f16s12", nontemporal=nt, xcd_chunk=chunk)
    for sweep in (lambda s: L.step(s, 4), lambda s: L.step_c16(s, comp, 4),
                  lambda s: L.step_c8(s, comp, 4), lambda s: L.step_c8(s, comp, 4, persistent=True)):
        st = state(L.init, prm)
        sweep(st)
        assert torch.equal(st.f[:, :n], one.f[:, :n])
