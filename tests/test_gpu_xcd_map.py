"""The library's own workgroup-to-XCD mapping (xcd_chunk = 0) at the sizes where
its runs end: fewer tiles than XCDs, whole and partial groups of runs, and both
sides of the state sizes at which it goes over from one run per XCD to short
runs and lets every other sweep run backwards.  Every form is bitwise the
hardware order (xcd_chunk = 1)."""
import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L
from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu

# cells of an all-fluid box: 1, 256, 257 (2 tiles), 7-9 tiles, 64 and 65 tiles,
# and about 240 and 384 MiB of state (2.7 and 3.3 M cells of 76 to 148 bytes)
BOXES = [(1, 1, 1), (16, 16, 1), (257, 1, 1), (16, 16, 7), (16, 16, 8), (16, 18, 8), (32, 32, 16),
         (33, 31, 17), (140, 139, 138), (150, 149, 147)]


@pytest.mark.parametrize("dims", BOXES)
@pytest.mark.parametrize("storage", ["f16s12", "f64s"])
def test_default_map_covers_every_cell_once(dims, storage):
    if storage == "f64s" and dims[0] > 140:
        pytest.skip("the smaller of the two large boxes is past the limit in FP64 already")
    print_case("xcd map", dims, storage)
    g = I.all_fluid(*dims)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    comp = L.narrow(L.compress(lat))
    n = lat.n_fluid
    gen = torch.Generator(device="cuda").manual_seed(5)
    f0 = 1e-2 * torch.randn((19, n), generator=gen, device="cuda")

    def states(chunk):
        prm = L.params(0.8, 3 / 16, (1e-5, 0, 0), storage, xcd_chunk=chunk)
        out = []
        for form in ("full", "c16", "c8", "inplace", "persistent", "inplace_full"):
            st = (L.init_inplace if form.startswith("inplace") else L.init)(lat, prm)
            st.f[:, :n] = f0
            if form == "full":
                L.step(st, 2)
            elif form == "c16":
                L.step_c16(st, comp, 2)
            elif form.startswith("inplace"):
                full = form.endswith("full")
                L.step_inplace(st, 2, None if full else comp, c8=not full)
            else:
                L.step_c8(st, comp, 2, persistent=form == "persistent")
            out.append(st.f[:, :n])
        if storage == "f64s":
            lam = torch.randn((19, lat.stride), generator=gen.manual_seed(6), device="cuda",
                              dtype=torch.float64)
            back = torch.full_like(lam, float("nan"))
            N._check("lbm_step_adjoint_c8", N.lbm_step_adjoint_c8(
                prm, n, lat.stride, comp.codes8, comp.codes, comp.tile_records, lat.adj, st.f,
                None, lam, back, None))
            out.append(back[:, :n])
        return out

    ref = states(1)
    for a in ref[1:6]:
        assert torch.equal(a, ref[0])
    for a, b in zip(states(0), ref):
        assert torch.equal(a, b)
