"""The assembly's walk over key positions and the code kernels at the sizes
where their pieces end: boxes of less than a row (64 positions), a tile (4096,
a 16^3 cube of the curves) and a few tiles; boxes that leave most of a curve's
cube empty, so that runs of 1, 8 and 64 tiles are passed over; block edges
below, at and above a row, with cut-off last blocks; row strides that do and
do not allow four cells per access."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import adj_u32, dev_flags, print_case
from test_gpu_compress import check_codes

pytestmark = pytest.mark.gpu

ORDERS = [("lex", 0), ("blocked", 2), ("blocked", 5), ("blocked", 16), ("blocked", 300),
          ("morton1", 0), ("morton2", 0), ("hilbert", 0), ("random", 9)]
BOXES = [(1, 1, 1), (2, 1, 3), (4, 4, 4), (5, 4, 4), (8, 8, 8), (9, 8, 7), (16, 16, 16),
         (17, 16, 15), (32, 32, 32), (33, 31, 34), (300, 3, 2), (2, 3, 270), (5, 140, 66)]


@pytest.mark.parametrize("order,param", ORDERS)
@pytest.mark.parametrize("dims", BOXES)
def test_numbering_and_adjacency(order, param, dims):
    print_case("walk", order, param, dims)
    g = I.random_flags(sum(dims), *dims, fluid_fraction=0.7, periodic=5)
    lat = L.build(dev_flags(g), g.periodic, order, param)
    sp = O.build(g.flags, g.periodic, order, param, stride=lat.stride)
    assert lat.n_fluid == sp.n_fluid == L.count_fluid(dev_flags(g), g.periodic, order, param)
    n = sp.n_fluid
    np.testing.assert_array_equal(lat.index_of.cpu().numpy(), sp.index_of)
    np.testing.assert_array_equal(lat.cell_of.cpu().numpy(), sp.cell_of)
    a = adj_u32(lat)
    np.testing.assert_array_equal(a[:, :n], sp.adj[:, :n])
    assert not a[:, n:].any()


@pytest.mark.parametrize("order", ["lex", "random"])  # no escapes; nearly all escapes
@pytest.mark.parametrize("pad", [0, 1, 2, 4])
@pytest.mark.parametrize("dims", [(9, 8, 7), (16, 16, 4), (34, 33, 32), (130, 40, 40)])
def test_codes_at_any_stride(order, pad, dims):
    """Strides of every residue modulo 4, the smallest ones ending with the
    list; the codes, the records and the columns left alone."""
    print_case("codes", order, pad, dims)
    g = I.random_flags(3, *dims, fluid_fraction=0.8, periodic=1)
    n = L.count_fluid(dev_flags(g), g.periodic, order, 4)
    stride = (n + 3) // 4 * 4 + pad
    lat = L.build(dev_flags(g), g.periodic, order, 4, stride=stride)
    comp = L.compress(lat)
    check_codes(lat, comp)
    L.narrow(comp)
    codes, c8 = comp.codes.cpu().numpy()[:, :n], comp.codes8.cpu().numpy()[:, :n]
    rec = comp.tile_records.cpu().numpy()
    narrow = 0
    for t in range(comp.n_tiles):
        c = codes[:, t * 256:(t + 1) * 256]
        fits = bool(np.all((c == -32768) | ((c >= -127) & (c <= 127))))
        assert rec[t, 19] == int(fits)
        want = np.where(c == -32768, -128, c) if fits else np.zeros_like(c)
        np.testing.assert_array_equal(c8[:, t * 256:(t + 1) * 256], want)
        narrow += int(fits)
    assert comp.n_narrow == narrow
    # the same call into filled arrays: columns past the list stay
    filled = torch.full((18, stride), 77, dtype=torch.int16, device="cuda")
    filled8 = torch.full((18, stride), 77, dtype=torch.int8, device="cuda")
    recs = torch.empty_like(comp.tile_records)
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda")
    st, esc, _ = N.lbm_compress_adjacency(n, stride, lat.adj, filled, recs, ws, 4096)
    assert st == 0 and esc == comp.n_escapes
    st, cnt, _ = N.lbm_narrow_codes(n, stride, filled, recs, filled8, ws, 4096)
    assert st == 0 and cnt == narrow
    assert bool((filled[:, n:] == 77).all()) and bool((filled8[:, n:] == 77).all())
    assert torch.equal(filled[:, :n], comp.codes[:, :n])
    assert torch.equal(recs, comp.tile_records)
