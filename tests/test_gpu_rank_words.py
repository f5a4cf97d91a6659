"""Large lexicographic lists, whose adjacency is found through rank words in
place of the index (from 40 Mi box cells on), against the same call with an
index that does not allow them (an odd 32-bit address): list, index and
adjacency are equal, with walls, periodic faces, faces of one cell's thickness
in x, and boxes that end inside a word."""
import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import lattice as L

from gpu_helpers import print_case

pytestmark = pytest.mark.gpu

CASES = [((351, 349, 347), 0, 0.5), ((351, 349, 347), 7, 0.5), ((352, 350, 348), 5, 0.9),
         ((2, 4700, 4501), 1, 0.7), ((1, 6501, 6503), 6, 0.6), ((41943041, 1, 1), 1, 0.5),
         ((512, 512, 400), 1, 0.7)]


@pytest.mark.parametrize("dims,periodic,por", CASES)
def test_rank_words_equal_the_index(dims, periodic, por):
    print_case("rank words", dims, periodic, por)
    nx, ny, nz = dims
    gen = torch.Generator(device="cuda").manual_seed(11)
    flags = (torch.rand((nz, ny, nx), generator=gen, device="cuda") < por).to(torch.uint8)
    box = nx * ny * nz
    assert box >= 40 << 20
    lat = L.build(flags, periodic, "lex")
    n = lat.n_fluid
    assert n == int(flags.sum())
    geom = N.lbm_geom(nx, ny, nz, periodic, 0, 0)
    room = torch.empty(box + 1, dtype=torch.int32, device="cuda")
    index = room[1:]  # 4 bytes past an aligned address
    cell = torch.empty_like(lat.cell_of)
    adj = torch.zeros_like(lat.adj)
    st, _, wsn = N.lbm_build_adjacency(geom, flags, 0, 0, index, None, None, 0, query=True)
    assert st == 0
    ws = torch.empty(wsn, dtype=torch.uint8, device="cuda")
    st, nf, _ = N.lbm_build_adjacency(geom, flags, 0, lat.stride, index, cell, adj, n, ws, wsn)
    assert st == 0 and nf == n
    assert torch.equal(index, lat.index_of)
    assert torch.equal(cell, lat.cell_of)
    assert torch.equal(adj, lat.adj)
    # and by the definition, on the index itself
    assert torch.equal(lat.index_of >= 0, flags.view(-1) != 0)
    assert torch.equal(lat.index_of[lat.cell_of.long()],
                       torch.arange(n, dtype=torch.int32, device="cuda"))
