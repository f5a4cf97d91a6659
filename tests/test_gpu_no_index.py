"""List and adjacency without an index array (index_of NULL, scratch in the
workspace), below and above the box size from which a lexicographic list looks
its neighbours up in rank words: as with one."""
import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import lattice as L

from gpu_helpers import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,order,param", [((33, 31, 34), "lex", 0), ((33, 31, 34), "hilbert", 0),
                                              ((351, 349, 347), "lex", 0)])
def test_list_without_index(dims, order, param):
    print_case("no index", dims, order)
    nx, ny, nz = dims
    gen = torch.Generator(device="cuda").manual_seed(12)
    flags = (torch.rand((nz, ny, nx), generator=gen, device="cuda") < 0.6).to(torch.uint8)
    lat = L.build(flags, 5, order, param)
    n = lat.n_fluid
    geom = N.lbm_geom(nx, ny, nz, 5, N.ORDERS[order], param)
    st, _, wsn = N.lbm_build_adjacency(geom, flags, 0, 0, None, None, None, 0, query=True)
    assert st == 0 and wsn >= 4 * nx * ny * nz
    ws = torch.empty(wsn, dtype=torch.uint8, device="cuda")
    cell, adj = torch.empty_like(lat.cell_of), torch.zeros_like(lat.adj)
    st, nf, _ = N.lbm_build_adjacency(geom, flags, 0, lat.stride, None, cell, adj, n, ws, wsn)
    assert st == 0 and nf == n
    assert torch.equal(cell, lat.cell_of) and torch.equal(adj, lat.adj)
