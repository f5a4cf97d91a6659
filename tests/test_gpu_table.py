"""The parameter table of a batch at the sizes where its launches end: one set
and one segment, 64 and 65 of each, more, empty members between others, and
segments that name few of many sets.  Every member is bitwise its solo run."""
import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu


def set_of(k):
    return L.params(0.6 + 0.003 * k, 3 / 16, (1e-4 * (k % 7), -2e-5 * k, 3e-5), "f64")


def start(st, base, n, k):
    gen = torch.Generator(device="cuda").manual_seed(100 + k)
    st.f[:, base:base + n] = 0.05 + 1e-3 * torch.randn((19, n), generator=gen, device="cuda",
                                                       dtype=torch.float64)


@pytest.mark.parametrize("members,sets,empty", [(1, 2, ()), (2, 2, (0,)), (64, 64, ()), (65, 65, ()),
                                                (65, 64, (3, 64)), (131, 200, (0, 1, 130)),
                                                (3, 1000, ())])
@pytest.mark.parametrize("persistent", [False, True])
def test_members_run_with_their_sets(members, sets, empty, persistent):
    print_case("table", members, sets, empty, persistent)
    g = I.random_flags(5, 9, 8, 7, fluid_fraction=0.8, periodic=1)
    wide = I.random_flags(6, 30, 9, 4, fluid_fraction=0.8, periodic=1)
    gone = I.Geometry("gone", g.flags * 0, 1)
    geoms = [gone if k in empty else (wide if k % 3 == 1 else g) for k in range(members)]
    b = L.Batch([dev_flags(x) for x in geoms], [1] * members, "lex", tile_align=True)
    prms = [set_of(k) for k in range(sets)]
    names = [(k * 17 + 1) % sets for k in range(members)]  # not 0 first: a table is needed
    segs = [(base, c, names[k]) for k, (base, c) in enumerate(b.segments)]
    st = L.init(b.lattice, prms, n=b.total, segments=segs)
    for k, (base, c, _) in enumerate(segs):
        start(st, base, c, k)
    L.step(st, 3, persistent=persistent)
    solo = {x.name + str(x.dims): L.build(dev_flags(x), 1, "lex") for x in (g, wide)}
    for k, (base, c, q) in enumerate(segs):
        if c == 0:
            continue
        one = L.init(solo[geoms[k].name + str(geoms[k].dims)], prms[q])
        start(one, 0, c, k)
        L.step(one, 3)
        assert torch.equal(st.f[:, base:base + c], one.f[:, :c]), k
