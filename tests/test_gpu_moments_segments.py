"""Totals of lbm_moments where its launches end: one cell, one tile, more tiles
than workgroups; empty segments; more segments than one launch takes; and a
workspace that holds only the largest segment's partials, so that the segments
are split over launches.  Fields are bitwise those of one segment; totals are
the exact sums of the fields (the double-double sums are within 1e-30 of them
before the final rounding, far inside the bound used: that of a float64
pairwise sum, 2^-53 log2 n of the sum of magnitudes)."""
import math

import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import inputs as I
from paper_1111_1129_amd import lattice as L

from gpu_helpers import dev_flags, print_case

pytestmark = pytest.mark.gpu

# segment lengths; each starts on the next tile
SEGMENTS = [[1], [256], [257], [0, 5, 0], [300, 0, 1, 256, 4000], [40 + 7 * k for k in range(64)],
            [11 + k % 5 * 300 for k in range(131)], [2_200_000, 3, 900_000]]


@pytest.mark.parametrize("storage", ["f64", "f16s12"])
@pytest.mark.parametrize("case", range(len(SEGMENTS)))
def test_totals_of_segments(storage, case):
    sizes = SEGMENTS[case]
    print_case("moments", storage, sizes[:6], len(sizes))
    segs, base = [], 0
    for k, c in enumerate(sizes):
        segs.append((base, c, k % 3))
        base += (c + 255) // 256 * 256
    n = base
    g = I.all_fluid(256, n // 256, 1)
    lat = L.build(dev_flags(g), g.periodic, "lex")
    prms = [L.params(0.8, 3 / 16, (1e-3 * k, 2e-3, -1e-3 * k), storage) for k in range(3)]
    st = L.init(lat, prms, n=n, segments=segs)
    gen = torch.Generator(device="cuda").manual_seed(3)
    st.f += 0.01 * torch.randn(st.f.shape, generator=gen, device="cuda")
    rho, u, tot = L.moments(st)
    J = L.objective(st)
    one = L.init(lat, L.params(storage=storage), n=n)  # no force: the gathered momentum
    one.f.copy_(st.f)
    rho1, u1, _ = L.moments(one)
    least = (max(1, (max(sizes) + 255) // 256) * 64 + 255) // 256 * 256
    small = torch.empty(least, dtype=torch.uint8, device="cuda")
    tot2 = torch.full_like(tot, float("nan"))
    rc, _ = N.lbm_moments(st.params, n, lat.stride, lat.adj, st.f, None, None, segs, tot2, small,
                          small.numel())
    assert rc == 0
    assert torch.equal(tot, tot2)
    noalloc = torch.full_like(tot, float("nan"))
    assert N.lbm_moments_noalloc(st.params, n, lat.stride, lat.adj, st.f, None, None, segs,
                                 noalloc) == 0
    for k, (b, c, q) in enumerate(segs):
        force = torch.tensor(list(prms[q].force), dtype=torch.float64, device="cuda")
        assert torch.equal(rho[b:b + c], rho1[b:b + c])
        want = torch.tensor([math.fsum(v.tolist()) for v in (rho[b:b + c], *u[:, b:b + c])],
                            dtype=torch.float64, device="cuda")
        # u of set q is the gathered momentum plus half its force (one rounding each)
        half = u1[:, b:b + c] + 0.5 * force[:, None]
        assert torch.allclose(u[:, b:b + c], half, rtol=0, atol=1e-16)
        scale = torch.stack([rho[b:b + c].abs().sum(), *u[:, b:b + c].abs().sum(1)])
        bits = max(1, c).bit_length() * 2.0 ** -53
        assert bool(((tot[k] - want).abs() <= bits * scale).all())
        # the two groupings of the same double-double sum: one final rounding
        assert bool(((tot[k] - noalloc[k]).abs() <= 2.0 ** -52 * tot[k].abs()).all())
        if c:
            assert J[k].item() == tot[k, 1].item() / c
        else:
            assert not tot[k].any() and torch.isnan(J[k])
