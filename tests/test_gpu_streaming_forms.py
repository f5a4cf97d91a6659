"""Every sweep form over lists larger than the last-level cache, or that it holds
most of, where the streaming kernels run: with and without launch hints, with a solid fraction,
over a list with narrow, 16-bit and escape tiles, with parameter sets, and the
adjoint in both of its builds.

The reference does not go through the launch choices under test: the same cells
are swept as sublists of 64 tiles, each a small launch of its own over the full
list (such launches are held against the CPU oracle elsewhere).  A sublist that
begins at column b is the call on the arrays from column b on, with b taken off
every adjacency entry.  Results are equal bit for bit."""
import dataclasses

import pytest
import torch

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import lattice as L

from gpu_helpers import print_case

pytestmark = pytest.mark.gpu

PIECE = 64 * 256
STEPS = 4


def flags_of(seed, nx, ny, nz, share):
    """Random cells, the last few made solid so that the count is whole tiles."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    flags = (torch.rand((nz, ny, nx), generator=gen, device="cuda") < share).to(torch.uint8)
    fluid = flags.view(-1).nonzero().view(-1)
    rest = fluid.numel() % 256
    if rest:
        flags.view(-1)[fluid[-rest:]] = 0
    return flags


def mixed_list(scale):
    """One list of three geometries: lexicographic, along a Hilbert curve, in
    random order.  (lattice, codes, the three column ranges)"""
    parts = [(flags_of(1, 60, 50, scale, 0.9), "lex", 0), (flags_of(2, 128, 128, scale, 0.8), "hilbert", 0),
             (flags_of(3, 40, 40, scale, 0.8), "random", 7)]
    counts = [int(f.sum()) for f, _, _ in parts]
    n = sum(counts)
    stride, adj, base, ranges = L.aligned_stride(n), None, 0, []
    for (flags, order, param), c in zip(parts, counts):
        lat = L.build(flags, 1, order, param, base=base, stride=stride, adj=adj)
        assert lat.n_fluid == c and c % 256 == 0
        adj = lat.adj
        ranges.append((base, c))
        base += c
    lat = dataclasses.replace(lat, base=0, n_fluid=n, index_of=None, cell_of=None)
    comp = L.narrow(L.compress(lat))
    rec = comp.tile_records
    narrow, escapes = int((rec[:, 19] != 0).sum()), int((rec[:, 18] != 0).sum())
    assert min(narrow, escapes, comp.n_tiles - narrow - escapes) > 100  # all three kinds
    return lat, comp, ranges


class Pieces:
    """Sublists of a list: (first column, cells), and its adjacency with the
    first column taken off."""

    def __init__(self, lat, ranges):
        self.S = lat.stride
        self.spans = [(b + o, min(PIECE, c - o)) for b, c in ranges for o in range(0, c, PIECE)]
        assert 19 * self.S < 2 ** 31
        self.adj = lat.adj.clone()
        for b, c in self.spans:
            self.adj[:, b:b + c] -= b

    def at(self, t, b):
        return None if t is None else t.data_ptr() + b * t.element_size()

    def step(self, prm_of, ns, src, dst):
        for b, c in self.spans:
            prm = prm_of(b)
            assert N.lbm_sweep_launch(prm, c, 1)[1] == (0, 0, 0)  # a small launch
            st, _ = N.lbm_step(prm, c, self.S, self.at(self.adj, b), self.at(ns, b), self.at(src, b),
                               self.at(dst, b), 1)
            assert st == N.LBM_OK

    def adjoint(self, prm, f, ns, lam, out, grad):
        for b, c in self.spans:
            assert N.lbm_step_adjoint(prm, c, self.S, self.at(self.adj, b), self.at(f, b),
                                      self.at(ns, b), self.at(lam, b), self.at(out, b),
                                      self.at(grad, b)) == N.LBM_OK


@pytest.fixture(scope="module")
def large():
    lat, comp, ranges = mixed_list(272)
    return lat, comp, ranges, Pieces(lat, ranges)


@pytest.fixture(scope="module")
def medium():
    lat, comp, ranges = mixed_list(76)
    return lat, comp, ranges, Pieces(lat, ranges)


def noise(shape, seed, dtype):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return (1e-2 * torch.randn(shape, generator=gen, device="cuda")).to(dtype)


def solid(lat):
    gen = torch.Generator(device="cuda").manual_seed(9)
    return torch.rand(lat.stride, generator=gen, device="cuda", dtype=torch.float64)


HINTS = [(False, 0), (True, 0), (True, 2), (False, 16), (True, 1)]


@pytest.mark.parametrize("pbb", [False, True])
@pytest.mark.parametrize("storage", ["f64s", "f32s", "f16s12"])
def test_sweeps_of_a_large_list(large, storage, pbb):
    lat, comp, _, pieces = large
    n = lat.n_fluid
    ns = solid(lat) if pbb else None
    plain = L.params(0.8, 3 / 16, (1e-5, 2e-6, 0), storage)
    dtype = N.STORAGE_DTYPE[plain.storage]
    f0 = noise((19, n), 5, dtype)
    a, b = (torch.zeros((19, lat.stride), dtype=dtype, device="cuda") for _ in range(2))
    a[:, :n] = f0
    for _ in range(STEPS):
        pieces.step(lambda _: plain, ns, a, b)
        a, b = b, a
    forms = [("full", 4, False), ("c16", 2, False), ("c8", 1, False), ("persistent", 1, False),
             ("inplace", 4, True), ("inplace_c16", 2, True), ("inplace_c8", 1, True)]
    for nt, chunk in HINTS:
        prm = L.params(0.8, 3 / 16, (1e-5, 2e-6, 0), storage, nontemporal=nt, xcd_chunk=chunk)
        for form, code_bytes, in_place in forms:
            launch = N.lbm_sweep_launch(prm, n, STEPS, code_bytes, in_place)[1]
            print_case("streaming", storage, pbb, nt, chunk, form, launch)
            assert launch[1] > 0  # none of them keeps the state in the cache
            st = (L.init_inplace if in_place else L.init)(lat, prm, ns=ns)
            st.f[:, :n] = f0
            if form == "full":
                L.step(st, STEPS)
            elif form == "c16":
                L.step_c16(st, comp, STEPS)
            elif in_place:
                L.step_inplace(st, STEPS, None if code_bytes == 4 else comp, c8=code_bytes == 1)
            else:
                L.step_c8(st, comp, STEPS, persistent=form == "persistent")
            assert torch.equal(st.f[:, :n], a[:, :n]), (form, nt, chunk)


# States that the cache holds most of: one run per XCD, plain stores, alternating
# directions without hints; (storage, third edge of the list's parts, forms)
NEAR = [("f64s", 60, ("full", "c16")), ("f64s", 120, ("inplace",)),
        ("f32s", 120, ("full", "c16")), ("f16s12", 120, ("full",))]


@pytest.mark.parametrize("pbb", [False, True])
@pytest.mark.parametrize("storage,scale,forms", NEAR)
def test_sweeps_of_a_list_near_the_cache(storage, scale, forms, pbb):
    lat, comp, ranges = mixed_list(scale)
    n, pieces = lat.n_fluid, Pieces(lat, ranges)
    ns = solid(lat) if pbb else None
    prm = L.params(0.8, 3 / 16, (1e-5, 2e-6, 0), storage)
    dtype = N.STORAGE_DTYPE[prm.storage]
    f0 = noise((19, n), 5, dtype)
    a, b = (torch.zeros((19, lat.stride), dtype=dtype, device="cuda") for _ in range(2))
    a[:, :n] = f0
    for _ in range(STEPS):
        pieces.step(lambda _: prm, ns, a, b)
        a, b = b, a
    for form in forms:
        in_place = form == "inplace"
        launch = N.lbm_sweep_launch(prm, n, STEPS, 2 if form == "c16" else 4, in_place)[1]
        print_case("near the cache", storage, scale, pbb, form, launch)
        assert launch == (0, 1, 1)
        st = (L.init_inplace if in_place else L.init)(lat, prm, ns=ns)
        st.f[:, :n] = f0
        if in_place:
            L.step_inplace(st, STEPS)
        elif form == "full":
            L.step(st, STEPS)
        else:
            L.step_c16(st, comp, STEPS)
        assert torch.equal(st.f[:, :n], a[:, :n]), form


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("storage", ["f64", "f32s"])
def test_parameter_sets_of_a_large_list(large, storage, persistent):
    lat, comp, ranges, pieces = large
    n = lat.n_fluid
    ns = solid(lat)
    for nt, chunk in HINTS[:3]:
        print_case("streaming table", storage, persistent, nt, chunk)
        sets = [L.params(0.7 + 0.1 * k, 3 / 16, (1e-5 * k, 2e-6, 0), storage, nontemporal=nt,
                         xcd_chunk=chunk) for k in range(4)]
        segs = [(b, c, 3 - k) for k, (b, c) in enumerate(ranges)]
        for use in (None, comp):
            st = L.init(lat, sets, ns=ns, segments=segs)
            assert N.lbm_sweep_launch(sets[0], n, STEPS, 4 if use is None else 1)[1][1] > 0
            st.f[:, :n] += noise((19, n), 6, st.f.dtype)
            a, b = st.f.clone(), torch.empty_like(st.f)
            quiet = [L.params(p.tau_plus, p.magic, tuple(p.force), storage) for p in sets]
            set_of = lambda col: quiet[next(q for b0, c, q in segs if b0 <= col < b0 + c)]
            for _ in range(STEPS):
                pieces.step(set_of, ns, a, b)
                a, b = b, a
            if use is None:
                L.step(st, STEPS, persistent=persistent)
            else:
                L.step_c8(st, use, STEPS, persistent=persistent)
            assert torch.equal(st.f[:, :n], a[:, :n]), (nt, chunk, use is None)


@pytest.mark.parametrize("pbb", [False, True])
@pytest.mark.parametrize("size", ["medium", "large"])  # three and two waves per SIMD
def test_adjoint_steps_of_a_large_list(size, pbb, request):
    lat, comp, _, pieces = request.getfixturevalue(size)
    n, S = lat.n_fluid, lat.stride
    assert (384 << 20) < n * 608 <= (960 << 20) if size == "medium" else n * 608 > (1280 << 20)
    ns = solid(lat) if pbb else None
    plain = L.params(0.8, 3 / 16, (1e-5, 2e-6, 0), "f64s")
    f = torch.zeros((19, S), dtype=torch.float64, device="cuda")
    f[:, :n] = noise((19, n), 5, f.dtype)
    lam0 = torch.zeros_like(f)
    lam0[:, :n] = noise((19, n), 8, f.dtype)

    def two_steps(step):
        # towards the other array and back: both directions where they alternate
        lam, other = lam0.clone(), torch.zeros_like(lam0)
        grad = torch.zeros(S, dtype=torch.float64, device="cuda") if pbb else None
        step(lam, other, grad)
        step(other, lam, grad)
        return lam[:, :n], None if grad is None else grad[:n]

    want, want_grad = two_steps(lambda x, y, g: pieces.adjoint(plain, f, ns, x, y, g))
    for nt, chunk in HINTS:
        prm = L.params(0.8, 3 / 16, (1e-5, 2e-6, 0), "f64s", nontemporal=nt, xcd_chunk=chunk)
        for form in ("full", "c16", "c8"):
            print_case("streaming adjoint", size, pbb, nt, chunk, form)

            def step(x, y, g):
                if form == "full":
                    rc = N.lbm_step_adjoint(prm, n, S, lat.adj, f, ns, x, y, g)
                elif form == "c16":
                    rc = N.lbm_step_adjoint_c16(prm, n, S, comp.codes, comp.tile_records, lat.adj, f,
                                                ns, x, y, g)
                else:
                    rc = N.lbm_step_adjoint_c8(prm, n, S, comp.codes8, comp.codes, comp.tile_records,
                                               lat.adj, f, ns, x, y, g)
                assert rc == N.LBM_OK

            got, grad = two_steps(step)
            assert torch.equal(got, want), (form, nt, chunk)
            assert grad is None or torch.equal(grad, want_grad), (form, nt, chunk)
