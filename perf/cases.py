"""Performance cases of the list-based D3Q19 TRT lattice Boltzmann framework.

Every case is one thing a program does with the public entry points of
``paper_1111_1129_amd.lattice`` and ``.adjoint``:

  sweep      n pull sweeps of one geometry, in one of the forms a program can
             choose: the full adjacency list, 16-bit or 8-bit codes, in place,
             one HIP graph, one persistent launch;
  batch      n sweeps of many uneven packings in one list, every member with
             its own parameters, and the members' totals;
  assemble   a new flag field to list, adjacency and adjacency codes;
  moments    density, velocity and totals of a state;
  adjoint    mean flux and its gradient with respect to the solid fraction.

Geometries are overlapping random spheres in a box with walls on the y and z
faces, periodic in x (the repository's packings), a tube along x filled with
such spheres, or the empty channel.  They are stamped on the GPU from the
seed: one placement per size, shifted along x and mirrored by the seed, so that
the fluid count does not depend on it.  Initial states are an equilibrium at a
random velocity with noise.
"""
import math

import torch

from paper_1111_1129_amd import adjoint as AD
from paper_1111_1129_amd import lattice as L

TAU, MAGIC = 0.8, 3.0 / 16.0
SIZE = {"f64": 8, "f64s": 8, "f32": 4, "f32s": 4, "f16s": 2, "f16s12": 2}


def listed():
    return [
        # the smallest calls: the 32^3 packing from the first configuration,
        # FP64, 100 sweeps by one call, library defaults
        dict(name="packing32_f64", kind="sweep", geom="spheres", nx=32, ny=32, nz=32, r0=4.0,
             r1=4.0, por=0.52, order="lex", param=0, storage="f64", form="full", steps=100,
             nt=False, chunk=0, pbb=False),
        # a small geometry stepped in a loop through one captured graph
        dict(name="packing64_f32s_graph", kind="sweep", geom="spheres", nx=64, ny=64, nz=64,
             r0=4.0, r1=10.0, por=0.45, order="lex", param=0, storage="f32s", form="graph_c8",
             steps=100, nt=True, chunk=1, pbb=False),
        # the packed tube as the usage example runs it: full list, launch
        # options given
        dict(name="tube_f64_full", kind="sweep", geom="tube", nx=256, ny=256, nz=256, r0=12.0,
             r1=12.0, por=0.65, order="lex", param=0, storage="f64", form="full", steps=20,
             nt=True, chunk=1, pbb=False),
        # the headline workload's form on half its box: FP64 over the codes,
        # the launch options the tuner picks there
        dict(name="packing512_f64_c8", kind="sweep", geom="spheres", nx=512, ny=512, nz=512,
             r0=8.0, r1=16.0, por=0.40, order="lex", param=0, storage="f64", form="c8", steps=4,
             nt=True, chunk=4, pbb=False),
        # shifted FP32 over the codes, an odd box, library defaults
        dict(name="packing301_f32s_c8", kind="sweep", geom="spheres", nx=301, ny=257, nz=403,
             r0=8.0, r1=16.0, por=0.40, order="lex", param=0, storage="f32s", form="c8", steps=10,
             nt=False, chunk=0, pbb=False),
        # scaled shifted FP16, one PDF array: the fastest reduced-precision
        # form of the precision workload
        dict(name="packing384_f16s12_inplace", kind="sweep", geom="spheres", nx=384, ny=384,
             nz=512, r0=8.0, r1=16.0, por=0.40, order="lex", param=0, storage="f16s12",
             form="inplace_c8", steps=10, nt=True, chunk=16, pbb=False),
        # the ordering study: blocked order, full list, library defaults
        dict(name="packing200_f64s_blocked", kind="sweep", geom="spheres", nx=200, ny=200, nz=200,
             r0=6.0, r1=12.0, por=0.45, order="blocked", param=16, storage="f64s", form="full",
             steps=20, nt=False, chunk=0, pbb=False),
        # the adjoint workload: forward and gradient with two-level checkpoints
        dict(name="adjoint128", kind="adjoint", nx=128, ny=128, nz=128, order="lex", param=0,
             storage="f64s", T=110, k=22, nt=True, chunk=1),
        # uneven packings with their own parameters, one launch per step over
        # the codes, then every member's totals
        dict(name="batch48_f32_c8", kind="batch", members=48, l0=48, l1=160, r0=4.0, r1=10.0,
             p0=0.3, p1=0.6, order="lex", storage="f32", form="c8", steps=10, nt=True, chunk=16),
        # a new large geometry: list, adjacency and both code forms
        dict(name="assemble384_lex", kind="assemble", geom="spheres", nx=384, ny=384, nz=512,
             r0=8.0, r1=16.0, por=0.40, order="lex", param=0),
        # the empty channel of the ordering study on a curve whose cube is
        # much larger than the box
        dict(name="assemble_channel_hilbert", kind="assemble", geom="channel", nx=500, ny=100,
             nz=100, r0=0.0, r1=0.0, por=1.0, order="hilbert", param=0),
        # fields and totals of a tube-sized state
        dict(name="moments_tube_f64", kind="moments", geom="tube", nx=256, ny=256, nz=256,
             r0=12.0, r1=12.0, por=0.65, order="lex", param=0, storage="f64", fields=True),
    ]


FORMS = ("full", "full", "c16", "c8", "c8", "inplace", "inplace_c8", "graph_c8", "persistent_c8")


def _edge(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _order(rng):
    return rng.choice((("lex", 0), ("lex", 0), ("lex", 0), ("blocked", rng.choice((8, 16, 32, 64))),
                       ("morton2", 0), ("hilbert", 0)))


def draw(rng):
    kind = rng.choice(("sweep", "sweep", "sweep", "batch", "assemble", "moments", "adjoint"))
    order, param = _order(rng)
    nt, chunk = rng.choice(((False, 0), (False, 0), (True, 1), (True, 4), (True, 16), (True, 64)))
    storage = rng.choice(("f64", "f64s", "f32", "f32s", "f16s", "f16s12"))
    if kind == "adjoint":
        k = rng.randint(3, 22)
        return dict(kind=kind, nx=_edge(rng, 24, 128), ny=_edge(rng, 24, 128),
                    nz=_edge(rng, 24, 128), order=order, param=param,
                    storage=rng.choice(("f64", "f64s")), T=rng.randint(k, min(110, 6 * k)), k=k,
                    nt=nt, chunk=chunk)
    if kind == "batch":
        return dict(kind=kind, members=rng.randint(2, 48), l0=32, l1=rng.randint(64, 160), r0=4.0,
                    r1=10.0, p0=0.3, p1=0.6, order=rng.choice(("lex", "lex", "blocked")),
                    storage=storage, form=rng.choice(("full", "c8", "c8", "persistent_c8")),
                    steps=rng.randint(2, 10), nt=nt, chunk=chunk)
    nx, ny, nz = (_edge(rng, 32, 400) for _ in range(3))
    geom = rng.choice(("spheres", "spheres", "spheres", "tube", "channel"))
    r0 = rng.choice((4.0, 6.0, 8.0, 12.0))
    case = dict(kind=kind, geom=geom, nx=nx, ny=ny, nz=nz, r0=r0,
                r1=r0 * rng.choice((1.0, 2.0)), por=rng.choice((0.35, 0.4, 0.5, 0.6)),
                order=order, param=param)
    if kind == "moments":
        case.update(storage=storage, fields=rng.random() < 0.5)
    if kind == "sweep":
        case.update(storage=storage, form=rng.choice(FORMS),
                    steps=2 * max(1, min(50, int(2e7 / (nx * ny * nz)))), nt=nt, chunk=chunk,
                    pbb=rng.random() < 0.2)
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _spheres(gen, nx, ny, nz, r0, r1, por, dev):
    """uint8 [nz][ny][nx], 1 = fluid: walls on the y and z faces and enough
    overlapping spheres, radius uniform in [r0, r1], that the expected fluid
    share of the interior is por."""
    flags = torch.zeros((nz, ny, nx), dtype=torch.uint8, device=dev)
    flags[1:nz - 1, 1:ny - 1, :] = 1
    if por >= 1.0:
        return flags
    r3 = r0 ** 3 if r1 == r0 else (r1 ** 4 - r0 ** 4) / (4.0 * (r1 - r0))
    count = max(1, round(math.log(1.0 / por) * nx * ny * nz / (4.0 / 3.0 * math.pi * r3)))
    c = torch.rand((count, 4), generator=gen, dtype=torch.float64).to(dev)
    box = torch.tensor([nx, ny, nz], dtype=torch.float64, device=dev)
    centre, rad = c[:, :3] * box, r0 + c[:, 3] * (r1 - r0)
    R = int(math.ceil(r1)) + 1
    o = torch.arange(-R, R + 1, device=dev)
    flat = flags.view(-1)
    per = max(1, (1 << 24) // (2 * R + 1) ** 3)
    for a in range(0, count, per):
        ct, rr = centre[a:a + per], rad[a:a + per]
        base = ct.floor().long()
        p = [base[:, d, None] + o for d in range(3)]
        d2 = [(p[d].double() - ct[:, d, None]) ** 2 for d in range(3)]
        solid = d2[0][:, None, None, :] + d2[1][:, None, :, None] + d2[2][:, :, None, None] \
            <= (rr * rr)[:, None, None, None]
        solid &= ((p[1] >= 0) & (p[1] < ny))[:, None, :, None]
        solid &= ((p[2] >= 0) & (p[2] < nz))[:, :, None, None]
        lin = (p[0] % nx)[:, None, None, :] + nx * (p[1][:, None, :, None] + ny * p[2][:, :, None, None])
        flat[lin[solid]] = 0
    return flags


def _shifted(flags, seed):
    """The same geometry, shifted along the periodic direction and mirrored."""
    gen = torch.Generator().manual_seed(seed)
    shift, my, mz = (int(torch.randint(0, m, (1,), generator=gen)) for m in (flags.shape[2], 2, 2))
    if my or mz:
        flags = flags.flip([d for d, on in ((1, my), (0, mz)) if on])
    return flags.roll(shift, 2).contiguous()


def _flags(case, seed, dev):
    return _shifted(_placed(case, dev), seed)


def _placed(case, dev):
    gen = torch.Generator().manual_seed(7)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["kind"] == "adjoint":
        return _spheres(gen, nx, ny, nz, 1.0, 1.0, 1.0, dev)
    if case["geom"] == "channel":
        # the empty channel with a few obstacles, so that the shift matters
        flags = _spheres(gen, nx, ny, nz, 1.0, 1.0, 1.0, dev)
        z, y, x = (torch.randint(1, n - 1, (8,), generator=gen) for n in (nz, ny, nx))
        flags[z.to(dev), y.to(dev), x.to(dev)] = 0
        return flags
    flags = _spheres(gen, nx, ny, nz, case["r0"], case["r1"], case["por"], dev)
    if case["geom"] == "tube":
        y = torch.arange(ny, device=dev) - (ny - 1) / 2.0
        z = torch.arange(nz, device=dev) - (nz - 1) / 2.0
        r = 0.46875 * min(ny, nz)
        flags *= (z[:, None] ** 2 + y[None, :] ** 2 <= r * r)[:, :, None]
    return flags


def _noise(n, seed, dev):
    """(u0, FP64 [19][n] relative deviations of the initial populations)."""
    gen = torch.Generator(device=dev).manual_seed(seed)
    u0 = (torch.rand(3, generator=gen, device=dev, dtype=torch.float64) - 0.5) * 2e-2
    return u0, 1e-3 * torch.randn((19, n), generator=gen, device=dev, dtype=torch.float64)


W = [1.0 / 3.0] + [1.0 / 18.0] * 6 + [1.0 / 36.0] * 12
C = [(0, 0, 0)]
for _c in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1),
           (0, 1, 1), (0, 1, -1)):
    C += [_c, tuple(-v for v in _c)]
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _stored(storage, n, seed, dev):
    """The initial populations [19][n] as the storage form holds them."""
    u0, noise = _noise(n, seed, dev)
    for i in range(19):
        cu = sum(C[i][d] * u0[d] for d in range(3))
        h = W[i] * (3.0 * cu + 4.5 * cu * cu - 1.5 * (u0 * u0).sum())
        noise[i] = h + W[i] * noise[i]
    if storage in ("f64", "f32"):
        noise += torch.tensor(W, dtype=torch.float64, device=dev)[:, None]
    if storage == "f16s12":
        noise *= 4096.0
    return noise if SIZE[storage] == 8 else noise.to(torch.float32 if SIZE[storage] == 4
                                                     else torch.float16)


def _solid_fraction(nx, ny, nz, seed, dev):
    """Smoothed random solid fraction in [0, 1], FP64 [nz][ny][nx]."""
    gen = torch.Generator(device=dev).manual_seed(seed)
    phi = torch.randn((1, 1, nz // 4 + 2, ny // 4 + 2, nx // 4 + 2), generator=gen, device=dev,
                      dtype=torch.float64)
    phi = torch.nn.functional.interpolate(phi, size=(nz, ny, nx), mode="trilinear")[0, 0]
    return (0.5 + 0.5 * phi).clamp(0.0, 1.0)


def _force(case):
    return (1e-6, 2e-7, 0.0) if case["kind"] == "batch" else (1e-6, 0.0, 0.0)


def _params(case, storage=None):
    return L.params(TAU, MAGIC, _force(case), storage or case["storage"],
                    nontemporal=case.get("nt", False), xcd_chunk=case.get("chunk", 0))


# the members of a batch: box edges, flag fields and parameters
def _members(case, seed, dev):
    gen = torch.Generator().manual_seed(7)
    sizes = torch.Generator().manual_seed(77)
    out = []
    for k in range(case["members"]):
        edge = int(torch.randint(case["l0"], case["l1"] + 1, (1,), generator=sizes))
        t = torch.rand(2, generator=sizes)
        por = case["p0"] + float(t[0]) * (case["p1"] - case["p0"])
        flags = _spheres(gen, edge, edge, edge, case["r0"], case["r1"], por, dev)
        out.append((_shifted(flags, seed + k), 0.7 + 0.4 * float(t[1]), (1e-6 * (1 + k % 5), 2e-7, 0.0)))
    return out


def prepare(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind == "batch":
        mem = _members(case, seed, dev)
        b = L.Batch([m[0] for m in mem], [1] * len(mem), case["order"],
                    16 if case["order"] == "blocked" else 0, tile_align=True)
        st = b.init([L.params(tau, MAGIC, g, case["storage"], nontemporal=case["nt"],
                              xcd_chunk=case["chunk"]) for _, tau, g in mem])
        for k, (base, cnt) in enumerate(b.segments):
            st.f[:, base:base + cnt] = _stored(case["storage"], cnt, seed + 1000 * k, dev)
        comp = None
        if case["form"] != "full":
            comp = L.narrow(L.compress(b.lattice, n=b.total))
        return dict(case=case, st=st, comp=comp, segments=b.segments)
    flags = _flags(case, seed, dev)
    if kind == "assemble":
        return dict(case=case, flags=flags)
    lat = L.build(flags, 1, case["order"], case["param"])
    n = lat.n_fluid
    if kind == "adjoint":
        ns = torch.zeros(lat.stride, dtype=torch.float64, device=dev)
        frac = _solid_fraction(case["nx"], case["ny"], case["nz"], seed, dev)
        ns[:n] = frac.view(-1)[lat.cell_of.long()]
        return dict(case=case, lat=lat, prm=_params(case), ns=ns.requires_grad_(True))
    prm = L.params(TAU, MAGIC, _force(case), case["storage"]) if kind == "moments" else _params(case)
    ns = None
    if case.get("pbb"):
        ns = torch.zeros(lat.stride, dtype=torch.float64, device=dev)
        frac = _solid_fraction(case["nx"], case["ny"], case["nz"], seed, dev)
        ns[:n] = frac.view(-1)[lat.cell_of.long()]
    form = case.get("form", "full")
    comp = L.compress(lat) if form.endswith(("c16", "c8")) else None
    if form.endswith("c8"):
        L.narrow(comp)
    st = (L.init_inplace if form.startswith("inplace") else L.init)(lat, prm, ns=ns)
    st.f[:, :n] = _stored(case["storage"], n, seed, dev)
    graph = L.StepGraph(st, case["steps"], comp) if form.startswith("graph") else None
    return dict(case=case, lat=lat, st=st, comp=comp, graph=graph)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "sweep":
        st, form, k = s["st"], case["form"], case["steps"]
        if form == "full":
            L.step(st, k)
        elif form == "c16":
            L.step_c16(st, s["comp"], k)
        elif form == "c8":
            L.step_c8(st, s["comp"], k)
        elif form == "persistent_c8":
            L.step_c8(st, s["comp"], k, persistent=True)
        elif form == "graph_c8":
            s["graph"].replay()
        else:
            L.step_inplace(st, k, s["comp"], c8=form.endswith("c8"))
        return st.f[:, :st.n]
    if kind == "batch":
        st = s["st"]
        if case["form"] == "full":
            L.step(st, case["steps"])
        else:
            L.step_c8(st, s["comp"], case["steps"], persistent=case["form"].startswith("persistent"))
        _, _, totals = L.moments(st, fields=False)
        return [totals] + [st.f[:, b:b + c] for b, c in s["segments"]]
    if kind == "assemble":
        lat = L.build(s["flags"], 1, case["order"], case["param"])
        comp = L.narrow(L.compress(lat))
        n = lat.n_fluid
        return dict(n=n, index_of=lat.index_of, cell_of=lat.cell_of, adj=lat.adj,
                    codes=comp.codes[:, :n], records=comp.tile_records, codes8=comp.codes8[:, :n],
                    escapes=comp.n_escapes, narrow=comp.n_narrow)
    if kind == "moments":
        rho, u, totals = L.moments(s["st"], fields=case["fields"])
        return dict(rho=rho, u=u, totals=totals)
    ns = s["ns"]
    ns.grad = None
    J = AD.PermeabilityFn.apply(ns, s["lat"], s["prm"], case["T"], case["k"])
    J.backward()
    return dict(J=J.detach(), grad=ns.grad[:s["lat"].n_fluid])


# --------------------------------------------------------------------------
# work
# --------------------------------------------------------------------------

def _cells(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["kind"] == "adjoint" or case["geom"] == "channel":
        return nx * (ny - 2) * (nz - 2)
    if case["geom"] == "tube":
        return case["por"] * nx * math.pi * (0.46875 * min(ny, nz)) ** 2
    return case["por"] * nx * (ny - 2) * (nz - 2)


def _index_bytes(form):
    """Adjacency bytes a cell update reads: 18 uint32, or 18 codes of two or
    one bytes; the in-place sweep reads them every other step."""
    per = 18.0 if form.endswith("c8") else 36.0 if form.endswith("c16") else 72.0
    return per / 2 if form.startswith("inplace") else per


def work(case):
    kind = case["kind"]
    if kind == "batch":
        edge = 0.5 * (case["l0"] + case["l1"])
        mean3 = edge ** 3 * (1 + ((case["l1"] - case["l0"]) / edge) ** 2 / 4)
        n = case["members"] * mean3 * 0.5 * (case["p0"] + case["p1"])
        sz = SIZE[case["storage"]]
        return {"bytes": n * (case["steps"] * (38 * sz + _index_bytes(case["form"])) + 19 * sz + 72),
                "flops": 200.0 * n * case["steps"]}
    n, box = _cells(case), case["nx"] * case["ny"] * case["nz"]
    if kind == "assemble":
        # flags in; index_of, cell_of, adjacency, 16-bit and 8-bit codes out
        return {"bytes": 5.0 * box + n * (4 + 72 + 36 + 18), "flops": 0.0}
    if kind == "moments":
        return {"bytes": n * (19 * SIZE[case["storage"]] + 72 + (32 if case["fields"] else 0)),
                "flops": 60.0 * n}
    if kind == "adjoint":
        # forward sweep and adjoint step per time step over one-byte codes
        return {"bytes": n * case["T"] * (312 + 18 + 498.0), "flops": 700.0 * n * case["T"]}
    per = 38 * SIZE[case["storage"]] + _index_bytes(case["form"]) + (8 if case["pbb"] else 0)
    return {"bytes": n * case["steps"] * per, "flops": 200.0 * n * case["steps"]}


# --------------------------------------------------------------------------
# the same in 64 bits, with plain torch
# --------------------------------------------------------------------------

def _hilbert(x, y, z, bits):
    X = [x.clone(), y.clone(), z.clone()]
    q = 1 << max(bits - 1, 0)
    while q > 1:
        p = q - 1
        for i in range(3):
            on = (X[i] & q) != 0
            t = (X[0] ^ X[i]) & p
            x0 = torch.where(on, X[0] ^ p, X[0] ^ t)
            if i:
                X[i] = torch.where(on, X[i], X[i] ^ t)
            X[0] = x0
        q >>= 1
    X[1] = X[1] ^ X[0]
    X[2] = X[2] ^ X[1]
    t = torch.zeros_like(x)
    q = 1 << max(bits - 1, 0)
    while q > 1:
        t = torch.where((X[2] & q) != 0, t ^ (q - 1), t)
        q >>= 1
    X = [v ^ t for v in X]
    key = torch.zeros_like(x)
    for j in range(bits):
        for d in range(3):
            key |= ((X[d] >> j) & 1) << (3 * j + 2 - d)
    return key


def _list(flags, order, param):
    """(cells in list order, source index [18][n], bounce-back [18][n])."""
    nz, ny, nx = flags.shape
    lin = flags.reshape(-1).nonzero()[:, 0]
    x, y, z = lin % nx, (lin // nx) % ny, lin // (nx * ny)
    if order == "blocked":
        b = param
        key = (z // b) * ((ny + b - 1) // b) + y // b
        key = key * ((nx + b - 1) // b) + x // b
        key = ((key * b + z % b) * b + y % b) * b + x % b
    elif order == "morton2":
        key = torch.zeros_like(lin)
        for k in range(6):
            for d, v in enumerate((x, y, z)):
                key |= ((v >> (2 * k)) & 3) << (6 * k + 2 * d)
    elif order == "hilbert":
        key = _hilbert(x, y, z, (max(nx, ny, nz) - 1).bit_length())
    else:
        key = lin
    at = torch.argsort(key)
    lin, x, y, z = lin[at], x[at], y[at], z[at]
    n = lin.numel()
    index = torch.full((nx * ny * nz,), -1, dtype=torch.int64, device=lin.device)
    index[lin] = torch.arange(n, device=lin.device)
    src, bounce = [], []
    for i in range(1, 19):
        px, py, pz = (x - C[i][0]) % nx, y - C[i][1], z - C[i][2]
        out = (py < 0) | (py >= ny) | (pz < 0) | (pz >= nz)
        j = index[px + nx * (py.clamp(0, ny - 1) + ny * pz.clamp(0, nz - 1))]
        bounce.append(out | (j < 0))
        src.append(j.clamp(min=0))
    return lin, src, bounce


def _gather(f, src, bounce):
    return [f[0]] + [torch.where(bounce[i - 1], f[OPP[i]], f[i][src[i - 1]]) for i in range(1, 19)]


def _moments(g):
    rho = sum(g)
    j = [sum(C[i][d] * g[i] for i in range(19) if C[i][d]) for d in range(3)]
    return rho, j


def _collide(g, tau, force, ns=None):
    sp = 1.0 / tau
    sm = 1.0 / (0.5 + MAGIC / (tau - 0.5))
    rho, j = _moments(g)
    jj = j[0] * j[0] + j[1] * j[1] + j[2] * j[2]
    out = []
    for i in range(19):
        o = OPP[i]
        cj = sum(C[i][d] * j[d] for d in range(3) if C[i][d]) if i else 0.0
        ep = W[i] * (rho + 4.5 * cj * cj - 1.5 * jj)
        em = 3.0 * W[i] * cj
        v = g[i] - sp * (0.5 * (g[i] + g[o]) - ep) - sm * (0.5 * (g[i] - g[o]) - em) \
            + 3.0 * W[i] * sum(C[i][d] * force[d] for d in range(3))
        out.append(v if ns is None else (1.0 - ns) * v + ns * g[o])
    return out


def _sweeps64(f, src, bounce, steps, tau, force, scale, ns=None):
    f = [r.double() / scale for r in f]
    for _ in range(steps):
        f = _collide(_gather(f, src, bounce), tau, force, ns)
    return f


def exact(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind == "assemble":
        return None  # whole numbers
    if kind == "batch":
        rows, tot = [], []
        scale = 4096.0 if case["storage"] == "f16s12" else 1.0
        for k, (flags, tau, force) in enumerate(_members(case, seed, dev)):
            lin, src, bounce = _list(flags, case["order"], 16)
            f = _stored(case["storage"], lin.numel(), seed + 1000 * k, dev)
            f = _sweeps64(f, src, bounce, case["steps"], tau, force, scale)
            rho, j = _moments(_gather(f, src, bounce))
            if case["storage"] not in ("f64", "f32"):
                rho = rho + 1.0
            tot.append(torch.stack([rho.sum()] + [(j[d] + 0.5 * force[d]).sum() for d in range(3)]))
            rows.append(torch.stack(f) * scale)
        return [torch.stack(tot)] + rows
    flags = _flags(case, seed, dev)
    lin, src, bounce = _list(flags, case["order"], case["param"])
    n = lin.numel()
    force = _force(case)
    if kind == "adjoint":
        ns = _solid_fraction(case["nx"], case["ny"], case["nz"], seed, dev).view(-1)[lin].clone()
        return _adjoint64(case, src, bounce, n, ns, force)
    f = _stored(case["storage"], n, seed, dev)
    scale = 4096.0 if case["storage"] == "f16s12" else 1.0
    if kind == "moments":
        rho, j = _moments(_gather([r.double() / scale for r in f], src, bounce))
        if case["storage"] not in ("f64", "f32"):
            rho = rho + 1.0
        u = torch.stack([j[d] + 0.5 * force[d] for d in range(3)])
        totals = torch.cat([rho.sum()[None], u.sum(1)])[None]
        return dict(rho=rho, u=u, totals=totals) if case["fields"] else dict(rho=None, u=None,
                                                                             totals=totals)
    ns = None
    if case["pbb"]:
        ns = _solid_fraction(case["nx"], case["ny"], case["nz"], seed, dev).view(-1)[lin]
    return torch.stack(_sweeps64(f, src, bounce, case["steps"], TAU, force, scale, ns)) * scale


def _adjoint64(case, src, bounce, n, ns, force):
    """Mean flux after T sweeps from rest and its gradient: reverse mode of
    the plain step, one step at a time from the stored states."""
    shift = case["storage"] == "f64s"
    f = torch.stack([torch.full((n,), 0.0 if shift else W[i], dtype=torch.float64, device=ns.device)
                     for i in range(19)])
    states = []
    for _ in range(case["T"]):
        states.append(f)
        f = torch.stack(_collide(_gather(f, src, bounce), TAU, force, ns))
    _, j = _moments(_gather(f, src, bounce))
    J = (j[0] + 0.5 * force[0]).sum() / n
    # dJ/df: the slot a cell pulls for direction i carries c_ix / n
    lam = _scatter([torch.full((n,), C[i][0] / n, dtype=torch.float64, device=ns.device)
                    for i in range(19)], src, bounce)
    grad = torch.zeros_like(ns)
    for f in reversed(states):
        g = [r.requires_grad_(True) for r in _gather(f, src, bounce)]
        s = ns.detach().clone().requires_grad_(True)
        out = torch.stack(_collide(g, TAU, force, s))
        d = torch.autograd.grad(out, g + [s], grad_outputs=lam)
        grad += d[-1]
        lam = _scatter(d[:-1], src, bounce)
    return dict(J=J, grad=grad)


def _scatter(d, src, bounce):
    """Transpose of _gather (every slot is pulled exactly once)."""
    lam = torch.zeros((19, d[0].numel()), dtype=torch.float64, device=d[0].device)
    lam[0] = d[0]
    for i in range(1, 19):
        b = bounce[i - 1]
        lam[OPP[i]][b] = d[i][b]
        lam[i][src[i - 1][~b]] = d[i][~b]
    return lam
