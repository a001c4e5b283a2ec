"""The work a user of this package has it do, as cases that can be timed and checked.

A case is a dict of plain values.  `listed()` names the ones that stand for the package's uses,
`draw(rng)` gives further ones of the same ranges, `prepare(case, seed)` makes what a program holds
before the call (inputs, operators, workspaces), `run(state)` is one pass through the public entry
points, `work(case)` the bytes and operations of the method itself, and `exact(case, seed)` the
results in 64 bits from plain torch.

Kinds of cases:
  lattice  one lattice solve and its density of states (`moments`, `dos`)
  batch    many perturbed spin cubes in one batched solve (`moments_batched`)
  serve    a stream of mixed requests through the server (`serve.Server`), all present at the start
  csr      one solve of a general sparse Hermitian matrix and its density of states
  dense    one solve of a dense symmetric matrix (`dense_moments`)
  green    site-diagonal Green's functions (`site_green`) or local densities of states (`ldos`)
  bounds   the spectral interval of a Hamiltonian (`lanczos_bounds`, clipped to Gershgorin)
"""
import math

import numpy as np
import torch

import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from paper_1105_5481_amd.serve import KPMRequest, Server

F64 = torch.float64
EPS = 0.01                       # spectral margin of the scale, the package's default


def device():
    return "cuda" if torch.cuda.is_available() else "cpu"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the paper-sized lattice: a call of well under a millisecond's work, latency counts
        dict(name="square_L32_f64", kind="lattice", Lx=32, Ly=32, Lz=0, spin=False, W=1.0, f64=True,
             M=256, R=8, K=1024),
        # a 3D spin texture in complex64, and the plain complex128 path users check it against
        dict(name="spin_cube_L64_c64", kind="lattice", Lx=64, Ly=64, Lz=64, spin=True, W=0.0, f64=False,
             M=1024, R=32, K=2048),
        dict(name="spin_cube_L64_c128", kind="lattice", Lx=64, Ly=64, Lz=64, spin=True, W=0.0, f64=True,
             M=1024, R=32, K=2048),
        # the largest single lattice: 4.2 million sites, 64 vectors streamed from HBM
        dict(name="anderson_L2048_f32", kind="lattice", Lx=2048, Ly=2048, Lz=0, spin=False, W=2.0, f64=False,
             M=4096, R=64, K=8192),
        # a 2D lattice of ordinary size with ragged extents and an odd vector count, in FP64
        dict(name="anderson_1001x750_f64", kind="lattice", Lx=1001, Ly=750, Lz=0, spin=False, W=2.0, f64=True,
             M=512, R=21, K=1024),
        # Monte-Carlo style batch: perturbed spin cubes of uneven size
        dict(name="batch256_L16-48_c64", kind="batch", count=256, Lmin=16, Lmax=48, f64=False, M=512, R=16),
        # serving: mixed 2D/3D, real/spin requests, all present when the server starts
        dict(name="serve_16req_logN12-18", kind="serve", n=16, logN_min=12.0, logN_max=18.0, mix=1005),
        # a general sparse matrix (13 entries per row, scattered columns)
        dict(name="csr_n100000_c64", kind="csr", n=100000, pairs=6, cplx=True, f64=False, M=512, R=16, K=1024),
        # the paper's dense experiments: the 10^3 lattice as a dense matrix, and the small matrix
        dict(name="dense_D1000_R1792", kind="dense", D=1000, M=1024, R=1792),
        dict(name="dense_D128_R1792", kind="dense", D=128, M=2048, R=1792),
        # Green's functions at 64 sites of a 3D spin texture
        dict(name="green_64sites_L48_c64", kind="green", Lx=48, Ly=48, Lz=48, spin=True, W=0.0, f64=False,
             M=1024, sites=64, ldos=False),
        # the spectral interval before a solve
        dict(name="lanczos_spin_L64_k100", kind="bounds", Lx=64, Ly=64, Lz=64, spin=True, W=0.0, k=100),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _extents(rng, lo, hi, dim):
    """Extents of a lattice of about N in [lo, hi] sites, its sides not quite equal."""
    L = _log(rng, lo, hi) ** (1.0 / dim)
    return [max(4, int(round(L * rng.uniform(0.75, 1.33)))) for _ in range(dim)] + [0] * (3 - dim)


def _seconds(updates, spin, f64, dim):
    """A rough cost of a lattice solve, to keep drawn cases below the largest listed one."""
    return updates / ((4.0e11 if spin else 6.0e11 if dim == 3 else 1.2e12) * (0.4 if f64 else 1.0))


def draw(rng):
    kind = rng.choice(["lattice"] * 5 + ["batch", "serve", "csr", "csr", "dense", "green", "bounds"])
    if kind == "lattice":
        dim, spin, f64 = rng.choice([2, 3]), rng.random() < 0.5, rng.random() < 0.35
        Lx, Ly, Lz = _extents(rng, 2.0 ** 10, 2.0 ** 22, dim)
        N = Lx * Ly * max(Lz, 1)
        R, M = int(round(_log(rng, 1, 64))), int(round(_log(rng, 64, 4096)))
        while _seconds(float(N) * R * M, spin, f64, dim) > 0.25:
            M, R = max(64, M // 2), R if M > 128 else max(1, R // 2)
        return dict(kind=kind, Lx=Lx, Ly=Ly, Lz=Lz, spin=spin, W=0.0 if spin else rng.choice([0.0, 1.0, 2.0]),
                    f64=f64, M=M, R=R, K=2 * M)
    if kind == "batch":
        count = int(round(_log(rng, 8, 256)))
        Lmin = rng.randint(8, 24)
        return dict(kind=kind, count=count, Lmin=Lmin, Lmax=Lmin + rng.randint(0, 24), f64=rng.random() < 0.25,
                    M=int(round(_log(rng, 64, 256 if count > 64 else 512))), R=rng.randint(4, 16))
    if kind == "serve":
        return dict(kind=kind, n=rng.randint(4, 16), logN_min=12.0, logN_max=rng.uniform(14.0, 17.0),
                    mix=rng.randrange(1 << 20))
    if kind == "csr":
        return dict(kind=kind, n=int(round(_log(rng, 2 ** 10, 2 ** 18))), pairs=rng.randint(2, 10),
                    cplx=rng.random() < 0.5, f64=rng.random() < 0.5, M=int(round(_log(rng, 64, 512))),
                    R=int(round(_log(rng, 1, 48))), K=1024)
    if kind == "dense":
        D, R = int(round(_log(rng, 32, 2048))), int(round(_log(rng, 16, 1792)))
        M = int(round(_log(rng, 64, 1024)))
        while 2.0 * D * D * R * (M // 2) > 4.0e12:
            M, R = max(64, M // 2), R if M > 128 else max(16, R // 2)
        return dict(kind=kind, D=D, M=M, R=R)
    spin, dim = rng.random() < 0.6, rng.choice([2, 3])
    if kind == "green":
        Lx, Ly, Lz = _extents(rng, 2.0 ** 10, 2.0 ** 17, dim)
        return dict(kind=kind, Lx=Lx, Ly=Ly, Lz=Lz, spin=spin, W=0.0 if spin else 2.0, f64=rng.random() < 0.35,
                    M=int(round(_log(rng, 128, 1024))), sites=int(round(_log(rng, 1, 64))), ldos=rng.random() < 0.5)
    Lx, Ly, Lz = _extents(rng, 2.0 ** 12, 2.0 ** 20, dim)
    return dict(kind=kind, Lx=Lx, Ly=Ly, Lz=Lz, spin=spin, W=0.0 if spin else 2.0, k=rng.randint(40, 200))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed, tag):
    g = torch.Generator(device="cpu")
    g.manual_seed((int(seed) * 1000003 + tag) & 0x7FFFFFFF)
    return g


def _rand(n, seed, tag):
    """n uniforms in [0, 1) as a device tensor; drawn on the host, so every run draws the same."""
    return torch.rand(n, dtype=F64, generator=_gen(seed, tag)).to(device())


def _spinor(u1, u2):
    """Spins uniform on the sphere as (cos(th/2), sin(th/2) cos(phi), sin(th/2) sin(phi))."""
    half, phi = torch.acos(1.0 - 2.0 * u1) / 2, 2.0 * math.pi * u2
    c, s = torch.cos(half), torch.sin(half)
    return torch.stack([c, s * torch.cos(phi), s * torch.sin(phi)], dim=1).contiguous()


def _lattice(Lx, Ly, Lz, spin, W, seed, tag=1):
    N = Lx * Ly * max(Lz, 1)
    lat = wl.Lattice(dim=3 if Lz else 2, L=(Lx, Ly, Lz if Lz else 1), t=1.0,
                     hop=wl.HOP_SPIN if spin else wl.HOP_REAL)
    if spin:
        lat.spinor = _spinor(_rand(N, seed, tag), _rand(N, seed, tag + 1))
    elif W > 0:
        lat.onsite = (_rand(N, seed, tag) - 0.5) * W
    return lat


def _batch_lattices(case, seed):
    """Perturbed textures: one spin per coordinate of the largest cube, restricted to each member's
    cube, with 1 to 8 spins of each drawn anew.  The sizes belong to the case."""
    n, top = case["count"], case["Lmax"]
    sizes = np.random.Generator(np.random.Philox(key=[1003, 5])).integers(case["Lmin"], top + 1, size=n)
    u = torch.stack([_rand(top ** 3, seed, 1), _rand(top ** 3, seed, 2)]).reshape(2, top, top, top)
    g = np.random.Generator(np.random.Philox(key=[int(seed), 3]))
    for L in (int(x) for x in sizes):
        w = u[:, :L, :L, :L].reshape(2, -1).contiguous()
        k = int(g.integers(1, 9))
        at = torch.from_numpy(g.choice(L ** 3, size=k, replace=False)).to(device())
        w[:, at] = torch.from_numpy(g.random(size=(2, k))).to(device())
        yield wl.Lattice(dim=3, L=(L, L, L), t=1.0, hop=wl.HOP_SPIN, spinor=_spinor(w[0], w[1]))


def _requests(case, seed):
    """Host-side requests of the serving recipe; shapes belong to the case, values to the seed."""
    shapes = wl.config5_stream(case["n"], rate=1.0, seed=case["mix"], logN_min=case["logN_min"],
                               logN_max=case["logN_max"], Ms=(256, 1024, 2048))
    out = []
    for r in shapes:
        rseed = (int(seed) * 65537 + r.rid) & 0x7FFFFFFF
        lat = r.lattice
        if lat.hop == wl.HOP_SPIN:
            th, ph = wl.spins_uniform(lat.N, rseed)
            lat = wl.Lattice(dim=lat.dim, L=lat.L, t=1.0, hop=wl.HOP_SPIN, spinor=wl.spinor_of(th, ph))
        else:
            lat = wl.Lattice(dim=lat.dim, L=lat.L, t=1.0, onsite=wl.anderson_onsite(lat.N, 2.0, rseed))
        out.append(KPMRequest(op=lat, M=r.M, R=r.R, vec=r.vec, seed=rseed, instance=0, arrival=0.0, rid=r.rid))
    return out


def _csr(case, seed):
    """A random sparse Hermitian matrix: the diagonal and, for each of `pairs` random permutations p,
    one entry at (i, p(i)) and its conjugate at (p(i), i).  Returns the CSR and its (n, 1 + 2 pairs)
    columns and values (duplicates add up)."""
    n, dev = case["n"], device()
    i = torch.arange(n, device=dev)
    cols, vals = [i], [torch.complex(_rand(n, seed, 1) - 0.5, torch.zeros(n, dtype=F64, device=dev))]
    for s in range(case["pairs"]):
        p = torch.randperm(n, generator=_gen(seed, 10 + s)).to(dev)
        q = torch.empty_like(p)
        q[p] = i
        re = 2.0 * _rand(n, seed, 100 + s) - 1.0
        im = 2.0 * _rand(n, seed, 200 + s) - 1.0 if case["cplx"] else torch.zeros_like(re)
        im = torch.where(p == i, torch.zeros_like(im), im)
        v = torch.complex(re, im)
        cols += [p, q]
        vals += [v, v[q].conj()]
    col, val = torch.stack(cols, 1), torch.stack(vals, 1)
    S = col.shape[1]
    rp = torch.arange(n + 1, dtype=torch.int64, device=dev) * S
    c = wl.CSR(n=n, row_ptr=rp, col=col.reshape(-1).to(torch.int32), val_re=val.real.reshape(-1).contiguous(),
               val_im=val.imag.reshape(-1).contiguous() if case["cplx"] else None)
    return c, col, val


def _dense(case, seed):
    """The 10 x 10 x 10 cube with unit hopping for D = 1000, else a Gaussian symmetric matrix; the
    cube with a little disorder, so that every seed is a matrix of its own."""
    D, dev = case["D"], device()
    if D == 1000:
        H = torch.diag((_rand(D, seed, 1) - 0.5) * 0.1)
        r = torch.arange(D, device=dev).reshape(10, 10, 10)
        for ax in range(3):
            for d in (-1, 1):
                H[r.reshape(-1), torch.roll(r, d, ax).reshape(-1)] -= 1.0
        return H.contiguous()
    X = torch.randn(D, D, dtype=F64, generator=_gen(seed, 1)).to(dev) / math.sqrt(2.0 * D)
    return (X + X.T).contiguous()


def _sites(case, seed):
    N = case["Lx"] * case["Ly"] * max(case["Lz"], 1)
    return np.random.Generator(np.random.Philox(key=[int(seed), 9])).choice(N, size=case["sites"], replace=False).tolist()


def _vec(spin):
    return kpm.VEC_PHASE if spin else kpm.VEC_RADEMACHER


def _prec(case):
    return kpm.F64 if case["f64"] else kpm.F32


def _build(op, prec):
    a, b = kpm.scale_from_bounds(*kpm.gershgorin(op), EPS)
    return kpm.Hamiltonian(op, a, b, prec)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=int(seed))
    if kind in ("lattice", "csr"):
        if kind == "lattice":
            op = _lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed)
            s["vec"] = _vec(case["spin"])
        else:
            op = _csr(case, seed)[0]
            s["vec"] = _vec(case["cplx"])
        s["ham"] = _build(op, _prec(case))
        n = s["ham"].workspace_bytes(case["M"], case["R"], s["vec"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["mu"] = torch.empty(case["M"], dtype=F64, device="cuda")
    elif kind == "batch":
        s["hams"] = [_build(lat, _prec(case)) for lat in _batch_lattices(case, seed)]
        s["mu"] = torch.empty(case["count"], case["M"], dtype=F64, device="cuda")
        s["seeds"] = [s["seed"] + i for i in range(case["count"])]
    elif kind == "serve":
        s["reqs"] = _requests(case, seed)
        s["server"] = Server(prec=kpm.F32, max_active=64, chunk=32)
    elif kind == "dense":
        s["H"] = _dense(case, seed)
        lim = float(s["H"].abs().sum(1).max()) if case["D"] == 1000 else 2.5
        s["a"], s["b"] = kpm.scale_from_bounds(-lim, lim, EPS)
        n = kpm.lib().kpm_dense_workspace_bytes(case["D"], case["M"], case["R"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    elif kind == "green":
        s["ham"] = _build(_lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed), _prec(case))
        s["sites"] = _sites(case, seed)
    else:
        op = _lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed)
        s["ham"] = kpm.Hamiltonian(op, 1.0, 0.0, kpm.F64)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind in ("lattice", "csr"):
        mu = kpm.moments(s["ham"], case["M"], case["R"], s["vec"], s["seed"], out=s["mu"], workspace=s["ws"])
        omega, rho = kpm.dos(mu, case["K"], s["ham"].a, s["ham"].b)
        return dict(mu=mu, omega=omega, rho=rho)
    if kind == "batch":
        kpm.moments_batched(s["hams"], case["M"], case["R"], kpm.VEC_PHASE, s["seeds"], outs=list(s["mu"]))
        return dict(mu=s["mu"])
    if kind == "serve":
        res = s["server"].run(s["reqs"], clock="chunks")
        return dict(mu=[r.mu for r in res], rho=[r.rho for r in res])
    if kind == "dense":
        return dict(mu=kpm.dense_moments(s["H"], s["a"], s["b"], case["M"], case["R"], seed=s["seed"],
                                         workspace=s["ws"]))
    if kind == "green":
        f = kpm.ldos if case["ldos"] else kpm.site_green
        omega, g = f(s["ham"], s["sites"], case["M"])
        return dict(omega=omega, g=g)
    r = kpm.lanczos_bounds(s["ham"], case["k"], s["seed"])
    return {k: r[k] for k in ("e_lo", "e_hi", "theta_min", "theta_max", "m", "alpha", "beta")}


# ---------------------------------------------------------------------------
# what the method cannot do without
# ---------------------------------------------------------------------------
def _solve_work(N, M, R, cplx, slots, spin_or_csr_bytes, onsite):
    """(bytes, flops): the operator's input and the moments; per vector element and step the stencil,
    2 v - r and the two dot products."""
    per = (8.0 * slots + 4.0 + 8.0) if cplx else (2.0 * slots + 2.0 + 4.0)
    return spin_or_csr_bytes + 8.0 * N * onsite + 8.0 * M, float(N) * R * (M // 2) * per


def _lattice_work(Lx, Ly, Lz, spin, W, M, R):
    N = Lx * Ly * max(Lz, 1)
    return _solve_work(N, M, R, spin, 6 if Lz else 4, 24.0 * N if spin else 0.0, 1 if W > 0 else 0)


def work(case):
    kind = case["kind"]
    if kind == "lattice":
        b, f = _lattice_work(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], case["M"], case["R"])
        b, f = b + 16.0 * case["K"], f + 2.0 * case["M"] * case["K"]
    elif kind == "csr":
        per = 1 + 2 * case["pairs"]
        b, f = _solve_work(case["n"], case["M"], case["R"], case["cplx"], per,
                           case["n"] * per * (4.0 + (16.0 if case["cplx"] else 8.0)), 0)
    elif kind == "batch":
        b = f = 0.0
        sizes = np.random.Generator(np.random.Philox(key=[1003, 5])).integers(case["Lmin"], case["Lmax"] + 1,
                                                                              size=case["count"])
        for L in (int(x) for x in sizes):
            x, y = _lattice_work(L, L, L, True, 0.0, case["M"], case["R"])
            b, f = b + x, f + y
    elif kind == "serve":
        b = f = 0.0
        for r in wl.config5_stream(case["n"], rate=1.0, seed=case["mix"], logN_min=case["logN_min"],
                                   logN_max=case["logN_max"], Ms=(256, 1024, 2048)):
            L = r.lattice.L
            x, y = _lattice_work(L[0], L[1], L[2] if r.lattice.dim == 3 else 0, r.lattice.hop == wl.HOP_SPIN, 2.0,
                                 r.M, r.R)
            b, f = b + x + 32.0 * r.M, f + y
    elif kind == "dense":
        D = float(case["D"])
        b, f = 8.0 * D * D + 8.0 * case["M"], (2.0 * D * D + 6.0 * D) * case["R"] * (case["M"] // 2)
    elif kind == "green":
        b, f = _lattice_work(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], case["M"], case["sites"])
        b += 32.0 * case["M"] * case["sites"]
    else:
        N = case["Lx"] * case["Ly"] * max(case["Lz"], 1)
        c = 2.0 if case["spin"] else 1.0
        b = (24.0 if case["spin"] else 8.0) * N
        f = N * case["k"] * c * ((8.0 if case["spin"] else 2.0) * (6 if case["Lz"] else 4) / c + 12.0)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
_LOW = 0xFFFFFFFF


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _mulhi(a, b):
    """High half of the unsigned 64 x 64 product of a tensor and a constant (int64 bit patterns)."""
    b0, b1 = b & _LOW, (b >> 32) & _LOW
    a0, a1 = a & _LOW, (a >> 32) & _LOW
    p00, p01, p10, p11 = a0 * b0, a0 * b1, a1 * b0, a1 * b1
    mid = ((p00 >> 32) & _LOW) + (p01 & _LOW) + (p10 & _LOW)
    return p11 + ((p01 >> 32) & _LOW) + ((p10 >> 32) & _LOW) + (mid >> 32)


def _philox(i, rq, seed, instance):
    """Philox4x64-10 (Salmon et al., SC'11), key (seed, 4), counter (i, rq, instance, 0)."""
    M0, M1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    c = [i, rq, torch.full_like(i, _signed(int(instance))), torch.zeros_like(i)]
    k0, k1 = int(seed), 4
    for _ in range(10):
        h0, h1 = _mulhi(c[0], M0), _mulhi(c[2], M1)
        l0, l1 = c[0] * _signed(M0), c[2] * _signed(M1)
        c = [h1 ^ c[1] ^ _signed(k0), l1, h0 ^ c[3] ^ _signed(k1), l0]
        k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    return c


def _start(N, R, phase, seed, instance=0):
    """The (N, R) start block: random phases or +-1."""
    i = torch.arange(N, device=device())
    cols = []
    for q in range((R + 3) // 4):
        for w in _philox(i, torch.full_like(i, q), seed, instance):
            if len(cols) < R:
                if phase:
                    a = ((w >> 34) & ((1 << 30) - 1)).to(F64) * (2.0 * math.pi / 2 ** 30)
                    cols.append(torch.complex(torch.cos(a), torch.sin(a)))
                else:
                    cols.append(torch.where(w < 0, -1.0, 1.0).to(F64))
    return torch.stack(cols, 1)


def _table(lat):
    """Neighbours (N, S), their hopping, and the diagonal of a lattice."""
    Lx, Ly, Lz = lat.L[0], lat.L[1], lat.L[2] if lat.dim == 3 else 1
    site = torch.arange(lat.N, device=device()).reshape(Lz, Ly, Lx)
    nb = torch.stack([torch.roll(site, d, ax).reshape(-1) for ax in (2, 1, 0)[:lat.dim] for d in (1, -1)], 1)
    if lat.hop == wl.HOP_SPIN:
        u = torch.as_tensor(lat.spinor, device=device())
        up = torch.complex(u[:, 1], u[:, 2])
        w = torch.stack([-(u[:, 0] * u[nb[:, s], 0] + up.conj() * up[nb[:, s]]) for s in range(nb.shape[1])], 1)
    else:
        w = torch.full(nb.shape, -1.0, dtype=F64, device=device())
    d = torch.zeros(lat.N, dtype=F64, device=device()) if lat.onsite is None else torch.as_tensor(lat.onsite, device=device())
    return nb, w, d


def _scale(d, w, off=None):
    r = w.abs().sum(1) if off is None else (w.abs() * off).sum(1)
    lo, hi = float((d - r).min()), float((d + r).max())
    return (hi - lo) / (2.0 - EPS), (hi + lo) / 2.0


def _dots(apply, v0, M, reduce):
    """Moments (unnormalised) by T_n T_n and T_{n+1} T_n, of start block v0, each dot product taken
    by `reduce` from the elementwise products."""
    mul = (lambda x, y: x.real * y.real + x.imag * y.imag) if v0.is_complex() else (lambda x, y: x * y)
    n0 = reduce(mul(v0, v0))
    mu = [n0]
    prev, cur = v0, apply(v0)
    n1 = reduce(mul(cur, prev))
    if M > 1:
        mu.append(n1)
    for n in range(1, M // 2 + 1):
        if 2 * n < M:
            mu.append(2.0 * reduce(mul(cur, cur)) - n0)
        if 2 * n + 1 < M:
            prev, cur = cur, apply(cur).mul_(2.0).sub_(prev)
            mu.append(2.0 * reduce(mul(cur, prev)) - n1)
    return torch.stack(mu[:M])


def _applier(nb, w, d, a, b):
    w, d = w / a, (d - b) / a

    def apply(v):
        out = d[:, None] * v
        for s in range(nb.shape[1]):
            out.addcmul_(w[:, s:s + 1].to(v.dtype), v[nb[:, s]])
        return out
    return apply


def _cheap(N, R, M, cplx, slots, limit=8.0):
    """Whether the plain evaluation stays within about `limit` seconds."""
    steps = M // 2
    return steps * (3 + 2 * slots) * max(1.2e-5, N * R * (16.0 if cplx else 8.0) * 3 / 2.5e12) < limit and \
        torch.cuda.is_available()


def _solve(op, M, R, seed):
    nb, w, d = op
    a, b = _scale(d, w)
    v = _start(nb.shape[0], R, w.is_complex(), seed)
    return _dots(_applier(nb, w, d, a, b), v, M, lambda x: x.sum()) / (nb.shape[0] * R), a, b


def _cosines(M, K):
    """(theta_k, n theta_k) of the K Chebyshev points, the product reduced exactly."""
    m = torch.arange(M, device=device())[None, :] * (2 * torch.arange(K, device=device())[:, None] + 1) % (4 * K)
    th = (torch.arange(K, dtype=F64, device=device()) + 0.5) * (math.pi / K)
    return th, m.to(F64) * (math.pi / (2 * K))


def _jackson(M):
    n = torch.arange(M, dtype=F64, device=device())
    q = math.pi / (M + 1)
    return ((M - n + 1) * torch.cos(q * n) + torch.sin(q * n) / math.tan(q)) / (M + 1)


def _dos(mu, K, a, b):
    """mu (..., M) -> omega (K), rho (..., K)."""
    M = mu.shape[-1]
    th, ang = _cosines(M, K)
    w = _jackson(M) * mu * 2.0
    w[..., 0] /= 2.0
    return a * torch.cos(th) + b, (w @ torch.cos(ang).T) / (math.pi * torch.sin(th)) / a


def _green(mu, K, a, b, lam=4.0):
    M = mu.shape[-1]
    th, ang = _cosines(M, K)
    n = torch.arange(M, dtype=F64, device=device())
    w = torch.sinh(lam * (1.0 - n / M)) / math.sinh(lam) * mu * 2.0
    w[..., 0] /= 2.0
    re, im = -(w @ torch.sin(ang).T) / torch.sin(th) / a, -(w @ torch.cos(ang).T) / torch.sin(th) / a
    return a * torch.cos(th) + b, torch.complex(re, im)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("lattice", "csr"):
        cplx = case["spin"] if kind == "lattice" else case["cplx"]
        N = case["Lx"] * case["Ly"] * max(case["Lz"], 1) if kind == "lattice" else case["n"]
        slots = (6 if case["Lz"] else 4) if kind == "lattice" else 2 * case["pairs"]
        if not _cheap(N, case["R"], case["M"], cplx, slots):
            return None
        if kind == "lattice":
            op = _table(_lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed))
        else:
            _, col, val = _csr(case, seed)
            # a permutation's fixed point is a second diagonal entry
            own = col == torch.arange(N, device=device())[:, None]
            d = (val.real * own).sum(1)
            op = (col, torch.where(own, torch.zeros_like(val), val), d)
            op = op if cplx else (col, op[1].real.contiguous(), d)
        mu, a, b = _solve(op, case["M"], case["R"], seed)
        omega, rho = _dos(mu, case["K"], a, b)
        return dict(mu=mu, omega=omega, rho=rho)
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "serve":
        mus, rhos, left = [], [], 10.0
        for r in _requests(case, seed):
            mu = rho = None
            N, cplx, slots = r.op.N, r.op.hop == wl.HOP_SPIN, 2 * r.op.dim
            cost = (r.M // 2) * (3 + 2 * slots) * max(1.2e-5, N * r.R * (16.0 if cplx else 8.0) * 3 / 2.5e12)
            if cost < left and torch.cuda.is_available():
                left -= cost
                mu, a, b = _solve(_table(r.op), r.M, r.R, r.seed)
                rho = _dos(mu, 2 * r.M, a, b)[1]
            mus.append(mu)
            rhos.append(rho)
        return dict(mu=mus, rho=rhos)
    if kind == "dense":
        D, R = case["D"], case["R"]
        if 2.0 * D * D * R * (case["M"] // 2) > 2.0e13 or not torch.cuda.is_available():
            return None
        H = _dense(case, seed)
        lim = float(H.abs().sum(1).max()) if D == 1000 else 2.5
        H = H / (2.0 * lim / (2.0 - EPS))
        v = _start(D, R, False, seed)
        return dict(mu=_dots(lambda x: H @ x, v, case["M"], lambda x: x.sum()) / (D * R))
    if kind == "green":
        N, S = case["Lx"] * case["Ly"] * max(case["Lz"], 1), case["sites"]
        if not _cheap(N, S, case["M"], case["spin"], 6 if case["Lz"] else 4):
            return None
        nb, w, d = _table(_lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed))
        a, b = _scale(d, w)
        v = torch.zeros(N, S, dtype=w.dtype, device=device())
        v[torch.tensor(_sites(case, seed), device=device()), torch.arange(S, device=device())] = 1.0
        mu = _dots(_applier(nb, w, d, a, b), v, case["M"], lambda x: x.sum(0)).T
        omega, g = (_dos if case["ldos"] else _green)(mu, 2 * case["M"], a, b)
        return dict(omega=omega, g=g)
    return _exact_bounds(case, seed)


def _exact_batch(case, seed):
    """All members as one block-diagonal operator."""
    parts, own, base = [], [], 0
    for h, lat in enumerate(_batch_lattices(case, seed)):
        nb, w, d = _table(lat)
        a, b = _scale(d, w)
        parts.append((nb + base, w / a, (d - b) / a, _start(lat.N, case["R"], True, int(seed) + h, h)))
        own.append(torch.full((lat.N,), h, device=device()))
        base += lat.N
    if not _cheap(base, case["R"], case["M"], True, 6, 15.0):
        return None
    nb, w, d, v = (torch.cat([p[k] for p in parts]) for k in range(4))
    own = torch.cat(own)
    count = torch.bincount(own, minlength=case["count"]).to(F64)
    del parts

    def reduce(x):
        return torch.zeros(case["count"], dtype=F64, device=device()).index_add_(0, own, x.sum(1))
    mu = _dots(_applier(nb, w, d, 1.0, 0.0), v, case["M"], reduce).T / (count * case["R"])[:, None]
    return dict(mu=mu.contiguous())


def _exact_bounds(case, seed):
    """The Lanczos interval; the coefficients themselves depend on rounding once the process loses
    orthogonality, so only the extreme Ritz values and the interval they give are compared."""
    nb, w, d = _table(_lattice(case["Lx"], case["Ly"], case["Lz"], case["spin"], case["W"], seed))
    glo, ghi = (lambda r: (float((d - r).min()), float((d + r).max())))(w.abs().sum(1))
    apply = _applier(nb, w, d, 1.0, 0.0)
    v = _start(nb.shape[0], 1, case["spin"], seed)
    v = v / torch.linalg.vector_norm(v)
    alpha, beta, prev = [], [], torch.zeros_like(v)
    for _ in range(case["k"]):
        u = apply(v)
        al = (u.conj() * v).sum().real
        u = u - al * v - (beta[-1] if beta else 0.0) * prev
        be = torch.linalg.vector_norm(u)
        alpha.append(al)
        beta.append(be)
        prev, v = v, u / be
    T = torch.diag(torch.stack(alpha)) + torch.diag(torch.stack(beta[:-1]), 1) + torch.diag(torch.stack(beta[:-1]), -1)
    th, y = (x.cpu() for x in torch.linalg.eigh(T.cpu()))
    res = float(beta[-1]) * y[-1].abs()
    wid = float(th[-1] - th[0])
    lo = float(th[0]) - max(float(res[0]), 0.005 * wid)
    hi = float(th[-1]) + max(float(res[-1]), 0.005 * wid)
    return dict(e_lo=max(lo, glo), e_hi=min(hi, ghi), theta_min=float(th[0]), theta_max=float(th[-1]),
                m=case["k"], alpha=None, beta=None)
