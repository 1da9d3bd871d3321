"""Performance cases of the grid-inference library: what its callers run, at the sizes they run it.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw()` more of the same ranges,
`prepare()` the inputs and handles a caller holds before the call, `run()` one pass through the public
entry points, `work()` the bytes and operations a pass cannot do without, and `exact()` the same
outputs from plain 64-bit torch.

Precision of what `run` returns: the network and the descriptors are single precision, so the DOS,
the density, the Fermi level and the forces behind them are handed on as float32, as a program does
that writes a volume file or moves atoms; the reductions of a stored LDOS are double precision
throughout and are returned as such.
"""
import functools
import itertools
import math
import struct

import numpy as np
import torch

import paper_2411_19617_amd as mala

A_AL = 4.05                     # fcc aluminium, Angstrom
A_LIQUID = 4.211                # the same number of atoms at 2.4 g/cc
RCUT = 4.67
EGRID = (-5.0, 0.1, 250)        # energies: first, spacing (eV), count
KB = 8.617333262e-5


# ------------------------------------------------------------------ the cases

def listed():
    solid = dict(cells=4, a=A_AL, jitter=0.1, vacuum=0.0, T=298.0)
    liquid = dict(cells=4, a=A_LIQUID, jitter=0.45, vacuum=0.0, T=933.0)
    cell32 = dict(cells=2, a=A_AL, jitter=0.1, vacuum=0.0, T=298.0)
    big = dict(nx=90, ny=90, nz=90)
    return [
        # the 32-atom cell on its own grid: the smallest call, a unit cell in a parameter scan
        dict(name="descriptors_cell32", kind="descriptors", twojmax=8, nx=20, ny=20, nz=20, begin=0, count=8000, **cell32),
        # a shard of the 256-atom liquid: an odd range of its 729,000 points, tiles crossing rows
        dict(name="descriptors_liquid", kind="descriptors", twojmax=10, begin=100_003, count=200_003, **big, **liquid),
        # the network alone over the 256-atom cell's grid with the whole LDOS stored
        dict(name="network_fp32", kind="network", precision="fp32", points=729_000, n_in=91, h1=400, h2=400),
        # the same in the BF16 form over a ragged batch of points
        dict(name="network_bf16", kind="network", precision="bf16", points=262_147, n_in=91, h1=400, h2=400),
        # the network factor of the forces
        dict(name="network_vjp", kind="network_vjp", points=100_003, n_in=91, h1=400, h2=400),
        # the descriptor factor of the forces, a shard of the solid's grid
        dict(name="descriptors_vjp", kind="descriptors_vjp", twojmax=10, begin=7, count=65_537, **big, **solid),
        # observables of a stored LDOS (a file's worth of points)
        dict(name="integrate", kind="integrate", points=500_009, T=298.0),
        # whole calls: the 32-atom cell (a step of a small molecular-dynamics run), ...
        dict(name="predict_cell32", kind="predict", precision="fp32", twojmax=8, h1=100, h2=100, nx=20, ny=20, nz=20, **cell32),
        # ... the 256-atom solid, ...
        dict(name="predict_solid", kind="predict", precision="fp32", twojmax=10, h1=400, h2=400, **big, **solid),
        # ... and a 16,384-atom slab between vacuum, BF16 network
        dict(name="predict_slab_bf16", kind="predict", precision="bf16", twojmax=10, h1=400, h2=400, nx=156, ny=180, nz=208,
             cells=16, a=A_AL, jitter=0.1, vacuum=10.0, T=298.0),
        # grid ACE descriptors of ranks 1-3, rows per point (the default), a shard
        dict(name="ace", kind="ace", nmax=4, lmax=4, planes=False, begin=50_001, count=300_007, **big, **solid),
        # and of rank 4
        dict(name="ace4", kind="ace4", nmax=3, lmax=3, planes=False, begin=0, count=150_001, **big, **liquid),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_snapshot(rng, pts_lo, pts_hi):
    """A cell of 32 to 500 atoms, solid or liquid, on a grid of about that many points, edges of any parity."""
    hot = rng.random() < 0.4
    n = rng.randint(2, 5)
    g = _log_int(rng, pts_lo, pts_hi) ** (1.0 / 3.0)
    nx, ny, nz = (max(8, int(round(g * math.exp(rng.uniform(-0.15, 0.15))))) for _ in range(3))
    return dict(cells=n, a=A_LIQUID if hot else A_AL, jitter=0.45 if hot else round(rng.uniform(0.05, 0.2), 3), vacuum=0.0,
                T=round(rng.uniform(600.0, 1000.0) if hot else rng.uniform(200.0, 600.0), 1), nx=nx, ny=ny, nz=nz)


def _draw_range(rng, s, most):
    total = s["nx"] * s["ny"] * s["nz"]
    count = min(total, most, max(1000, int(total * rng.uniform(0.3, 1.0))))
    return dict(begin=rng.randint(0, total - count), count=count)


def draw(rng):
    kind = rng.choice(["descriptors", "descriptors", "network", "network", "network_vjp", "descriptors_vjp", "integrate",
                       "predict", "predict", "ace", "ace4"])
    if kind == "descriptors":
        s = _draw_snapshot(rng, 4_000, 600_000)
        return dict(kind=kind, twojmax=rng.choice([2, 4, 6, 8, 10]), **s, **_draw_range(rng, s, 400_000))
    if kind == "descriptors_vjp":
        s = _draw_snapshot(rng, 4_000, 200_000)
        return dict(kind=kind, twojmax=rng.choice([2, 4, 6, 8, 10]), **s, **_draw_range(rng, s, 100_000))
    if kind == "network":
        return dict(kind=kind, precision=rng.choice(["fp32", "bf16"]), points=_log_int(rng, 8_000, 700_000),
                    n_in=rng.choice([55, 91]), h1=_log_int(rng, 64, 448), h2=_log_int(rng, 64, 448))
    if kind == "network_vjp":
        return dict(kind=kind, points=_log_int(rng, 8_000, 300_000), n_in=rng.choice([55, 91]), h1=_log_int(rng, 64, 416),
                    h2=_log_int(rng, 64, 416))
    if kind == "integrate":
        return dict(kind=kind, points=_log_int(rng, 8_000, 700_000), T=round(rng.uniform(200.0, 1000.0), 1))
    if kind == "predict":
        return dict(kind=kind, precision=rng.choice(["fp32", "bf16"]), twojmax=rng.choice([8, 10]), h1=_log_int(rng, 64, 448),
                    h2=_log_int(rng, 64, 448), **_draw_snapshot(rng, 6_000, 700_000))
    s = _draw_snapshot(rng, 4_000, 500_000)
    if kind == "ace":
        return dict(kind=kind, nmax=rng.randint(2, 4), lmax=rng.randint(2, 4), planes=rng.random() < 0.4, **s,
                    **_draw_range(rng, s, 300_000))
    return dict(kind=kind, nmax=rng.randint(2, 3), lmax=rng.randint(2, 3), planes=rng.random() < 0.4, **s,
                **_draw_range(rng, s, 200_000))


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=None)
def _context():
    """The process's one library context, as a program keeps it."""
    return mala.Context(0)


def _snapshot(case, seed):
    """fcc cells, every coordinate displaced; a slab has vacuum on both sides along z."""
    n, a = case["cells"], case["a"]
    g = np.arange(n)
    corner = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 1, 3)
    basis = np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
    pos = ((corner + basis).reshape(-1, 3) + 0.1) * a
    rng = np.random.default_rng([seed, 1])
    pos = pos + case["jitter"] * rng.standard_normal(pos.shape)
    L = np.array([n * a] * 3)
    pos[:, 2] += case["vacuum"]
    L[2] += 2.0 * case["vacuum"]
    return np.mod(pos, L), L, (case["nx"], case["ny"], case["nz"])


def _net(n_in, h1, h2, seed, scaler=None):
    """Xavier-uniform weights; the output map puts 3 electrons per fcc atom below 6.2 eV."""
    rng = np.random.default_rng([seed, 2])
    w = [n_in, h1, h2, EGRID[2]]
    W, b = [], []
    for i in range(3):
        lim = math.sqrt(6.0 / (w[i] + w[i + 1]))
        W.append(rng.uniform(-lim, lim, (w[i + 1], w[i])).astype(np.float32).astype(np.float64))
        b.append(rng.uniform(-0.1, 0.1, w[i + 1]).astype(np.float32).astype(np.float64))
    if scaler is None:      # components of a descriptor row spread over orders of magnitude
        mean = 10.0 ** rng.uniform(0.0, 3.0, n_in)
        scaler = mean, mean * rng.uniform(0.05, 0.3, n_in)
    e = EGRID[0] + EGRID[1] * np.arange(EGRID[2])
    shift = 3.0 / (16.61 * (2.0 / 3.0) * 11.7 ** 1.5) * np.sqrt(e + 5.5)
    return dict(widths=w, W=W, b=b, mean=np.asarray(scaler[0], np.float32).astype(np.float64),
                std=np.asarray(scaler[1], np.float32).astype(np.float64), scale=(0.1 * shift).astype(np.float32).astype(np.float64),
                shift=shift.astype(np.float32).astype(np.float64), slope=0.01)


def _blob(net):
    f8 = lambda a: np.asarray(a, "<f8").tobytes()  # noqa: E731
    out = [b"MALANET1", struct.pack("<4id4i", 1, 3, 1, 0, net["slope"], *net["widths"]), f8(net["mean"]), f8(net["std"])]
    for W, b in zip(net["W"], net["b"]):
        out += [f8(W), f8(b)]
    return b"".join(out + [f8(net["scale"]), f8(net["shift"]), struct.pack("<Q", 0)])


def _net_state(case, seed):
    """Network, descriptor rows x0 ~ N(0, 1) around its scaler, a vector over the energies."""
    net = _net(case["n_in"], case["h1"], case["h2"], seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    mean, std = (torch.tensor(net[k], device="cuda", dtype=torch.float32) for k in ("mean", "std"))
    B = mean + std * torch.randn((case["points"], case["n_in"]), generator=g, device="cuda")
    if case["kind"] == "network_vjp":
        # the derivative jumps where a unit crosses its kink: rows within rounding of one are
        # replaced by rows that are not (to the left of the jump and to the right are both right)
        for _ in range(8):
            bad = torch.nonzero(_margin(net, B) < 1e-5).reshape(-1)
            if not len(bad):
                break
            B[bad] = mean + std * torch.randn((len(bad), case["n_in"]), generator=g, device="cuda")
    v = torch.randn((case["points"], EGRID[2]), generator=g, device="cuda") if case["kind"] == "network_vjp" else None
    return net, B, v


def _electrons(case):
    return 3.0 * 4 * case["cells"] ** 3


def _scaler(case, seed):
    """Mean and spread of the descriptors over a sample of the snapshot's grid points."""
    pos, L, N = _snapshot(case, seed)
    total = N[0] * N[1] * N[2]
    pts = np.sort(np.random.default_rng([seed, 3]).choice(total, min(total, 2048), replace=False))
    B = _exact_descriptors(pos, L, N, case["twojmax"], torch.as_tensor(pts, device="cuda"))
    return B.mean(0).cpu().numpy(), (B.std(0) + 1e-3).cpu().numpy()


def prepare(case, seed):
    ctx, kind = _context(), case["kind"]
    s = dict(case=case, ctx=ctx)
    if kind in ("network", "network_vjp"):
        net, s["B"], s["v"] = _net_state(case, seed)
        s["weights"] = ctx.weights(_blob(net), mala.PREC_BF16 if case.get("precision") == "bf16" else mala.PREC_FP32)
    elif kind == "integrate":
        s["ldos"], s["dV"], s["ne"] = _ldos(case, seed)
    else:
        s["pos"], s["L"], s["N"] = _snapshot(case, seed)
        if kind == "descriptors_vjp":
            g = torch.Generator(device="cuda").manual_seed(seed)
            s["g"] = torch.randn((case["count"], mala.n_descriptors(case["twojmax"])), generator=g, device="cuda")
        if kind == "predict":
            net = _net(mala.n_descriptors(case["twojmax"]), case["h1"], case["h2"], seed, _scaler(case, seed))
            s["weights"] = ctx.weights(_blob(net), mala.PREC_BF16 if case["precision"] == "bf16" else mala.PREC_FP32)
    return s


def _ldos(case, seed):
    """A free-electron-like LDOS with every point's own 10% scatter."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    e = EGRID[0] + EGRID[1] * torch.arange(EGRID[2], device="cuda")
    base = 3.0 / (16.61 * (2.0 / 3.0) * 11.7 ** 1.5) * torch.sqrt(e + 5.5)
    ldos = base * (1.0 + 0.1 * torch.randn((case["points"], EGRID[2]), generator=g, device="cuda"))
    return ldos, 16.61 / 2800.0, 3.0 * case["points"] / 2800.0


# ------------------------------------------------------------------ one pass

def run(s):
    case, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind == "network":
        return ctx.mala_ldos_infer(s["weights"], s["B"], EGRID[2])
    if kind == "network_vjp":
        return ctx.mala_ldos_vjp(s["weights"], s["B"], s["v"])
    if kind == "integrate":
        dos, dens, res = ctx.mala_integrate(s["ldos"], s["dV"], EGRID, case["T"], s["ne"])
        return {"dos": dos, "density": dens, "e_fermi": res.view(torch.float64)[:1]}
    if kind == "predict":
        dos, dens, res = ctx.mala_predict(s["weights"], s["pos"], s["L"], s["N"], RCUT, case["twojmax"], EGRID, case["T"],
                                          _electrons(case))
        return {"dos": dos.float(), "density": dens.float(), "e_fermi_e_band": res.view(torch.float64)[:2].float()}
    end = case["begin"] + case["count"]
    if kind == "descriptors":
        return ctx.mala_descriptors(s["pos"], s["L"], s["N"], RCUT, case["twojmax"], case["begin"], end)
    if kind == "descriptors_vjp":
        return -ctx.mala_descriptors_vjp(s["pos"], s["L"], s["N"], RCUT, case["twojmax"], s["g"], case["begin"], end).float()
    f = ctx.mala_ace_descriptors if kind == "ace" else ctx.mala_ace4_descriptors
    return f(s["pos"], s["L"], s["N"], RCUT, case["nmax"], case["lmax"], case["begin"], end, descriptor_major=case["planes"])


# ------------------------------------------------------------------ what a pass cannot do without

@functools.lru_cache(maxsize=None)
def _descriptor_flops(tj):
    """(per neighbour, per point): 22 per stored element of u, 10 per coupling term, 4 per product with u."""
    half = sum((J // 2 + 1) * (J + 1) for J in range(tj + 1))
    z = b = 0
    for j1, j2, j in _triples(tj):
        D = (j1 + j2 - j) // 2
        b += (j // 2 + 1) * (j + 1)
        rows = sum(1 for m in range(j // 2 + 1) for m1 in range(j1 + 1) if 0 <= m - m1 + D <= j2)
        cols = sum(min(j1, m + D) - max(0, m + D - j2) + 1 for m in range(j + 1))
        z += rows * cols
    return 22.0 * half, 10.0 * z + 4.0 * b


def work(case):
    kind = case["kind"]
    if kind in ("network", "network_vjp"):
        w = [case["n_in"], case["h1"], case["h2"], EGRID[2]]
        macs = w[0] * w[1] + w[1] * w[2] + w[2] * w[3]
        vjp = kind == "network_vjp"
        el = 2 if case.get("precision") == "bf16" else 4
        return {"bytes": 4.0 * case["points"] * ((2 if vjp else 1) * w[0] + w[3]) + el * macs,
                "flops": (4.0 if vjp else 2.0) * macs * case["points"]}
    if kind == "integrate":
        n = case["points"]
        return {"bytes": 4.0 * n * EGRID[2] + 8.0 * n, "flops": 4.0 * n * EGRID[2]}
    atoms = 4 * case["cells"] ** 3
    volume = (case["cells"] * case["a"]) ** 2 * (case["cells"] * case["a"] + 2.0 * case["vacuum"])
    nbr = 4.0 / 3.0 * math.pi * RCUT ** 3 * atoms / volume
    if kind in ("ace", "ace4"):
        n = mala.ace_count(case["nmax"], case["lmax"]) if kind == "ace" else mala.ace4_count(case["nmax"], case["lmax"])
        basis = case["nmax"] * (case["lmax"] + 1) * (case["lmax"] + 2) / 2
        return {"bytes": 4.0 * case["count"] * n + 24.0 * atoms, "flops": case["count"] * (4.0 * basis * nbr + 40.0 * n)}
    tj = case["twojmax"]
    per_nbr, per_pt = _descriptor_flops(tj)
    nB = len(_triples(tj))
    if kind == "predict":
        n = case["nx"] * case["ny"] * case["nz"]
        macs = nB * case["h1"] + case["h1"] * case["h2"] + case["h2"] * EGRID[2]
        return {"bytes": 8.0 * n + 24.0 * atoms + 4.0 * macs, "flops": n * (per_nbr * nbr + per_pt + 2.0 * macs)}
    vjp = kind == "descriptors_vjp"
    return {"bytes": 4.0 * case["count"] * nB + 24.0 * atoms * (2 if vjp else 1),
            "flops": case["count"] * (per_nbr * nbr + per_pt) * (3.0 if vjp else 1.0)}


# ------------------------------------------------------------------ 64 bits, plain torch

def _triples(tj):
    return [(a, b, c) for a in range(tj + 1) for b in range(a + 1) for c in range(a - b, min(tj, a + b) + 1, 2) if c >= a]


def _neighbours(pos, L, N, pts):
    """Displacements [points][k][3] to the atom images within the cutoff (padded: distance 2 rcut) and the atoms' indices."""
    dev = pts.device
    shifts = [range(-int(math.ceil(RCUT / L[d])), int(math.ceil(RCUT / L[d])) + 1) for d in range(3)]
    sh = np.array(list(itertools.product(*shifts))) * L
    img = (pos[None] + sh[:, None]).reshape(-1, 3)
    idx = np.tile(np.arange(len(pos)), len(sh))
    near = np.all((img > -RCUT) & (img < L + RCUT), axis=1)
    img, idx = torch.tensor(img[near], device=dev), torch.tensor(idx[near], device=dev)
    h = [L[d] / N[d] for d in range(3)]
    ijk = [torch.div(pts, N[1] * N[2], rounding_mode="floor"), torch.div(pts, N[2], rounding_mode="floor") % N[1], pts % N[2]]
    r = torch.stack([ijk[d].double() * h[d] for d in range(3)], 1)
    keep = ((img > r.min(0).values - RCUT) & (img < r.max(0).values + RCUT)).all(1)
    img, idx = img[keep], idx[keep]
    d2 = sum((img[None, :, d] - r[:, None, d]) ** 2 for d in range(3))
    k = max(1, int((d2 < RCUT * RCUT).sum(1).max())) if img.shape[0] else 0
    if k == 0:
        return torch.full((len(pts), 1, 3), 2.0 * RCUT, device=dev, dtype=torch.float64), torch.zeros((len(pts), 1), device=dev, dtype=torch.long)
    at = torch.topk(d2, k, dim=1, largest=False).indices
    d = img[at] - r[:, None, :]
    out = torch.gather(d2, 1, at) >= RCUT * RCUT
    d[out] = torch.tensor([2.0 * RCUT, 0.0, 0.0], device=dev, dtype=torch.float64)
    return d, idx[at]


@functools.lru_cache(maxsize=2)
def _sphere(tj):
    """Exact quadrature on S^3 for even polynomials of degree 3 tj, and the zonal functions U_j(q.s) of its nodes as
    coefficients over the monomials of q (degree <= tj)."""
    nt, na = (3 * tj // 2 + 2) // 2 + 1, 3 * tj // 2 + 1
    x, w = np.polynomial.legendre.leggauss(nt)
    t, w = 0.5 * (x + 1.0), 0.5 * w
    al = 2.0 * math.pi * np.arange(na) / na
    T, A, G = np.meshgrid(t, al, al, indexing="ij")
    Wt = (np.meshgrid(w, al, al, indexing="ij")[0] / (na * na)).reshape(-1)
    p1, p2 = 0.5 * (A + G), 0.5 * (A - G)
    S = np.stack([np.sqrt(1 - T) * np.cos(p1), np.sqrt(1 - T) * np.sin(p1), np.sqrt(T) * np.cos(p2), np.sqrt(T) * np.sin(p2)], -1).reshape(-1, 4)
    mono = [m for m in itertools.product(range(tj + 1), repeat=4) if sum(m) <= tj]
    deg = np.array([sum(m) for m in mono])
    multi = np.array([math.factorial(sum(m)) / math.prod(math.factorial(k) for k in m) for m in mono])
    sp = S[:, :, None] ** np.arange(tj + 1)
    sm = np.stack([sp[:, 0, m[0]] * sp[:, 1, m[1]] * sp[:, 2, m[2]] * sp[:, 3, m[3]] for m in mono], 0) * multi[:, None]
    cheb = [np.array([1.0]), np.array([0.0, 2.0])]
    while len(cheb) <= tj:
        c = np.concatenate([[0.0], 2.0 * cheb[-1]])
        c[: len(cheb[-2])] -= cheb[-2]
        cheb.append(c)
    C = [sm * np.pad(cheb[j], (0, tj + 1 - len(cheb[j])))[deg][:, None] for j in range(tj + 1)]
    dev = torch.device("cuda")
    return (torch.tensor(np.concatenate(C, 1), device=dev), torch.tensor(Wt, device=dev), torch.tensor(np.array(mono), device=dev), len(Wt))


def _bispectrum(d, tj):
    """B [points][triples] of displacements d: u^j is a function on S^3, f_j(s) = U_j(1.s) + sum_k fc_k U_j(q_k.s), and
    B(j1, j2, j) = (j + 1) times the mean of f_j1 f_j2 f_j over the sphere."""
    C, Wt, mono, ns = _sphere(tj)
    r = d.square().sum(-1).sqrt()
    fc = torch.where(r < RCUT, 0.5 * (torch.cos(math.pi * r / RCUT) + 1.0), torch.zeros_like(r))
    th = 0.99363 * math.pi / RCUT * r
    q = torch.cat([torch.cos(th)[..., None], (torch.sin(th) / r)[..., None] * d], -1)
    pw = [torch.ones_like(q)]
    for _ in range(tj):
        pw.append(pw[-1] * q)
    pw = torch.stack(pw, -1)
    M = (fc[..., None] * pw[:, :, 0][..., mono[:, 0]] * pw[:, :, 1][..., mono[:, 1]] * pw[:, :, 2][..., mono[:, 2]] * pw[:, :, 3][..., mono[:, 3]]).sum(1)
    M = M + (mono[:, 1:].sum(1) == 0).double()
    f = (M @ C).reshape(-1, tj + 1, ns)
    out, pair = [], {}
    for a, b, c in _triples(tj):
        if (a, b) not in pair:
            pair = {(a, b): f[:, a] * f[:, b] * Wt}
        out.append((c + 1) * (pair[a, b] * f[:, c]).sum(1))
    return torch.stack(out, 1)


def _exact_descriptors(pos, L, N, tj, pts, chunk=4096):
    return torch.cat([_bispectrum(_neighbours(pos, L, N, pts[k:k + chunk])[0], tj) for k in range(0, len(pts), chunk)])


def _exact_descriptors_vjp(pos, L, N, tj, pts, g, chunk=1024):
    out = torch.zeros((len(pos), 3), device=pts.device, dtype=torch.float64)
    for k in range(0, len(pts), chunk):
        d, idx = _neighbours(pos, L, N, pts[k:k + chunk])
        d = d.detach().requires_grad_(True)
        (_bispectrum(d, tj) * g[k:k + chunk].double()).sum().backward()
        out.index_add_(0, idx.reshape(-1), d.grad.reshape(-1, 3))
    return out


def _t(a):
    return torch.tensor(a, device="cuda", dtype=torch.float64)


def _forward(net, B):
    """LDOS of rows B, with every unit's pre-activation and the size of its terms."""
    x, zs = (B.double() - _t(net["mean"])) / _t(net["std"]), []
    for W, b in zip(net["W"], net["b"]):
        z = x @ _t(W).T + _t(b)
        zs.append((z, x))
        x = torch.where(z > 0, z, net["slope"] * z)
    return _t(net["scale"]) * x + _t(net["shift"]), zs


def _margin(net, B, chunk=65536):
    out = []
    for k in range(0, len(B), chunk):
        m = None
        for (z, x), W, b in zip(_forward(net, B[k:k + chunk])[1], net["W"], net["b"]):
            v = (z.abs() / (x.abs() @ _t(W).abs().T + _t(b).abs())).min(1).values
            m = v if m is None else torch.minimum(m, v)
        out.append(m)
    return torch.cat(out)


def _exact_network(net, B, chunk=65536):
    return torch.cat([_forward(net, B[k:k + chunk])[0] for k in range(0, len(B), chunk)])


def _exact_network_vjp(net, B, v, chunk=65536):
    out = []
    for k in range(0, len(B), chunk):
        zs = _forward(net, B[k:k + chunk])[1]
        d = v[k:k + chunk].double() * _t(net["scale"])
        for (z, _), W in zip(zs[::-1], net["W"][::-1]):
            d = (d * torch.where(z > 0, 1.0, net["slope"]).double()) @ _t(W)
        out.append(d / _t(net["std"]))
    return torch.cat(out)


def _fermi_weights(mu, T):
    """int f D = w.D and int f e D = v.D for D linear between the energies: 48-point Gauss-Legendre on every interval."""
    e0, de, n = EGRID
    x, wx = np.polynomial.legendre.leggauss(48)
    t, wx = 0.5 * (x + 1.0), 0.5 * de * wx
    e = e0 + de * (np.arange(n - 1)[:, None] + t)
    f = 1.0 / (1.0 + np.exp(np.clip((e - mu) / (KB * T), -700, 700)))
    w, v = np.zeros(n), np.zeros(n)
    for out, y in ((w, f), (v, f * e)):
        out[:-1] += (y * (1.0 - t) * wx).sum(1)
        out[1:] += (y * t * wx).sum(1)
    return w, v


def _exact_observables(ldos, dV, T, ne):
    """DOS, density, E_F and band energy of an LDOS given as a list of blocks of rows."""
    D = sum(b.double().sum(0) for b in ldos) * dV
    Dn = D.cpu().numpy()
    lo, hi = EGRID[0], EGRID[0] + EGRID[1] * (EGRID[2] - 1)
    for _ in range(70):
        mu = 0.5 * (lo + hi)
        lo, hi = (mu, hi) if _fermi_weights(mu, T)[0] @ Dn < ne else (lo, mu)
    w, v = _fermi_weights(0.5 * (lo + hi), T)
    return D, torch.cat([b.double() @ _t(w) for b in ldos]), 0.5 * (lo + hi), float(v @ Dn)


def _fact(n):
    return math.factorial(n)


@functools.lru_cache(maxsize=None)
def _w3j(a, b, c, x, y, z):
    if x + y + z or c < abs(a - b) or c > a + b or abs(x) > a or abs(y) > b or abs(z) > c:
        return 0.0
    tri = _fact(a + b - c) * _fact(a - b + c) * _fact(-a + b + c) / _fact(a + b + c + 1)
    pre = math.sqrt(tri * _fact(a + x) * _fact(a - x) * _fact(b + y) * _fact(b - y) * _fact(c + z) * _fact(c - z))
    s = 0.0
    for k in range(a + b + c + 1):
        t = (k, a + b - c - k, a - x - k, b + y - k, c - b + x + k, c - a - y + k)
        if min(t) >= 0:
            s += (-1) ** k / math.prod(_fact(i) for i in t)
    return (-1) ** (a - b - z) * pre * s


def _cg(a, x, b, y, c, z):
    return (-1) ** (a - b + z) * math.sqrt(2 * c + 1) * _w3j(a, b, c, x, y, -z)


def _ace_basis(d, nmax, lmax):
    """A[n, l, m] [points] complex: Chebyshev polynomials times the cosine cutoff, spherical harmonics, and the point's own term."""
    r = d.square().sum(-1).sqrt()
    fc = torch.where(r < RCUT, 0.5 * (torch.cos(math.pi * r / RCUT) + 1.0), torch.zeros_like(r))
    x = torch.clamp(2.0 * r / RCUT - 1.0, -1.0, 1.0)
    R = [torch.cos(n * torch.acos(x)) * fc for n in range(nmax)]
    ct = d[..., 2] / r
    xy = torch.complex(d[..., 0], d[..., 1]) / r
    A = {}
    for l in range(lmax + 1):
        for m in range(l + 1):
            p = torch.zeros_like(r)      # m-th derivative of the Legendre polynomial
            for k in range(l // 2 + 1):
                e = l - 2 * k
                if e >= m:
                    p = p + (-1) ** k * math.comb(l, k) * math.comb(2 * l - 2 * k, l) / 2.0 ** l * _fact(e) / _fact(e - m) * ct ** (e - m)
            Y = (-1) ** m * math.sqrt((2 * l + 1) / (4 * math.pi) * _fact(l - m) / _fact(l + m)) * p * xy ** m
            for n in range(nmax):
                a = (R[n] * Y).sum(1)
                if l == 0:
                    a = a + (-1) ** n / math.sqrt(4 * math.pi)
                A[n, l, m] = a
                if m:
                    A[n, l, -m] = (-1) ** m * a.conj()
    return A


def _ace_rows(d, nmax, lmax):
    A = _ace_basis(d, nmax, lmax)
    out = [A[n, 0, 0].real for n in range(nmax)]
    for l in range(lmax + 1):
        for n1, n2 in itertools.combinations_with_replacement(range(nmax), 2):
            out.append(sum((-1) ** m * (A[n1, l, m] * A[n2, l, -m]).real for m in range(-l, l + 1)))
    keys = [(n, l) for n in range(nmax) for l in range(lmax + 1)]
    for (n1, l1), (n2, l2), (n3, l3) in itertools.combinations_with_replacement(keys, 3):
        if l3 < abs(l1 - l2) or l3 > l1 + l2 or (l1 + l2 + l3) % 2:
            continue
        s = 0.0
        for m3 in range(-l3, l3 + 1):
            p = 0.0
            for m1 in range(max(-l1, -m3 - l2), min(l1, -m3 + l2) + 1):
                p = p + _w3j(l1, l2, l3, m1, -m1 - m3, m3) * A[n1, l1, m1] * A[n2, l2, -m1 - m3]
            s = s + (p * A[n3, l3, m3]).real
        out.append(s)
    return torch.stack(out, 1)


@functools.lru_cache(maxsize=None)
def _couplings(ls, same):
    """The intermediate couplings of four angular momenta whose invariants, summed over exchanges of equal keys, are independent."""
    perms = [p for p in itertools.permutations(range(4)) if all(same[p[i]] == same[i] for i in range(4))]
    kept, out = [], []
    for L in range(max(abs(ls[0] - ls[1]), abs(ls[2] - ls[3])), min(ls[0] + ls[1], ls[2] + ls[3]) + 1):
        T = np.zeros([2 * l + 1 for l in ls])
        for m in itertools.product(*(range(-l, l + 1) for l in ls[:3])):
            m4 = -sum(m)
            if abs(m4) <= ls[3] and abs(m[0] + m[1]) <= L:
                M = m[0] + m[1]
                T[m[0] + ls[0], m[1] + ls[1], m[2] + ls[2], m4 + ls[3]] = (_cg(ls[0], m[0], ls[1], m[1], L, M) * (-1) ** (L - M)
                                                                           * _cg(ls[2], m[2], ls[3], m4, L, -M) / math.sqrt(2 * L + 1))
        v = sum(np.transpose(T, p) for p in perms).ravel() / len(perms)
        sv = np.linalg.svd(np.array(kept + [v]), compute_uv=False)
        if np.sum(sv > 1e-9 * max(1.0, sv[0])) > len(kept):
            kept.append(v)
            out.append(L)
    return out


def _ace4_rows(d, nmax, lmax):
    A = _ace_basis(d, nmax, lmax)
    keys = [(n, l) for n in range(nmax) for l in range(lmax + 1)]
    pairs = {}

    def pair(p, q, L):
        if (p, q, L) not in pairs:
            (n1, l1), (n2, l2) = keys[p], keys[q]
            pairs[p, q, L] = [sum(_cg(l1, m, l2, M - m, L, M) * A[n1, l1, m] * A[n2, l2, M - m]
                                  for m in range(max(-l1, M - l2), min(l1, M + l2) + 1)) for M in range(-L, L + 1)]
        return pairs[p, q, L]

    out = []
    for ps in itertools.combinations_with_replacement(range(len(keys)), 4):
        ls = tuple(keys[p][1] for p in ps)
        if sum(ls) % 2:
            continue
        for L in _couplings(ls, tuple(ps.index(p) for p in ps)):
            a, b = pair(ps[0], ps[1], L), pair(ps[2], ps[3], L)
            out.append(sum((-1) ** (L - M) * (a[M + L] * b[L - M]).real for M in range(-L, L + 1)) / math.sqrt(2 * L + 1))
    return torch.stack(out, 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("network", "network_vjp"):
        net, B, v = _net_state(case, seed)
        return _exact_network(net, B) if v is None else _exact_network_vjp(net, B, v)
    if kind == "integrate":
        ldos, dV, ne = _ldos(case, seed)
        D, n, ef, _ = _exact_observables([ldos], dV, case["T"], ne)
        return {"dos": D, "density": n, "e_fermi": _t([ef])}
    pos, L, N = _snapshot(case, seed)
    if kind == "predict":
        if case["precision"] == "bf16" or N[0] * N[1] * N[2] > 1_000_000:      # 64 bits say little about BF16, and take long on the slab
            return None
        net = _net(len(_triples(case["twojmax"])), case["h1"], case["h2"], seed, _scaler(case, seed))
        total = N[0] * N[1] * N[2]
        B = _exact_descriptors(pos, L, N, case["twojmax"], torch.arange(total, device="cuda"))
        ldos = [_exact_network(net, B[k:k + 65536]) for k in range(0, total, 65536)]
        D, n, ef, eb = _exact_observables(ldos, float(np.prod(L)) / total, case["T"], _electrons(case))
        return {"dos": D, "density": n, "e_fermi_e_band": _t([ef, eb])}
    pts = torch.arange(case["begin"], case["begin"] + case["count"], device="cuda")
    if kind == "descriptors":
        return _exact_descriptors(pos, L, N, case["twojmax"], pts)
    if kind == "descriptors_vjp":
        g = torch.Generator(device="cuda").manual_seed(seed)
        g = torch.randn((case["count"], len(_triples(case["twojmax"]))), generator=g, device="cuda")
        return -_exact_descriptors_vjp(pos, L, N, case["twojmax"], pts, g)
    rows = _ace_rows if kind == "ace" else _ace4_rows
    B = torch.cat([rows(_neighbours(pos, L, N, pts[k:k + 16384])[0], case["nmax"], case["lmax"]) for k in range(0, len(pts), 16384)])
    return B.T.contiguous() if case["planes"] else B
