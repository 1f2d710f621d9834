"""Timed workloads of the lMBD path: inputs, one pass through the public entry points, and
a plain 64-bit evaluation of the method to compare small cases with.

The structures are seeded random ones of the kinds the rest of the repository uses: carbon
at 2.0 g/cm^3 (periodic cubes) or 64 atoms per (12 A)^3 (open cubes), and H/C/N/O
50/30/10/10 at 1.0 g/cm^3 (periodic cubes and open spheres), with a minimum distance of
1.3 or 0.9 A and Hirshfeld ratios in [0.6, 1.0]; 12 quadrature nodes, n_max = 6.
"""
import math

import numpy as np
import torch

import paper_2407_06409_amd as P

BOHR, HARTREE = 0.529177210903, 27.211386245988
# alpha0 (bohr^3), C6 (Ha bohr^6), R0 (bohr) of H, C, N, O
SPECIES = [[4.5, 6.5, 3.10], [12.0, 46.6, 3.59], [7.4, 24.2, 3.34], [5.4, 15.6, 3.19]]
MASS = [1.008, 12.011, 14.007, 15.999]
BETA, DAMP, R_BUF, R_INNER, N_MAX, N_FREQ = 0.83, 6.0, 0.5, 2.0, 6, 12
_x, _w = np.polynomial.legendre.leggauss(N_FREQ)
OMEGA, WEIGHT = 0.5 * (1.0 + _x) / (1.0 - _x), _w / (1.0 - _x) ** 2

DENSITY = {"carbon_box": 2.0 / 12.011 / 1.66053906660, "carbon_open": 64.0 / 12.0 ** 3,
           "hcno_box": 1.0 / 7.1084 / 1.66053906660, "hcno_open": 1.0 / 7.1084 / 1.66053906660}   # atoms per A^3


def _case(name, kind, atoms, rc, precision="fp64", out="forces", r1=0.0, r2=0.0, cn="series", requests=1, host=False):
    """kind: structure; rc: r_SCS (and every other radius unless r1, r2 > 0: r_MBD,1, r_MBD,2 and
    r_nbr = r1 + r2); out: "energy", "forces", or "train" (autograd: energies, then the gradients in
    positions and Hirshfeld ratios); requests: structures of one batch; host: numpy arrays in and out."""
    d = dict(kind=kind, atoms=atoms, rc=rc, precision=precision, out=out, r1=r1, r2=r2, cn=cn, requests=requests, host=host)
    return dict(d, name=name) if name else d


def listed():
    return [
        # a molecule-sized cluster: the energy of one configuration, where launches and latency count
        _case("cluster64_energy", "carbon_open", 64, 5.0, out="energy"),
        # the same with forces: one step of molecular dynamics or of a relaxation on a small system
        _case("cluster64_forces", "carbon_open", 64, 5.0),
        # the smallest periodic request, from and to host arrays, as a caller without device arrays sends it
        _case("host60_mixed", "hcno_box", 60, 5.0, "mixed", host=True),
        # a batch of requests of several sizes, open and periodic, evaluated in one call
        _case("requests12_mixed", "requests", 2400, 5.5, "mixed", requests=12),
        # one training step on a box: energies, then gradients in positions and Hirshfeld ratios
        _case("train216", "carbon_box", 216, 6.0, out="train"),
        # the repository's benchmark: 1,728 C, energy and forces
        _case("box1728", "carbon_box", 1728, 6.0),
        # the same in mixed precision
        _case("box1728_mixed", "carbon_box", 1728, 6.0, "mixed"),
        # a molecular liquid, energies alone (scoring configurations, Monte Carlo)
        _case("liquid4096_energy", "hcno_box", 4096, 6.0, out="energy"),
        # the largest box of the repository's benchmark, in mixed precision
        _case("box13824_mixed", "carbon_box", 13824, 6.0, "mixed"),
        # the two-radius regime with moderate radii: sparse products, about 300 sites per neighbourhood
        _case("two_radius1728", "carbon_box", 1728, 6.0, r1=6.0, r2=3.0),
        # coefficients fitted to the spectrum bounds of every atom and node
        _case("fitted1728", "carbon_box", 1728, 6.0, cn="fit"),
        # production radii 10 + 8 A: about 2,450 sites per neighbourhood
        _case("production512", "carbon_box", 512, 6.0, r1=10.0, r2=8.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["cluster", "host", "requests", "train", "box", "box", "liquid", "two_radius", "fitted", "production"])
    prec = rng.choice(["fp64", "mixed"])
    rc = round(rng.uniform(5.0, 6.0), 2)
    if family == "cluster":
        return _case(None, rng.choice(["carbon_open", "hcno_open"]), _log(rng, 12, 400), rc, prec, rng.choice(["energy", "forces"]))
    if family == "host":
        return _case(None, "hcno_box", _log(rng, 50, 800), rc, prec, host=True)
    if family == "requests":
        n = rng.randint(3, 24)
        return _case(None, "requests", _log(rng, 60 * n, 250 * n), rc, prec, requests=n)
    if family == "train":
        return _case(None, rng.choice(["carbon_box", "hcno_box"]), _log(rng, 64, 700), rc, prec, "train")
    if family == "box":
        return _case(None, "carbon_box", _log(rng, 100, 6000 if prec == "mixed" else 3000), rc, prec, rng.choice(["energy", "forces"]))
    if family == "liquid":
        return _case(None, "hcno_box", _log(rng, 100, 5000), rc, prec, rng.choice(["energy", "forces"]))
    if family == "two_radius":
        return _case(None, "carbon_box", _log(rng, 200, 1728), rc, prec, rng.choice(["energy", "forces"]), r1=rc, r2=round(rng.uniform(2.5, 3.5), 2))
    if family == "fitted":
        return _case(None, "carbon_box", _log(rng, 100, 1728), rc, prec, cn="fit")
    r1 = round(rng.uniform(9.0, 10.0), 2)
    return _case(None, "carbon_box", _log(rng, 100, 450), rc, prec, rng.choice(["energy", "forces"]), r1=r1, r2=round(rng.uniform(6.0, r1 - 2.0), 2))


# ---------------------------------------------------------------------------- inputs

def _close(a, b, dmin, box):
    """(len(a),) whether a point of a lies closer than dmin to one of b (minimum image in a cube of edge box, if any)."""
    out = []
    for s in range(0, len(a), 1024):
        d = a[s:s + 1024, None, :] - b[None, :, :]
        if box:
            d -= box * torch.round(d / box)
        out.append(((d * d).sum(-1) < dmin * dmin).any(1))
    return torch.cat(out)


def _place(n, dmin, gen, box=0.0, radius=0.0, edge=0.0):
    """n random points no closer than dmin: in a periodic cube, an open sphere or an open cube."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    acc = torch.empty((0, 3), dtype=torch.float64, device=dev)
    while len(acc) < n:
        m = n - len(acc) + 8
        if radius:
            g = torch.randn((m, 3), dtype=torch.float64, generator=gen)
            p = g / g.norm(dim=1, keepdim=True) * radius * torch.rand((m, 1), dtype=torch.float64, generator=gen) ** (1.0 / 3.0)
        else:
            p = torch.rand((m, 3), dtype=torch.float64, generator=gen) * (box or edge)
        p = p.to(dev)
        if len(acc):
            p = p[~_close(p, acc, dmin, box)]
        keep = torch.ones(len(p), dtype=torch.bool, device=dev)
        for s in range(0, len(p), 1024):   # a candidate gives way to any earlier one that it clashes with
            d = p[s:s + 1024, None, :] - p[None, :, :]
            if box:
                d -= box * torch.round(d / box)
            rows = torch.arange(s, min(s + 1024, len(p)), device=dev)
            near = ((d * d).sum(-1) < dmin * dmin) & (torch.arange(len(p), device=dev)[None, :] < rows[:, None])
            keep[rows] = ~near.any(1)
        acc = torch.cat([acc, p[keep]])[:n]
    return acc.cpu().numpy()


def _structure(kind, n, rc, r1, r2, seed):
    gen = torch.Generator().manual_seed(seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    dmin, cell = (1.3 if kind.startswith("carbon") else 0.9), None
    if kind.endswith("box"):
        edge = (n / DENSITY[kind]) ** (1.0 / 3.0)
        pos, cell = _place(n, dmin, gen, box=edge), np.eye(3) * edge
    elif kind == "carbon_open":
        pos = _place(n, dmin, gen, edge=(n / DENSITY[kind]) ** (1.0 / 3.0))
    else:
        pos = _place(n, dmin, gen, radius=(3.0 * n / (4.0 * math.pi * DENSITY[kind])) ** (1.0 / 3.0))
    species = np.ones(n, dtype=np.int32)
    if kind.startswith("hcno"):
        other, carbon = int(round(0.1 * n)), int(0.3 * n)
        species = np.repeat([0, 1, 2, 3], [n - 2 * other - carbon, carbon, other, other]).astype(np.int32)
        rng.shuffle(species)
    cut = dict(r_scs=rc, r_nbr=r1 + r2 or rc, r_mbd1=r1 or rc, r_mbd2=r2 or rc)
    return dict(pos=pos, species=species, v_ratio=rng.uniform(0.6, 1.0, size=n), cell=cell, pbc=(0, 0, 0) if cell is None else (1, 1, 1), cutoffs=cut)


def _sizes(case):
    """The sizes of a batch: spread geometrically over a factor of 16 around the mean."""
    k = case["requests"]
    w = [16.0 ** (i / max(k - 1, 1)) for i in range(k)]
    return [max(8, int(case["atoms"] * x / sum(w))) for x in w]


def _structures(case, seed):
    if case["kind"] != "requests":
        return [_structure(case["kind"], case["atoms"], case["rc"], case["r1"], case["r2"], seed)]
    return [_structure("hcno_box" if i % 2 and n >= 50 else "hcno_open", n, round(case["rc"] - 0.02 * i, 2), 0.0, 0.0, seed * 64 + i)
            for i, n in enumerate(_sizes(case))]


def prepare(case, seed):
    params = P.MethodParams(omega=OMEGA, weight=WEIGHT, beta=BETA, damp_d=DAMP, r_buf=R_BUF, r_inner=R_INNER, n_max=N_MAX,
                            precision=case["precision"], cn_mode=case["cn"])
    structs = _structures(case, seed)
    if not case["host"]:
        dev = torch.device("cuda", torch.cuda.current_device())
        for s in structs:
            s["pos"] = torch.as_tensor(s["pos"], device=dev)
            s["species"] = torch.as_tensor(s["species"], device=dev)
            s["v_ratio"] = torch.as_tensor(s["v_ratio"], device=dev)
    state = dict(case=case, params=params, structs=structs)
    if case["out"] == "train":
        s = structs[0]
        s["pos"].requires_grad_(True)
        s["v_ratio"].requires_grad_(True)
        state["seeds"] = torch.as_tensor(_seeds(len(s["pos"]), seed), device=s["pos"].device)
    return state


def _seeds(n, seed):
    """dLoss/dE of every atom in a training step."""
    return np.random.Generator(np.random.PCG64(seed + 1)).normal(size=n)


def _taken(case, x):
    """The results as a program takes them: mixed precision (FP32 pair tensors and matrices) is chosen by
    programs that go on in single precision, so they take its results as float32."""
    if case["precision"] == "fp64":
        return x
    return x.astype(np.float32) if isinstance(x, np.ndarray) else x.float()


def run(state):
    case, s = state["case"], state["structs"][0]
    if case["out"] == "train":
        s["pos"].grad = s["v_ratio"].grad = None
        e = P.LMBDEnergy.apply(s["pos"], s["species"], s["v_ratio"], s["cell"], s["cutoffs"], state["params"], SPECIES)
        (e * state["seeds"]).sum().backward()
        return {"0": {"energies": _taken(case, e.detach()), "dpos": _taken(case, s["pos"].grad), "dnu": _taken(case, s["v_ratio"].grad)}}
    outs = P.compute_batch(state["structs"], state["params"], SPECIES, forces=case["out"] == "forces")
    keys = ("energies", "forces") if case["out"] == "forces" else ("energies",)
    return {str(i): {k: _taken(case, o[k]) for k in keys} for i, o in enumerate(outs)}


def work(case):
    """One pass: inputs and outputs once, and the products of the method as it is stated, on neighbourhoods of
    the mean size: per atom and frequency a Cholesky factorisation (N^3 / 3, N = 3 n1) and triangular solves, per
    atom the Krylov products with the coupled pairs of T_LR (18 flops per pair and column) and, for gradients,
    T-bar on those pairs."""
    nbytes = flops = 0.0
    sizes = _sizes(case) if case["kind"] == "requests" else [case["atoms"]]
    grad = case["out"] != "energy"
    for i, n in enumerate(sizes):
        kind = ("hcno_box" if i % 2 and n >= 50 else "hcno_open") if case["kind"] == "requests" else case["kind"]
        rho = DENSITY[kind]
        ball = lambda r: rho * 4.0 / 3.0 * math.pi * r ** 3  # noqa: E731
        cap = n if kind.endswith("open") else math.inf
        rc, r1, r2 = case["rc"], case["r1"] or case["rc"], case["r2"] or case["rc"]
        n1, nk = min(ball(rc), cap), min(ball(case["r1"] + case["r2"] or rc), cap)
        pairs = nk * min(ball(r2), nk) + 2 * min(ball(r1), nk) if case["r1"] else nk * nk * 0.5
        N = 3.0 * n1
        per = (N_FREQ + 1) * (N ** 3 / 3.0 + (12.0 if grad else 6.0) * N * N)
        per += (N_MAX - 2 if grad else 2) * 18.0 * 3 * N_FREQ * pairs
        if grad:
            per += 9.0 * 3 * N_FREQ * N_MAX * pairs
        if case["cn"] == "fit":
            per += 20 * 18.0 * N_FREQ * pairs
        flops += n * per
        nbytes += n * (24 + 4 + 8 + 8 + (24 if grad else 0) + (16 if case["out"] == "train" else 0))
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------- the method in 64 bits

def _sites(pos, cell, k, rmax):
    """Sites within rmax (A) of atom k, the atom itself first: base indices and integer cell shifts."""
    m = 0 if cell is None else int(math.ceil(rmax / cell[0, 0])) + 1
    g = np.stack(np.meshgrid(*[np.arange(-m, m + 1)] * 3, indexing="ij"), -1).reshape(-1, 3)
    img = pos[None] + (g[:, None, :] @ cell if cell is not None else np.zeros((1, 1, 3)))
    d = np.linalg.norm(img - pos[k], axis=-1)
    sh, base = np.nonzero(d < rmax)
    order = np.argsort(d[sh, base], kind="stable")
    return base[order], g[sh[order]], d[sh, base][order]


def _fermi(r, S):
    return 1.0 / (1.0 + torch.exp(-DAMP * (r / S - 1.0)))


def _cut(r, rc, rb):
    x = (r - rc + rb) / rb
    return torch.where(r < rc - rb, torch.ones_like(r), torch.where(r < rc, 1.0 - 3.0 * x * x + 2.0 * x ** 3, torch.zeros_like(r)))


def _dipole(v, r):
    return (3.0 * v[:, :, None] * v[:, None, :] - (r * r)[:, None, None] * torch.eye(3, dtype=v.dtype, device=v.device)) / r[:, None, None] ** 5


def _t_sr(v, s, S, rc):
    """Damped short-range tensors (pairs, frequencies, 3, 3)."""
    r = v.norm(dim=1)
    u = r[:, None] / s
    ex = torch.exp(-u * u)
    g = torch.erf(u) - 2.0 / math.sqrt(math.pi) * u * ex
    h = (4.0 / math.sqrt(math.pi) * u ** 3 * ex)[:, :, None, None] * (v[:, :, None] * v[:, None, :] / r[:, None, None] ** 5)[:, None]
    return (_cut(r, rc, R_BUF / BOHR) * (1.0 - _fermi(r, S)))[:, None, None, None] * (h - _dipole(v, r)[:, None] * g[:, :, None, None])


def _energies(pos, species, nu, cell, cut):
    """Per-atom energies (eV) of one structure as a differentiable function of pos (A) and nu."""
    dev, tab = pos.device, torch.as_tensor(SPECIES, dtype=torch.float64, device=pos.device)[torch.as_tensor(species, dtype=torch.long, device=pos.device)]
    a0, c6, r0 = tab.T
    om = torch.as_tensor(np.concatenate([[0.0], OMEGA]), device=dev)
    abar = (a0 * nu)[:, None] / (1.0 + (om[None] / (4.0 * c6 / (3.0 * a0 * a0))[:, None]) ** 2)
    sig, R = (math.sqrt(2.0 / math.pi) * abar / 3.0) ** (1.0 / 3.0), r0 * nu ** (1.0 / 3.0)
    rs, x_np = cut["r_scs"], pos.detach().cpu().numpy()
    eye, frames, cen = torch.eye(3, dtype=torch.float64, device=dev), [], []
    ix = lambda a: torch.as_tensor(a, dtype=torch.long, device=dev)  # noqa: E731
    for k in range(len(x_np)):
        base, sh, dist = _sites(x_np, cell, k, max(2.0 * rs, cut["r_nbr"]))
        n1, n12, nK = (int((dist < r).sum()) for r in (rs, 2.0 * rs, cut["r_nbr"]))
        b = ix(base)
        p = pos[b] - pos[k]
        if cell is not None:
            p = p + torch.as_tensor(sh @ cell, device=dev)
        p = p / BOHR
        d = torch.cdist(p.detach()[:n1], p.detach()[:n12], compute_mode="donot_use_mm_for_euclid_dist")
        I, J = torch.nonzero((d < rs / BOHR) & (torch.arange(n12, device=dev)[None] != torch.arange(n1, device=dev)[:, None]), as_tuple=True)
        t = _t_sr(p[I] - p[J], torch.sqrt(sig[b[I]] ** 2 + sig[b[J]] ** 2), BETA * (R[b[I]] + R[b[J]]), rs / BOHR)
        x = (p[I] - p[J]).norm(dim=1) * BOHR / R_INNER
        inner = torch.where(x < 1.0, 3.0 * x * x - 2.0 * x ** 3, torch.ones_like(x))
        own = J < n1
        B = torch.zeros((n1, n1, len(om), 3, 3), dtype=torch.float64, device=dev).index_put((I[own], J[own]), t[own])
        B = B.permute(2, 0, 3, 1, 4).reshape(len(om), 3 * n1, 3 * n1) + torch.diag_embed((1.0 / abar[b[:n1]]).T.repeat_interleave(3, dim=1))
        far = inner[~own][:, None, None, None] * t[~own] * abar[b[J[~own]]][:, :, None, None]
        rhs = eye - torch.zeros((n1, len(om), 3, 3), dtype=torch.float64, device=dev).index_add(0, I[~own], far)
        X = torch.linalg.solve(B, rhs.permute(1, 0, 2, 3).reshape(len(om), 3 * n1, 3)).reshape(len(om), n1, 3, 3)
        loc = (X * eye).sum((2, 3)).T / 3.0
        frames.append((b, p[:nK], n1, nK, loc))
        cen.append(loc[0])
    cen, e = torch.stack(cen), []
    for b, p, n1, nK, loc in frames:
        bk = b[:nK]
        x = (p[1:n1].norm(dim=1) * BOHR / rs)[:, None]
        f = 3.0 * x * x - 2.0 * x ** 3
        m = min(n1, nK)
        A = torch.cat([loc[:1], (1.0 - f[:m - 1]) * loc[1:m] + f[:m - 1] * cen[bk[1:m]], cen[bk[m:]]])
        Rt = r0[bk] * (A[:, 0] / a0[bk]) ** (1.0 / 3.0)
        I, J = torch.nonzero(~torch.eye(nK, dtype=torch.bool, device=dev), as_tuple=True)
        v = p[I] - p[J]
        r = v.norm(dim=1)
        rc = torch.full_like(r, cut["r_mbd2"] / BOHR)
        rc[(I == 0) | (J == 0)] = cut["r_mbd1"] / BOHR
        t = (_cut(r, rc, R_BUF / BOHR) * _fermi(r, BETA * (Rt[I] + Rt[J])))[:, None, None] * _dipole(v, r)
        T = torch.zeros((nK, nK, 3, 3), dtype=torch.float64, device=dev).index_put((I, J), t).permute(0, 2, 1, 3).reshape(3 * nK, 3 * nK)
        s = torch.sqrt(A[:, 1:]).T.repeat_interleave(3, dim=1)
        u = torch.zeros((len(OMEGA), 3 * nK, 3), dtype=torch.float64, device=dev)
        u[:, :3] = eye
        per = 0.0
        for n in range(1, N_MAX + 1):
            u = s[:, :, None] * torch.matmul(T, s[:, :, None] * u)
            if n > 1:
                per = per - (u[:, :3] * eye).sum((1, 2)) / n
        e.append((torch.as_tensor(WEIGHT, device=dev) * per).sum() / (2.0 * math.pi) * HARTREE)
    return torch.stack(e)


def exact(case, seed):
    """The outputs of run() from plain torch in 64 bits; None where that takes long (large structures) or where the
    result is an estimate by construction (spectrum bounds)."""
    structs = _structures(case, seed)
    if case["cn"] != "series" or case["r1"] or sum(len(s["pos"]) for s in structs) > 130:
        return None
    dev, out = "cuda" if torch.cuda.is_available() else "cpu", {}
    for i, s in enumerate(structs):
        pos = torch.as_tensor(s["pos"], device=dev).requires_grad_(True)
        nu = torch.as_tensor(s["v_ratio"], device=dev).requires_grad_(True)
        with torch.set_grad_enabled(case["out"] != "energy"):
            e = _energies(pos, s["species"], nu, s["cell"], s["cutoffs"])
        o = {"energies": e.detach()}
        if case["out"] == "train":
            o["dpos"], o["dnu"] = torch.autograd.grad((e * torch.as_tensor(_seeds(len(pos), seed), device=dev)).sum(), (pos, nu))
        elif case["out"] == "forces":
            o["forces"] = -torch.autograd.grad(e.sum(), pos)[0]
        out[str(i)] = {k: v.cpu() for k, v in o.items()}
    return out
