"""Workloads of the library, through its public Python entry points.

Every system is the seeded tight-binding model of the repository's benchmark (two orbitals per
site, onsite -1.5 / +1.5 eV +- 0.1, hopping -0.3 exp(-r / 1.5 A) below 6 A, sites uniform in a
periodic cube at 0.1 per A^3 and Morton sorted, or 70 % of them in dense spheres in a dilute
background), built here on the GPU from the seed.  The kinds of work:

  step      one whole density matrix from a new Hamiltonian: graph, cores, SP2, D
  density   D on cores that are kept (the same system under many Hamiltonians)
  md        one step along a trajectory: graph from the previous D, the cores carried over, D
  gradient  D and the adjoint of a scalar of D with respect to H
  foe       the finite-temperature density matrix (Chebyshev expansion, mu solved)
  cores     graph and cores alone

Mixed precision gives D to 1e-6, so programs that use it keep D in single precision; FP64 D
stays double.  D and index buffers have the room that a program leaves for the next system of the
same kind.
"""
import math

import numpy as np
import torch

import paper_1603_00937_amd as gb

TAU = 1e-5
MIXED = ("fp16x3", "bf16x6", "fp32")


def listed():
    return [
        # a unit cell's worth of orbitals, where launches and host time count
        {"name": "step_fp64_n256", "kind": "step", "sites": 128, "density": 0.05, "clustered": False,
         "core": 16, "method": "block", "precision": "fp64"},
        # the plain method at the size where whole-matrix diagonalisation is still the check
        {"name": "step_fp64_n1024", "kind": "step", "sites": 512, "density": 0.1, "clustered": False,
         "core": 16, "method": "block", "precision": "fp64"},
        # the mixed default on a small odd system (block cores, a ragged last core)
        {"name": "step_fp16x3_n2050", "kind": "step", "sites": 1025, "density": 0.1,
         "clustered": False, "core": 32, "method": "block", "precision": "fp16x3"},
        # the benchmark: the whole path at N = 18000 on communities
        {"name": "step_fp16x3_n18000", "kind": "step", "sites": 9000, "density": 0.1,
         "clustered": False, "core": 32, "method": "multilevel", "precision": "fp16x3"},
        # the heterogeneous system (uneven subgraphs), the largest the benchmark runs
        {"name": "step_fp16x3_n100000", "kind": "step", "sites": 50000, "density": 0.03,
         "clustered": True, "core": 32, "method": "multilevel", "precision": "fp16x3"},
        # double precision throughout, on kept communities
        {"name": "density_fp64_n18000", "kind": "density", "sites": 9000, "density": 0.1,
         "clustered": False, "core": 32, "method": "multilevel", "precision": "fp64"},
        # the split-bf16 alternative of the mixed path, on kept blocks of an odd size
        {"name": "density_bf16x6_n6014", "kind": "density", "sites": 3007, "density": 0.1,
         "clustered": False, "core": 32, "method": "block", "precision": "bf16x6"},
        # native FP32 squares with small cores
        {"name": "density_fp32_n3000", "kind": "density", "sites": 1500, "density": 0.1,
         "clustered": False, "core": 16, "method": "block", "precision": "fp32"},
        # molecular dynamics: graph from the previous D, communities carried over
        {"name": "md_fp16x3_n4096", "kind": "md", "sites": 2048, "density": 0.1,
         "clustered": False, "core": 32, "method": "multilevel", "precision": "fp16x3"},
        # training-style use: D and the gradient with respect to H
        {"name": "gradient_n1800", "kind": "gradient", "sites": 900, "density": 0.1,
         "clustered": False, "core": 32, "method": "block", "precision": "fp64"},
        # finite temperature
        {"name": "foe_n1024", "kind": "foe", "sites": 512, "density": 0.1, "clustered": False,
         "core": 16, "method": "block", "precision": "fp64", "beta": 8.0, "order": 160},
        # graph and cores of a system past the sizes whose vertex sets fit LDS bitmaps
        {"name": "cores_n160002", "kind": "cores", "sites": 80001, "density": 0.1,
         "clustered": False, "core": 32, "method": "block", "precision": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "density", "density", "md", "gradient", "foe",
                       "cores"])
    c = {"kind": kind, "density": 0.1, "clustered": False, "core": rng.choice([16, 24, 32]),
         "method": rng.choice(["block", "multilevel"]), "precision": "fp64"}
    if kind == "step":
        c["precision"] = rng.choice(["fp64", "fp16x3", "fp16x3", "bf16x6"])
        c["clustered"] = rng.random() < 0.3
        lo, hi = (4000, 40000) if c["clustered"] else (130, 9000)
        if c["precision"] == "fp64":
            lo, hi = min(lo, hi // 2), hi // 3
        c["sites"] = _log_int(rng, lo, hi)
        if c["clustered"]:
            c.update(density=0.03, core=32, method="multilevel")
        elif c["sites"] < 400:
            c["density"] = 0.05
    elif kind == "density":
        c["precision"] = rng.choice(["fp64", "fp16x3", "bf16x6", "fp32"])
        c["sites"] = _log_int(rng, 300, 3500)
    elif kind == "md":
        c["precision"] = rng.choice(["fp64", "fp16x3", "fp16x3"])
        c["sites"] = _log_int(rng, 300, 4000)
    elif kind == "gradient":
        c["sites"] = _log_int(rng, 150, 1200)
        if c["sites"] < 400:
            c["density"] = 0.05
    elif kind == "foe":
        c.update(sites=_log_int(rng, 150, 520), beta=round(rng.uniform(3.0, 10.0), 2),
                 order=rng.randrange(40, 151))
        if c["sites"] < 400:
            c["density"] = 0.05
    else:
        c.update(sites=_log_int(rng, 1000, 100000), core=32, method="block")
    return c


# ---- systems ---------------------------------------------------------------------------------

def _positions(case, rng):
    n = case["sites"]
    if not case["clustered"]:
        L = round((n / case["density"]) ** (1.0 / 3.0), 9)
        return rng.uniform(0.0, L, (n, 3)), L
    per, rho = 500, 0.15
    n_sph = max(1, (7 * n // 10) // per)
    n_dil = n - n_sph * per
    vol = per / rho
    R = (3.0 * vol / (4.0 * math.pi)) ** (1.0 / 3.0)
    L = round((n_sph * vol + n_dil / case["density"]) ** (1.0 / 3.0), 9)
    centres = np.zeros((0, 3))
    while len(centres) < n_sph:
        c = rng.uniform(0.0, L, 3)
        d = centres - c
        d -= L * np.rint(d / L)
        if not (np.einsum("ij,ij->i", d, d) <= 4.0 * R * R).any():
            centres = np.vstack([centres, c])
    pts = []
    for c in centres:
        u = rng.uniform(-R, R, (4 * per, 3))
        u = u[np.einsum("ij,ij->i", u, u) < R * R][:per]
        pts.append((c + u) % L)
    dil = np.zeros((0, 3))
    while len(dil) < n_dil:
        u = rng.uniform(0.0, L, (2 * n_dil, 3))
        keep = np.ones(len(u), dtype=bool)
        for c in centres:
            d = u - c
            d -= L * np.rint(d / L)
            keep &= np.einsum("ij,ij->i", d, d) >= R * R
        dil = np.vstack([dil, u[keep]])
    return np.vstack(pts + [dil[:n_dil]]), L


def _morton(pos, L):
    q = np.minimum((pos / L * 1024.0).astype(np.int64), 1023)
    code = np.zeros(len(pos), dtype=np.int64)
    for b in range(10):
        for d in range(3):
            code |= ((q[:, d] >> b) & 1) << (3 * b + d)
    return np.argsort(code, kind="stable")


def _hamiltonian(pos, L, onsite):
    """ELL arrays (columns ascending, padding -1 / 0) of the model at the given positions."""
    x = torch.from_numpy(pos).cuda()
    n = x.shape[0]
    rows, cols, dist = [], [], []
    step = max(1, (1 << 26) // n)
    for a in range(0, n, step):
        r2 = torch.zeros((min(step, n - a), n), dtype=torch.float64, device="cuda")
        for k in range(3):
            d = x[a:a + step, k, None] - x[None, :, k]
            d = d - L * torch.round(d / L)
            r2 += d * d
        i, j = torch.nonzero(r2 < 36.0, as_tuple=True)
        rows.append(i + a)
        cols.append(j)
        dist.append(r2[i, j].sqrt())
    i, j, r = torch.cat(rows), torch.cat(cols), torch.cat(dist)
    t = torch.where(i == j, torch.zeros_like(r), -0.3 * torch.exp(-r / 1.5))
    onsite = torch.from_numpy(onsite).cuda()
    ri, cj, tv = [], [], []
    for a in (0, 1):
        for b in (0, 1):
            m = (i != j) if a != b else torch.ones_like(i, dtype=torch.bool)
            ri.append(2 * i[m] + a)
            cj.append(2 * j[m] + b)
            v = t[m]
            tv.append(torch.where(i[m] == j[m], onsite[2 * i[m] + a], v) if a == b else v)
    ri, cj, tv = torch.cat(ri), torch.cat(cj), torch.cat(tv)
    N = 2 * n
    order = torch.argsort(ri * N + cj)
    ri, cj, tv = ri[order], cj[order], tv[order]
    count = torch.bincount(ri, minlength=N)
    start = torch.cumsum(count, 0) - count
    slot = torch.arange(len(ri), device="cuda") - start[ri]
    W = int(count.max())
    col = torch.full((N, W), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros((N, W), dtype=torch.float64, device="cuda")
    col[ri, slot] = cj.to(torch.int32)
    val[ri, slot] = tv
    return col, val


def _system(case, seed):
    rng = np.random.default_rng([seed, case["sites"]])
    pos, L = _positions(case, rng)
    pos = np.ascontiguousarray(pos[_morton(pos, L)])
    n = case["sites"]
    onsite = np.tile([-1.5, 1.5], n) + rng.uniform(-0.1, 0.1, 2 * n)
    return rng, pos, L, onsite


# ---- what a program holds before the call ------------------------------------------------------

def _room(case):
    """Columns of the D buffers: the largest subgraph of such a system, with headroom."""
    N = 2 * case["sites"]
    return min(N, 2304 if case["clustered"] or case["method"] == "multilevel" else 3072)


def _widened(col, val, case):
    """ELL arrays with the room a row needs as sites move (five standard deviations)."""
    m = case["density"] * 905.0
    W = max(col.shape[1], min(2 * case["sites"], 2 * int(m + 5.0 * math.sqrt(m) + 1.0)))
    pad = (0, W - col.shape[1])
    return (torch.nn.functional.pad(col, pad, value=-1).contiguous(),
            torch.nn.functional.pad(val, pad).contiguous())


def prepare(case, seed):
    rng, pos, L, onsite = _system(case, seed)
    n = case["sites"]
    st = {"case": case, "n_occ": n}
    if case["kind"] == "md":  # the starting point's D (FP64) and cores, then the sites move
        col, val = _hamiltonian(pos, L, onsite)
        st["part"] = gb.partition(gb.build_graph(col, val, TAU), case["core"], case["method"])
        st["D"] = gb.density(col, val, n, TAU, partition=st["part"])[:2]
        pos = (pos + rng.normal(0.0, 0.02, pos.shape)) % L
    st["col"], st["val"] = _hamiltonian(pos, L, onsite)
    N, room = 2 * n, _room(case)
    if case["kind"] == "cores":
        n_sub = -(-N // case["core"])
        st["adj"] = torch.zeros(N * min(N, 768), dtype=torch.int32, device="cuda")
        st["sub"] = torch.zeros(n_sub * min(N, 2304), dtype=torch.int32, device="cuda")
        return st
    st["out"] = (torch.zeros((N, room), dtype=torch.int32, device="cuda"),
                 torch.zeros((N, room), dtype=torch.float64, device="cuda"))
    if case["kind"] == "gradient":
        st["col"], st["val"] = _widened(st["col"], st["val"], case)
    if case["kind"] in ("density", "gradient"):
        st["part"] = gb.partition(gb.build_graph(st["col"], st["val"], TAU), case["core"],
                                  case["method"])
    if case["kind"] == "gradient":
        st["val"].requires_grad_(True)
        g = torch.from_numpy(rng.normal(0.0, 1.0, (2 * n, st["part"].max_sub)))
        st["G"] = g.cuda()
    return st


def _result(case, D_col, D_val):
    return {"col": D_col, "val": D_val.float() if case["precision"] in MIXED else D_val}


def run(st):
    case, col, val, n_occ = st["case"], st["col"], st["val"], st["n_occ"]
    kind = case["kind"]
    if kind == "step":
        g = gb.build_graph(col, val, TAU)
        p = gb.partition(g, case["core"], case["method"])
        D_col, D_val, _ = gb.density(col, val, n_occ, TAU, partition=p,
                                     precision=case["precision"], D=st["out"])
        return _result(case, D_col, D_val)
    if kind == "density":
        D_col, D_val, _ = gb.density(col, val, n_occ, TAU, partition=st["part"],
                                     precision=case["precision"], D=st["out"])
        return _result(case, D_col, D_val)
    if kind == "md":
        g = gb.build_graph(col, val, TAU, mode="dprev", aux=st["D"], tau_aux=1e-4)
        p = gb.partition_update(g, st["part"])
        D_col, D_val, _ = gb.density(col, val, n_occ, TAU, partition=p,
                                     precision=case["precision"], D=st["out"])
        return _result(case, D_col, D_val)
    if kind == "gradient":
        D_col, D_val, _ = gb.density_with_grad(col, val, n_occ, TAU, partition=st["part"])
        grad, = torch.autograd.grad(D_val, val, st["G"])
        out_col, out_val = st["out"]
        out_col[:, :D_col.shape[1]] = D_col
        out_val[:, :D_col.shape[1]] = D_val.detach()
        return {"col": out_col, "val": out_val, "grad": grad}
    if kind == "foe":
        g = gb.build_graph(col, val, TAU)
        p = gb.partition(g, case["core"], case["method"])
        D_col, D_val, info = gb.foe_density(col, val, n_occ, TAU, case["beta"], case["order"],
                                            partition=p, D=st["out"])
        return {"col": D_col, "val": D_val, "mu": info["mu"]}
    g = gb.build_graph(col, val, TAU)
    p = gb.partition(g, case["core"], case["method"])
    row_ptr, adj = g.arrays()
    core_ptr, sub_ptr, sub_idx = p.arrays()
    st["adj"][:len(adj)] = adj
    st["sub"][:len(sub_idx)] = sub_idx
    return {"row_ptr": row_ptr, "col": st["adj"], "core_ptr": core_ptr, "sub_ptr": sub_ptr,
            "sub_idx": st["sub"]}


# ---- what one pass cannot do without -----------------------------------------------------------

def _sizes(case):
    """Typical H row length and subgraph size of the model (orbitals)."""
    rho = 0.075 if case["clustered"] else case["density"]
    N = 2 * case["sites"]
    width = min(N, 2 * rho * 905.0)                   # sites within 6 A
    reach = 7.5 + (3.8 if case["method"] == "multilevel" else 4.5) * (case["core"] / 32) ** 0.33
    sub = min(0.9 * N, 2 * rho * 4.19 * reach ** 3)   # a core and its two-hop halo
    return N, width, sub


def work(case):
    N, width, sub = _sizes(case)
    cores = N / case["core"]
    H, D = 12.0 * N * width, 12.0 * N * sub
    pairs = 2.0 * N * width * width                   # products of the graph's X0^2
    square = sub * sub * (sub + 1)                    # a symmetric block square
    kind = case["kind"]
    if kind == "cores":
        return {"bytes": H + 4.0 * N * sub + 4.0 * cores * sub, "flops": pairs}
    if kind == "foe":                                 # core rows times a sparse H per term
        return {"bytes": H + D, "flops": pairs + case["order"] * 2.0 * N * sub * width}
    flops = cores * 20 * square + (pairs if kind in ("step", "md") else 0.0)
    if kind == "gradient":
        flops += cores * 20 * 2 * square
    return {"bytes": H + D + (D if kind in ("md", "gradient") else 0.0) +
            (H if kind == "gradient" else 0.0), "flops": flops}


# ---- the values in 64 bits ---------------------------------------------------------------------

def _blocks(col, val, case):
    """X0, its bounds and the subgraphs (core first, then halo, both ascending) of block cores."""
    N = col.shape[0]
    r, s = torch.nonzero(col >= 0, as_tuple=True)
    H = torch.zeros((N, N), dtype=torch.float64, device="cuda")
    H[r, col[r, s].long()] = val[r, s]
    d = H.diagonal()
    off = H.abs().sum(1) - d.abs()
    emin, emax = float((d - off).min()), float((d + off).max())
    X0 = (emax * torch.eye(N, dtype=torch.float64, device="cuda") - H) / (emax - emin)
    S = (X0 @ X0).abs() >= TAU
    S.fill_diagonal_(True)
    subs = []
    for a in range(0, N, case["core"]):
        b = min(a + case["core"], N)
        near = S[a:b].any(0)
        near[a:b] = False
        subs.append((b - a, torch.cat([torch.arange(a, b, device="cuda"),
                                       torch.nonzero(near)[:, 0]])))
    return H, X0, emin, emax, subs


def _to_ell(case, subs, rows):
    """Core rows of every block as column-ELL values (rows ascending per column)."""
    out = torch.zeros((2 * case["sites"], _room(case)), dtype=torch.float64, device="cuda")
    for (k, ix), v in zip(subs, rows):
        o = torch.argsort(ix)
        out[ix[:k], :len(ix)] = v[:, o]
    return out


def _sp2(X0, subs, n_occ, tape=False):
    """Every block's SP2 expansion with one branch sequence from the summed core traces."""
    xs = [X0[ix][:, ix] for _, ix in subs]
    N = X0.shape[0]
    steps, kept = [], []
    while True:
        t1 = sum(float(x.diagonal()[:k].sum()) for (k, _), x in zip(subs, xs))
        t2 = sum(float((x[:k] ** 2).sum()) for (k, _), x in zip(subs, xs))
        if abs(t1 - t2) <= 1e-10 * N / 1024.0 or len(steps) >= 100:
            return xs, steps, kept
        lin = not abs(t2 - n_occ) < abs(2.0 * t1 - t2 - n_occ)
        if tape:
            kept.append(xs)
        steps.append(lin)
        xs = [2.0 * x - x @ x if lin else x @ x for x in xs]


def exact(case, seed):
    """Dense FP64 linear algebra per block, for block cores up to N = 6200 (communities and
    larger systems: none).  Index outputs have no such value."""
    limit = {"step": 3100, "density": 3100, "gradient": 1000, "foe": 1600}.get(case["kind"], 0)
    if case["method"] != "block" or case["clustered"] or case["sites"] > limit:
        return None
    rng, pos, L, onsite = _system(case, seed)
    col, val = _hamiltonian(pos, L, onsite)
    if case["kind"] == "gradient":
        col, val = _widened(col, val, case)
    N, n_occ = col.shape[0], case["sites"]
    H, X0, emin, emax, subs = _blocks(col, val, case)
    if case["kind"] == "foe":
        return _exact_foe(case, H, emin, emax, subs, n_occ)
    if case["kind"] != "gradient":
        xs, _, _ = _sp2(X0, subs, n_occ)
        return {"col": None, "val": _to_ell(case, subs, [x[:k] for (k, _), x in zip(subs, xs)])}
    xs, steps, kept = _sp2(X0, subs, n_occ, tape=True)
    width = max(len(ix) for _, ix in subs)
    G = torch.from_numpy(rng.normal(0.0, 1.0, (N, width))).cuda()
    dH = torch.zeros_like(X0)
    for q, (k, ix) in enumerate(subs):
        rank = torch.argsort(torch.argsort(ix))
        g = torch.zeros_like(xs[q])
        g[:, :k] = G[ix[:k]][:, rank].T
        g = 0.5 * (g + g.T)
        for x, lin in zip(reversed([layer[q] for layer in kept]), reversed(steps)):
            p = g @ x + x @ g
            g = 2.0 * g - p if lin else p
        dH[ix[:, None], ix[None, :]] -= g / (emax - emin)
    r, s = torch.nonzero(col >= 0, as_tuple=True)
    grad = torch.zeros_like(val)
    grad[r, s] = dH[r, col[r, s].long()]
    return {"col": None, "val": _to_ell(case, subs, [x[:k] for (k, _), x in zip(subs, xs)]),
            "grad": grad}


def _exact_foe(case, H, emin, emax, subs, n_occ):
    M, beta = case["order"], case["beta"]
    mid, half = 0.5 * (emax + emin), 0.5 * (emax - emin)
    eye = torch.eye(H.shape[0], dtype=torch.float64, device="cuda")
    Ht = (2.0 * H - (emax + emin) * eye) / (emax - emin)
    terms, traces = [], np.zeros(M + 1)
    for k, ix in subs:
        h = Ht[ix][:, ix]
        v = torch.empty((M + 1, k, len(ix)), dtype=torch.float64, device="cuda")
        v[0] = torch.eye(len(ix), dtype=torch.float64, device="cuda")[:k]
        v[1] = h[:k]
        for m in range(2, M + 1):
            v[m] = 2.0 * (v[m - 1] @ h) - v[m - 2]
        traces += v[:, :, :k].diagonal(dim1=1, dim2=2).sum(1).cpu().numpy()
        terms.append(v)
    K = max(4 * (M + 1), 1024)
    th = math.pi * (np.arange(K) + 0.5) / K
    e = mid + half * np.cos(th)
    basis = np.cos(np.outer(np.arange(M + 1), th))

    def coefficients(mu):
        f = 1.0 / (1.0 + np.exp(beta * (e - mu)))
        c = basis @ f * (2.0 / K)
        c[0] *= 0.5
        return c

    lo, hi = emin, emax
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        if not lo < mu < hi:
            break
        lo, hi = (mu, hi) if float(coefficients(mu) @ traces) < n_occ else (lo, mu)
    mu = 0.5 * (lo + hi)
    c = torch.from_numpy(coefficients(mu)).cuda()
    rows = [(c[:, None, None] * v).sum(0) for v in terms]
    return {"col": None, "val": _to_ell(case, subs, rows), "mu": mu}
