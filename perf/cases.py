"""Performance cases: what a user of the library has it do, and its FP64 values.

A case is one pass of a user's program on a live handle: advance a batch by a
number of time steps (with the statistics sampled every 10 steps, or none) and
read results back: the statistics, and the fields looked at, of some or all
realisations.  A pass continues from where the last one ended.  Two kinds:

  rods   1D batches.  Instances share a shape, or (``ragged``) have lengths
         log-uniform up to ``n`` and a random mix of FE and PC.  Equations: heat,
         Dean-Kawasaki species, Burgers; schemes FE, PC and the implicit BE and
         CN; periodic or Dirichlet; uniform or composite material.
  grid   2D / 3D periodic batches of one grid.

Statistics (``stats``): "none", "moments" (1D per-cell mean and variance),
"corr" (1D covariance and S_k as well), "spatial" (2D / 3D spatial mean and
variance) and "sk" (2D radially binned S(k) as well).
``looks`` realisations, spread over the batch, are read back after a pass;
``fields`` says whether their fields are read too.

Every realisation starts from its steady profile plus a random perturbation and
draws its noise from its seed, so the seed alone makes the inputs.
"""
import math

import numpy as np
import torch

from paper_2406_12157_amd import she

EVERY = 10  # steps between samples, as in the workloads and the benchmark


def listed():
    return [
        # The smallest job: one short ring in double precision, all statistics.
        # A program that watches its convergence reads them back often.
        _rods("ring64_f64_corr", 64, 1, 1000, f64=True, stats="corr"),
        # One rod between two temperatures, predictor-corrector, with the full
        # covariance: the long-range correlation study.
        _rods("rod128_pc_corr", 128, 1, 5000, scheme="pc", dirichlet=True, stats="corr"),
        # The same study as an ensemble: many realisations of one rod.
        _rods("rod128_pc_x1024", 128, 1024, 2000, scheme="pc", dirichlet=True, stats="moments"),
        # A parameter sweep in one batch: 1000 rods of all lengths, FE and PC.
        _rods("ragged4096_x1000", 4096, 1000, 1000, dirichlet=True, ragged=True),
        # The sweep with per-cell statistics.
        _rods("ragged4096_x1000_moments", 4096, 1000, 1000, dirichlet=True, ragged=True, stats="moments"),
        # Stochastic Burgers rings, an ensemble.
        _rods("burgers256_x1024", 256, 1024, 1000, eq="burgers", stats="moments"),
        # Implicit rods: large time steps, an ensemble.
        _rods("rod256_cn_x1024", 256, 1024, 200, scheme="cn", dirichlet=True, r=2.0),
        # One small plane with its structure factor: launches and latency count.
        _grid("plane128_sk", (128, 128), 1, 200, stats="sk"),
        # Planes in double precision, predictor-corrector, a height that no
        # power of two divides.
        _grid("plane256x130_f64_pc_x16", (256, 130), 16, 100, scheme="pc", f64=True, stats="spatial"),
        # The benchmark: 256 planes of 512 x 512 with S(k).
        _grid("plane512_x256_sk", (512, 512), 256, 200, stats="sk", fields=False),
        # A large box of the species equation.
        _grid("box256_dk", (256, 256, 256), 1, 500, eq="species", stats="spatial", fields=False),
        # Small boxes, predictor-corrector.
        _grid("box64_pc_x4", (64, 64, 64), 4, 50, scheme="pc", stats="spatial"),
    ]


def _rods(name, n, count, steps, eq="heat", scheme="fe", dirichlet=False, f64=False, stats="none", ragged=False,
          composite=False, r=None, fields=True):
    if r is None:
        r = {"heat": 0.2 if scheme == "fe" and not ragged else 0.05, "species": 0.1, "burgers": 0.25}[eq]
    if ragged:
        r = 0.1
    return dict(name=name, kind="rods", n=n, count=count, steps=steps, eq=eq, scheme=scheme, dirichlet=dirichlet,
                f64=f64, stats=stats, ragged=ragged, composite=composite, r=r, looks=min(count, 8), fields=fields)


def _grid(name, n, count, steps, eq="heat", scheme="fe", f64=False, stats="none", r=None, fields=True):
    n = tuple(n) + (1,) * (3 - len(n))
    if r is None:
        r = 0.1 if n[2] == 1 else 0.05
    return dict(name=name, kind="grid", nx=n[0], ny=n[1], nz=n[2], count=count, steps=steps, eq=eq, scheme=scheme,
                f64=f64, stats=stats, r=r, looks=min(count, 4), fields=fields)


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    family = rng.choice(["rods", "rods", "ragged", "implicit", "plane", "plane", "box"])
    f64 = rng.random() < 0.3
    if family == "rods":
        eq = rng.choice(["heat", "heat", "species", "burgers"])
        n = _log(rng, 16, 2048)
        count = _log(rng, 1, max(2, min(1024, 2 ** 18 // n)))
        stats = rng.choice(["none", "moments", "corr"] if n <= 160 and count <= 64 else ["none", "moments"])
        dirichlet = eq != "burgers" and rng.random() < 0.6
        composite = eq == "heat" and dirichlet and rng.random() < 0.25
        scheme = rng.choice(["fe", "pc"])
        return _unnamed(_rods("", n, count, _log(rng, 100, 2000), eq=eq, scheme=scheme, dirichlet=dirichlet, f64=f64,
                              stats=stats, composite=composite, r=0.05 if composite else None))
    if family == "ragged":
        return _unnamed(_rods("", _log(rng, 300, 4096), _log(rng, 50, 1000), _log(rng, 100, 1000), dirichlet=True,
                              ragged=True, f64=f64, stats=rng.choice(["none", "moments"])))
    if family == "implicit":
        n = _log(rng, 16, 512)
        return _unnamed(_rods("", n, _log(rng, 1, 1024), _log(rng, 50, 300), eq=rng.choice(["heat", "species"]),
                              scheme=rng.choice(["be", "cn"]), dirichlet=rng.random() < 0.5, f64=f64,
                              stats=rng.choice(["none", "moments"]), r=rng.choice([0.5, 1.0, 2.0, 4.0])))
    scheme, eq = rng.choice(["fe", "pc"]), rng.choice(["heat", "heat", "species"])
    if family == "plane":
        stats = rng.choice(["spatial", "sk"])
        nx = 2 ** rng.randint(4, 10)
        ny = 2 ** rng.randint(4, 10) if stats == "sk" else _log(rng, 8, 1024)
        count = _log(rng, 1, max(2, min(256, 2 ** 23 // (nx * ny))))
        return _unnamed(_grid("", (nx, ny), count, _log(rng, 20, 100), eq=eq, scheme=scheme, f64=f64, stats=stats))
    nx, ny, nz = 2 ** rng.randint(3, 8), 4 * _log(rng, 2, 48), _log(rng, 8, 192)
    count = _log(rng, 1, max(2, min(16, 2 ** 23 // (nx * ny * nz))))
    return _unnamed(_grid("", (nx, ny, nz), count, _log(rng, 20, 60), eq=eq, scheme=scheme, f64=f64, stats="spatial"))


def _unnamed(case):
    del case["name"]
    return case


# ------------------------------------------------------------------ instances

_EQ = {"heat": she.HEAT, "species": she.SPECIES, "burgers": she.BURGERS}
_SCHEME = {"fe": she.EM, "pc": she.HEUN, "be": she.BE, "cn": she.CN}
_STATS = {"none": 0, "moments": she.STAT_MOMENTS, "corr": she.STAT_MOMENTS | she.STAT_CORR, "spatial": she.STAT_SPATIAL,
          "sk": she.STAT_SPATIAL | she.STAT_SK}


def _params(case, seed):
    """One dict per realisation, in the ranges of the repository's workloads."""
    eq, count = case["eq"], case["count"]
    u0, eps, gap = {"heat": (1.0, 1e-2, 0.1), "species": (100.0, 1.0, 20.0), "burgers": (0.15, 1e-4, 0.0)}[eq]
    sd = math.sqrt(eps * {"heat": u0 * u0, "species": u0, "burgers": u0 * (1.0 - u0)}[eq])
    if case["kind"] == "grid":
        if eq == "species" and case["nz"] > 1:
            u0, sd = 1e3, math.sqrt(1e3)
        n = (case["nx"], case["ny"]) + ((case["nz"],) if case["nz"] > 1 else ())
        return [dict(n=n, eq=_EQ[eq], scheme=_SCHEME[case["scheme"]], r=case["r"], eps=eps, u0=u0, init_sd=sd, seed=seed,
                     realisation=q) for q in range(count)]
    out = []
    rng = np.random.default_rng(case["n"])  # the sweep's lengths and schemes are the case's, its noise the seed's
    for q in range(count):
        n, scheme, d = case["n"], _SCHEME[case["scheme"]], gap
        if case["ragged"]:
            lo = min(64, n // 4)
            n, scheme = int(round(lo * (n / lo) ** rng.random())), int(rng.random() < 0.5)
            d = 0.15 * rng.random()
        p = dict(n=(n,), eq=_EQ[eq], scheme=scheme, r=case["r"], eps=1e-3 if eq == "heat" and scheme else eps, u0=u0,
                 init_sd=sd, seed=seed, realisation=q, bc=she.PERIODIC)
        if case["dirichlet"]:
            p.update(bc=she.DIRICHLET, u_left=u0 + d, u_right=u0 - d)
        if eq == "burgers":
            p.update(nu=0.6)
        if case["composite"]:
            h = n // 2
            p.update(cond=[1.0] * h + [3.0] * (n - h), cap=[1.0] * h + [0.7] * (n - h))
        out.append(p)
    return out


def _looks(case):
    """The realisations read back: spread over the batch, its ends among them."""
    k, c = case["looks"], case["count"]
    return sorted({(i * (c - 1)) // max(1, k - 1) for i in range(k)}) if c > 1 else [0]


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, s.looks = case, _looks(case)
    s.handle = she.Handle([she.Instance(**p) for p in _params(case, seed)], precision=she.F64 if case["f64"] else she.F32,
                          burn_in=0, sample_every=EVERY, stats=_STATS[case["stats"]])
    return s


def run(s):
    c, h = s.case, s.handle
    out = {}
    if c["stats"] == "none":
        h.step(c["steps"])
    else:
        h.run(c["steps"])
        got = [h.stats(i, corr=c["stats"] == "corr", sk=c["stats"] in ("corr", "sk")) for i in s.looks]
        for key in ("mean", "var", "corr", "sk"):
            if key in got[0]:
                out[key] = np.concatenate([g[key].reshape(-1) for g in got])
        for key in ("sum_u", "spatial_var", "n_samples"):
            out[key] = np.array([g[key] for g in got])
    if c["fields"]:
        out["field"] = np.concatenate([h.read_field(i) for i in s.looks])
    return out


def work(case):
    """State read once and written once, statistics written once; per cell and
    step one number per face (ten Philox rounds of four operations for four
    numbers, five for each Box-Muller number), four operations per face flux and
    two per direction for the update (twice the stencil for PC)."""
    es = 8 if case["f64"] else 4
    if case["kind"] == "rods":
        dim, cells = 1, sum(p["n"][0] for p in _params(case, 0))
        stat = {"none": 0, "moments": 16 * cells, "corr": 16 * cells + 8 * cells * case["n"]}[case["stats"]]
    else:
        dim = 2 if case["nz"] == 1 else 3
        cells = case["nx"] * case["ny"] * case["nz"] * case["count"]
        stat = 8 * case["count"] * (2 + (she.n_shells((case["nx"], case["ny"])) if case["stats"] == "sk" else 0))
    stencil = dim * 6 * (1.5 if case["kind"] == "rods" and case["ragged"] else 2 if case["scheme"] == "pc" else 1)
    if case["scheme"] in ("be", "cn"):
        stencil += 8  # tridiagonal solve
    return {"bytes": 2 * es * cells + stat, "flops": cells * case["steps"] * (dim * 15 + stencil)}


# ------------------------------------------------------------------ values in 64 bits

_M32 = 0xFFFFFFFF


def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _normals(block, step, tag, real, seed):
    """The four normals of Philox4x32-10 blocks (last axis): int64 tensors that
    broadcast against each other."""
    block, step, real = torch.broadcast_tensors(block, step, real)
    c0, c1, c2, c3 = block & _M32, step & _M32, ((step >> 32) & 0xFFFF) | (tag << 16), real & _M32
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    out = []
    for a, b in ((c0, c1), (c2, c3)):
        rho = torch.sqrt(-2.0 * torch.log(((a >> 9).double() + 0.5) * 2.0 ** -23))
        ang = (b >> 9).double() * (2.0 * math.pi * 2.0 ** -23)
        out += [rho * torch.cos(ang), rho * torch.sin(ang)]
    return torch.stack(out, -1)


def _amp(eq, v):
    if eq == she.HEAT:
        return v
    return torch.sqrt(torch.clamp(v if eq == she.SPECIES else v * (1.0 - v), min=0.0))


def exact(case, seed):
    if case["kind"] == "rods":
        return _exact_rods(case, seed)
    if case["nx"] * case["ny"] * case["nz"] * case["count"] * case["steps"] > 2 ** 34:
        return None
    return _exact_grid(case, seed)


def _exact_rods(case, seed):
    looks = _looks(case)
    ps = [_params(case, seed)[q] for q in looks]
    dev, eq, B = _dev(), ps[0]["eq"], len(ps)
    N = torch.tensor([p["n"][0] for p in ps], device=dev)
    nm = int(N.max())
    dirichlet, theta = case["dirichlet"], {"be": 1.0, "cn": 0.5}.get(case["scheme"], 0.0)

    def col(f):
        return torch.tensor([float(f(p)) for p in ps], device=dev, dtype=torch.float64)[:, None]

    u0 = col(lambda p: p["u0"])
    uL, uR = col(lambda p: p.get("u_left", p["u0"])), col(lambda p: p.get("u_right", p["u0"]))
    nu = ps[0].get("nu", 0.0)
    i = torch.arange(nm, device=dev)[None, :]
    inside = i < N[:, None]
    ref = uL + (uR - uL) * (i + 0.5) / N[:, None] if dirichlet else u0.expand(B, nm)
    # conductance and noise factor of each face, capacity factor of each cell
    rf, sf, wc = np.zeros((B, nm + 1)), np.zeros((B, nm + 1)), np.ones((B, nm))
    for b, p in enumerate(ps):
        n = p["n"][0]
        lam = np.asarray(p["cond"]) if "cond" in p else np.ones(n)
        lf = np.empty(n + 1)
        lf[1:n] = 2.0 * lam[:-1] * lam[1:] / (lam[:-1] + lam[1:])
        lf[0], lf[n] = (lam[0], lam[-1]) if dirichlet else (2.0 * lam[0] * lam[-1] / (lam[0] + lam[-1]),) * 2
        rf[b, :n + 1] = p["r"] * lf
        sf[b, :n + 1] = np.sqrt(2.0 * p["r"] * lf * p["eps"])
        if "cap" in p:
            wc[b, :n] = 1.0 / np.asarray(p["cap"])
    rf, sf, wc = (torch.tensor(v, device=dev) for v in (rf, sf, wc))
    pc = torch.tensor([p["scheme"] == she.HEUN for p in ps], device=dev)[:, None]
    rows, last = torch.arange(B, device=dev), N - 1

    def div(U, z, ex):
        F = torch.zeros(B, nm + 1, device=dev, dtype=torch.float64)
        lo, hi = (U[:, :-1], U[:, 1:]) if dirichlet else (torch.cat([U[:, -1:], U[:, :-1]], 1), U)
        o = 1 if dirichlet else 0
        c = 0.5 * (lo + hi)
        F[:, o:nm] = ex * rf[:, o:nm] * (hi - lo) + sf[:, o:nm] * _amp(eq, c) * z[:, o:nm] - nu * c * (1.0 - c)
        if dirichlet:
            s2 = math.sqrt(2.0)
            F[:, 0] = (2.0 * rf[:, 0] * (ex * U[:, 0] - uL[:, 0]) + s2 * sf[:, 0] * _amp(eq, uL[:, 0]) * z[:, 0]
                       - nu * uL[:, 0] * (1.0 - uL[:, 0]))
            F[rows, N] = (2.0 * rf[rows, N] * (uR[:, 0] - ex * U[rows, last])
                          + s2 * sf[rows, N] * _amp(eq, uR[:, 0]) * z[rows, N] - nu * uR[:, 0] * (1.0 - uR[:, 0]))
        else:
            F[:, nm] = F[:, 0]
        return torch.where(inside, wc * (F[:, 1:] - F[:, :-1]), 0.0)

    minv = None
    if theta:  # (1 - theta A) is the same for every realisation
        n = nm
        A = torch.zeros(n, n, device=dev, dtype=torch.float64)
        for f in range(1, n):
            r = float(rf[0, f])
            A[f, f] -= r
            A[f, f - 1] += r
            A[f - 1, f - 1] -= r
            A[f - 1, f] += r
        r0, rn = float(rf[0, 0]), float(rf[0, n])
        if dirichlet:
            A[0, 0] -= 2.0 * r0
            A[n - 1, n - 1] -= 2.0 * rn
        else:
            A[0, 0] -= r0
            A[0, n - 1] += r0
            A[n - 1, n - 1] -= r0
            A[n - 1, 0] += r0
        minv = torch.linalg.inv(torch.eye(n, device=dev, dtype=torch.float64) - theta * A).T.contiguous()

    real = torch.tensor([p["realisation"] for p in ps], device=dev)[:, None]
    nb = (nm + 1 + 3) // 4
    blk = torch.arange(nb, device=dev)[None, :]
    zi = _normals(blk, torch.zeros((), device=dev, dtype=torch.int64), 1, real, seed).reshape(B, -1)[:, :nm]
    U = torch.where(inside, ref + col(lambda p: p["init_sd"]) * zi, 0.0)
    chunk = max(1, 2 ** 22 // (B * nb))
    samples, every = [], EVERY
    for t0 in range(0, case["steps"], chunk):
        m = min(chunk, case["steps"] - t0)
        z = _normals(blk[None], torch.arange(t0, t0 + m, device=dev)[:, None, None], 0, real[None], seed)
        z = z.reshape(m, B, -1)[:, :, :nm + 1]
        for k in range(m):
            if theta:
                U = (U + div(U, z[k], 1.0 - theta)) @ minv
            else:
                P = U + div(U, z[k], 1.0)
                U = torch.where(pc, 0.5 * (U + P + div(P, z[k], 1.0)), P) if bool(pc.any()) else P
            if case["stats"] != "none" and (t0 + k + 1) % every == 0:
                samples.append(torch.where(inside, U - ref, 0.0))
    out = {}
    sizes = [p["n"][0] for p in ps]

    def flat(v):
        return torch.cat([v[b, :n] for b, n in enumerate(sizes)]).cpu().numpy()

    if case["stats"] != "none" and samples:
        D = torch.stack(samples)  # [samples, B, nm]
        M, Nf = len(samples), N.double()
        m1, m2 = D.mean(0), (D * D).mean(0)
        out["mean"], out["var"] = flat(ref + m1), flat(m2 - m1 * m1)
        a, b = D.sum(2) / Nf, (D * D).sum(2) / Nf
        out["spatial_var"] = (b - a * a).mean(0).cpu().numpy()
        out["sum_u"] = torch.where(inside, U, 0.0).sum(1).cpu().numpy()
        out["n_samples"] = np.full(B, M)
        if case["stats"] == "corr":
            C = D.permute(1, 2, 0) @ D.permute(1, 0, 2).contiguous() / M - m1[:, :, None] * m1[:, None, :]
            out["corr"] = C.reshape(-1).cpu().numpy()
            out["sk"] = (torch.fft.fft(D + ref, dim=2).abs() ** 2).mean(0).reshape(-1).cpu().numpy()
    elif case["stats"] != "none":
        return None
    if case["fields"]:
        out["field"] = flat(U)
    return out


def _exact_grid(case, seed):
    looks = _looks(case)
    allp = _params(case, seed)
    parts = []
    for q in looks:
        parts.append(_exact_field(case, allp[q], seed))
    out = {}
    for key in parts[0]:
        out[key] = np.concatenate([np.atleast_1d(p[key]) for p in parts])
    return out


def _exact_field(case, p, seed):
    dev = _dev()
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    dim, eq, r = (2 if nz == 1 else 3), p["eq"], p["r"]
    sigma = math.sqrt(2.0 * r * p["eps"])
    real = torch.tensor(p["realisation"], device=dev)
    cells = nx * ny * nz
    zero = torch.zeros((), device=dev, dtype=torch.int64)
    zi = _normals(torch.arange(cells // 4, device=dev), zero, 1, real, seed).reshape(nz, ny, nx)
    U = p["u0"] + p["init_sd"] * zi
    blk = torch.arange(nz * ny * dim * nx // 4, device=dev)

    def div(V, z):
        tot = torch.zeros_like(V)
        for e in range(dim):
            ax = 2 - e
            lo = torch.roll(V, 1, ax)
            F = r * (V - lo) + sigma * _amp(eq, 0.5 * (lo + V)) * z[:, :, e]
            tot += torch.roll(F, -1, ax) - F
        return tot

    shells = None
    if case["stats"] == "sk":
        nb = she.n_shells((nx, ny))
        kx, ky = (torch.fft.fftfreq(n, 1.0 / n, device=dev, dtype=torch.float64) for n in (nx, ny))
        shells = torch.floor(torch.sqrt(kx[None, :] ** 2 + ky[:, None] ** 2) + 0.5).long().reshape(-1)
        modes = torch.bincount(shells, minlength=nb).double()
        sk = torch.zeros(nb, device=dev, dtype=torch.float64)
    sm = sv = 0.0
    count = 0
    for t in range(case["steps"]):
        z = _normals(blk, torch.full((), t, device=dev, dtype=torch.int64), 0, real, seed).reshape(nz, ny, dim, nx)
        P = U + div(U, z)
        U = 0.5 * (U + P + div(P, z)) if p["scheme"] == she.HEUN else P
        if case["stats"] != "none" and (t + 1) % EVERY == 0:
            count += 1
            d = U - p["u0"]
            a, b = d.mean(), (d * d).mean()
            sm, sv = sm + a, sv + (b - a * a)
            if shells is not None:
                sk += torch.zeros_like(sk).index_add_(0, shells, (torch.fft.fft2(U[0]).abs() ** 2).reshape(-1))
    out = {}
    if case["stats"] != "none":
        out["mean"], out["var"] = float(p["u0"] + sm / count), float(sv / count)
        if shells is not None:
            out["sk"] = torch.where(modes > 0, sk / (count * modes.clamp(min=1)), 0.0).cpu().numpy()
        out["sum_u"], out["spatial_var"], out["n_samples"] = float(U.sum()), float(sv / count), count
    if case["fields"]:
        out["field"] = U.reshape(-1).cpu().numpy()
    return out
