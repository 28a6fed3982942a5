"""The framework's performance cases: what a user's program has it do, over
the sizes that the repository's workloads span, each through the public
binding (``paper_cs_0703028_amd.rtlbl.Tracer``).

Four kinds of work:

``step``    the whole path on one grid: clear the tallies, kappa table, rays,
            powers per cell.  A flow solver calls it once per outer iteration.
``kappa``   one kappa (and Planck) table of a grid, in one of the line sum's
            forms: a program that keeps or studies spectra.
``trace``   rays through a table in hand, and their powers: more rays until
            the noise is low enough.
``batch``   one prepared graph launch over several receiver cases, and its
            results.

Powers of the plain form (``TALLY_F32``: an FP32 march with FP32 partial sums,
which the caller chose) are handed on as float32 fields, as a solver stores
them; those of the precision form (``TALLY_F64``) as float64.

Spectra follow the repository's laws: Lorentz lines with log-normal strengths,
a 5 cm^-1 cutoff, points at ``dnu``; ``density`` is lines per cm^-1.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_cs_0703028_amd import inputs as I
from paper_cs_0703028_amd import rtlbl as R

MODES = {"plain": R.KAPPA_PLAIN, "compensated": R.KAPPA_COMPENSATED,
         "table16": R.KAPPA_TABLE16, "adaptive": R.KAPPA_ADAPTIVE,
         "wings": R.KAPPA_ADAPTIVE_WINGS}


def _case(kind, nx, ny, nz, n_nu, density, **kw):
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "field": "hot", "n_nu": n_nu, "dnu": 0.01,
         "density": density, "density2": 0.0, "p": 1.0, "T_wall": 0.0, "mode": "plain",
         "planck": False, "prec": "f32", "eps": 1e-3, "rays": 0, "n_cases": 1}
    c.update(kw)
    return c


def listed():
    return [
        # a coarse receptor model called from a control loop: everything is latency
        _case("step", 5, 6, 7, 3037, 15.5, field="linear", p=1.3, T_wall=1100.0, rays=700,
              name="step_5x6x7_ragged"),
        # the small workload: one outer iteration of a coarse flow solution
        _case("step", 8, 8, 8, 10000, 5.0, field="linear", rays=1024, name="step_8cube"),
        # the same in the precision form (compensated sums, Planck table, FP64 sums)
        _case("step", 8, 8, 8, 10000, 5.0, field="linear", rays=1024, mode="compensated",
              planck=True, prec="f64", name="step_8cube_precision"),
        # the headline workload: one outer iteration of a resolved flow solution
        _case("step", 32, 32, 32, 50000, 40.0, rays=1 << 20, name="step_32cube"),
        # spectra of a receiver case of the batched workload
        _case("kappa", 24, 24, 24, 20000, 25.0, name="kappa_24cube"),
        # a dense line list on a small grid (200 lines per cm^-1)
        _case("kappa", 8, 8, 8, 10000, 200.0, field="linear", name="kappa_8cube_dense"),
        # two absorbing gases, as the paper's listing pairs H2O and CO2
        _case("kappa", 16, 16, 16, 20000, 25.0, density2=12.5, name="kappa_16cube_two_gases"),
        # the precision form's tables (kappa and Planck)
        _case("kappa", 16, 16, 16, 20000, 25.0, mode="compensated", planck=True,
              name="kappa_16cube_precision"),
        # adaptive windows with wing return on the headline grid
        _case("kappa", 32, 32, 32, 50000, 40.0, mode="wings", eps=1e-3, name="kappa_32cube_wings"),
        # the paper's own 16-point profile on the headline grid
        _case("kappa", 32, 32, 32, 50000, 40.0, mode="table16", name="kappa_32cube_table16"),
        # more rays in the precision form through tables in hand
        _case("trace", 24, 24, 24, 20000, 25.0, mode="compensated", planck=True, prec="f64",
              rays=1 << 14, name="trace_24cube_precision"),
        # a design study: several receiver cases in one prepared launch
        _case("batch", 24, 24, 24, 20000, 25.0, rays=1 << 15, n_cases=6, name="batch_6_cases"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "kappa", "kappa", "kappa", "trace", "batch"])
    dnu = rng.choice([0.005, 0.01, 0.01, 0.02, 0.05])
    density = math.exp(rng.uniform(math.log(3.0), math.log(200.0)))
    kw = {"dnu": dnu, "field": rng.choice(["hot", "linear"]), "p": round(rng.uniform(0.5, 2.0), 3),
          "T_wall": rng.choice([0.0, 0.0, round(rng.uniform(400.0, 1500.0), 1)])}
    if rng.random() < 0.5:  # a cube, or a box with odd sizes
        nx = ny = nz = _log_int(rng, 4, 28)
    else:
        nx, ny, nz = (_log_int(rng, 3, 28) for _ in range(3))
    n_nu = _log_int(rng, 1500, 40000)
    cells = nx * ny * nz
    # keep a drawn case below the largest listed one: line evaluations, updates
    most = 1.2e11
    evals = cells * n_nu * density * 10.0
    if evals > most:
        density = max(3.0, density * most / evals)
    density = round(density, 2)
    precise = rng.random() < 0.35
    segs = 3.0 / (1.0 / nx + 1.0 / ny + 1.0 / nz)
    rays = min(_log_int(rng, 300, 1 << 18), max(64, int(3e11 / (segs * n_nu))))
    if kind == "kappa":
        kw["mode"] = rng.choice(["plain", "plain", "compensated", "table16", "adaptive", "wings"])
        kw["eps"] = rng.choice([1e-2, 1e-3, 1e-4, 1e-5])
        kw["planck"] = kw["mode"] == "compensated" or rng.random() < 0.2
        if kw["mode"] in ("plain", "compensated", "table16") and rng.random() < 0.3:
            kw["density2"] = round(0.5 * density, 2)
    elif kind == "batch":
        kw["n_cases"] = rng.randint(2, 8)
        rays = max(64, rays // kw["n_cases"])
        nx = ny = nz = min(28, max(4, nx))
        kw["rays"] = rays
        kw["mode"] = "compensated" if precise else "plain"
    else:
        if precise:
            kw.update(mode="compensated", planck=True, prec="f64")
        elif rng.random() < 0.25:
            kw.update(mode=rng.choice(["table16", "wings"]))
        kw["rays"] = rays
    return _case(kind, nx, ny, nz, n_nu, density, **kw)


# ------------------------------------------------------------------- inputs
def _grid(c, seed, k=0):
    """Case k's grid: a hot spot or a linear temperature field, mole fractions
    drawn per cell.  Later cases of a batch are smaller and larger in turn."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    if c["kind"] == "batch":
        nx = ny = nz = max(2, nx + (k % 3 - 1) * (nx // 3))
    n = nx * ny * nz
    h = 1.0 / max(nx, ny, nz)
    i = np.arange(n)
    ix, iy, iz = i % nx, (i // nx) % ny, i // (nx * ny)
    if c["field"] == "hot":
        r2 = sum(((a + 0.5) / m - 0.5) ** 2 for a, m in ((ix, nx), (iy, ny), (iz, nz)))
        T = 400.0 + 1400.0 * np.exp(-r2 / (2.0 * 0.15 ** 2))
    else:
        T = 300.0 + 1200.0 * ix / max(nx - 1, 1)
    x = I.rng(seed + 7919 * k, I.STREAM_XH2O).uniform(0.05, 0.2, n)
    return I.Grid(nx, ny, nz, h, T.astype(np.float64), x, np.full(n, c["p"]), c["T_wall"])


def _lines(c, seed):
    span = c["n_nu"] * c["dnu"]
    return I.line_list(max(1, int(c["density"] * span)), 1000.0, 1000.0 + span, seed=seed,
                       dnu=c["dnu"], n_nu=c["n_nu"])


def _gas2(c, seed, grid):
    span = c["n_nu"] * c["dnu"]
    L = I.line_list(max(1, int(c["density2"] * span)), 1000.0, 1000.0 + span,
                    seed=seed + I.GAS2_SEED_OFFSET, dnu=c["dnu"], n_nu=c["n_nu"], s_median=3e-22,
                    gamma_lo=0.06, gamma_hi=0.09, n_exp=0.75)
    x = I.rng(seed, I.STREAM_XGAS).uniform(0.05, 0.15, grid.n_cells)
    return I.Gas(x=x, lines=L)


def prepare(case, seed):
    c = case
    s = {"case": c, "seed": seed, "tracer": R.Tracer(0)}
    t, L = s["tracer"], _lines(c, seed)
    if c["kind"] == "batch":
        t.setup_lines(L)
        cases = [I.Workload("case%d" % k, _grid(c, seed, k), L, c["rays"] * (1 + k % 2), seed + k)
                 for k in range(c["n_cases"])]
        s["workspace"] = t.batch_prepare(cases, kappa_mode=MODES[c["mode"]])
        return s
    g = _grid(c, seed)
    t.setup_grid(g)
    t.setup_lines(L)
    if c["density2"]:
        t.setup_gas(1, _gas2(c, seed, g))
    if c["mode"] in ("adaptive", "wings"):
        t.set_line_tolerance(c["eps"])
    ld = t.required_pitch()
    s["kappa"] = torch.empty((g.n_cells, ld), dtype=torch.float32, device="cuda")
    s["planck"] = torch.empty_like(s["kappa"]) if c["planck"] else None
    if c["kind"] == "trace":
        t.compute_kappa(MODES[c["mode"]], s["kappa"], s["planck"])
    return s


def _powers(c, parts):
    if c["prec"] == "f64":
        return parts
    return [tuple(np.asarray(a, np.float32) for a in p) for p in parts]


def run(state):
    c, t = state["case"], state["tracer"]
    if c["kind"] == "batch":
        t.batch_launch()
        return _powers(c, t.batch_results())
    if c["kind"] in ("step", "kappa"):
        t.compute_kappa(MODES[c["mode"]], state["kappa"], state["planck"])
    if c["kind"] == "kappa":
        return (state["kappa"], state["planck"]) if c["planck"] else state["kappa"]
    t.reset_tally()
    t.trace_rays(state["seed"], c["rays"], prec=R.TALLY_F64 if c["prec"] == "f64" else R.TALLY_F32)
    return _powers(c, [t.tally()])


# --------------------------------------------------------------------- work
def work(case):
    c = case
    K = 5.0 / c["dnu"]
    grids = [_grid(c, 1, k) for k in range(c["n_cases"])]
    cells = sum(g.n_cells for g in grids)
    n_nu, span = c["n_nu"], c["n_nu"] * c["dnu"]
    lines = c["density"] * span
    lines2 = c["density2"] * span
    flops = nbytes = 0.0
    if c["kind"] != "trace":
        if c["mode"] == "table16":     # a multiply-add at 16 points
            flops += 2.0 * 16 * (lines + lines2) * cells
        else:                          # d^2 + g^2, a reciprocal, a multiply-add
            pts = min(2 * K + 1, n_nu) * min(1.0, 1.0 - 0.25 * min(2 * K, n_nu) / n_nu)
            if c["mode"] in ("adaptive", "wings"):  # the points kept near T_ref
                L = _lines(c, 1)
                w2 = L.S * L.gamma / (math.pi * c["eps"] * L.S.sum() / span) - L.gamma ** 2
                pts = min(pts, float(np.mean(2.0 * np.minimum(np.sqrt(np.maximum(w2, 0.0)) / c["dnu"], K))))
            flops += 4.0 * pts * (lines + lines2) * cells
        nbytes += 48.0 * (lines + lines2) + 24.0 * cells
    if c["kind"] == "kappa":
        nbytes += 4.0 * cells * n_nu * (2 if c["planck"] else 1)
    else:
        for k, g in enumerate(grids):
            rays = c["rays"] * (1 + k % 2 if c["kind"] == "batch" else 1)
            segs = 3.0 / (1.0 / g.nx + 1.0 / g.ny + 1.0 / g.nz) * rays
            flops += 9.0 * segs * n_nu
        # the table is read once (and, where it is made here, written once)
        if c["kind"] != "batch":
            nbytes += 4.0 * cells * n_nu * (2 if c["planck"] else 1) * (2 if c["kind"] == "step" else 1)
        nbytes += 16.0 * cells
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------ the same in 64 bits (torch)
_H, _C, _KB, _ATM = 6.62607015e-34, 299792458.0, 1.380649e-23, 101325.0
_C2, _C1 = _H * _C / _KB * 100.0, 2.0 * _H * _C * _C * 1e8


def _dev(a):
    return torch.as_tensor(np.asarray(a, np.float64),
                           device="cuda" if torch.cuda.is_available() else "cpu")


def _ratio(L, T):
    """Eq. (1): strength ratio S(T)/S(T_ref), [cells, lines]."""
    nu, E = _dev(L.nu), _dev(L.E_lower)
    T = T[:, None]
    return ((L.T_ref / T) ** 1.5 * torch.exp(-_C2 * E * (1.0 / T - 1.0 / L.T_ref))
            * torch.expm1(-_C2 * nu / T) / torch.expm1(-_C2 * nu / L.T_ref))


def _exact_kappa(c, g, L, x, mode):
    """Eq. (2) of one gas, [cells, n_nu]."""
    n_nu, dnu = L.n_nu, L.dnu
    K = int(round(L.cutoff / dnu))
    order = np.argsort(L.nu, kind="stable")
    L = I.Lines(L.nu[order], L.S[order], L.gamma[order], L.n_T[order], L.E_lower[order], L.T_ref,
                L.cutoff, L.nu0, dnu, n_nu)
    r = (L.nu - L.nu0) / dnu
    meets = (np.floor(r) + K >= 0) & (np.ceil(r - K) <= n_nu - 1)
    L = I.Lines(*(a[meets] for a in (L.nu, L.S, L.gamma, L.n_T, L.E_lower)), L.T_ref, L.cutoff,
                L.nu0, dnu, n_nu)
    r = r[meets]
    T, p = _dev(g.T), _dev(g.p)
    u = _dev(x) * p * _ATM / (_KB * T) * 1e-6
    out = torch.zeros((g.n_cells, n_nu), dtype=torch.float64, device=T.device)
    rt, S = _dev(r), _dev(L.S)
    if mode == "table16":
        amp = u[:, None] * S * _ratio(L, T)
        m = np.floor(r)
        for k in range(16):
            j = m + (k - 7)
            ok = (j >= 0) & (j < n_nu)
            d = (j - r) * dnu
            f = _dev(L.gamma / (math.pi * (d * d + L.gamma ** 2)))
            out.index_add_(1, torch.as_tensor(j[ok].astype(np.int64), device=out.device),
                           (amp * f)[:, torch.as_tensor(ok, device=out.device)])
        return out
    gam = _dev(L.gamma) * p[:, None] * (L.T_ref / T[:, None]) ** _dev(L.n_T)
    s = S * _ratio(L, T)
    hw = None
    if mode in ("adaptive", "wings"):
        sbar = s.sum(1, keepdim=True) / (n_nu * dnu)
        w2 = s * gam / (math.pi * c["eps"] * sbar) - gam * gam
        w = torch.where(w2 < 0, -torch.ones_like(w2), torch.sqrt(w2.clamp(min=0)) / dnu)
        n8 = -(-g.n_cells // 8)
        pad = torch.full((n8 * 8, w.shape[1]), -1.0, dtype=w.dtype, device=w.device)
        pad[:g.n_cells] = w
        hw = pad.view(n8, 8, -1).amax(1).clamp(max=float(K)).repeat_interleave(8, 0)[:g.n_cells]
    amp = u[:, None] * s * gam / math.pi
    lost = torch.zeros(g.n_cells, dtype=torch.float64, device=T.device)
    step = 250
    for j0 in range(0, n_nu, step):
        j = torch.arange(j0, min(j0 + step, n_nu), device=T.device, dtype=torch.float64)
        a, b = (int(v) for v in np.searchsorted(r, (j0 - K - 1, j0 + step + K + 1)))
        block = max(1, int(6e7 / max(1, (b - a) * step)))
        for c0 in range(0, g.n_cells, block):
            q = slice(c0, c0 + block)
            d = j[None, :] - rt[a:b, None]
            keep = (d.abs() <= K)[None]
            if hw is not None:
                keep = keep & (d.abs()[None] <= hw[q, a:b, None])
            v = amp[q, a:b, None] / ((d * dnu)[None] ** 2 + gam[q, a:b, None] ** 2)
            out[q, j0:j0 + step] = torch.where(keep, v, torch.zeros_like(v)).sum(1)
    if mode == "wings":
        r_, m = rt, torch.floor(rt)
        h0 = torch.ceil(r_ - K).clamp(min=0)
        h1 = (m + K).clamp(max=n_nu - 1)
        k0 = torch.maximum(torch.ceil(r_ - hw), h0)
        k1 = torch.minimum(torch.floor(r_ + hw), h1)
        none = (hw < 0) | (k0 > k1)
        k0, k1 = torch.where(none, h1 + 1, k0), torch.where(none, h1, k1)
        u_ = u[:, None] * s / math.pi
        for lo, hi in ((h0.expand_as(k0), k0 - 1), (k1 + 1, h1.expand_as(k1))):
            mass = u_ * (torch.atan((hi + 0.5 - r_) * dnu / gam)
                         - torch.atan((lo - 0.5 - r_) * dnu / gam)) / dnu
            lost += torch.where(lo <= hi, mass, torch.zeros_like(mass)).sum(1)
        out += (lost / n_nu)[:, None]
    return out


def _planck(T, nu):
    return _C1 * nu ** 3 / torch.expm1(_C2 * nu / T)


_M0, _M1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
_W0, _W1 = 0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B


def _mulhilo(a, b):
    """128-bit products of uint64 arrays a by the constant (or array) b."""
    lo32 = np.uint64(0xFFFFFFFF)
    s = np.uint64(32)
    b = np.uint64(b)
    al, ah, bl, bh = a & lo32, a >> s, b & lo32, b >> s
    ll, lh, hl, hh = al * bl, al * bh, ah * bl, ah * bh
    mid = (ll >> s) + (lh & lo32) + (hl & lo32)
    return hh + (lh >> s) + (hl >> s) + (mid >> s), a * b


def _philox(seed, r, block):
    """Philox4x64-10 (Salmon et al., SC'11), key (seed, 1), counter (r, block, 0, 0)."""
    x = [r.copy(), np.full_like(r, block), np.zeros_like(r), np.zeros_like(r)]
    k0, k1 = seed, 1
    for _ in range(10):
        h0, l0 = _mulhilo(x[0], _M0)
        h1, l1 = _mulhilo(x[2], _M1)
        x = [h1 ^ x[1] ^ np.uint64(k0), l1, h0 ^ x[3] ^ np.uint64(k1), l0]
        k0, k1 = (k0 + _W0) % 2 ** 64, (k1 + _W1) % 2 ** 64
    return x


def _exact_rays(seed, n_rays, nx, ny, nz):
    """Origins (units of a cell) and directions of the set's rays."""
    r = np.arange(n_rays, dtype=np.uint64)
    w = _philox(seed, r, 0)
    n = np.array([nx, ny, nz])
    areas = [ny * nz, ny * nz, nz * nx, nz * nx, nx * ny, nx * ny]
    pick, _ = _mulhilo(w[0], sum(areas))
    face = np.searchsorted(np.cumsum(areas), pick.astype(np.int64), side="right")
    axis, side = face // 2, face % 2
    O, D = np.zeros((n_rays, 3)), np.zeros((n_rays, 3))
    t1, t2 = (axis + 1) % 3, (axis + 2) % 3
    i = np.arange(n_rays)
    O[i, axis] = np.where(side == 1, n[axis], 0)
    for t, v in ((t1, w[1]), (t2, w[2])):
        hi = np.array([int(a) * (int(n[b]) << 20) >> 64 for a, b in zip(v, t)])
        O[i, t] = (2 * hi + 1) / 2.0 ** 21
    R1 = 1 << 20
    A, B = np.zeros(n_rays, np.int64), np.zeros(n_rays, np.int64)
    open_ = np.ones(n_rays, bool)
    words = [w[3]]
    for k in range(61):
        if k > 0 and (k - 1) % 4 == 0:
            if not open_.any():
                break
            words = _philox(seed, r, 1 + (k - 1) // 4)
        v = words[0 if k == 0 else (k - 1) % 4]
        a = (v & np.uint64(2 * R1 - 1)).astype(np.int64) - R1
        b = ((v >> np.uint64(21)) & np.uint64(2 * R1 - 1)).astype(np.int64) - R1
        ok = open_ & (a * a + b * b < R1 * R1)
        A[ok], B[ok] = a[ok], b[ok]
        open_ &= ~ok
    rest = R1 * R1 - A * A - B * B
    Cn = np.floor(np.sqrt(rest.astype(np.float64))).astype(np.int64)
    Cn -= Cn * Cn > rest
    Cn += (Cn + 1) ** 2 <= rest
    D[i, axis] = np.where(side == 1, -Cn, Cn)
    D[i, t1], D[i, t2] = A, B
    return O, D


def _exact_powers(g, L, seed, n_rays, kappa):
    """Eq. (3) cell after cell: absorbed, emitted, {entering, emitted, absorbed, escaped}."""
    dev = kappa.device
    O, D = _exact_rays(seed, n_rays, g.nx, g.ny, g.nz)
    ts = []
    with np.errstate(divide="ignore", invalid="ignore"):
        for k, n in enumerate((g.nx, g.ny, g.nz)):
            t = (np.arange(n + 1)[None, :] - O[:, k:k + 1]) / D[:, k:k + 1]
            ts.append(np.where(np.isfinite(t) & (t > 0), t, np.inf))
    # the exit: the first axis whose last plane is reached
    last = np.stack([np.where(np.isfinite(t).any(1), np.where(np.isfinite(t), t, -np.inf).max(1),
                              np.inf) for t in ts])
    t_out = last.min(0)
    t = np.sort(np.concatenate(ts, axis=1), axis=1)
    t = np.concatenate([np.zeros((n_rays, 1)), t], axis=1)
    inside = t[:, 1:] <= t_out[:, None]
    with np.errstate(invalid="ignore"):
        mid = 0.5 * (t[:, 1:] + t[:, :-1])
    mid = np.where(inside, mid, 0.0)
    pos = [np.clip(np.floor(O[:, k:k + 1] + mid * D[:, k:k + 1]), 0, n - 1).astype(np.int64)
           for k, n in enumerate((g.nx, g.ny, g.nz))]
    cell = pos[0] + g.nx * (pos[1] + g.ny * pos[2])
    norm = np.sqrt((D ** 2).sum(1, keepdims=True))
    with np.errstate(invalid="ignore"):
        length = np.where(inside, (t[:, 1:] - t[:, :-1]), 0.0) * norm * g.cell_m * 100.0
    nu = L.nu0 + L.dnu * torch.arange(L.n_nu, dtype=torch.float64, device=dev)
    area = 2.0 * g.cell_m ** 2 * (g.nx * g.ny + g.ny * g.nz + g.nz * g.nx)
    wgt = math.pi * area * L.dnu / n_rays
    wall = _planck(g.T_wall, nu) if g.T_wall > 0 else torch.zeros_like(nu)
    T = _dev(g.T)
    ab = torch.zeros(g.n_cells, dtype=torch.float64, device=dev)
    em, bal = torch.zeros_like(ab), [wgt * n_rays * float(wall.sum()), 0.0, 0.0, 0.0]
    block = max(1, int(4e7 / L.n_nu))
    for r0 in range(0, n_rays, block):
        q = slice(r0, r0 + block)
        Ib = wall.expand(len(range(*q.indices(n_rays))), -1).clone()
        for k in range(cell.shape[1]):
            hit = np.nonzero(length[q, k] > 0)[0]
            if not len(hit):
                continue
            h = torch.as_tensor(hit, device=dev)
            cs = torch.as_tensor(cell[q, k][hit], device=dev)
            a = -torch.expm1(-kappa[cs] * _dev(length[q, k][hit])[:, None])
            B = _planck(T[cs][:, None], nu[None])
            I0 = Ib[h]
            ab.index_add_(0, cs, (I0 * a).sum(1))
            em.index_add_(0, cs, (B * a).sum(1))
            Ib[h] = I0 - (I0 - B) * a
        bal[3] += wgt * float(Ib.sum())
    ab, em = ab * wgt, em * wgt
    bal[1], bal[2] = float(em.sum()), float(ab.sum())
    return ab, em, torch.tensor(bal, dtype=torch.float64)


def exact(case, seed):
    c = case
    L = _lines(c, seed)
    K2 = 2 * 5.0 / c["dnu"]
    grids = [_grid(c, seed, k) for k in range(c["n_cases"])]
    cells = sum(g.n_cells for g in grids)
    pairs = cells * c["n_nu"] * (c["density"] + c["density2"]) * c["dnu"] * (K2 + 250)
    updates = 0.0
    if c["kind"] != "kappa":
        for k, g in enumerate(grids):
            updates += (3.0 / (1.0 / g.nx + 1.0 / g.ny + 1.0 / g.nz) * c["n_nu"]
                        * c["rays"] * (1 + k % 2 if c["kind"] == "batch" else 1))
    if pairs > 2e11 or updates > 4e10 or cells * c["n_nu"] > 1.2e9:  # over 20 seconds
        return None
    mode = "plain" if c["mode"] == "compensated" else c["mode"]
    outs = []
    for k, g in enumerate(grids):
        kap = _exact_kappa(c, g, L, g.x, mode)
        if c["density2"]:
            G2 = _gas2(c, seed, g)
            kap += _exact_kappa(c, g, G2.lines, G2.x, mode)
        if c["kind"] == "kappa":
            def pitched(v):
                ld = -(-c["n_nu"] // R.MARCH_CHUNK) * R.MARCH_CHUNK
                return torch.nn.functional.pad(v, (0, ld - c["n_nu"]))
            if not c["planck"]:
                return pitched(kap)
            nu = L.nu0 + L.dnu * torch.arange(L.n_nu, dtype=torch.float64, device=kap.device)
            return pitched(kap), pitched(_planck(_dev(g.T)[:, None], nu[None]))
        s = seed + k if c["kind"] == "batch" else seed
        rays = c["rays"] * (1 + k % 2 if c["kind"] == "batch" else 1)
        outs.append(_exact_powers(g, L, s, rays, kap))
    return outs
