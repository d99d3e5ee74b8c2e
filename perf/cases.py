"""The calls whose speed matters to a user of this package, as cases that can be timed and checked.

A case is a plain dict; ``prepare`` makes what a program holds before the call (states, contexts, weights), ``run``
makes one pass through the public entry points, ``work`` states the bytes and operations such a pass cannot do
without, and ``exact`` gives the same result in 64-bit torch, written from the equations.

Kinds of case:

* ``step``      one time step of a whole level (``Solver.advance``: CFL reduction and update),
* ``list``      the same for the listed patch groups of a refined level,
* ``hierarchy`` one root step of a refined hierarchy, replayed from its HIP graph,
* ``train``     one optimizer step of the learned flux,
* ``infer``     the network on a validation set,
* ``diag``      the diagnostics of a level (volume totals, divergence of B, CFL step).

The states are those of the paper's ABC box in motion: the force-free field plus smooth density, pressure and
velocity modes, a diagonal drift and i.i.d. velocity noise.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

GAMMA = 5.0 / 3.0
COURANT = 0.5
NOISE = 0.003
DTYPES = {"f64": torch.float64, "f32": torch.float32, "f32_mixed": torch.float32}
# operations of one cell update (all directions): reconstruction, tracing, two Riemann fluxes per direction, EMFs
FLOPS_STEP = {"ctu": 4000.0, "vl": 2200.0}
MLP_FLOPS = 2.0 * (15 * 64 + 64 * 64 + 64 * 7)
SHAPES = [(15, 64), (64,), (64, 64), (64,), (64, 7), (7,)]
NPARAM = sum(math.prod(s) for s in SHAPES)


def listed():
    def step(name, scheme, prec, nx, ny, nz):
        recon, riemann = {"ctu": ("ppm", "hlld"), "vl": ("plm", "roe"), "mlp": ("ppm", "mlp")}[scheme]
        return {"name": name, "kind": "step", "scheme": "vl" if scheme == "vl" else "ctu", "recon": recon,
                "riemann": riemann, "prec": prec, "nx": nx, "ny": ny, "nz": nz}

    return [
        # the plain method's configuration: 32^3 in double; a step is a handful of short launches
        step("vl_f64_32", "vl", "f64", 32, 32, 32),
        # the precision form's 128^3 box, in both precisions: what most runs spend their time on
        step("ctu_f32_128", "ctu", "f32", 128, 128, 128),
        step("ctu_f64_128", "ctu", "f64", 128, 128, 128),
        # the paper's own benchmark scheme
        step("vl_f32_128", "vl", "f32", 128, 128, 128),
        # the largest uniform run of the relaxation study
        step("ctu_f32_256", "ctu", "f32", 256, 256, 256),
        # a box whose sides are no multiples of anything, double energy beside single fields
        step("ctu_mixed_odd", "ctu", "f32_mixed", 97, 61, 83),
        # the learned flux in place of HLLD
        step("mlp_f32_128", "mlp", "f32", 128, 128, 128),
        # one refined level of uneven group count: the work unit of an AMR run
        {"name": "list_f32_191", "kind": "list", "scheme": "ctu", "recon": "ppm", "riemann": "hlld", "prec": "f32",
         "nx": 256, "ny": 256, "nz": 256, "groups": 191},
        # a whole hierarchy step: ghosts, updates, corrections, restriction
        {"name": "amr_f32_64", "kind": "hierarchy", "prec": "f32", "root": 64, "level1": 31, "level2": 67,
         "subcycle": False},
        # the training driver's batch
        {"name": "train_4096", "kind": "train", "rows": 4096},
        # the training driver's validation pass at the end of an epoch
        {"name": "infer_250k", "kind": "infer", "rows": 250_000},
        # what a run writes down every so many steps
        {"name": "diag_f64_128", "kind": "diag", "prec": "f64", "nx": 128, "ny": 128, "nz": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["step"] * 6 + ["list", "list", "hierarchy", "train", "infer", "diag"])
    if kind == "step":
        scheme, recon, riemann = rng.choice([("ctu", "ppm", "hlld")] * 3 + [("vl", "plm", "roe")] * 2 +
                                            [("ctu", "ppm", "mlp"), ("ctu", "plm", "roe"), ("vl", "ppm", "hlld")])
        prec = "f32" if riemann == "mlp" else rng.choice(["f32", "f32", "f64", "f64", "f32_mixed"])
        nx, ny, nz = (_log_int(rng, 16, 160) for _ in range(3))
        return {"kind": kind, "scheme": scheme, "recon": recon, "riemann": riemann, "prec": prec,
                "nx": nx, "ny": ny, "nz": nz}
    if kind == "list":
        prec = rng.choice(["f32", "f32", "f64"])
        n = 16 * rng.randint(4, 12)
        return {"kind": kind, "scheme": "ctu", "recon": "ppm", "riemann": "hlld", "prec": prec, "nx": n, "ny": n,
                "nz": 16 * rng.randint(4, 12), "groups": min(_log_int(rng, 4, 300), n // 16 * (n // 16) * 3)}
    if kind == "hierarchy":
        return {"kind": kind, "prec": rng.choice(["f32", "f32", "f64"]), "root": 16 * rng.randint(2, 4),
                "level1": _log_int(rng, 3, 48), "level2": _log_int(rng, 5, 96), "subcycle": rng.random() < 0.5}
    if kind == "diag":
        nx, ny, nz = (_log_int(rng, 16, 200) for _ in range(3))
        return {"kind": kind, "prec": rng.choice(["f32", "f64"]), "nx": nx, "ny": ny, "nz": nz}
    return {"kind": kind, "rows": _log_int(rng, 256, 16384) if kind == "train" else _log_int(rng, 1000, 600_000)}


# ------------------------------------------------------------------ inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _primitives(nx, ny, nz, seed):
    """rho, v, p at cells and the divergence-free field on the lower faces, in double."""
    dev = _device()
    rng = random.Random(seed)
    L = max(nx, ny, nz)
    # whole numbers of periods along each side
    x, y, z = (((torch.arange(n, dtype=torch.float64, device=dev) + 0.5) * (2 * math.pi / n)).reshape(shape)
               for n, shape in ((nx, (1, 1, nx)), (ny, (1, ny, 1)), (nz, (nz, 1, 1))))

    def modes(amp):
        out = torch.zeros((nz, ny, nx), dtype=torch.float64, device=dev)
        for _ in range(3):
            k = [rng.randint(0, 2) for _ in range(3)]
            out += amp / 3 * torch.cos(k[0] * x + k[1] * y + k[2] * z + rng.uniform(0, 2 * math.pi))
        return out

    gen = torch.Generator(device=dev).manual_seed(seed)
    noise = (torch.rand((3, nz, ny, nx), generator=gen, dtype=torch.float64, device=dev) * 2 - 1) * NOISE
    rho, p = 1 + modes(0.2), 1 + modes(0.2)
    v = [modes(0.15) + drift + noise[a] for a, drift in enumerate((0.08, 0.11, 0.06))]
    s = [rng.uniform(0, 2 * math.pi) for _ in range(3)]
    full = (nz, ny, nx)
    b = [torch.sin(z + s[2]) + torch.cos(y + s[1]), torch.sin(x + s[0]) + torch.cos(z + s[2]),
         torch.sin(y + s[1]) + torch.cos(x + s[0])]
    return rho, v, p, torch.stack([c.expand(full) for c in b]), 1.0 / L


def _up(q, a):
    """the neighbour one cell up along axis a (0: x, 1: y, 2: z), periodic"""
    return torch.roll(q, -1, dims=q.dim() - 1 - a)


def _down(q, a):
    return torch.roll(q, 1, dims=q.dim() - 1 - a)


def _conserved(nx, ny, nz, prec, seed):
    """U (5, ...), face B (3, ...) in the level's type, the double energy, and dx."""
    rho, v, p, B, dx = _primitives(nx, ny, nz, seed)
    B = B.to(DTYPES[prec])
    Bd = B.double()
    bc = [0.5 * (Bd[a] + _up(Bd[a], a)) for a in range(3)]
    e = p / (GAMMA - 1) + 0.5 * rho * sum(c * c for c in v) + 0.5 * sum(c * c for c in bc)
    U = torch.stack([rho, *(rho * c for c in v), e]).to(DTYPES[prec])
    return U.contiguous(), B.contiguous(), e.contiguous(), dx


def _group_origins(case, seed):
    g = [case[k] // 16 for k in ("nx", "ny", "nz")]
    pick = random.Random(seed).sample(range(g[0] * g[1] * g[2]), case["groups"])
    return torch.tensor([[16 * (q % g[0]), 16 * (q // g[0] % g[1]), 16 * (q // (g[0] * g[1]))] for q in pick],
                        dtype=torch.int32)


def _weights(seed):
    """Packed network weights of a surrogate that behaves: a GELU pair (g(x) - g(-x) = x) carries each of the seven
    unit jumps through both hidden layers to a dissipation of about the fast speed, small seeded weights elsewhere."""
    gen = torch.Generator().manual_seed(seed)
    w = [0.02 * (torch.rand(s, generator=gen) * 2 - 1) for s in SHAPES]
    w[4] *= 0.5
    gain = [-1.2, -1.2, -1.2, -1.2, -1.8, -1.2, -1.2]
    for q in range(7):
        for h, sign in ((2 * q, 1.0), (2 * q + 1, -1.0)):
            w[0][7 + q, h] += sign
            w[2][2 * q, h] += sign
            w[2][2 * q + 1, h] -= sign
            w[4][h, q] += sign * gain[q]
    return torch.cat([x.reshape(-1) for x in w]).to(torch.float32)


def _training(rows, seed):
    """Features as the interface normalisation gives them, targets, and a run's weights and Adam moments."""
    gen = torch.Generator().manual_seed(seed)
    mean = torch.randn((rows, 7), generator=gen) * torch.tensor([0.0, 0.3, 0.3, 0.3, 0.0, 1.0, 1.0])
    mean[:, 0] = 1.0
    mean[:, 4] = torch.exp(torch.rand(rows, generator=gen) * 5 - 6)        # jump sizes 2e-3 .. 0.4
    jump = torch.nn.functional.normalize(torch.randn((rows, 7), generator=gen), dim=1)
    X = torch.cat([mean, jump, torch.randn((rows, 1), generator=gen)], dim=1).contiguous()
    T = -1.2 * jump * torch.tensor([1, 1, 1, 1, 1.5, 1, 1.0]) * (1 + 0.2 * mean[:, 5:6] ** 2)
    m = 1e-3 * torch.randn(NPARAM, generator=gen)
    v = 1e-6 * (0.5 + torch.rand(NPARAM, generator=gen))
    return X, T.contiguous(), _weights(seed + 1), m, v


# ------------------------------------------------------------------ cases
def prepare(case, seed):
    from paper_1804_03479_amd.mhd import Level, MlpOps, Solver
    kind = case["kind"]
    if kind in ("train", "infer"):
        ops = MlpOps(Solver("ctu", "ppm", "mlp", "f32"))
        X, T, P, m, v = (t.cuda() for t in _training(case["rows"], seed))
        s = {"kind": kind, "ops": ops, "X": X, "P": P}
        if kind == "train":
            s.update(T=T, m=m, v=v, g=torch.zeros_like(P), step=100, loss=torch.zeros(1, device="cuda"))
        return s
    if kind == "hierarchy":
        from paper_1804_03479_amd import inputs
        from paper_1804_03479_amd.amr import Hierarchy
        n = case["root"]
        rho, v, p, B, dx = _primitives(n, n, n, seed)
        f = {"rho": rho, "vx": v[0], "vy": v[1], "vz": v[2], "p": p, "bx": B[0], "by": B[1], "bz": B[2]}
        problem = inputs.Problem({k: t.cpu().numpy() for k, t in f.items()}, dx=dx)
        h = Hierarchy(n, [case["level1"], case["level2"]], prec=case["prec"], seed=seed, subcycle=case["subcycle"],
                      problem=problem)
        return {"kind": kind, "h": h, "graph": h.capture()}
    U, B, e, dx = _conserved(case["nx"], case["ny"], case["nz"], case["prec"], seed)
    mixed = case["prec"] == "f32_mixed"
    if kind == "diag":
        return {"kind": kind, "solver": Solver("ctu", "ppm", "hlld", case["prec"]), "level": Level(U, B, dx)}
    groups = _group_origins(case, seed).cuda() if kind == "list" else None
    s = Solver(case["scheme"], case["recon"], case["riemann"], case["prec"], courant=COURANT, gamma=GAMMA)
    if case["riemann"] == "mlp":
        MlpOps(s).set_weights(_weights(seed).cuda())
    return {"kind": kind, "solver": s, "level": Level(U, B, dx, groups, 16, E64=e if mixed else None),
            "t": torch.zeros(1, dtype=torch.float64, device="cuda"), "double": case["prec"] == "f64"}


def run(state):
    kind = state["kind"]
    if kind in ("step", "list"):
        lv = state["level"]
        state["solver"].advance(lv, t_dev=state["t"])
        # a single-precision run keeps its clock in a double too, but to the accuracy of its wave speeds; the mixed
        # form's energy is mirrored into U
        return {"U": lv.U, "B": lv.B, "t": state["t"]} if state["double"] else {"U": lv.U, "B": lv.B}
    if kind == "hierarchy":
        h = state["h"]
        h.replay(state["graph"])
        torch.cuda.current_stream().wait_stream(h.stream)
        return [t for lv in h.levels for t in (lv.U, lv.B)]
    ops = state.get("ops")
    if kind == "train":
        state["step"] += 1
        ops.train_step(state["P"], state["m"], state["v"], state["g"], state["step"], state["X"], state["T"], 1e-3,
                       state["loss"])
        return {k: state[k] for k in ("P", "m", "v", "g", "loss")}
    if kind == "infer":
        return ops.forward(state["P"], state["X"])
    s, lv = state["solver"], state["level"]
    return {"sums": s.sums(lv), "divb": list(s.divb(lv)), "dt": s.cfl_dt(lv)}


def work(case):
    kind = case["kind"]
    if kind in ("train", "infer"):
        n = case["rows"]
        if kind == "infer":
            return {"bytes": 4.0 * (22 * n + NPARAM), "flops": MLP_FLOPS * n}
        return {"bytes": 4.0 * (22 * n + 7 * NPARAM), "flops": 3 * MLP_FLOPS * n}
    word = 8.0 if case["prec"] == "f64" else 4.0
    if kind == "hierarchy":
        cells = [case["root"] ** 3] + [case[k] * 4096 * (2 ** (l + 1) if case["subcycle"] else 1)
                                       for l, k in enumerate(("level1", "level2"))]
        return {"bytes": 16 * word * sum(cells), "flops": FLOPS_STEP["ctu"] * sum(cells)}
    cells = case["groups"] * 4096.0 if kind == "list" else float(case["nx"] * case["ny"] * case["nz"])
    if kind == "diag":
        return {"bytes": 8 * word * cells, "flops": 120.0 * cells}
    flops = FLOPS_STEP[case["scheme"]] + (6 * MLP_FLOPS if case["riemann"] == "mlp" else 0.0)
    # U and B in and out; the mixed form's double energy as well
    return {"bytes": (16 * word + (16 if case["prec"] == "f32_mixed" else 0)) * cells, "flops": flops * cells}


# ------------------------------------------------------------------ the same in 64 bits
def _flux(w, bn):
    """conserved state and flux along the normal of w = (rho, vn, v1, v2, p, b1, b2)"""
    d, vn, v1, v2, p, b1, b2 = w
    bb = bn * bn + b1 * b1 + b2 * b2
    e = p / (GAMMA - 1) + 0.5 * d * (vn * vn + v1 * v1 + v2 * v2) + 0.5 * bb
    pt, vb = p + 0.5 * bb, vn * bn + v1 * b1 + v2 * b2
    u = torch.stack([d, d * vn, d * v1, d * v2, e, b1, b2])
    f = torch.stack([d * vn, d * vn * vn + pt - bn * bn, d * vn * v1 - bn * b1, d * vn * v2 - bn * b2,
                     (e + pt) * vn - bn * vb, b1 * vn - bn * v1, b2 * vn - bn * v2])
    return u, f, pt


def _fast(d, p, bn, b1, b2):
    a2, t2 = GAMMA * p / d, (b1 * b1 + b2 * b2) / d
    n2 = bn * bn / d
    return torch.sqrt(0.5 * (a2 + n2 + t2 + torch.sqrt((a2 - n2 - t2) ** 2 + 4 * a2 * t2)))


def _hlld(wl, wr, bn):
    (ul, fl, ptl), (ur, fr, ptr) = _flux(wl, bn), _flux(wr, bn)
    c = torch.maximum(_fast(wl[0], wl[4], bn, wl[5], wl[6]), _fast(wr[0], wr[4], bn, wr[5], wr[6]))
    sl, sr = torch.minimum(wl[1], wr[1]) - c, torch.maximum(wl[1], wr[1]) + c
    ml, mr = wl[0] * (sl - wl[1]), wr[0] * (sr - wr[1])
    sm = (mr * wr[1] - ml * wl[1] - ptr + ptl) / (mr - ml)
    pts = ptl + ml * (sm - wl[1])

    def star(w, u, s, pt):
        d, vn = w[0], w[1]
        sv, ss = s - vn, s - sm
        ds, den = d * sv / ss, d * sv * ss - bn * bn
        flat = den.abs() <= 1e-12 * ((d * sv * ss).abs() + bn * bn)
        safe = torch.where(flat, torch.ones_like(den), den)
        mf = torch.where(flat, torch.zeros_like(den), bn * (sm - vn) / safe)
        bf = torch.where(flat, torch.ones_like(den), (d * sv * sv - bn * bn) / safe)
        v1, v2, b1, b2 = w[2] - w[5] * mf, w[3] - w[6] * mf, w[5] * bf, w[6] * bf
        vb, vbs = vn * bn + w[2] * w[5] + w[3] * w[6], sm * bn + v1 * b1 + v2 * b2
        es = (sv * u[4] - pt * vn + pts * sm + bn * (vb - vbs)) / ss
        return torch.stack([ds, ds * sm, ds * v1, ds * v2, es, b1, b2]), v1, v2

    usl, v1l, v2l = star(wl, ul, sl, ptl)
    usr, v1r, v2r = star(wr, ur, sr, ptr)
    dl, dr = torch.sqrt(usl[0]), torch.sqrt(usr[0])
    sls, srs = sm - bn.abs() / dl, sm + bn.abs() / dr
    sg = torch.where(bn >= 0, 1.0, -1.0)
    i = 1 / (dl + dr)
    v1, v2 = (dl * v1l + dr * v1r + (usr[5] - usl[5]) * sg) * i, (dl * v2l + dr * v2r + (usr[6] - usl[6]) * sg) * i
    b1 = (dl * usr[5] + dr * usl[5] + dl * dr * (v1r - v1l) * sg) * i
    b2 = (dl * usr[6] + dr * usl[6] + dl * dr * (v2r - v2l) * sg) * i
    vb = sm * bn + v1 * b1 + v2 * b2
    ussl = torch.stack([usl[0], usl[1], usl[0] * v1, usl[0] * v2,
                        usl[4] - dl * (sm * bn + v1l * usl[5] + v2l * usl[6] - vb) * sg, b1, b2])
    ussr = torch.stack([usr[0], usr[1], usr[0] * v1, usr[0] * v2,
                        usr[4] + dr * (sm * bn + v1r * usr[5] + v2r * usr[6] - vb) * sg, b1, b2])
    fsl, fsr = fl + sl * (usl - ul), fr + sr * (usr - ur)
    f = torch.where(sm >= 0, fsl + sls * (ussl - usl), fsr + srs * (ussr - usr))
    f = torch.where(sls >= 0, fsl, torch.where(srs <= 0, fsr, f))
    return torch.where(sl >= 0, fl, torch.where(sr <= 0, fr, f))


def _alphas(asq, cfsq, cssq):
    """fast and slow weights of Roe & Balsara's normalisation"""
    one, zero = torch.ones_like(asq), torch.zeros_like(asq)
    gap = cfsq - cssq
    inv = 1 / torch.where(gap > 0, gap, one)
    af, sl = torch.sqrt(((asq - cssq) * inv).clamp(min=0)), torch.sqrt(((cfsq - asq) * inv).clamp(min=0))
    af, sl = torch.where(cfsq - asq <= 0, one, af), torch.where(cfsq - asq <= 0, zero, sl)
    af, sl = torch.where(asq - cssq <= 0, zero, af), torch.where(asq - cssq <= 0, one, sl)
    return torch.where(gap <= 0, one, af), torch.where(gap <= 0, zero, sl)


def _roe(wl, wr, bn):
    (ul, fl, ptl), (ur, fr, ptr) = _flux(wl, bn), _flux(wr, bn)
    g1, g2 = GAMMA - 1, GAMMA - 2
    rl, rr = torch.sqrt(wl[0]), torch.sqrt(wr[0])
    i = 1 / (rl + rr)
    d = rl * rr
    vx, vy, vz = ((rl * wl[k] + rr * wr[k]) * i for k in (1, 2, 3))
    h = (rl * ((ul[4] + ptl) / wl[0]) + rr * ((ur[4] + ptr) / wr[0])) * i
    by, bz = ((rr * wl[k] + rl * wr[k]) * i for k in (5, 6))
    X = 0.5 * ((wr[5] - wl[5]) ** 2 + (wr[6] - wl[6]) ** 2) * i * i
    vsq, btsq = vx * vx + vy * vy + vz * vz, by * by + bz * bz
    ca2, ct2 = bn * bn / d, btsq / d
    hp = h - ca2 - ct2
    asq = g1 * (hp - 0.5 * vsq) - g2 * X
    cfsq = 0.5 * (ca2 + ct2 + asq + torch.sqrt((ca2 + ct2 - asq) ** 2 + 4 * asq * ct2))
    cssq = asq * ca2 / cfsq
    cf, cs, ca, a, bt = cfsq.sqrt(), cssq.sqrt(), ca2.sqrt(), asq.sqrt(), btsq.sqrt()
    ib = 1 / torch.where(bt > 0, bt, torch.ones_like(bt))
    b2, b3 = (torch.where(bt > 0, q * ib, torch.full_like(bt, math.sqrt(0.5))) for q in (by, bz))
    af, sl = _alphas(asq, cfsq, cssq)
    sq = d.sqrt()
    s = torch.where(bn >= 0, 1.0, -1.0)
    qf, qs, afp, asp = cf * af * s, cs * sl * s, af * a / sq, sl * a / sq
    vb = vy * b2 + vz * b3
    n = 0.5 / asq
    Cff, Css, Qf, Qs, Af, As = n * af * cf, n * sl * cs, n * qf, n * qs, n * af * a * sq, n * sl * a * sq
    gf, gs, hv = g1 * n * af, g1 * n * sl, vsq - hp
    lf, ls = n * afp * bt, n * asp * bt
    z = torch.zeros_like(d)
    waves = []
    for sg, cfast in ((-1, cf), (1, cf)):
        waves.append((vx + sg * cfast,
                      [gf * hv + Cff * (cf - sg * vx) + sg * Qs * vb - ls, -gf * vx + sg * Cff, -gf * vy - sg * Qs * b2,
                       -gf * vz - sg * Qs * b3, gf, As * b2 - gf * by, As * b3 - gf * bz],
                      [af, af * (vx + sg * cf), af * vy - sg * qs * b2, af * vz - sg * qs * b3,
                       af * (hp + sg * vx * cf) - sg * qs * vb + asp * bt, asp * b2, asp * b3]))
        waves.append((vx + sg * ca,
                      [-sg * 0.5 * (vy * b3 - vz * b2), z, sg * 0.5 * b3, -sg * 0.5 * b2, z, -0.5 * sq * b3 * s,
                       0.5 * sq * b2 * s],
                      [z, z, sg * b3, -sg * b2, sg * (vy * b3 - vz * b2), -s * b3 / sq, s * b2 / sq]))
        waves.append((vx + sg * cs,
                      [gs * hv + Css * (cs - sg * vx) - sg * Qf * vb + lf, -gs * vx + sg * Css, -gs * vy + sg * Qf * b2,
                       -gs * vz + sg * Qf * b3, gs, -Af * b2 - gs * by, -Af * b3 - gs * bz],
                      [sl, sl * (vx + sg * cs), sl * vy + sg * qf * b2, sl * vz + sg * qf * b3,
                       sl * (hp + sg * vx * cs) + sg * qf * vb - afp * bt, -afp * b2, -afp * b3]))
    waves.append((vx, [1 - (0.5 * g1 * vsq - g2 * X) / asq, g1 * vx / asq, g1 * vy / asq, g1 * vz / asq, -g1 / asq,
                       g1 * by / asq, g1 * bz / asq],
                  [torch.ones_like(d), vx, vy, vz, 0.5 * vsq + g2 * X / g1, z, z]))
    du = ur - ul
    f = 0.5 * (fl + fr)
    for lam, left, right in waves:
        f = f - 0.5 * (lam.abs() * sum(p * q for p, q in zip(left, du))) * torch.stack(right)
    return f


def _learned(P):
    """the learned flux with these weights: the exact central part and the network's dissipation"""
    net = _network(P)

    def flux(wl, wr, bn):
        (_, fl, _), (_, fr, _) = _flux(wl, bn), _flux(wr, bn)
        rho0, p0 = 0.5 * (wl[0] + wr[0]), 0.5 * (wl[4] + wr[4])
        v0, b0 = torch.sqrt(p0 / rho0), torch.sqrt(p0)
        sc = torch.stack([rho0, v0, v0, v0, p0, b0, b0])
        jump = (wr - wl) / sc
        s = jump.square().sum(0).sqrt()
        x = 0.5 * (wl + wr) / sc
        x[4] = s
        X = torch.cat([x, jump / s.clamp(min=1e-300), (bn / b0)[None]])
        y = net(X.reshape(15, -1).T).T.reshape(wl.shape)
        return 0.5 * (fl + fr) + y * s * torch.stack([rho0 * v0, p0, p0, p0, p0 * v0, b0 * v0, b0 * v0])

    return flux


def _network(P):
    w, at = [], 0
    for shape in SHAPES:
        n = math.prod(shape)
        w.append(P[at:at + n].reshape(shape))
        at += n

    def gelu(x):
        return torch.nn.functional.gelu(x, approximate="tanh")

    return lambda X: gelu(gelu(X @ w[0] + w[1]) @ w[2] + w[3]) @ w[4] + w[5]


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))


def _edges(q, a, recon):
    """limited lower and upper edge values of each cell along axis a"""
    dl, dr = q - _down(q, a), _up(q, a) - q
    if recon == "plm":
        s = _minmod(dl, dr)
        return q - 0.5 * s, q + 0.5 * s
    s = _minmod(0.5 * (dl + dr), 2 * _minmod(dl, dr))
    lo = 0.5 * (_down(q, a) + q) - (s - _down(s, a)) / 6
    hi = _up(lo, a)
    flat = (hi - q) * (q - lo) <= 0
    d, c = hi - lo, q - 0.5 * (lo + hi)
    new_lo = torch.where(d * c > d * d / 6, 3 * q - 2 * hi, lo)
    new_hi = torch.where(-d * d / 6 > d * c, 3 * q - 2 * lo, hi)
    return torch.where(flat, q, new_lo), torch.where(flat, q, new_hi)


def _trace(c, lo, hi, bn_lo, bn_hi, r, every):
    """edge states of a cell half a step on: each wave takes the average of the parabola over what it sweeps"""
    d, u, p, by, bz = c[0], c[1], c[4], c[5], c[6]
    dq, q6 = hi - lo, 6 * (c - 0.5 * (lo + hi))
    bn = 0.5 * (bn_lo + bn_hi)
    sd = d.sqrt()
    asq, btsq = GAMMA * p / d, by * by + bz * bz
    ca2, ct2 = bn * bn / d, btsq / d
    cfsq = 0.5 * (asq + ca2 + ct2 + torch.sqrt((ca2 + ct2 - asq) ** 2 + 4 * asq * ct2))
    cssq = asq * ca2 / cfsq
    cf, cs, ca, a, bt = cfsq.sqrt(), cssq.sqrt(), bn.abs() / sd, asq.sqrt(), btsq.sqrt()
    ib = 1 / torch.where(bt > 0, bt, torch.ones_like(bt))
    b2, b3 = (torch.where(bt > 0, q * ib, torch.full_like(bt, math.sqrt(0.5))) for q in (by, bz))
    af, sl = _alphas(asq, cfsq, cssq)
    sg = torch.where(bn >= 0, 1.0, -1.0)
    Qf, Qs, Af, As = cf * af * sg, cs * sl * sg, a * af * sd, a * sl * sd
    n = 0.5 / asq
    z, one = torch.zeros_like(d), torch.ones_like(d)
    waves = [(u, [one, z, z, z, -1 / asq, z, z], [one, z, z, z, z, z, z])]
    for w in (-1, 1):
        waves.append((u + w * cf, [z, w * n * cf * af, -w * n * Qs * b2, -w * n * Qs * b3, n * af / d, n * As * b2 / d,
                                   n * As * b3 / d],
                      [d * af, w * cf * af, -w * Qs * b2, -w * Qs * b3, d * asq * af, As * b2, As * b3]))
        waves.append((u + w * cs, [z, w * n * cs * sl, w * n * Qf * b2, w * n * Qf * b3, n * sl / d, -n * Af * b2 / d,
                                   -n * Af * b3 / d],
                      [d * sl, w * cs * sl, w * Qf * b2, w * Qf * b3, d * asq * sl, -Af * b2, -Af * b3]))
        waves.append((u + w * ca, [z, z, 0.5 * w * b3, -0.5 * w * b2, z, -0.5 * sg * b3 / sd, 0.5 * sg * b2 / sd],
                      [z, z, w * b3, -w * b2, z, -sg * sd * b3, sg * sd * b2]))
    for lam, left, right in waves:
        xi = lam * r
        ad, a6 = (sum(g * q for g, q in zip(left, x)) for x in (dq, q6))
        up, dn = (xi, -xi) if every else (xi.clamp(min=0), (-xi).clamp(min=0))
        right = torch.stack(right)
        hi = hi - 0.5 * up * (ad - (1 - 2 / 3 * xi) * a6) * right
        lo = lo + 0.5 * dn * (ad + (1 + 2 / 3 * xi) * a6) * right
    hb = 0.5 * r * (bn_hi - bn_lo)
    src = torch.stack([z, z, z, z, z, hb * c[2], hb * c[3]])
    return lo + src, hi + src


def _frame(W, a):
    """(rho, vn, v1, v2, p, b1, b2) of W = (rho, vx, vy, vz, p, bx, by, bz) along axis a"""
    b, c = (a + 1) % 3, (a + 2) % 3
    return torch.stack([W[0], W[1 + a], W[1 + b], W[1 + c], W[4], W[5 + b], W[5 + c]])


def _to_box(f, a):
    """mass, momentum x, y, z, energy, and the two EMFs the a-face carries: E_b = F[B_c], E_c = -F[B_b]"""
    b, c = (a + 1) % 3, (a + 2) % 3
    out = [f[0], None, None, None, f[4], f[6], -f[5]]
    out[1 + a], out[1 + b], out[1 + c] = f[1], f[2], f[3]
    return torch.stack(out)


def _prims(U, B):
    bc = [0.5 * (B[a] + _up(B[a], a)) for a in range(3)]
    v = [U[1 + a] / U[0] for a in range(3)]
    p = (GAMMA - 1) * (U[4] - 0.5 * U[0] * sum(c * c for c in v) - 0.5 * sum(c * c for c in bc))
    return torch.stack([U[0], *v, p, *bc])


def _emfs(F, W):
    """upwind corner EMFs from the face values and the cells' -v x B"""
    out = []
    for a in range(3):
        b, c = (a + 1) % 3, (a + 2) % 3
        r11 = W[1 + c] * W[5 + b] - W[1 + b] * W[5 + c]
        r01, r10 = _down(r11, b), _down(r11, c)
        r00 = _down(r01, c)
        eb1, mb1, ec1, mc1 = F[b][6], F[b][0], F[c][5], F[c][0]
        eb0, mb0, ec0, mc0 = _down(eb1, c), _down(mb1, c), _down(ec1, b), _down(mc1, b)

        def pick(m, pos, neg):
            return torch.where(m > 0, pos, torch.where(m < 0, neg, 0.5 * (pos + neg)))

        out.append(0.25 * (eb0 + eb1 + ec0 + ec1) +
                   0.25 * (pick(mb0, ec0 - r00, ec1 - r10) - pick(mb1, r01 - ec0, r11 - ec1) +
                           pick(mc0, eb0 - r00, eb1 - r01) - pick(mc1, r10 - eb0, r11 - eb1)))
    return out


def _update(U, B, F, E, r):
    U = U - r * sum(_up(F[a][:5], a) - F[a][:5] for a in range(3))
    Bn = []
    for a in range(3):
        b, c = (a + 1) % 3, (a + 2) % 3
        Bn.append(B[a] - r * (_up(E[c], b) - E[c]) + r * (_up(E[b], c) - E[b]))
    return U, torch.stack(Bn)


def _correct(s, a, F, E, bn, bnh, dbn, hr):
    """transverse update of the states of the a-edges of their own cells, from field bn to the half-step field bnh"""
    b, c = (a + 1) % 3, (a + 2) % 3
    bf = [bn, s[5], s[6]]
    v = s[1:4]
    vb = sum(p * q for p, q in zip(v, bf))
    e = s[4] / (GAMMA - 1) + 0.5 * s[0] * sum(q * q for q in v) + 0.5 * sum(q * q for q in bf) + hr * dbn * vb
    m = [s[0] * v[k] + hr * dbn * bf[k] for k in range(3)]
    df = sum(_up(F[t][:5], t) - F[t][:5] for t in (b, c))
    rho = s[0] - hr * df[0]
    m = [m[k] - hr * df[1 + ax] for k, ax in enumerate((a, b, c))]
    e = e - hr * df[4]
    Ea = E[a]

    def mean_up(ax):                      # E_a averaged along ax
        return 0.5 * (Ea + _up(Ea, ax))

    b1 = bf[1] - hr * (_up(mean_up(b), c) - mean_up(b))     # the b field feels dE_a/dc, averaged over its two faces
    b2 = bf[2] + hr * (_up(mean_up(c), b) - mean_up(c))
    v = [q / rho for q in m]
    p = (GAMMA - 1) * (e - 0.5 * rho * sum(q * q for q in v) - 0.5 * (bnh * bnh + b1 * b1 + b2 * b2))
    out = torch.stack([rho, *v, p, b1, b2])
    return torch.where((rho > 0) & (p > 0), out, s)


def _signal(W):
    return sum(W[1 + a].abs() + _fast(W[0], W[4], W[5 + a], W[5 + (a + 1) % 3], W[5 + (a + 2) % 3]) for a in range(3))


def _step64(case, U, B, dx, seed, where=None):
    """one step of the whole periodic grid in double; the CFL maximum over the cells `where` (all of them)"""
    W = _prims(U, B)
    sig = _signal(W)
    dt = COURANT * dx / float((sig if where is None else sig[where]).max())
    r = dt / dx
    solver = {"hlld": _hlld, "roe": _roe}.get(case["riemann"])
    if solver is None:
        solver = _learned(_weights(seed).double().to(U.device))
    if case["scheme"] == "vl":
        F = [_to_box(solver(_frame(_down(W, a), a), _frame(W, a), B[a]), a) for a in range(3)]
        Uh, Bh = _update(U, B, F, _emfs(F, W), 0.5 * r)
        Wh = _prims(Uh, Bh)
        F = []
        for a in range(3):
            lo, hi = _edges(_frame(Wh, a), a, case["recon"])
            F.append(_to_box(solver(_down(hi, a), lo, Bh[a]), a))
    else:
        states, F = [], []
        for a in range(3):
            q = _frame(W, a)
            lo, hi = _edges(q, a, case["recon"])
            lo, hi = _trace(q, lo, hi, B[a], _up(B[a], a), r, case["riemann"] != "roe")
            states.append((lo, hi))
            F.append(_to_box(solver(_down(hi, a), lo, B[a]), a))
        E = _emfs(F, W)
        Uh, Bh = _update(U, B, F, E, 0.5 * r)
        Wh = _prims(Uh, Bh)
        F2 = []
        for a in range(3):
            lo, hi = states[a]
            dbn = _up(B[a], a) - B[a]
            lo = _correct(lo, a, F, E, B[a], Bh[a], dbn, 0.5 * r)
            hi = _correct(hi, a, F, E, _up(B[a], a), _up(Bh[a], a), dbn, 0.5 * r)
            F2.append(_to_box(solver(_down(hi, a), lo, Bh[a]), a))
        F = F2
    U, B = _update(U, B, F, _emfs(F, Wh), r)
    return U, B, dt


def exact(case, seed):
    kind = case["kind"]
    if kind == "hierarchy":
        return None          # a whole engine: prolongation, correction and restriction around the steps above
    if kind in ("train", "infer"):
        X, T, P, m, v = (t.double().to(_device()) for t in _training(case["rows"], seed))
        if kind == "infer":
            return _network(P)(X)
        P.requires_grad_(True)
        loss = (_network(P)(X) - T).square().mean()
        g, = torch.autograd.grad(loss, P)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        new = P.detach() - 1e-3 * (m / (1 - 0.9 ** 101)) / ((v / (1 - 0.999 ** 101)).sqrt() + 1e-8)
        return {"P": new, "m": m, "v": v, "g": g, "loss": loss.detach().reshape(1)}
    U, B, e, dx = _conserved(case["nx"], case["ny"], case["nz"], case["prec"], seed)
    U, B = U.double(), B.double()
    if case["prec"] == "f32_mixed":
        U[4] = e
    if kind == "diag":
        W = _prims(U, B)
        tot = [float(q.sum()) * dx ** 3 for q in U]
        tot += [0.5 * float(W[5:].square().sum()) * dx ** 3, 0.5 * float((U[1:4].square().sum(0) / U[0]).sum()) * dx ** 3]
        div = sum((_up(B[a], a) - B[a]) / dx for a in range(3)).abs()
        # the divergence is rounding noise: it has no value of its own
        return {"sums": tot, "divb": [None, None] if float(div.max()) < 1e-8 / dx else [float(div.max()),
                float(div.mean())], "dt": COURANT * dx / float(_signal(W).max())}
    if kind == "step":
        U, B, dt = _step64(case, U, B, dx, seed)
    else:
        on = torch.zeros(U.shape[1:], dtype=torch.bool, device=U.device)
        for x, y, z in _group_origins(case, seed).tolist():
            on[z:z + 16, y:y + 16, x:x + 16] = True
        near = on.clone()
        for a in range(3):            # the step length looks at the groups and their four ghost layers
            dim = 2 - a
            near = torch.stack([torch.roll(near, k, dims=dim) for k in range(-4, 5)]).any(0)
        Un, Bn, dt = _step64(case, U, B, dx, seed, near)
        U = torch.where(on, Un, U)
        B = torch.stack([torch.where(on | _down(on, a), Bn[a], B[a]) for a in range(3)])
    t = torch.tensor([dt], dtype=torch.float64)
    return {"U": U, "B": B, "t": t} if case["prec"] == "f64" else {"U": U, "B": B}
