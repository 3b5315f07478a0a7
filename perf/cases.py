"""Performance cases of the MHD step: what a user of this package has it do.

A case names a path, a grid and the scheme options:

* ``step``    one time step as a time loop takes it (``Context.step`` with the
              CFL maxima and conservation sums read back for the next one);
* ``advance`` a short run through the time loop (``rollout.advance``);
* ``adjoint`` one step of the hand-written adjoint given the stage states
              (``Context.step_adjoint``), FP64 cotangents.

``prepare`` makes the initial state on the GPU from the seed, ``run`` is one
pass, ``work`` the bytes and operations it cannot do without, and ``exact``
the same step written with plain torch operations in FP64.
"""
import math

import torch

from paper_2510_24175_amd import workloads
from paper_2510_24175_amd.mhd import Context
from paper_2510_24175_amd.rollout import advance

DEV = "cuda"
TDTYPE = {"f32": torch.float32, "f64": torch.float64}
WENO_EPS = {"f32": 1e-30, "f64": 1e-40}


def _case(path, fields, n, dtype, riemann="hlld", limiter="minmod", bc="periodic", order=2, div="glm", steps=1):
    return {"path": path, "fields": fields, "nx": n[0], "ny": n[1], "nz": n[2], "dtype": dtype,
            "riemann": riemann, "limiter": limiter, "bc": bc, "order": order, "div": div, "steps": steps}


def listed():
    paper = dict(limiter="wenoz", order=3)
    cases = {
        # the 1D shock tube of the tests, marched ten steps: launches, read-backs and the loop itself
        "tube_400_f64": _case("advance", "tube", (400, 1, 1), "f64", riemann="hll", bc="outflow", steps=10),
        # the 2D Orszag-Tang vortex at its usual resolution
        "vortex2d_1024_f32": _case("step", "vortex", (1024, 1024, 1), "f32"),
        # a small 3D box, as in parameter studies
        "turbulence_64_f32": _case("step", "turbulence", (64, 64, 64), "f32"),
        # a box with open boundaries, odd sizes, and the other limiter and solver
        "outflow_odd_f32": _case("step", "turbulence", (203, 131, 89), "f32", riemann="hll", limiter="mc", bc="outflow"),
        # the double-precision turbulence configuration
        "turbulence_128_f64": _case("step", "turbulence", (128, 128, 128), "f64"),
        # the benchmark's headline grid
        "turbulence_512_f32": _case("step", "turbulence", (512, 512, 512), "f32"),
        # the paper's scheme with GLM at its per-GPU share of the strong-scaling grid, in the paper's precision
        "paper_416_f64": _case("step", "vortex", (416, 416, 416), "f64", **paper),
        # the same scheme in single precision on a smaller grid
        "paper_208_f32": _case("step", "vortex", (208, 208, 208), "f32", **paper),
        # the paper's weak-scaling share with constrained transport, mean edge EMF
        "ct_mean_352_f64": _case("step", "vortex", (352, 352, 352), "f64", div="ct_mean", **paper),
        # constrained transport with the upwind edge EMF, single precision, a quarter of that share per axis pair
        "ct_upwind_176_f32": _case("step", "vortex", (176, 176, 176), "f32", div="ct_upwind", **paper),
        # the adjoint configuration of the gradient runs
        "adjoint_128_f32": _case("adjoint", "turbulence", (128, 128, 128), "f32"),
        # a double-precision gradient on a ragged box
        "adjoint_odd_f64": _case("adjoint", "turbulence", (150, 110, 70), "f64"),
    }
    return [dict(c, name=k) for k, c in cases.items()]


def draw(rng):
    """One more case: a path, its options and a grid of the listed range (log-uniform cell count, any shape)."""
    kind = rng.choice(["tube", "plane", "plm", "plm", "plm", "weno", "weno", "ct", "ct", "adjoint", "adjoint"])
    dtype = rng.choice(["f32", "f64"])
    riemann = rng.choice(["hlld", "hlld", "hlld", "hll"])
    plm = rng.choice(["minmod", "minmod", "mc"])

    def grid(lo, hi, ndim):
        cells = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = cells ** (1.0 / ndim)
        n = [max(8, int(side * math.exp(rng.uniform(-0.35, 0.35)))) for _ in range(ndim)]
        if rng.random() < 0.4:  # aligned sizes are the common choice
            n = [max(16, (v + 8) // 16 * 16) for v in n]
        return tuple(n) + (1,) * (3 - ndim)

    if kind == "tube":
        return _case("advance", "tube", grid(100, 8000, 1), dtype, riemann, rng.choice([plm, "wenoz"]), "outflow",
                     rng.choice([2, 3]), steps=rng.randint(4, 12))
    if kind == "plane":
        return _case("step", "vortex", grid(1e4, 3e6, 2), dtype, riemann, rng.choice([plm, "wenoz"]), "periodic",
                     rng.choice([2, 3]))
    if kind == "plm":
        return _case("step", "turbulence", grid(3e4, 5e7, 3), dtype, riemann, plm,
                     rng.choice(["periodic", "periodic", "outflow"]))
    if kind == "weno":
        return _case("step", rng.choice(["vortex", "turbulence"]), grid(3e4, 2e7, 3), dtype, riemann, "wenoz",
                     "periodic", 3)
    if kind == "ct":
        return _case("step", "vortex", grid(3e4, 1.5e7, 3), dtype, riemann, rng.choice(["wenoz", "wenoz", "minmod"]),
                     "periodic", 3, div=rng.choice(["ct_mean", "ct_upwind"]))
    return _case("adjoint", "turbulence", grid(2e4, 6e6, 3), dtype, riemann, plm,
                 rng.choice(["periodic", "periodic", "outflow"]))


# ------------------------------------------------------------------ inputs --

def _n(case):
    return case["nx"], case["ny"], case["nz"]


def _ndim(case):
    return 3 if case["nz"] > 1 else (2 if case["ny"] > 1 else 1)


def _gamma(case):
    return 2.0 if case["fields"] == "tube" else 5.0 / 3.0


def _courant(case):
    return 0.3 if _ndim(case) == 3 else 0.4


def _ct(case):
    return case["div"] != "glm"


def _setup(case):
    s = workloads.make_setup(case["fields"], _ndim(case), _n(case), gamma=_gamma(case), cfl=_courant(case),
                             riemann=case["riemann"], limiter=case["limiter"], bc=((case["bc"],) * 2,) * 3,
                             glm=not _ct(case), time_order=case["order"])
    if _ct(case):
        s["ct"], s["ct_emf"] = True, case["div"][3:]
    return s


def _modes(n, gen, power, off, curl=False):
    """Three fields, each a Gaussian sum of the Fourier modes 1 <= |k| <= 4 with |k|^power amplitudes (or, with
    curl, the curl of such a vector potential), sampled at the cell centres displaced by off cells."""
    K = 9
    k = torch.arange(K, dtype=torch.float64) - 4
    kz, ky, kx = torch.meshgrid(k, k, k, indexing="ij")
    k2 = kx * kx + ky * ky + kz * kz
    amp = torch.where((k2 >= 1) & (k2 <= 16), k2.clamp(min=1.0) ** (0.5 * power), torch.zeros_like(k2))
    C = torch.randn(3, K, K, K, 2, generator=gen, dtype=torch.float64)
    C = torch.complex(C[..., 0], C[..., 1]) * amp
    if curl:
        kv = (kx, ky, kz)
        C = torch.stack([2j * math.pi * (kv[(a + 1) % 3] * C[(a + 2) % 3] - kv[(a + 2) % 3] * C[(a + 1) % 3])
                         for a in range(3)])
    C = C.to(DEV)
    E = [torch.exp(2j * math.pi * (k[:, None] * ((torch.arange(m, dtype=torch.float64) + 0.5 + off) / m)[None])).to(DEV)
         for m in n]
    nx, ny, nz = n
    out = torch.empty(3, nz, ny, nx, dtype=torch.float64, device=DEV)
    Ey, Az = E[1].T.contiguous(), torch.cat([E[2].real, -E[2].imag]).T.contiguous()
    for a in range(3):
        G = torch.stack([Ey @ (C[a, z] @ E[0]) for z in range(K)]).reshape(K, ny * nx)
        torch.matmul(Az, torch.cat([G.real, G.imag]), out=out[a].view(nz, ny * nx))
    return out


def _primitives(case, seed, off=0.0):
    """FP64 primitive fields (9, or 12 with the face field, components) on the device."""
    nx, ny, nz = n = _n(case)
    gen = torch.Generator().manual_seed(int(seed))
    V = torch.zeros(12 if _ct(case) else 9, nz, ny, nx, dtype=torch.float64, device=DEV)
    tp = 2 * math.pi
    if case["fields"] == "turbulence":
        # decaying turbulence once its density and pressure have left their uniform start
        v, b, s = _modes(n, gen, -1.0, off), _modes(n, gen, -2.0, off, curl=True), _modes(n, gen, -1.0, off)
        V[1:4] = v * (0.5 / v.square().sum(0).mean().sqrt())
        V[5:8] = b * (0.5 / b.square().sum(0).mean().sqrt())
        s /= s.abs().amax(dim=(1, 2, 3), keepdim=True)
        V[0], V[4], V[8] = 1.0 + 0.3 * s[0], 1.0 + 0.3 * s[1], 0.02 * s[2]
        return V
    u = (1.0 + 0.05 * (2.0 * torch.rand(8, generator=gen, dtype=torch.float64) - 1.0)).tolist()
    ph = torch.rand(3, generator=gen, dtype=torch.float64).tolist()

    def x(m, o=0.5):
        return (torch.arange(m, dtype=torch.float64, device=DEV) + o) / m

    if case["fields"] == "tube":
        # a Brio-Wu-type shock tube
        left = x(nx) < 0.45 + 0.1 * ph[0]
        for q, (a, b) in {0: (1.0, 0.125), 4: (1.0, 0.1), 6: (1.0, -1.0)}.items():
            V[q, 0, 0] = torch.where(left, a * u[q], b * u[q])
        V[5] = 0.75 * u[1]
        return V
    # Orszag-Tang vortex, in 3D with the velocity modulated along z
    X, Y, Z = x(nx).view(1, 1, nx) + ph[0], x(ny).view(1, ny, 1) + ph[1], x(nz).view(nz, 1, 1) + ph[2]
    eps, b0 = (0.2 if nz > 1 else 0.0), 1.0 / math.sqrt(4 * math.pi)
    mz = 1.0 + eps * torch.sin(tp * Z)
    V[0], V[4] = 25.0 / (36.0 * math.pi), 5.0 / (12.0 * math.pi)
    V[1] = -u[0] * mz * torch.sin(tp * Y)
    V[2] = u[1] * mz * torch.sin(tp * X)
    V[3] = eps * torch.sin(tp * Z)
    V[5] = -u[2] * b0 * torch.sin(tp * Y)
    V[6] = u[3] * b0 * torch.sin(2 * tp * X)
    if _ct(case):  # each face component is independent of its own coordinate: no discrete divergence
        V[9:12] = V[5:8]
    return V


def _cons(V, g, ct=False):
    U = V.clone()
    if ct:
        for d in range(3):
            U[5 + d] = 0.5 * (V[9 + d] + V[9 + d].roll(-1, 2 - d))
    U[1:4] = V[0] * V[1:4]
    U[4] = V[4] / (g - 1.0) + 0.5 * V[0] * V[1:4].square().sum(0) + 0.5 * U[5:8].square().sum(0)
    return U


def _prim(U, g):
    v = U[1:4] / U[0]
    p = (g - 1.0) * (U[4] - 0.5 * (U[1:4] * v).sum(0) - 0.5 * U[5:8].square().sum(0))
    return torch.cat([U[:1], v, p[None], U[5:9]])


def _slabs(nz, cells):
    kz = max(1, min(nz, int(6e6 // max(1, cells // nz))))
    return [(k, min(nz, k + kz)) for k in range(0, nz, kz)]


def _cfl(U, case):
    """(dt, c_h) of a state by the Courant condition on the fast speed."""
    n, g = _n(case), _gamma(case)
    s = c = 0.0
    for k0, k1 in _slabs(n[2], U[0].numel()):
        W = _prim(U[:, k0:k1].double(), g)
        for d in range(_ndim(case)):
            lam = (W[1 + d].abs() + _fast(W[0], W[4], W[5:8], d, g)).max().item()
            s, c = max(s, lam * n[d]), max(c, lam)
    return _courant(case) / s, c


def prepare(case, seed):
    setup = _setup(case)
    adj = case["path"] == "adjoint"
    ctx = Context(setup, case["dtype"], adjoint=adj)
    U = ctx.prim_to_cons(_primitives(case, seed))
    if case["path"] == "advance":
        return {"path": "advance", "ctx": ctx, "U": U, "steps": case["steps"]}
    dt, ch = _cfl(U, case)
    st = {"path": case["path"], "ctx": ctx, "U": U, "dt": dt, "ch": ch}
    if adj:
        # the stage-1 state of the step (the fields a fraction of a cell on) and the cotangent carried so far
        st["U1"] = ctx.prim_to_cons(_primitives(case, seed, off=0.1))
        st["lam"], st["lam_n"] = _cotangent(case, seed), ctx.empty(torch.float64)
    else:
        st["out"] = torch.empty_like(U)
    return st


def _cotangent(case, seed):
    gen = torch.Generator().manual_seed(int(seed) + 7919)
    return torch.cat([_modes(_n(case), gen, -1.0, 0.0) for _ in range(3)])


def run(state):
    ctx = state["ctx"]
    if state["path"] == "advance":
        U, _, hist = advance(ctx, state["U"], nsteps=state["steps"])
        return {"U": U, "dt": torch.tensor([h[0] for h in hist], dtype=ctx.tdtype)}
    if state["path"] == "adjoint":
        dt, ch = state["dt"], state["ch"]
        return {"lam": ctx.step_adjoint(state["U"], state["U1"], state["lam"], state["lam_n"], dt, ch,
                                        ctx.damp(dt, ch))}
    ctx.step(state["U"], state["out"], state["dt"], state["ch"])
    dt, ch, sums = ctx.step_info()
    return {"U": state["out"], "info": torch.tensor([dt, ch, *sums], dtype=ctx.tdtype)}


def work(case):
    cells = case["nx"] * case["ny"] * case["nz"]
    b = 4 if case["dtype"] == "f32" else 8
    weno, nd = case["limiter"] == "wenoz", _ndim(case)
    # per cell and axis: a limited slope and two face states of 9 components (PLM 5, WENO-Z 50 operations each),
    # one Riemann problem; per cell and stage: the primitive map and the update
    stage = nd * (9 * (50 if weno else 5) + (180 if case["riemann"] == "hlld" else 110) + 18) + 60
    if _ct(case):
        stage += 60 if case["div"] == "ct_mean" else 450
    if case["path"] == "adjoint":
        # two states and the cotangent in, the cotangent out; a reversed stage costs about three forward ones
        return {"bytes": cells * 9 * (2 * b + 16), "flops": cells * 2 * 3 * stage}
    return {"bytes": cells * 2 * b * (12 if _ct(case) else 9) * case["steps"],
            "flops": cells * case["order"] * stage * case["steps"]}


# ------------------------------------------- the same step in plain torch --

def _fast(rho, p, B, d, g):
    a2, b2, bn2 = g * p / rho, B.square().sum(0) / rho, B[d].square() / rho
    disc = ((a2 - b2).square() + 4.0 * a2 * (b2 - bn2)).clamp(min=0.0)
    return (0.5 * (a2 + b2 + disc.sqrt())).sqrt()


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() <= b.abs(), a, b), torch.zeros_like(a))


def _weno(v0, v1, v2, v3, v4, eps):
    b0 = 13 / 12 * (v0 - 2 * v1 + v2).square() + 0.25 * (v0 - 4 * v1 + 3 * v2).square() + eps
    b1 = 13 / 12 * (v1 - 2 * v2 + v3).square() + 0.25 * (v1 - v3).square() + eps
    b2 = 13 / 12 * (v2 - 2 * v3 + v4).square() + 0.25 * (3 * v2 - 4 * v3 + v4).square() + eps
    t = (b0 - b2).abs()
    a0, a1, a2 = 0.1 * (1 + t / b0), 0.6 * (1 + t / b1), 0.3 * (1 + t / b2)
    return (a0 * (2 * v0 - 7 * v1 + 11 * v2) + a1 * (5 * v2 + 2 * v3 - v1) + a2 * (2 * v2 + 5 * v3 - v4)) / (6 * (a0 + a1 + a2))


def _face_states(W, ax, case):
    """States left and right of the n + 1 faces along axis ax of W, which carries the ghost cells of that axis."""
    m = W.shape[ax]
    if case["limiter"] == "wenoz":
        v = [W.narrow(ax, k, m - 4) for k in range(5)]
        eps = WENO_EPS[case["dtype"]]
        hi, lo = _weno(*v, eps), _weno(*v[::-1], eps)
    else:
        w = W.narrow(ax, 1, m - 2)
        a, b = w - W.narrow(ax, 0, m - 2), W.narrow(ax, 2, m - 2) - w
        s = _minmod(a, b) if case["limiter"] == "minmod" else _minmod(2 * a, _minmod(2 * b, 0.5 * (a + b)))
        hi, lo = w + 0.5 * s, w - 0.5 * s
    f = hi.shape[ax] - 1
    return hi.narrow(ax, 0, f), lo.narrow(ax, 1, f)


def _flux(VL, VR, d, case, ch, bnf):
    """Riemann flux (9 components) between two primitive face states along axis d."""
    g, glm = _gamma(case), not _ct(case)
    d1, d2 = (d + 1) % 3, (d + 2) % 3
    if glm:
        bn = 0.5 * (VL[5 + d] + VR[5 + d]) - 0.5 / ch * (VR[8] - VL[8])
        psi = 0.5 * (VL[8] + VR[8]) - 0.5 * ch * (VR[5 + d] - VL[5 + d])
    else:
        bn = bnf

    def side(V):
        B = torch.stack([bn, V[5 + d1], V[5 + d2]])
        q = {"r": V[0], "u": V[1 + d], "v": (V[1 + d1], V[1 + d2]), "p": V[4], "b": (B[1], B[2])}
        bsq = B.square().sum(0)
        q["E"] = q["p"] / (g - 1) + 0.5 * q["r"] * (q["u"] ** 2 + q["v"][0] ** 2 + q["v"][1] ** 2) + 0.5 * bsq
        q["pt"] = q["p"] + 0.5 * bsq
        q["vb"] = q["u"] * bn + q["v"][0] * B[1] + q["v"][1] * B[2]
        q["c"] = _fast(q["r"], q["p"], B, 0, g)
        r, u, (v1, v2), (b1, b2) = q["r"], q["u"], q["v"], q["b"]
        q["U"] = [r, r * u, r * v1, r * v2, q["E"], b1, b2]
        q["F"] = [r * u, r * u * u + q["pt"] - bn * bn, r * u * v1 - bn * b1, r * u * v2 - bn * b2,
                  (q["E"] + q["pt"]) * u - bn * q["vb"], u * b1 - v1 * bn, u * b2 - v2 * bn]
        return q

    L, R = side(VL), side(VR)
    if case["riemann"] == "hll":
        sL = torch.minimum(L["u"] - L["c"], R["u"] - R["c"]).clamp(max=0.0)
        sR = torch.maximum(L["u"] + L["c"], R["u"] + R["c"]).clamp(min=0.0)
        f = [(sR * a - sL * b + sL * sR * (y - x)) / (sR - sL) for a, b, x, y in zip(L["F"], R["F"], L["U"], R["U"])]
    else:
        cm = torch.maximum(L["c"], R["c"])
        L["S"], R["S"] = torch.minimum(L["u"], R["u"]) - cm, torch.maximum(L["u"], R["u"]) + cm
        mL, mR = (L["S"] - L["u"]) * L["r"], (R["S"] - R["u"]) * R["r"]
        sM = (mR * R["u"] - mL * L["u"] - R["pt"] + L["pt"]) / (mR - mL)
        pts = (mR * L["pt"] - mL * R["pt"] + mL * mR * (R["u"] - L["u"])) / (mR - mL)
        sg = torch.where(bn >= 0, 1.0, -1.0)
        for q, m in ((L, mL), (R, mR)):
            q["rs"] = m / (q["S"] - sM)
            mm = m * (q["S"] - sM)
            D = mm - bn * bn
            deg = D.abs() <= 16 * 2.220446049250313e-16 * (mm.abs() + bn * bn)
            D = torch.where(deg, torch.ones_like(D), D)
            cv = torch.where(deg, torch.zeros_like(D), bn * (sM - q["u"]) / D)
            cb = torch.where(deg, torch.ones_like(D), (m * (q["S"] - q["u"]) - bn * bn) / D)
            q["vs"] = [v - b * cv for v, b in zip(q["v"], q["b"])]
            q["bs"] = [b * cb for b in q["b"]]
            q["sq"] = q["rs"].sqrt()
            q["vbs"] = sM * bn + q["vs"][0] * q["bs"][0] + q["vs"][1] * q["bs"][1]
            q["Es"] = ((q["S"] - q["u"]) * q["E"] - q["pt"] * q["u"] + pts * sM + bn * (q["vb"] - q["vbs"])) / (q["S"] - sM)
        a, b = L["sq"], R["sq"]
        vss = [(a * L["vs"][i] + b * R["vs"][i] + (R["bs"][i] - L["bs"][i]) * sg) / (a + b) for i in (0, 1)]
        bss = [(a * R["bs"][i] + b * L["bs"][i] + a * b * (R["vs"][i] - L["vs"][i]) * sg) / (a + b) for i in (0, 1)]
        vbss = sM * bn + vss[0] * bss[0] + vss[1] * bss[1]
        left = sM >= 0
        f = None
        for q, s in ((L, -1.0), (R, 1.0)):
            ss = sM + s * bn.abs() / q["sq"]
            outer, dbl = (q["S"] >= 0, ss < 0) if s < 0 else (q["S"] <= 0, ss >= 0)
            us = [q["rs"], q["rs"] * sM, q["rs"] * q["vs"][0], q["rs"] * q["vs"][1], q["Es"], *q["bs"]]
            Ess = q["Es"] + s * q["sq"] * (q["vbs"] - vbss) * sg
            uss = [q["rs"], q["rs"] * sM, q["rs"] * vss[0], q["rs"] * vss[1], Ess, *bss]
            a1 = torch.where(outer, torch.zeros_like(ss), q["S"])
            a2 = torch.where(outer | ~dbl, torch.zeros_like(ss), ss)
            h = [F + a1 * (y - x) + a2 * (z - y) for F, x, y, z in zip(q["F"], q["U"], us, uss)]
            f = h if f is None else [torch.where(left, x, y) for x, y in zip(f, h)]
    F = [None] * 9
    F[0], F[1 + d], F[1 + d1], F[1 + d2], F[4], F[5 + d1], F[5 + d2] = f
    zero = torch.zeros_like(bn)
    F[5 + d], F[8] = (psi, ch * ch * bn) if glm else (zero, zero)
    return torch.stack(F)


def _rate(U, case, ch):
    """dU/dt of the 9 cell components and, with constrained transport, the face fluxes of the transverse field."""
    n, nd, g = _n(case), _ndim(case), _gamma(case)
    H = 3 if case["limiter"] == "wenoz" else 2
    ghost = []
    for m in n:
        i = torch.arange(-H, m + H, device=DEV)
        ghost.append(i % m if case["bc"] == "periodic" else i.clamp(0, m - 1))
    rates, flx = [], [[] for _ in range(6)]
    for k0, k1 in _slabs(n[2], U[0].numel()):
        W = _prim(U[:9, k0:k1], g)
        r = torch.zeros_like(W)
        for d in range(nd):
            ax = -1 - d
            if d == 2:
                X = _prim(U[:9].index_select(1, ghost[2][k0:k1 + 2 * H]), g)
            else:
                X = W.index_select(W.dim() + ax, ghost[d])
            bnf = None
            if _ct(case):
                i = torch.arange(k0, k1 + 1, device=DEV) % n[2] if d == 2 else torch.arange(n[d] + 1, device=DEV) % n[d]
                bf = U[9 + d] if d == 2 else U[9 + d, k0:k1]
                bnf = bf.index_select(bf.dim() + ax, i)
            F = _flux(*_face_states(X, ax, case), d, case, ch, bnf)
            m = F.shape[ax] - 1
            r = r - (F.narrow(ax, 1, m) - F.narrow(ax, 0, m)) * float(n[d])
            if _ct(case):
                for e, q in enumerate([q for q in (5, 6, 7) if q != 5 + d]):
                    flx[2 * d + e].append(F[q].narrow(ax, 0, m))
        rates.append(r)
    return torch.cat(rates, 1), [torch.cat(f) if f else None for f in flx]


def _back(a, d):
    return a.roll(1, 2 - d)


def _emf(U, flx, case):
    """Edge EMFs on each cell's lower edges."""
    if case["div"] == "ct_mean":
        xy, xz, yx, yz, zx, zy = flx
        return [0.25 * (_back(zy, 1) + zy - _back(yz, 2) - yz), 0.25 * (_back(xz, 2) + xz - _back(zx, 0) - zx),
                0.25 * (_back(yx, 0) + yx - _back(xy, 1) - xy)]
    W = _prim(U[:9], _gamma(case))
    out = []
    for e in range(3):
        p, q = (e + 1) % 3, (e + 2) % 3

        def slope(f, d):
            return _minmod(f - _back(f, d), f.roll(-1, 2 - d) - f)

        def at(f, a, b):  # the field of cell (a, b) around the edge
            f = f if a else _back(f, p)
            return f if b else _back(f, q)

        vp, vq = W[1 + p], W[1 + q]
        cp, cq = (_fast(W[0], W[4], W[5:8], d, _gamma(case)) for d in (p, q))
        cells = [(a, b) for a in (0, 1) for b in (0, 1)]
        ap, am, bp, bm = (torch.stack([at(f, a, b) for a, b in cells]).amax(0).clamp(min=0.0)
                          for f in (vp + cp, cp - vp, vq + cq, cq - vq))
        fq, fp = U[9 + q], U[9 + p]
        Bq = [(at(fq, a, 1) + (0.5 - a) * at(slope(fq, p), a, 1)) for a in (0, 1)]
        Bp = [(at(fp, 1, b) + (0.5 - b) * at(slope(fp, q), 1, b)) for b in (0, 1)]
        E = ap * am / (ap + am) * (Bq[1] - Bq[0]) - bp * bm / (bp + bm) * (Bp[1] - Bp[0])
        for a, b in cells:
            x, y = (at(v, a, b) + (0.5 - a) * at(slope(v, p), a, b) + (0.5 - b) * at(slope(v, q), a, b) for v in (vp, vq))
            E = E + (am if a else ap) / (ap + am) * (bm if b else bp) / (bp + bm) * (y * Bp[b] - x * Bq[a])
        out.append(E)
    return out


def _stage(Un, U, case, dt, ch, a, b):
    """a Un + b (U + dt L(U))."""
    r, flx = _rate(U, case, ch)
    out = U.clone()
    out[:9] = U[:9] + dt * r
    if _ct(case):
        E, n = _emf(U, flx, case), _n(case)
        for d in range(3):
            d1, d2 = (d + 1) % 3, (d + 2) % 3
            out[9 + d] = U[9 + d] - dt * ((E[d2].roll(-1, 2 - d1) - E[d2]) * n[d1] - (E[d1].roll(-1, 2 - d2) - E[d1]) * n[d2])
    out = b * out + (a * Un if a else 0.0)
    if _ct(case):
        for d in range(3):
            out[5 + d] = 0.5 * (out[9 + d] + out[9 + d].roll(-1, 2 - d))
    return out


def _damp(case, dt, ch):
    n = _n(case)[:_ndim(case)]
    return math.exp(-0.1 * ch * dt * max(n)) if not _ct(case) else 1.0


def _step(U, case, dt, ch):
    weights = [(0, 1), (0.5, 0.5)] if case["order"] == 2 else [(0, 1), (0.75, 0.25), (1 / 3, 2 / 3)]
    W = U
    for a, b in weights:
        W = _stage(U, W, case, dt, ch, a, b)
    W[8] *= _damp(case, dt, ch)
    return W


def _state(case, seed, off=0.0):
    """The state that a context of the case's type holds, in FP64."""
    return _cons(_primitives(case, seed, off), _gamma(case), _ct(case)).to(TDTYPE[case["dtype"]]).double()


def exact(case, seed):
    cells = case["nx"] * case["ny"] * case["nz"]
    if case["path"] == "adjoint":
        if cells > 3_000_000:
            return None  # the tape of the reversed step would not fit
        Un, U1, lam = _state(case, seed), _state(case, seed, 0.1), _cotangent(case, seed)
        dt, ch = _cfl(Un, case)
        mu = lam.clone()
        mu[8] *= _damp(case, dt, ch)

        def vjp(U, v):
            U = U.clone().requires_grad_()
            return torch.autograd.grad(_rate(U, case, ch)[0], U, v)[0]

        lam1 = 0.5 * mu + 0.5 * dt * vjp(U1, mu)
        return {"lam": 0.5 * mu + lam1 + dt * vjp(Un, lam1)}
    with torch.no_grad():
        U = _state(case, seed)
        if case["path"] == "advance":
            dts = []
            for _ in range(case["steps"]):
                dt, ch = _cfl(U, case)
                U = _step(U, case, dt, ch)
                dts.append(dt)
            return {"U": U, "dt": torch.tensor(dts, dtype=torch.float64)}
        U = _step(U, case, *_cfl(U, case))
        dt, ch = _cfl(U, case)
        sums = [U[q].sum().item() / cells for q in range(9)]
        return {"U": U, "info": torch.tensor([dt, ch, *sums], dtype=torch.float64)}
