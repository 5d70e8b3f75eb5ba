"""The work a program has the library do, as cases that can be timed and checked.

Every case is one pass through the public entry points of
``paid_1610_09991_amd`` on the GPU.  The integrations are the library's main
path: an fRG step asks, at one or several flow scales, for every bubble of a
grid of transfer momenta, with the 9-function box basis, the five form factors
or the 25-function box basis, one error criterion and the launch profile that
the package ships.  The rest are the steps beside it: the contraction with the
couplings, the flow driver, inference with the subdivision model and one step
of its training.  Sizes are those of the workloads, the tests and the
benchmark, cut to a part of the grid where the full one adds nothing but time.
"""
from __future__ import annotations

import json
import math
import os

import numpy as np
import torch

import paid_1610_09991_amd as P
import workloads as W
from paid_1610_09991_amd import seed_model as SM

DEV = "cuda:0"
# region pool of one context: three contexts and what runs beside them share
# the card, as a solver with other arrays in memory would have it
POOL_GIB = 56.0


def listed():
    return [
        # one transfer momentum at one flow scale, both channels: the smallest
        # call a solver makes (a single point looked at, a line search over q);
        # launches and latency decide
        dict(name="one momentum", op="integrate", rows="fixed", n_rows=1, tp=-0.25, mu=-0.95,
             T=0.05, omega=0.3, grid=1, basis="box1", channels=3, rtol=1e-6),
        # the small lattice of the tests: 8 x 8 momenta, five form factors
        dict(name="8x8 five form factors", op="integrate", rows="fixed", n_rows=1, tp=0.0, mu=0.0,
             T=0.1, omega=0.1, grid=8, basis="five", channels=3, rtol=1e-6),
        # one flow scale of the benchmark's workload: the call a flow makes at
        # every step (24 x 24 momenta, 9 form factors, low temperature)
        dict(name="one flow scale 24x24", op="integrate", rows="fixed", n_rows=1, tp=-0.25,
             mu=-0.95, T=0.01, omega=0.128, grid=24, basis="box1", channels=3, rtol=1e-6),
        # the benchmark's workload: 20 flow scales in one call, 23,040 containers
        dict(name="20 flow scales 24x24", op="integrate", rows="scales", n_rows=20, tp=-0.25,
             mu=-0.95, T=0.01, omega=10.0, grid=24, basis="box1", channels=3, rtol=1e-6),
        # a parameter scan: random rows, started from the shipped subdivision model
        dict(name="16 rows 12x12 seeded", op="integrate", rows="random", n_rows=16, grid=12,
             basis="box1", channels=3, rtol=1e-6, seeded=True),
        # every integral held to its own tolerance, the comparison mode
        dict(name="8x8 per integral", op="integrate", rows="fixed", n_rows=1, tp=-0.25, mu=-0.95,
             T=0.02, omega=0.1, grid=8, basis="box1", channels=3, rtol=1e-6, err_mode=1),
        # the 25-function box basis (325 integrals per momentum) at the lowest temperature
        dict(name="8x8 25 form factors", op="integrate", rows="fixed", n_rows=1, tp=-0.3, mu=-1.1,
             T=0.005, omega=0.1, grid=8, basis="box2", channels=3, rtol=1e-6),
        # the right-hand sides of the flow for all scales and momenta of the benchmark
        dict(name="contract 11520 of 9", op="contract", n=11520, M=9),
        # and for the 25-function basis on a 32 x 32 grid
        dict(name="contract 1024 of 25", op="contract", n=1024, M=25),
        # the flow driver on a small lattice, one decade of the scale
        dict(name="flow 4x4", op="flow", grid=4, tp=0.0, mu=0.0, T=0.1, omega0=1.0, omega1=0.3,
             rtol=1e-5),
        # predicted subdivision of every container of the benchmark's workload
        dict(name="model forward 23040", op="forward", n=23040),
        # one training step of the subdivision model: loss, gradient, Adam
        dict(name="model training step 256", op="train", n=256),
    ]


def draw(rng):
    """A case of the same ranges: integrations mostly, then the steps beside them."""
    def logu(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    op = rng.choice(["integrate"] * 7 + ["contract", "contract", "forward", "train", "train"])
    if op == "contract":
        M = rng.choice([1, 5, 9, 9, 16, 17, 25, 32])
        return dict(op=op, n=int(logu(1, 12000 if M <= 16 else 4000)), M=M)
    if op == "forward":
        return dict(op=op, n=int(logu(1, 40000)))
    if op == "train":
        return dict(op=op, n=int(logu(1, 2048)))
    basis = rng.choice(["box1", "box1", "box1", "box1", "five", "box2", "box0", "mixed"])
    err = rng.choice([0, 0, 0, 0, 1]) if basis != "box2" else 0
    seeded = basis == "box1" and err == 0 and rng.random() < 0.2
    n_rows = int(logu(1, 8))
    # momenta: any number from one to a 24 x 24 grid's, less where each costs more
    n_q = int(logu(1, (576 if err == 0 and basis != "box2" else 64) / n_rows + 1))
    return dict(op="integrate", rows="random", n_rows=n_rows, n_q=n_q, basis=basis,
                channels=rng.choice([1, 2, 3, 3, 3]), rtol=rng.choice([1e-6, 1e-6, 1e-7]),
                err_mode=err, seeded=bool(seeded),
                T_min=0.02 if err or basis == "box2" else 0.01)


# ------------------------------------------------------------------ inputs
def _basis(name):
    if name == "five":
        return W.ff5(), 1
    if name == "mixed":  # a general orthonormal set: no definite parity, no symmetry
        r = np.random.default_rng(11)
        return np.linalg.qr(r.normal(size=(9, 9)))[0][:6].copy(), 1
    L = int(name[-1])
    return W.ff_box(L), L


def _integrals(case, seed):
    """Parameter rows, momenta and form factors of an integration.  The seed
    moves the chemical potential (and the random rows), as a scan over fillings
    does."""
    rng = np.random.default_rng(seed)
    if case["rows"] == "random":
        n = case["n_rows"]
        T = np.exp(rng.uniform(math.log(case.get("T_min", 0.01)), math.log(0.1), n))
        om = np.exp(rng.uniform(math.log(0.05), math.log(10.0), n))
        p = np.stack([np.ones(n), rng.uniform(-0.35, 0.0, n), rng.uniform(-1.2, 0.0, n), T, om],
                     axis=1)
    else:
        n = case["n_rows"]
        om = (case["omega"] * 10.0 ** (-3.0 * np.arange(n) / (n - 1)) if case["rows"] == "scales"
              else np.array([case["omega"]]))
        mu = case["mu"] + 0.02 * rng.uniform(-1.0, 1.0)
        p = np.array([[1.0, case["tp"], mu, case["T"], o] for o in om])
    if "n_q" in case:
        q = rng.uniform(-math.pi, math.pi, (case["n_q"], 2))
    elif case["grid"] == 1:
        q = rng.uniform(-math.pi, math.pi, (1, 2))
    else:
        q = W.q_grid(case["grid"])
    ff, L = _basis(case["basis"])
    return p, q, ff, L


def _f32(rng, shape, scale=1.0):
    return (scale * rng.normal(size=shape)).astype(np.float32)


def _mlp_slices():
    dims, out, off = [7, 128, 128, 128, 256], [], 0
    for l in range(4):
        ni, no = dims[l], dims[l + 1]
        out.append((off, off + no * ni, no, ni))
        off += no * ni + no
    return out


def _model_inputs(case, seed, labels):
    """Features of containers drawn from the batched workload's distribution,
    and labels of the size that converged trees give."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    ax, ay = rng.uniform(0, 1, n), rng.uniform(0, 1, n)
    x = np.stack([np.maximum(ax, ay), np.minimum(ax, ay), rng.uniform(-1.2, 0.0, n),
                  rng.uniform(math.log10(0.005), -1.0, n), rng.uniform(-0.35, 0.0, n),
                  rng.uniform(-2.0, 1.0, n), rng.choice([-1.0, 1.0], n)], axis=1)
    y = np.abs(rng.normal(3.0, 2.0, (n, 256))) if labels else None
    return x.astype(np.float32), None if y is None else y.astype(np.float32)


def _flow_inputs(case, seed):
    rng = np.random.default_rng(seed)
    q = W.q_grid(case["grid"])
    V = [rng.normal(size=(len(q), 5, 5)) for _ in range(3)]
    S = [rng.normal(size=(len(q), 5, 5)) for _ in range(3)]
    mu = case["mu"] + 0.05 * rng.uniform(-1.0, 1.0)
    return (1.0, case["tp"], mu, case["T"]), q, V, S


def _couplings(case, seed):
    rng = np.random.default_rng(seed)
    n, M = case["n"], case["M"]
    chi = rng.normal(size=(n, 2, M, M))
    return [0.5 * (chi + chi.swapaxes(-1, -2))] + [rng.normal(size=(n, M, M)) for _ in range(3)]


def _profile():
    with open(os.path.join(os.path.dirname(P.__file__), "tuned_c2.json")) as f:
        return json.load(f)["config"]


def prepare(case, seed):
    op = case["op"]
    if op == "integrate":
        p, q, ff, L = _integrals(case, seed)
        nch = 2 if case["channels"] == 3 else 1
        n_ctr = len(p) * len(q) * nch
        # the shipped launch profile and graph replay where containers are
        # many, the defaults where they are few
        kw = dict(_profile(), graph=1) if n_ctr > 512 else {}
        ctx = P.Context(max_regions=(1 << 17) if case.get("err_mode", 0) == 0 else (1 << 18),
                        pool_gib=POOL_GIB, err_mode=case.get("err_mode", 0), **kw)
        if case.get("seeded"):
            w, meta = SM.load()
            ctx.set_seed_model(w, kappa=meta["kappa"])
        out = torch.empty((len(p), len(q), nch, len(ff), len(ff)), dtype=torch.float64, device=DEV)
        return dict(op=op, ctx=ctx, p=p, q=q, ff=ff, L=L, channels=case["channels"],
                    rtol=case["rtol"], out=out)
    if op == "flow":
        base, q, V, S = _flow_inputs(case, seed)
        return dict(op=op, ctx=P.Context(max_regions=1 << 16, pool_gib=POOL_GIB), base=base, q=q, V=V, S=S,
                    om=(case["omega0"], case["omega1"]), rtol=case["rtol"])
    ctx = P.Context()
    if op == "contract":
        a = [torch.tensor(x, device=DEV) for x in _couplings(case, seed)]
        return dict(op=op, ctx=ctx, a=a)
    w = torch.tensor(SM.load()[0], device=DEV)
    x, y = _model_inputs(case, seed, op == "train")
    if op == "forward":
        return dict(op=op, ctx=ctx, w=w, x=torch.tensor(x, device=DEV),
                    y=torch.empty((case["n"], 256), dtype=torch.float32, device=DEV))
    return dict(op=op, ctx=ctx, w=w, x=torch.tensor(x, device=DEV), y=torch.tensor(y, device=DEV),
                g=torch.empty_like(w), m=torch.zeros_like(w), v=torch.zeros_like(w), t=0)


def run(s):
    c, op = s["ctx"], s["op"]
    if op == "integrate":
        out, _, _, _ = c.integrate(s["p"], s["q"], s["ff"], s["L"], s["channels"], rtol=s["rtol"],
                                   out=s["out"])
        return out
    if op == "flow":
        return c.flow(s["base"], s["q"], W.ff5(), 1, *s["V"], *s["S"], omega0=s["om"][0],
                      omega1=s["om"][1], rtol=s["rtol"], rtol_int=0.01 * s["rtol"])[:3]
    if op == "contract":
        return c.contract(*s["a"])
    if op == "forward":
        return c.mlp_forward(s["w"], s["x"], s["y"])
    s["t"] += 1
    loss = c.mlp_loss_grad_noalloc(s["w"], s["x"], s["y"], s["g"])
    c.mlp_adam(s["w"], s["g"], s["m"], s["v"], s["t"], 1e-4)
    return dict(loss=loss, g=s["g"], w=s["w"], m=s["m"], v=s["v"])


# ------------------------------------------------------------------ work
def _leaves(T, om, rtol):
    """Leaves of a converged tree, a law through the workloads' counts at rtol
    1e-6 (240 at Omega 10, 1,300 at 1, 15,000 at 0.1, temperature capping the
    growth at 3 T), growing as rtol^-0.27."""
    return (120.0 + 1350.0 / math.hypot(om, 3.0 * T) ** 1.04) * (1e-6 / rtol) ** 0.27


def work(case):
    op = case["op"]
    if op == "contract":
        n, M = case["n"], case["M"]
        return {"bytes": 8.0 * n * 8 * M * M, "flops": 7.0 * 2 * n * M ** 3}
    per = 2.0 * (7 * 128 + 2 * 128 * 128 + 128 * 256)
    if op == "forward":
        return {"bytes": 4.0 * (case["n"] * 263 + 67072), "flops": per * case["n"]}
    if op == "train":
        return {"bytes": 4.0 * (case["n"] * 263 + 9 * 67072), "flops": 3 * per * case["n"]}
    if op == "flow":
        n_ctr, leaves, M, L, evals = 2 * case["grid"] ** 2, _leaves(case["T"], 0.5, 1e-7), 5, 1, 13
    else:
        ff, L = _basis(case["basis"])
        M = len(ff)
        n_q = case["n_q"] if "n_q" in case else case["grid"] ** 2
        n_ctr, evals = n_q * (2 if case["channels"] == 3 else 1), 1
        if case["rows"] == "scales":
            om = [case["omega"] * 10.0 ** (-3.0 * k / (case["n_rows"] - 1))
                  for k in range(case["n_rows"])]
            leaves = sum(_leaves(case["T"], o, case["rtol"]) for o in om)
        elif case["rows"] == "random":
            leaves = case["n_rows"] * _leaves(0.03, 0.7, case["rtol"])
        else:
            leaves = _leaves(case["T"], case["omega"], case["rtol"])
        leaves *= 6.0 if case.get("err_mode", 0) == 1 else 1.0
        n_ctr_out = n_ctr * case["n_rows"]
        out_bytes = 8.0 * n_ctr_out * M * M
    # a split: 289 nodes of the integrand (72 flops) and the separable sums
    npr = (2 * L + 1) * (L + 1)
    split = 289 * 72 + 2 * 17 * npr * 27 + 2 * 9 * npr * 10 + 4 * npr * npr * 42 + 6 * M * (M + 1)
    if op == "flow":
        out_bytes = 8.0 * n_ctr / 2 * 9 * M * M
    return {"bytes": out_bytes, "flops": evals * n_ctr * leaves / 3.0 * split}


# ------------------------------------------------------------------ 64-bit values
def _bubbles(row, q, ff, L, channels, kind="dot"):
    """chi^pp and chi^ph [n_q][n_ch][M][M] of one parameter row by the
    periodic trapezoid rule in p (exponentially accurate: the integrand is
    analytic in a strip of width ~ pi T / |grad eps|) and the Matsubara sum of
    the regulated product, its tail expanded in 1/w^2 and summed with Hurwitz
    zeta values."""
    t, tp, mu, T, om = (float(v) for v in row)
    D = dict(dtype=torch.float64, device=DEV)
    G = 2 * int(math.ceil(20.0 * (2 * t + 4 * abs(tp) + 0.5) / (math.pi * T) / 2))
    G = max(G, 128)
    x = -math.pi + 2 * math.pi * torch.arange(G, **D) / G
    u = [torch.ones_like(x)]
    for k in range(1, L + 1):
        u += [math.sqrt(2.0) * torch.cos(k * x), math.sqrt(2.0) * torch.sin(k * x)]
    u = torch.stack(u)                                   # [nb][G]
    nb = 2 * L + 1
    ffc = torch.tensor(np.asarray(ff), **D)
    top = max(4 * abs(t) + 4 * abs(tp) + abs(mu), om)
    nm = max(8, int(math.ceil(2.5 * top / (math.pi * T))))
    K = 28
    z = [0.0] + [float(torch.special.zeta(torch.tensor(2.0 * k, dtype=torch.float64),
                                          torch.tensor(nm + 0.5, dtype=torch.float64)))
                 * (2 * math.pi * T) ** (-2 * k) for k in range(1, K + 1)]
    # weight W(w) as a series in v = 1/w^2
    wser = [0.0] * (K + 1)
    if kind == "dot":
        wser[1], nom = -4.0 * om, 3
    else:
        wser[0], nom = 1.0, 2
    for _ in range(nom):
        for k in range(1, K + 1):
            wser[k] -= om * om * wser[k - 1]
    res = []
    for l in np.asarray(q):
        def eps(sx, sy):
            cx, cy = torch.cos(sx)[:, None], torch.cos(sy)[None, :]
            return -2 * t * (cx + cy) - 4 * tp * cx * cy - mu
        a, b = eps(l[0] / 2 + x, l[1] / 2 + x), eps(l[0] / 2 - x, l[1] / 2 - x)
        a2, b2, ab = a * a, b * b, a * b
        s1 = torch.zeros_like(a)  # sum W w^2 / ((w^2+a^2)(w^2+b^2))
        s0 = torch.zeros_like(a)  # sum W / ((w^2+a^2)(w^2+b^2))
        for n in range(nm - 1, -1, -1):
            w2 = ((2 * n + 1) * math.pi * T) ** 2
            wt = -4 * om * w2 * w2 / (w2 + om * om) ** 3 if kind == "dot" else \
                w2 * w2 / (w2 + om * om) ** 2
            r = wt / ((w2 + a2) * (w2 + b2))
            s1 += w2 * r
            s0 += r
        # tail: 1/((1+a^2 v)(1+b^2 v)) = sum (-v)^k h_k, h_k = a^2 h_{k-1} + b^(2k)
        h, bp = torch.ones_like(a), torch.ones_like(a)
        for k in range(0, K - 1):
            c1 = sum(wser[j] * z[j + k + 1] for j in range(K + 1) if j + k + 1 <= K)
            c0 = sum(wser[j] * z[j + k + 2] for j in range(K + 1) if j + k + 2 <= K)
            sg = -1.0 if k & 1 else 1.0
            s1 += sg * c1 * h
            s0 += sg * c0 * h
            bp = bp * b2
            h = a2 * h + bp
        row_out = []
        for ch, sgn in ((1, 1.0), (2, -1.0)):
            if not channels & ch:
                continue
            g = 2.0 * T * (ab * s0 + sgn * s1)
            # sum_p g u_a u_c (x) u_b u_d (y)
            pr = (u[:, None, :] * u[None, :, :]).reshape(nb * nb, G)
            Gm = (pr @ g @ pr.T / (G * G)).reshape(nb, nb, nb, nb)  # [a][c][b][d]
            box = Gm.permute(0, 2, 1, 3).reshape(nb * nb, nb * nb)
            row_out.append(ffc @ box @ ffc.T)
        res.append(torch.stack(row_out))
    return torch.stack(res)


def _gelu(z):
    return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _mlp(w, x):
    for l, (a, b, no, ni) in enumerate(_mlp_slices()):
        x = x @ w[a:b].reshape(no, ni).T + w[b:b + no]
        x = _gelu(x) if l < 3 else x
    return x


def _contraction(chi, VP, VC, VD):
    pp, ph = chi[:, 0].contiguous(), chi[:, 1].contiguous()
    mm = torch.matmul
    return (mm(mm(VP, pp), VP), -mm(mm(VC, ph), VC),
            2 * mm(mm(VD, ph), VD) - mm(mm(VC, ph), VD) - mm(mm(VD, ph), VC))


def exact(case, seed):
    op = case["op"]
    D = dict(dtype=torch.float64, device=DEV)
    if op == "contract":
        return _contraction(*[torch.tensor(x, **D) for x in _couplings(case, seed)])
    if op == "forward":
        return _mlp(torch.tensor(SM.load()[0], **D),
                    torch.tensor(_model_inputs(case, seed, False)[0], **D))
    if op == "train":
        w = torch.tensor(SM.load()[0], **D).requires_grad_(True)
        x, y = (torch.tensor(v, **D) for v in _model_inputs(case, seed, True))
        loss = ((_mlp(w, x) - y) ** 2).mean()
        loss.backward()
        g = w.grad
        m, v = 0.1 * g, 0.001 * g * g
        wn = w.detach() - 1e-4 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
        return dict(loss=float(loss), g=g, w=wn, m=m, v=v)
    if op == "flow":
        base, q, V, S = _flow_inputs(case, seed)
        ff, L = _basis("five")
        chi = [_bubbles((*base, o), q, ff, L, 3, kind="plain")
               for o in (case["omega0"], case["omega1"])]
        d = _contraction(chi[1] - chi[0], *[torch.tensor(v, **D) for v in V])
        return tuple(torch.tensor(s, **D) + x for s, x in zip(S, d))
    p, q, ff, L = _integrals(case, seed)
    # seconds of the trapezoid rule: grid points times frequencies
    cost = sum((20.0 * 3.9 / (math.pi * r[3])) ** 2 * (2.5 * max(6.7, r[4]) / (math.pi * r[3]) + 100)
               for r in p) * len(q) * 1.2e-10
    if cost > 12.0:
        return None
    return torch.stack([_bubbles(r, q, ff, L, case["channels"]) for r in p])
