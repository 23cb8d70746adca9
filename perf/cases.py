"""Workloads for timing the library: what a program that uses it has it do, from
the smallest call to the paper-scale one.

Families (the "call" of a case):

  sox       Plan.sigma (+ Plan.energy where the whole grid is evaluated): the
            exchange self-energy of one Green's function, in each precision, for
            symmetric (physical) and general G, with or without Sigma in the THC
            basis, on the whole tau grid or on one GPU's slice of it
  direct    Plan.sigma_direct added onto an exchange term, and the energy of the sum
  screened  Plan.static_screening, then Plan.sigma_screened with its core
  loop      the loop's control path for a few iterations: Dyson step, then DIIS
            on Sigma (Pulay's residual or the commutator)
  train     minibatch Adam steps of the warm-start network, then the gradient on
            a held-out batch
  infer     a learned start: pair profiles of a THC self-energy, the bf16 forward
            and the back-projection of what it predicts

The inputs follow the generators of ``paper_2404_17744_amd.synth`` (independent
particles in random orthogonal orbitals, X ~ N(0, 1/n), V = L L^T / naux), drawn
on the device.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2404_17744_amd import synth, thcsox, warmstart

DEV = "cuda:0"
BETA = 100.0


def listed():
    return [
        # one evaluation at the smallest size in use (interactive checks, unit
        # tests): launches and latency are all of it
        {"name": "sox_n8_fp64", "call": "sox", "n": 8, "naux": 32, "ntau": 12, "k1": 12,
         "precision": "fp64", "sym": True, "thc": False},
        # one loop evaluation of a warm-start system (n = 40 .. 160, naux = 5 n, 64
        # tau points), odd in every dimension, with Sigma in the THC basis
        {"name": "sox_n97_fp16x2_thc", "call": "sox", "n": 97, "naux": 485, "ntau": 64, "k1": 64,
         "precision": "fp16x2", "sym": True, "thc": True},
        # the throughput workload
        {"name": "sox_n300_fp16x2", "call": "sox", "n": 300, "naux": 1800, "ntau": 100, "k1": 100,
         "precision": "fp16x2", "sym": True, "thc": False},
        # two tau points of the paper-scale system (one GPU's share, cut to two)
        {"name": "sox_n1100_fp16x2_slice", "call": "sox", "n": 1100, "naux": 5500, "ntau": 100,
         "k1": 2, "precision": "fp16x2", "sym": True, "thc": False},
        # the reference precision on a mid-size system, a slice of the grid
        {"name": "sox_n200_fp64_slice", "call": "sox", "n": 200, "naux": 1100, "ntau": 100, "k1": 20,
         "precision": "fp64", "sym": True, "thc": False},
        # FP32 on sizes that divide nothing, G without symmetry (every tile of D)
        {"name": "sox_n149_fp32_general", "call": "sox", "n": 149, "naux": 797, "ntau": 33, "k1": 33,
         "precision": "fp32", "sym": False, "thc": False},
        # screened exchange on three bf16 planes: polarisation, solve, second U, both
        # placements of the screened line
        {"name": "screened_n120_bf16x3", "call": "screened", "n": 120, "naux": 600, "ntau": 64,
         "k1": 16, "precision": "bf16x3", "kind": "sosex"},
        # the direct term of full second order at the throughput size
        {"name": "direct_n300", "call": "direct", "n": 300, "naux": 1800, "ntau": 100, "k1": 100,
         "precision": "fp16x2"},
        # three loop iterations' Dyson steps and commutator DIIS at the throughput size
        {"name": "loop_n300_commutator", "call": "loop", "n": 300, "ntau": 100, "nfreq": 256,
         "depth": 3, "kind": "commutator"},
        # the same for a warm-start system, Pulay's residual
        {"name": "loop_n77_pulay", "call": "loop", "n": 77, "ntau": 64, "nfreq": 256, "depth": 3,
         "kind": "pulay"},
        # training of the warm-start network at its default sizes
        {"name": "train_h512_b4096", "call": "train", "m": 64, "hidden": 512, "batch": 4096,
         "steps": 4},
        # a learned start for a system of n = 101
        {"name": "infer_n101_h512", "call": "infer", "n": 101, "naux": 505, "m": 64, "hidden": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.5:
        prec = rng.choice(["fp16x2", "fp16x2", "fp64", "bf16x3", "fp32"])
        n = _log(rng, 8, 420)
        naux = max(4, int(n * rng.uniform(3.0, 8.0)))
        ntau = rng.randint(8, 100)
        # at most about a tenth of a second: the slice of the grid that fits
        rate = {"fp16x2": 2.5e14, "bf16x3": 1.2e14, "fp32": 8e13, "fp64": 2.5e13}[prec]
        k1 = max(1, min(ntau, int(0.1 * rate / (4.0 * (naux * n) ** 2))))
        return {"call": "sox", "n": n, "naux": naux, "ntau": ntau, "k1": k1, "precision": prec,
                "sym": rng.random() < 0.7, "thc": rng.random() < 0.3}
    if u < 0.6:
        n = _log(rng, 12, 320)
        ntau = rng.randint(8, 100)
        return {"call": "direct", "n": n, "naux": int(n * rng.uniform(3.0, 6.5)), "ntau": ntau,
                "k1": rng.randint(1, ntau), "precision": rng.choice(["fp16x2", "fp64"])}
    if u < 0.7:
        n = _log(rng, 16, 160)
        ntau = rng.randint(8, 64)
        return {"call": "screened", "n": n, "naux": int(n * rng.uniform(3.0, 6.0)), "ntau": ntau,
                "k1": rng.randint(1, min(ntau, 16)),
                "precision": rng.choice(["fp16x2", "bf16x3", "fp32", "fp64"]),
                "kind": rng.choice(["sosex", "g3w2"])}
    if u < 0.8:
        return {"call": "loop", "n": _log(rng, 8, 320), "ntau": rng.randint(24, 100),
                "nfreq": rng.choice([128, 149, 256]), "depth": rng.randint(2, 4),
                "kind": rng.choice(["pulay", "commutator"])}
    if u < 0.9:
        return {"call": "train", "m": rng.choice([12, 32, 64, 95, 100]),
                "hidden": rng.choice([64, 128, 200, 256, 512]), "batch": _log(rng, 64, 8192),
                "steps": rng.randint(1, 6)}
    n = rng.randint(40, 160)
    return {"call": "infer", "n": n, "naux": 5 * n, "m": rng.choice([32, 64]),
            "hidden": rng.choice([128, 256, 512])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, *shape, scale=1.0, dtype=torch.float64):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype) * scale


def _orbitals(n, seed):
    """Random orthogonal orbitals, their energies and the chemical potential."""
    rng = np.random.default_rng(seed)
    q, r = np.linalg.qr(rng.standard_normal((n, n)))
    q = q * np.sign(np.diag(r))
    eps = np.concatenate([rng.uniform(-1.5, -0.3, n // 2), rng.uniform(0.1, 2.0, n - n // 2)])
    mu = 0.5 * (eps[:n // 2].max() + eps[n // 2:].min())
    return torch.from_numpy(q).to(DEV), torch.from_numpy(eps).to(DEV), float(mu)


def _g0(Q, eps, mu, tau):
    """G(tau) of independent particles, [ntau, n, n]."""
    xi = eps - mu
    t = torch.from_numpy(np.asarray(tau)).to(DEV)[:, None]
    ex = torch.where(xi >= 0, -xi * t, xi * (BETA - t))
    g = -torch.exp(ex) / (1.0 + torch.exp(-BETA * xi.abs()))
    out = torch.empty((len(tau), len(eps), len(eps)), dtype=torch.float64, device=DEV)
    for k in range(len(tau)):
        out[k] = (Q * g[k]) @ Q.T
    return out


def _system(c, seed):
    """X, V, tau, weights and G of a SOX-type case."""
    n, naux = c["n"], c["naux"]
    g = _gen(seed)
    X = _randn(g, n, naux, scale=1.0 / math.sqrt(n))
    L = _randn(g, naux, naux)
    V = L @ L.T / naux
    V = 0.5 * (V + V.T)
    tau, w = synth.cheb_tau_grid(c["ntau"], BETA)
    if c.get("sym", True):
        G = _g0(*_orbitals(n, seed), tau)
    else:
        G = _randn(g, c["ntau"], n, n, scale=0.3)
    return X.contiguous(), V.contiguous(), tau, w, G


def _pole_sigmas(c, seed):
    """depth pairs (Sigma_in, Sigma_out): sums of symmetric poles, the second
    near the first as in a converging loop."""
    n, m = c["n"], c["ntau"]
    g = _gen(seed + 1)
    tau, _ = synth.cheb_tau_grid(m, BETA)
    t = torch.from_numpy(tau).to(DEV)
    pairs = []
    for _ in range(c["depth"]):
        two = []
        for scale in (0.05, 0.01):
            S = torch.zeros((m, n, n), dtype=torch.float64, device=DEV)
            for w in (0.4, 1.1, -0.6, -1.7):
                A = _randn(g, n, n, scale=scale / math.sqrt(n))
                k = torch.exp(-t * w) / (1 + math.exp(-BETA * w)) if w >= 0 else \
                    torch.exp(w * (BETA - t)) / (1 + math.exp(BETA * w))
                S -= k[:, None, None] * (0.5 * (A + A.T))
            two.append(S)
        pairs.append((two[0], two[0] + two[1]))
    return tau, pairs


def _net_params(c, seed):
    rng = np.random.default_rng(seed)
    p = warmstart.init_params(c["m"], c["hidden"], seed)
    p["W3"] = p["W3"] * 10.0             # past the first epochs: no longer the identity
    for b in ("b1", "b2", "b3"):
        p[b] = 0.05 * rng.standard_normal(p[b].shape)
    return {k: np.asarray(v, dtype=np.float32) for k, v in p.items()}


def _profiles(c, rows, g):
    """Pair profiles over tau (largest magnitude 1) and nearby targets."""
    m = c["m"]
    t = torch.linspace(0.0, 1.0, m, device=DEV)
    a = torch.rand(rows, 2, generator=g, device=DEV) * 40 + 1
    s = torch.randn(rows, 2, generator=g, device=DEV)
    x = s[:, :1] * torch.exp(-a[:, :1] * t) + s[:, 1:] * torch.exp(-a[:, 1:] * (1 - t))
    x = x / x.abs().amax(dim=1, keepdim=True)
    y = x * (1 + 0.1 * torch.randn(rows, 1, generator=g, device=DEV)) + 0.02 * x.flip(1)
    return x.contiguous(), y.contiguous()


def prepare(case, seed):
    c, s = case, {"case": case}
    if c["call"] in ("sox", "direct", "screened"):
        X, V, tau, w, G = _system(c, seed)
        s["plan"] = thcsox.Plan(X, V, tau, w, BETA, precision=c["precision"])
        s["G"], s["S"] = G, torch.zeros_like(G)
        if c.get("thc"):
            s["Sthc"] = torch.zeros((c["ntau"], c["naux"], c["naux"]), dtype=torch.float64, device=DEV)
        if c["call"] == "direct":
            s["S_sox"] = _randn(_gen(seed + 2), *G.shape, scale=0.01)
    elif c["call"] == "loop":
        Q, eps, mu = _orbitals(c["n"], seed)
        tau, s["pairs"] = _pole_sigmas(c, seed)
        s["dyson"] = thcsox.Dyson((Q * eps) @ Q.T, mu, tau, BETA, c["nfreq"])
        like = s["pairs"][0][0]
        s["next"], s["G"] = torch.empty_like(like), torch.empty_like(like)
        if c["kind"] == "commutator":
            s["e"] = torch.empty((2, c["nfreq"], c["n"], c["n"]), dtype=torch.float64, device=DEV)
            s["diis"] = thcsox.Diis(like, depth=c["depth"], residual_like=s["e"])
        else:
            s["diis"] = thcsox.Diis(like, depth=c["depth"])
    elif c["call"] == "train":
        s["net"] = thcsox.MLP(c["m"], c["hidden"], _net_params(c, seed), max_batch=c["batch"])
        g = _gen(seed)
        s["batches"] = [_profiles(c, c["batch"], g) for _ in range(c["steps"] + 1)]
    else:
        X, V, tau, w, _ = _system({**c, "ntau": c["m"]}, seed)
        s["plan"] = thcsox.Plan(X, V, tau, w, BETA, precision="fp16x2")
        s["net"] = thcsox.MLP(c["m"], c["hidden"], _net_params(c, seed))
        s["Sthc"] = _thc_sigma(c, seed)
        s["pred"] = torch.empty_like(s["Sthc"])
        s["S"] = torch.empty((c["m"], c["n"], c["n"]), dtype=torch.float64, device=DEV)
    return s


def _thc_sigma(c, seed):
    """A THC-basis self-energy: decaying from both ends of the grid, magnitudes
    spread over pairs."""
    g = _gen(seed + 3)
    A = c["naux"]
    t = torch.linspace(0.0, 1.0, c["m"], device=DEV, dtype=torch.float64)[:, None, None]
    out = torch.zeros((c["m"], A, A), dtype=torch.float64, device=DEV)
    for rate in (3.0, 11.0):
        M = _randn(g, A, A) * torch.exp(_randn(g, A, A))
        M = 0.5 * (M + M.T)
        out += M * torch.exp(-rate * t) + 0.7 * M.T.flip(0) * torch.exp(-rate * (1 - t))
    return out


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    c = state["case"]
    if c["call"] == "sox":
        plan, G, S = state["plan"], state["G"], state["S"]
        out = {"sigma": S}
        if c["thc"]:
            plan.sigma(G, 0, c["k1"], thc=True, out=S, out_thc=state["Sthc"])
            out["sigma_thc"] = state["Sthc"]
        else:
            plan.sigma(G, 0, c["k1"], out=S)
        if c["k1"] == c["ntau"]:
            out["energy"] = plan.energy(G, S)
        return out
    if c["call"] == "direct":
        plan, G, S = state["plan"], state["G"], state["S"]
        S.copy_(state["S_sox"])
        plan.sigma_direct(G, 0, c["k1"], out=S, accumulate=True)
        return {"sigma": S, "energy": plan.energy(G, S)}
    if c["call"] == "screened":
        plan, G, S = state["plan"], state["G"], state["S"]
        W = plan.static_screening(G)
        plan.sigma_screened(G, W, c["kind"], 0, c["k1"], out=S)
        return {"W": W, "sigma": S}
    if c["call"] == "loop":
        dyson, diis = state["dyson"], state["diis"]
        energies = []
        for S_in, S_out in state["pairs"]:
            G, gamma = dyson.step(S_in, G_out=state["G"])
            energies.append(dyson.onebody(gamma))
            if c["kind"] == "commutator":
                e = dyson.commutator(S_in, S_out, out=state["e"])
                diis.step_res(e, S_out, state["next"])
            else:
                diis.step(S_in, S_out, state["next"])
        out = {"G": G, "gamma": gamma, "E1": energies, "sigma_next": state["next"]}
        if c["kind"] == "commutator":
            out["e"] = state["e"]
        return out
    if c["call"] == "train":
        net = state["net"]
        losses = [net.train_step(x, t, 3e-4) for x, t in state["batches"][:-1]]
        loss, grads = net.gradients(*state["batches"][-1])
        return {"losses": losses, "loss": loss, "grads": grads}
    Sthc, pred = state["Sthc"], state["pred"]
    scale = warmstart.pair_scale(Sthc)
    x = warmstart.pair_profiles(Sthc, scale)
    y = state["net"].forward_bf16(x)
    thcsox.thcsox_pair_scatter(c["m"], c["naux"], y.data_ptr(), scale.data_ptr(), pred.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    state["plan"].backproject(pred, out=state["S"])
    return {"y": y, "sigma_thc": pred, "sigma": state["S"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c = case
    if c["call"] in ("sox", "direct", "screened"):
        n, a, m, k1 = float(c["n"]), float(c["naux"]), c["ntau"], c["k1"]
        inp = 8.0 * (n * a + a * a + m * n * n)
        if c["call"] == "sox":
            # half of the B, C products where D is symmetric
            fused = 2 * a * a * n * n * (0.5 * (1 + 1 / a) if c["sym"] else 1.0)
            mac = fused + a * n ** 3 + 2 * a * a * n + 3 * a * n * n
            return {"bytes": inp + 8.0 * k1 * (n * n + (a * a if c["thc"] else 0)),
                    "flops": 2.0 * mac * k1}
        if c["call"] == "direct":
            mac = 2 * a ** 3 + 3 * a * a * n + 3 * a * n * n
            return {"bytes": inp + 16.0 * k1 * n * n, "flops": 2.0 * mac * k1}
        sox = 2 * a * a * n * n * (2.0 if c["kind"] == "sosex" else 0.5) + \
            a * n ** 3 * (2 if c["kind"] == "sosex" else 1) + 2 * a * a * n
        mac = m * (2 * a * a * n + 2 * a * n * n) + 3 * a ** 3 + a * a * n * n + sox * k1
        return {"bytes": inp + 8.0 * (a * a + k1 * n * n), "flops": 2.0 * mac}
    if c["call"] == "loop":
        n, m, w, d = float(c["n"]), c["ntau"], c["nfreq"], c["depth"]
        mac = 2 * w * m * n * n * 2 + 4 * w * n ** 3
        byt = 8.0 * n * n * (2 * m + m + m)
        if c["kind"] == "commutator":
            mac += 2 * w * m * n * n + 8 * w * n ** 3
            byt += 8.0 * n * n * 2 * w
        return {"bytes": d * byt, "flops": 2.0 * mac * d}
    if c["call"] == "train":
        m, H, B, st = c["m"], c["hidden"], c["batch"], c["steps"] + 1
        return {"bytes": st * (8.0 * B * m + 28.0 * (2 * m * H + H * H)),
                "flops": st * 6.0 * B * (2 * m * H + H * H)}
    m, H, a, n = c["m"], c["hidden"], float(c["naux"]), float(c["n"])
    return {"bytes": 16.0 * m * a * a + 8.0 * m * n * n,
            "flops": 2.0 * a * a * (2 * m * H + H * H) + 2.0 * m * (n * a * a + n * n * a)}


# ---------------------------------------------------------------------------
# the same in 64 bits, from the definitions
# ---------------------------------------------------------------------------

def _u(X, V):
    """U[P, q, s] = sum_Q V_PQ X_qQ X_sQ."""
    n, a = X.shape
    U = torch.empty((a, n, n), dtype=torch.float64, device=DEV)
    step = max(1, int(5e8 / (8 * n * a)))
    for q in range(0, n, step):
        kr = (X[q:q + step, None, :] * X[None, :, :]).reshape(-1, a)
        U[:, q:q + step] = (V @ kr.T).view(a, -1, n)
    return U


def _exchange(X, Ua, Uc, Gk, Gb):
    """(Sigma_RP in the THC basis, Sigma) with core a on A, core c on C."""
    n, a = X.shape
    Gt, GX = X.T @ Gk, (Gk @ X).T
    S = torch.zeros((a, a), dtype=torch.float64, device=DEV)
    outer, inner = max(1, int(6e9 / (8 * a * n))), max(1, int(2e9 / (16 * a * a)))
    for v0 in range(0, n, outer):
        A = (Ua.view(a * n, n) @ Gb[:, v0:v0 + outer].contiguous()).view(a, n, -1)
        A = A.permute(2, 0, 1).contiguous()
        C0 = Uc[:, v0:v0 + outer].permute(1, 0, 2).contiguous()
        for v in range(0, len(A), inner):
            B = A[v:v + inner] @ Gt.T.contiguous()       # [v, P, R]
            C = C0[v:v + inner] @ GX.T.contiguous()      # [v, R, P]
            S -= (C * B.transpose(1, 2)).sum(0)
    return S, X @ S @ X.T


def _trace_energy(G, S, w):
    m = len(w)
    tr = [(G[m - 1 - k].T * S[k]).sum().item() for k in range(m)]
    return -0.5 * float(np.dot(w, tr))


def _maps(m, nfreq):
    """Chebyshev nodes to Matsubara values and the least-squares way back
    (values at the nodes, and at beta^-)."""
    x, gw = np.polynomial.legendre.leggauss(2400)
    wn = (2 * np.arange(nfreq) + 1) * np.pi / BETA
    Tl = np.polynomial.chebyshev.chebvander(x, m - 1)
    T = (np.exp(1j * np.outer(wn, 0.5 * BETA * (1 + x))) * gw * 0.5 * BETA) @ Tl
    nodes = -np.cos((2 * np.arange(m) + 1) * np.pi / (2 * m))
    Tn = np.polynomial.chebyshev.chebvander(nodes, m - 1)
    Wf = T @ ((2.0 - (np.arange(m) == 0))[:, None] / m * Tn.T)
    A = np.vstack([T.real, T.imag])
    q, r = np.linalg.qr(A)
    P = np.linalg.solve(r, q.T)
    return Wf, np.vstack([Tn, np.ones(m)]) @ P


def _net64(p, x):
    z1 = x @ p["W1"].T + p["b1"]
    h1 = z1 * torch.sigmoid(z1)
    z2 = h1 @ p["W2"].T + p["b2"]
    return x + (z2 * torch.sigmoid(z2)) @ p["W3"].T + p["b3"]


def _exact_loop(c, seed):
    n, m, nf = c["n"], c["ntau"], c["nfreq"]
    Q, eps, mu = _orbitals(n, seed)
    F = (Q * eps) @ Q.T
    _, pairs = _pole_sigmas(c, seed)
    Wf, Wb = (torch.from_numpy(v).to(DEV) for v in _maps(m, nf))
    iw = 1j * (2 * torch.arange(nf, device=DEV, dtype=torch.float64) + 1) * math.pi / BETA
    eye = torch.eye(n, dtype=torch.complex128, device=DEV)

    def freq(S):
        S = S.reshape(m, n * n)
        return torch.complex(Wf.real.contiguous() @ S, Wf.imag.contiguous() @ S).view(nf, n, n)

    res, outs, e1 = [], [], []
    for S_in, S_out in pairs:
        Giw = torch.linalg.inv(((iw + mu)[:, None, None] * eye - F - freq(S_in)).cpu()).to(DEV)
        both = Wb @ torch.cat([Giw.real.reshape(nf, -1), Giw.imag.reshape(nf, -1)])
        G, gamma = both[:m].view(m, n, n), -both[m].view(n, n)
        e1.append((F * gamma.T).sum().item())
        if c["kind"] == "commutator":
            D = freq(S_out - S_in)
            e = Giw @ D - D @ Giw
            res.append(torch.stack([e.real, e.imag]))
        else:
            res.append(S_out - S_in)
        outs.append(S_out)
    k = len(res)
    B = np.ones((k + 1, k + 1))
    B[k, k] = 0.0
    for i in range(k):
        for j in range(k):
            B[i, j] = (res[i] * res[j]).sum().item()
    top = max(B[i, i] for i in range(k))
    B[:k, :k] /= top
    cf = np.linalg.solve(B, np.eye(k + 1)[k])[:k]
    out = {"G": G, "gamma": gamma, "E1": e1,
           "sigma_next": sum(float(x) * S for x, S in zip(cf, outs))}
    if c["kind"] == "commutator":
        out["e"] = res[-1]
    return out


def _exact_train(c, seed):
    p = {k: torch.from_numpy(v).to(DEV).double().requires_grad_() for k, v in _net_params(c, seed).items()}
    g = _gen(seed)
    batches = [tuple(v.double() for v in _profiles(c, c["batch"], g)) for _ in range(c["steps"] + 1)]
    opt = torch.optim.Adam(p.values(), lr=3e-4)
    losses = []
    for x, t in batches:
        opt.zero_grad()
        loss = ((_net64(p, x) - t) ** 2).mean()
        loss.backward()
        losses.append(loss.item())
        if len(losses) <= c["steps"]:
            opt.step()
    return {"losses": losses[:-1], "loss": losses[-1], "grads": {k: v.grad for k, v in p.items()}}


def exact(case, seed):
    c = case
    if c["call"] == "loop":
        return _exact_loop(c, seed)
    if c["call"] == "train":
        return _exact_train(c, seed)
    if c["call"] == "infer":
        X = _system({**c, "ntau": c["m"]}, seed)[0]
        p = {k: torch.from_numpy(v).to(DEV).double() for k, v in _net_params(c, seed).items()}
        S = _thc_sigma(c, seed)
        scale = S.abs().amax(0).reshape(-1)
        x = (S.reshape(c["m"], -1) / scale).T.contiguous()
        y = torch.cat([_net64(p, b) for b in x.split(65536)])
        pred = (y.T * scale).reshape(S.shape).contiguous()
        return {"y": y, "sigma_thc": pred, "sigma": torch.stack([X @ P @ X.T for P in pred])}
    X, V, tau, w, G = _system(c, seed)
    m, k1 = c["ntau"], c["k1"]
    S = torch.zeros_like(G)
    if c["call"] == "direct":
        S = _randn(_gen(seed + 2), *G.shape, scale=0.01)
        for k in range(k1):
            Gt, Gbt = X.T @ G[k] @ X, X.T @ G[m - 1 - k] @ X
            S[k] += X @ ((V @ (Gt * Gbt.T) @ V) * Gt) @ X.T
        return {"sigma": S, "energy": _trace_energy(G, S, w)}
    U = _u(X, V)
    if c["call"] == "screened":
        Pi0 = torch.zeros_like(V)
        for k in range(m):
            Pi0 += float(w[k]) * (X.T @ G[k] @ X) * (X.T @ G[m - 1 - k] @ X).T
        W = torch.linalg.solve(torch.eye(c["naux"], dtype=torch.float64, device=DEV) + V @ Pi0, V)
        Uw = _u(X, W)
        for k in range(k1):
            g = G[k], G[m - 1 - k]
            if c["kind"] == "sosex":
                S[k] = 0.5 * (_exchange(X, U, Uw, *g)[1] + _exchange(X, Uw, U, *g)[1])
            else:
                S[k] = _exchange(X, Uw, Uw, *g)[1]
        return {"W": W, "sigma": S}
    thc = torch.zeros((m, c["naux"], c["naux"]), dtype=torch.float64, device=DEV) if c["thc"] else None
    for k in range(k1):
        t, S[k] = _exchange(X, U, U, G[k], G[m - 1 - k])
        if c["thc"]:
            thc[k] = t
    out = {"sigma": S}
    if c["thc"]:
        out["sigma_thc"] = thc
    if k1 == m:
        out["energy"] = _trace_energy(G, S, w)
    return out
