"""DIIS histories longer than one pass of the kernels takes (eight entries), lengths
that divide nothing, both residual kinds and an output that aliases an input,
against the oracle's extrapolation; and the traces of the energies at sizes around
the blocks of 32 and 64 that a wavefront takes.  Bars: 1e-11 as for the shorter
histories; 1e-13 for a sum of n^2 products in FP64."""
import numpy as np
import pytest
import torch

from oracle import loopctl as olc
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,steps,shape", [(1, 3, (2, 3, 3)), (8, 11, (3, 17, 17)),
                                               (9, 14, (5, 41, 41)), (17, 18, (2, 9, 9))])
@pytest.mark.parametrize("kind", ["pulay", "explicit"])
def test_long_histories(dev, depth, steps, shape, kind):
    rng = np.random.default_rng(depth + steps)
    print(f"case diis depth{depth} {kind} {shape}", flush=True)
    like = torch.empty(shape, dtype=torch.float64, device=dev)
    res_shape = (2, 7, 13)
    res_like = torch.empty(res_shape, dtype=torch.float64, device=dev) if kind == "explicit" else None
    diis = thcsox.Diis(like, depth=depth, residual_like=res_like)
    ins, outs, ress = [], [], []
    for _ in range(steps):
        a, b, r = (rng.standard_normal(s) for s in (shape, shape, res_shape))
        ins.append(a); outs.append(b); ress.append(r)
        ad, bd = torch.from_numpy(a).to(dev), torch.from_numpy(b).to(dev)
        if kind == "pulay":
            diis.step(ad, bd, ad)          # the output aliases the input
            ref = olc.diis_next(ins[-depth:], outs[-depth:])
        else:
            diis.step_res(torch.from_numpy(r).to(dev), bd, ad)
            ref = olc.cdiis_next(ress[-depth:], outs[-depth:])
        got = ad.cpu().numpy()
        assert np.abs(got - ref).max() <= 1e-11 * max(1.0, np.abs(ref).max())
    diis.close()


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 130, 300])
def test_energy_traces(dev, n):
    m = 3
    X, V = synth.thc_factors(n, 2, seed=1)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=n)
    S = synth.random_general_g(n, m, seed=n + 1)
    print(f"case traces n{n}", flush=True)
    Gd, Sd = torch.from_numpy(G).to(dev), torch.from_numpy(S).to(dev)
    plan = thcsox.Plan(torch.from_numpy(X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    E = plan.energy(Gd, Sd)
    plan.close()
    terms = [w[k] * G[m - 1 - k].T * S[k] for k in range(m)]
    assert abs(E + 0.5 * sum(t.sum() for t in terms)) <= 1e-13 * sum(np.abs(t).sum() for t in terms)
    d = thcsox.Dyson(Gd[0].contiguous(), 0.1, tau, 100.0, 4)
    e1 = d.onebody(Sd[0].contiguous())
    d.close()
    t = G[0] * S[0].T
    assert abs(e1 - t.sum()) <= 1e-13 * np.abs(t).sum()
