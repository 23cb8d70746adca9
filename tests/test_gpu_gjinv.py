"""The blocked Gauss-Jordan inversion at the edges of its blocking, complex (the Dyson
step) and real (the static screening): one column or row more or less than a panel
(32, 16, 8 and 4 columns, by size), than a wavefront, than a 64-column trailing
block, and each register blocking.  Random matrices far from diagonal dominance, so
that pivots are taken all over the rows; the bar of 1e-10 is n eps times a condition
number of a few thousand."""
import numpy as np
import pytest
import torch

from oracle import screened as osc
from oracle import transforms as otr
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 97, 128, 300, 511, 512, 513, 1024,
                               1025, 2049])
def test_complex_inverse_block_edges(dev, n):
    rng = np.random.default_rng(n)
    F = rng.standard_normal((n, n))
    F = 0.5 * (F + F.T)
    S = 10.0 * rng.standard_normal((4, n, n))
    tau, _ = synth.cheb_tau_grid(4, 100.0)
    print(f"case inverse complex n{n}", flush=True)
    Tm = otr.cheb_to_matsubara(4, 3, 100.0)
    G_ref, gam_ref, _ = otr.loop_step(F, 0.1, 100.0, S, Tm)
    d = thcsox.Dyson(torch.from_numpy(F).to(dev), 0.1, tau, 100.0, 3)
    G, gam = d.step(torch.from_numpy(S).to(dev))
    d.close()
    assert _rel(G.cpu().numpy(), G_ref) < 1e-10
    assert _rel(gam.cpu().numpy(), gam_ref) < 1e-10


@pytest.mark.parametrize("naux", [1, 2, 31, 32, 33, 64, 65, 129, 512, 513, 1025, 2049])
def test_real_inverse_block_edges(dev, naux):
    """W = (1 + V Pi0)^-1 V with a general G (Pi0 of no definite sign)."""
    n, m = 3, 4
    X, V = synth.thc_factors(n, naux, seed=naux)
    G = synth.random_general_g(n, m, seed=2)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    print(f"case inverse real naux{naux}", flush=True)
    plan = thcsox.Plan(torch.from_numpy(X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    W = plan.static_screening(torch.from_numpy(G).to(dev)).cpu().numpy()
    plan.close()
    ref = osc.screened_core(V, osc.static_polarization(X, G, w))
    assert _rel(W, ref) < 1e-10


def test_singular_matrix_is_refused(dev):
    """A zero column in one frequency's matrix."""
    n = 40
    tau, _ = synth.cheb_tau_grid(4, 100.0)
    d = thcsox.Dyson(torch.zeros((n, n), dtype=torch.float64, device=dev), 0.0, tau, 100.0, 2)
    S = torch.zeros((4, n, n), dtype=torch.float64, device=dev)
    S[:, 7, 7] = float("inf")
    print("case inverse singular", flush=True)
    with pytest.raises(thcsox.ThcsoxError):
        d.step(S)
    d.close()
