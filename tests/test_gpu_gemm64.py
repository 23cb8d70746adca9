"""The direct term and the FP64 matrix-core GEMM under it.  The GEMM at the sizes where its tiling can go wrong, through
the direct term (every operand orientation: X^T G, T X, V Pi, W V, X H, T X^T) against
the oracle: extents of 1, odd extents (8-byte aligned rows), one element more or
less than a tile edge of 32, 64 and 128, partial last k steps, and enough tiles for
each tile edge to be picked.  FP64 sums of at most 520 products: 520 eps ~ 1e-13 of
the largest term, with a factor of ten for the four products in a row.

Mirrored tau points share one W where V is symmetric; a V with a rounding-level or a
visible asymmetry takes either route and gives the same self-energy."""
import numpy as np
import pytest
import torch

from oracle import direct as od
from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,naux,m", [
    (1, 1, 2), (1, 2, 3), (2, 1, 2), (2, 3, 4), (7, 31, 5), (15, 33, 4), (17, 32, 6),
    (31, 65, 5), (33, 63, 16), (64, 128, 8), (65, 127, 16), (63, 129, 9), (129, 515, 20),
    (130, 520, 24), (128, 512, 16),
])
def test_direct_term_tile_edges(dev, n, naux, m):
    X, V = synth.thc_factors(n, naux, seed=n + naux)
    G = synth.random_general_g(n, m, seed=n * 7 + m)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    print(f"case direct tiles n{n} naux{naux} m{m}", flush=True)
    ref = osox.sigma_all_tau(od.sigma_direct_thc, G, X, V)
    plan = thcsox.Plan(torch.from_numpy(X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    S = plan.sigma_direct(torch.from_numpy(G).to(dev)).cpu().numpy()
    plan.close()
    assert np.abs(S - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("m", [1, 2, 5, 8])
@pytest.mark.parametrize("asym", [0.0, 1e-16, 1e-13])
def test_direct_term_mirrored_pairs(dev, m, asym):
    """Every slice [a, b) of the grid against the oracle, and bitwise equal to the same
    points of the whole; general G; V as given, symmetric or not."""
    n, naux = 9, 37
    X, V = synth.thc_factors(n, naux, seed=3)
    V = V + asym * np.abs(V).max() * np.triu(np.ones_like(V), 1)
    G = synth.random_general_g(n, m, seed=5)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    print(f"case direct pairs m{m} asym{asym}", flush=True)
    ref = osox.sigma_all_tau(od.sigma_direct_thc, G, X, V)
    plan = thcsox.Plan(torch.from_numpy(X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    Gd = torch.from_numpy(G).to(dev)
    whole = plan.sigma_direct(Gd).cpu().numpy()
    assert np.abs(whole - ref).max() <= 1e-12 * np.abs(ref).max()
    for a in range(m):
        for b in range(a + 1, m + 1):
            part = torch.zeros_like(Gd)
            part[a:b] = 1.0
            plan.sigma_direct(Gd, a, b, out=part, accumulate=True)
            part = part.cpu().numpy()
            assert np.array_equal(part[a:b], 1.0 + whole[a:b]) and not part[:a].any() and not part[b:].any()
    plan.close()
