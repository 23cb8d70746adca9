"""The FP64 exchange path (A stage, fused stage with memory-to-LDS loads, reduction) at
the edges of its blocking: one k or THC point more or less than a 16-wide k stage
and a 64-wide tile, odd and even numbers of stages per v, v ranges left empty, and
several tau points per launch; symmetric G (half of the tiles skipped) and general.
Bar 1e-12 of max |Sigma|: FP64 sums of at most n^2 naux^2 products."""
import numpy as np
import pytest
import torch

from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("n,naux,m", [(1, 1, 1), (2, 63, 3), (15, 64, 2), (16, 65, 5), (17, 127, 4),
                                      (31, 129, 7), (33, 50, 18), (47, 192, 2), (49, 30, 3)])
def test_fp64_exchange_edges(dev, n, naux, m, general):
    if n == 1:
        X, V = synth.thc_factors(1, naux, seed=4)
        general = True
    else:
        s = synth.make_system(n, naux, seed=n)
        X, V = s.X, s.V
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=m) if general else synth.g0_tau(s, tau, 100.0)
    print(f"case fp64 n{n} naux{naux} m{m} general={general}", flush=True)
    ref = osox.sigma_all_tau(osox.sigma_thc_paper, G, X, V)
    plan = thcsox.Plan(torch.from_numpy(X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    S = plan.sigma(torch.from_numpy(G).to(dev)).cpu().numpy()
    plan.close()
    assert np.abs(S - ref).max() <= 1e-12 * np.abs(ref).max()
