"""The direct term on every range [a, b) of the tau grid: mirrored pairs wholly and half
inside the range, the middle point of an odd grid, and V symmetric (pairs) or not (points
one by one).  Points outside the range keep what they held; inside it the result is the
whole grid's, or is added to what was there."""
import numpy as np
import pytest
import torch

from oracle import direct as od
from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("symmetric_v", [True, False])
@pytest.mark.parametrize("m", [1, 2, 5, 6, 19])
def test_every_range(dev, m, symmetric_v):
    n, naux = 7, 33
    s = synth.make_system(n, naux, seed=m)
    V = s.V.copy()
    if not symmetric_v:
        V[0, 1] += 1e-3 * abs(V).max()
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=m)
    ref = osox.sigma_all_tau(od.sigma_direct_thc, G, s.X, V)
    plan = thcsox.Plan(torch.from_numpy(s.X).to(dev), torch.from_numpy(V).to(dev), tau, w, 100.0)
    Gd = torch.from_numpy(G).to(dev)
    bar = 1e-11 * np.abs(ref).max()
    ranges = [(a, b) for a in range(m) for b in range(a + 1, m + 1) if m < 10 or (a * 7 + b) % 5 == 0]
    print(f"case direct n{n} naux{naux} m{m} symmetric_v={symmetric_v}", flush=True)
    for a, b in ranges:
        S = torch.full_like(Gd, 3.0)
        plan.sigma_direct(Gd, a, b, out=S)
        plan.sigma_direct(Gd, a, b, out=S, accumulate=True)
        S = S.cpu().numpy()
        assert np.all(S[:a] == 3.0) and np.all(S[b:] == 3.0)
        assert np.abs(S[a:b] - 2.0 * ref[a:b]).max() <= bar, (a, b)
    plan.close()
