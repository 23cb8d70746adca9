"""Ranges of the direct term on one side of the tau grid, where a batch holds more pairs
(three buffers each) than one of whole pairs (four): sizes of the range around a batch of
either kind, on both sides, against the whole grid's bits."""
import numpy as np
import pytest
import torch

from oracle import direct as od
from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit_matrices", [0, 7, 13])
@pytest.mark.parametrize("m", [44, 45])
def test_one_sided_ranges(dev, m, limit_matrices):
    """Without a limit a batch holds 12 pairs or 16 points; with room for 13 matrices 3 pairs
    or 4 points, for 7 one pair or one point."""
    n, naux = 5, 290
    s = synth.make_system(n, naux, seed=m)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=m)
    on = lambda a: torch.from_numpy(a).to(dev)
    X, V, Gd = on(s.X), on(s.V), on(G)
    ref = osox.sigma_all_tau(od.sigma_direct_thc, G, s.X, s.V)
    plan = thcsox.Plan(X, V, tau, w, 100.0)
    whole = plan.sigma_direct(Gd)
    assert np.abs(whole.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()
    if limit_matrices:
        # (what the plan takes under a limit depends on it: find one that leaves that room)
        taken, one = plan.info()["bytes"], 8 * naux * naux
        plan.close()
        limit = taken + limit_matrices * one
        while True:
            plan = thcsox.Plan(X, V, tau, w, 100.0, workspace_limit=limit)
            room = limit - plan.info()["bytes"]
            if room <= (limit_matrices + 0.5) * one:
                break
            plan.close()
            limit -= max(room - int((limit_matrices + 0.5) * one), 256)
        assert room >= 3.5 * one
    half = (m + 1) // 2
    print(f"case direct one side m{m} limit {limit_matrices}", flush=True)
    for k in (1, 3, 4, 5, 12, 13, 16, 17, half - 1, half):
        for a, b in ((0, k), (m - k, m), (half - k, half), (half, min(m, half + k))):
            S = torch.full_like(Gd, 3.0)
            plan.sigma_direct(Gd, a, b, out=S)
            assert torch.equal(S[a:b], whole[a:b]), (a, b)
            assert bool((S[:a] == 3.0).all()) and bool((S[b:] == 3.0).all()), (a, b)
    plan.close()
