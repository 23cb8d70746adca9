"""The direct term's use of V's symmetry: two uncoupled systems of very different
interaction strength in one plan, the weak one with a V that is symmetric, symmetric up to
the last bits or not symmetric at all.  Each system's self-energy is held to its own
largest element; the bar is 20 000 times the unit rounding for sums of at most a few
hundred products in three successive matrix products."""
import numpy as np
import pytest
import torch

from oracle import direct as od
from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weak", ["symmetric", "last bits", "general"])
@pytest.mark.parametrize("m", [4, 7])
def test_weak_block_beside_a_strong_one(dev, m, weak):
    n1, a1, n2, a2 = 4, 21, 5, 37
    rng = np.random.default_rng(m)
    X1, V1 = synth.thc_factors(n1, a1, seed=1)
    X2, V2 = synth.thc_factors(n2, a2, seed=2)
    V1 = V1 * (1e10 / np.abs(V1).max())
    V2 = V2 * (1e-6 / np.abs(V2).max())
    if weak == "last bits":
        up = np.triu(rng.integers(-2, 3, V2.shape), 1)
        V2 = V2 * (1.0 + up * 2.0 ** -52)
    elif weak == "general":
        V2 = rng.uniform(-1e-6, 1e-6, V2.shape)
    X = np.zeros((n1 + n2, a1 + a2))
    V = np.zeros((a1 + a2, a1 + a2))
    X[:n1, :a1], X[n1:, a1:] = X1, X2
    V[:a1, :a1], V[a1:, a1:] = V1, V2
    G = np.zeros((m, n1 + n2, n1 + n2))
    G[:, :n1, :n1] = synth.random_general_g(n1, m, seed=3)
    G[:, n1:, n1:] = synth.random_general_g(n2, m, seed=4)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    on = lambda a: torch.from_numpy(a).to(dev)
    print(f"case direct weak block m{m} {weak}", flush=True)
    plan = thcsox.Plan(on(X), on(V), tau, w, 100.0)
    S = plan.sigma_direct(on(G)).cpu().numpy()
    plan.close()
    ref1 = osox.sigma_all_tau(od.sigma_direct_thc, G[:, :n1, :n1], X1, V1)
    ref2 = osox.sigma_all_tau(od.sigma_direct_thc, G[:, n1:, n1:], X2, V2)
    bar = 20000 * 2.0 ** -53
    assert np.abs(S[:, :n1, :n1] - ref1).max() <= bar * np.abs(ref1).max()
    assert np.abs(S[:, n1:, n1:] - ref2).max() <= bar * np.abs(ref2).max()
    assert not S[:, :n1, n1:].any() and not S[:, n1:, :n1].any()
