"""The fused stage of every precision where the last block of THC points is not full: 1, 2
and 3 of its four 32-wide strips hold a point, at the first and the last point of a
strip, as columns, rows (general G, where the blocks below the diagonal are formed too)
and the corner; and full blocks.  Against the oracle; bars as fractions of max |Sigma|: 2e-6
for fp16x2, FP32 and bf16x3 (two FP16 planes carry 22 bits, FP32 and three bf16 planes
24, over sums of at most n naux products whose roundings do not align), 1e-12 for FP64
(64-wide blocks of two strips)."""
import numpy as np
import pytest
import torch

from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("precision", ["fp16x2", "fp32", "bf16x3", "fp64"])
@pytest.mark.parametrize("naux", [1, 33, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257])
def test_partial_blocks(dev, naux, precision, general):
    n, m = 10, 3
    s = synth.make_system(n, naux, seed=naux)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=m) if general else synth.g0_tau(s, tau, 100.0)
    print(f"case {precision} n{n} naux{naux} general={general}", flush=True)
    ref = osox.sigma_all_tau(osox.sigma_thc_paper, G, s.X, s.V)
    plan = thcsox.Plan(torch.from_numpy(s.X).to(dev), torch.from_numpy(s.V).to(dev), tau, w, 100.0,
                       precision=precision)
    S = plan.sigma(torch.from_numpy(G).to(dev)).cpu().numpy()
    plan.close()
    assert np.abs(S - ref).max() <= (1e-12 if precision == "fp64" else 2e-6) * np.abs(ref).max()
