"""The register-resident A stage at odd numbers of 32-wide k chunks (1, 3, 5, 7 and 9;
fp16x2 and FP32), through Sigma against the oracle: the last chunk full and with a
single orbital, symmetric G and general, an odd number of tau points (the last launch
holds a single one); and past 320 orbitals, where the streaming fp16x2 kernel pads to an
even number of chunks that the fused stage does not walk (n = 330: 11 of 12).  Bar 2e-6
of max |Sigma|: two FP16 planes carry 22 bits, FP32 24, over sums of at most n naux
products whose roundings do not align."""
import numpy as np
import pytest
import torch

from oracle import sox as osox
from paper_2404_17744_amd import synth, thcsox

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp16x2", "fp32"])
@pytest.mark.parametrize("n,naux", [(5, 9), (32, 33), (65, 40), (96, 31), (129, 24), (160, 17),
                                    (193, 20), (224, 15), (257, 12), (288, 19), (330, 11)])
def test_odd_chunk_counts(dev, n, naux, precision):
    m, general = 3, n % 2 == 0
    s = synth.make_system(n, naux, seed=n)
    tau, w = synth.cheb_tau_grid(m, 100.0)
    G = synth.random_general_g(n, m, seed=m) if general else synth.g0_tau(s, tau, 100.0)
    print(f"case {precision} n{n} naux{naux} general={general}", flush=True)
    ref = osox.sigma_all_tau(osox.sigma_thc_paper, G, s.X, s.V)
    plan = thcsox.Plan(torch.from_numpy(s.X).to(dev), torch.from_numpy(s.V).to(dev), tau, w, 100.0,
                       precision=precision)
    S = plan.sigma(torch.from_numpy(G).to(dev)).cpu().numpy()
    plan.close()
    assert np.abs(S - ref).max() <= 2e-6 * np.abs(ref).max()
