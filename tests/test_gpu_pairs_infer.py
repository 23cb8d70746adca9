"""The learned start's kernels at the edges of their blocking: pair gather and scatter
(blocks of 64 pairs x 64 tau points, with and without a pair list, pairs outside the
array) exactly, and the bf16 forward at batches around 64 and 128 rows and on both
sides of the switch to 128 rows a workgroup, against the oracle's bf16 forward (half
a bf16 unit of the residual branch, as the other parity tests) and bitwise between
the two row blockings."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from paper_2404_17744_amd import thcsox, warmstart

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,A", [(1, 1), (3, 5), (12, 8), (63, 9), (64, 11), (65, 7), (130, 23)])
def test_gather_scatter_blocks(dev, m, A):
    rng = np.random.default_rng(m * A)
    print(f"case pairs m{m} A{A}", flush=True)
    Sn = rng.standard_normal((m, A * A))
    S = torch.from_numpy(Sn.reshape(m, A, A)).to(dev)
    scale = warmstart.pair_scale(S)
    sc = scale.cpu().numpy()
    assert np.array_equal(sc, np.abs(Sn).max(0))
    x = warmstart.pair_profiles(S, scale)
    ref = (Sn / sc).astype(np.float32).T
    assert np.array_equal(x.cpu().numpy(), ref)
    pairs = rng.integers(-2, A * A + 2, size=2 * A * A + 1)
    got = warmstart.pair_profiles(S, scale, torch.from_numpy(pairs.astype(np.int64)).to(dev)).cpu().numpy()
    ok = (pairs >= 0) & (pairs < A * A)
    assert np.array_equal(got[ok], ref[pairs[ok]]) and not got[~ok].any()
    out = torch.empty_like(S)
    thcsox.thcsox_pair_scatter(m, A, x.data_ptr(), scale.data_ptr(), out.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    assert np.array_equal(out.cpu().numpy().reshape(m, -1), x.cpu().numpy().T.astype(np.float64) * sc)


@pytest.mark.parametrize("m,H", [(32, 256), (64, 256), (32, 512), (64, 512), (64, 128)])
def test_bf16_forward_row_blocks(dev, m, H):
    rng = np.random.default_rng(m + H)
    p = {k: v.astype(np.float32) for k, v in warmstart.init_params(m, H, 3).items()}
    p["W3"] = p["W3"] * 30
    B = 2 * 256 * 128
    print(f"case bf16 rows m{m} H{H}", flush=True)
    x = torch.from_numpy(rng.standard_normal((B + 77, m)).astype(np.float32)).to(dev)
    net = thcsox.MLP(m, H, p, max_batch=16)
    y = net.forward_bf16(x)
    for n in (1, 63, 64, 65, 127, 128, 129, 1000, B - 1, B):
        assert torch.equal(net.forward_bf16(x[:n].contiguous()), y[:n]), n
    net.close()
    s = slice(B - 300, B + 77)
    ref = omlp.forward_bf16({k: v.astype(np.float64) for k, v in p.items()}, x[s].cpu().numpy().astype(np.float64))
    xs = x[s].cpu().numpy()
    branch = np.abs(ref - xs).max()
    assert np.abs(y[s].cpu().numpy() - ref).max() <= 2.0 ** -9 * branch
