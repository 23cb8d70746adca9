"""Both forms of the pair kernels (one thread per element, and by blocks of 64 pairs and 64
tau points) on either side of the rules that choose between them, with ragged blocks, against the same FP64
and FP32 arithmetic in torch; every value is rounded once, so they agree to the bit."""
import pytest
import torch

from paper_2404_17744_amd import thcsox

pytestmark = pytest.mark.gpu


def _inputs(dev, naux, m):
    g = torch.Generator(device=dev).manual_seed(naux + m)
    S = torch.randn(m, naux * naux, dtype=torch.float64, device=dev, generator=g)
    return S, S.abs().amax(0), torch.cuda.current_stream().cuda_stream


# naux, tau points: few points, few pairs, and by blocks in gather, scatter or both
@pytest.mark.parametrize("naux,m", [(9, 3), (101, 64), (101, 65), (141, 45), (143, 44), (211, 24),
                                    (253, 23), (253, 24), (274, 11), (275, 12), (397, 97)])
def test_all_pairs_forms(dev, naux, m):
    S, scale, s = _inputs(dev, naux, m)
    aa = naux * naux
    print(f"case pair forms naux{naux} m{m}", flush=True)
    sc = torch.empty_like(scale)
    thcsox.thcsox_pair_scale(m, naux, S.data_ptr(), sc.data_ptr(), s)
    assert torch.equal(sc, scale)
    x = torch.full((aa, m), 9.0, dtype=torch.float32, device=dev)
    thcsox.thcsox_pair_gather(m, naux, S.data_ptr(), sc.data_ptr(), None, aa, x.data_ptr(), s)
    assert torch.equal(x, (S / scale).T.float())
    back = torch.zeros_like(S)
    thcsox.thcsox_pair_scatter(m, naux, x.data_ptr(), sc.data_ptr(), back.data_ptr(), s)
    assert torch.equal(back, x.T.double() * scale)


@pytest.mark.parametrize("n,m", [(1, 5), (4099, 70), (32767, 65), (32771, 65), (131071, 48),
                                 (131101, 47), (131101, 48)])
def test_listed_pairs_forms(dev, n, m):
    naux = 60
    S, scale, s = _inputs(dev, naux, m)
    aa = naux * naux
    g = torch.Generator(device=dev).manual_seed(n)
    pairs = torch.randint(-2, aa + 2, (n,), device=dev, generator=g)
    print(f"case listed pair forms n{n} m{m}", flush=True)
    x = torch.full((n, m), 9.0, dtype=torch.float32, device=dev)
    thcsox.thcsox_pair_gather(m, naux, S.data_ptr(), scale.data_ptr(), pairs.data_ptr(), n,
                              x.data_ptr(), s)
    inside = (pairs >= 0) & (pairs < aa)
    want = (S / scale).T.float()[pairs.clamp(0, aa - 1)] * inside[:, None]
    assert torch.equal(x, want)
