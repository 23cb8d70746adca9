"""The pair kernels of the learned start beyond 2^30 pairs (naux > 32768), where a launch
cannot have a workgroup for every block of 64 pairs.  One tau point, so that the scale of
a pair is its magnitude and its profile is its sign; everything is compared on the device."""
import pytest
import torch

from paper_2404_17744_amd import thcsox

pytestmark = pytest.mark.gpu
NAUX = 32781
STEP = 1 << 26


def _chunks(n):
    return [slice(a, min(a + STEP, n)) for a in range(0, n, STEP)]


def test_all_pairs(dev):
    aa = NAUX * NAUX
    assert aa > 1 << 30 and aa % 64 != 0
    S = torch.empty(aa, dtype=torch.float64, device=dev)
    for c in _chunks(aa):
        i = torch.arange(c.start, c.stop, device=dev)
        S[c] = (i % 1013 - 506).double() * 0.25
    scale = torch.empty_like(S)
    x = torch.full((aa,), 9.0, dtype=torch.float32, device=dev)
    s = torch.cuda.current_stream().cuda_stream
    print(f"case all pairs naux{NAUX}", flush=True)
    thcsox.thcsox_pair_scale(1, NAUX, S.data_ptr(), scale.data_ptr(), s)
    thcsox.thcsox_pair_gather(1, NAUX, S.data_ptr(), scale.data_ptr(), None, aa, x.data_ptr(), s)
    for c in _chunks(aa):
        assert torch.equal(x[c], torch.sign(S[c]).float()), c
    back = torch.zeros_like(S)
    thcsox.thcsox_pair_scatter(1, NAUX, x.data_ptr(), scale.data_ptr(), back.data_ptr(), s)
    for c in _chunks(aa):
        assert torch.equal(back[c], S[c]), c


def test_more_listed_pairs_than_a_launch_has_threads_for(dev):
    naux, n = 5, (1 << 30) + 77
    S = torch.arange(-12, 13, dtype=torch.float64, device=dev)
    scale = torch.ones_like(S)
    pairs = torch.empty(n, dtype=torch.int64, device=dev)
    for c in _chunks(n):
        pairs[c] = torch.arange(c.start, c.stop, device=dev) % 27 - 1   # -1 and 25: outside
    x = torch.full((n,), 9.0, dtype=torch.float32, device=dev)
    s = torch.cuda.current_stream().cuda_stream
    print("case listed pairs", flush=True)
    thcsox.thcsox_pair_gather(1, naux, S.data_ptr(), scale.data_ptr(), pairs.data_ptr(), n,
                              x.data_ptr(), s)
    want = torch.cat([torch.zeros(1, device=dev), S.float(), torch.zeros(1, device=dev)])
    for c in _chunks(n):
        assert torch.equal(x[c], want[pairs[c] + 1]), c


def test_blocks_in_several_launches(dev):
    """Sixteen tau points of 2^29 pairs and more, the first size at which the forms by blocks
    take two launches; values that FP32 holds exactly, so that they come back as they were."""
    naux, m = 23171, 16
    aa = naux * naux
    assert aa > 1 << 29 and aa % 64 != 0

    def values(k, c):
        i = torch.arange(c.start, c.stop, device=dev)
        return ((i * 7 + k * 13) % 2047 - 1023).double() * 0.25

    S = torch.empty((m, aa), dtype=torch.float64, device=dev)
    for k in range(m):
        for c in _chunks(aa):
            S[k, c] = values(k, c)
    scale = torch.full((aa,), 2.0, dtype=torch.float64, device=dev)
    x = torch.full((aa, m), 9.0, dtype=torch.float32, device=dev)
    s = torch.cuda.current_stream().cuda_stream
    print(f"case blocks naux{naux} m{m}", flush=True)
    thcsox.thcsox_pair_gather(m, naux, S.data_ptr(), scale.data_ptr(), None, aa, x.data_ptr(), s)
    for k in (0, 7, m - 1):
        for c in _chunks(aa):
            assert torch.equal(x[c, k], 0.5 * values(k, c).float()), (k, c)
    S.zero_()
    thcsox.thcsox_pair_scatter(m, naux, x.data_ptr(), scale.data_ptr(), S.data_ptr(), s)
    for k in range(m):
        for c in _chunks(aa):
            assert torch.equal(S[k, c], values(k, c)), (k, c)
