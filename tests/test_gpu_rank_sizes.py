"""Channel rankings (O_act and Algorithm 1) at the sizes where their kernels begin and end, with
ties, zeros, unaligned inputs and outputs, against a plain sort."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("d_in", [1, 2, 7, 8, 9, 63, 1023, 1025, 8191, 8192, 8193, 32768, 32769])
def test_rankings_at_the_edges(d_in):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_in)
    s = rng.lognormal(0, 2, d_in + 1).astype(np.float32)
    s[rng.random(d_in + 1) < 0.3] = s[0]                       # many ties
    s[rng.random(d_in + 1) < 0.1] = 0.0
    s[rng.random(d_in + 1) < 0.02] = 1e-40                     # subnormal
    for offset in (0, 1):
        stat = torch.from_numpy(s).to(DEV)[offset:offset + d_in]
        order = np.argsort(-s[offset:offset + d_in], kind="stable")
        for k in sorted({0, 1, d_in // 200, d_in // 3, d_in}):
            idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
            around = torch.full((d_in + 8,), 5, dtype=torch.uint8, device=DEV)
            mask = around[3 + offset:3 + offset + d_in]
            B.extract_channel_outliers(stat, k, idx, mask, ws)
            want = np.zeros(d_in, np.uint8)
            want[order[:k]] = 1
            assert np.array_equal(mask.cpu().numpy(), want)
            assert np.array_equal(idx.cpu().numpy(), np.flatnonzero(want))
            assert bool((around[:3 + offset] == 5).all()) and bool((around[3 + offset + d_in:] == 5).all())
            d_eff = d_in - k
            live = order[k:]
            for bit_set, avg in (((2, 3, 4), 2.6), ((2, 3, 4), 3.0), ((3, 4), 4.0), ((1, 2), 1.0)):
                around.fill_(5)
                bits = around[3 + offset:3 + offset + d_in]
                counts = B.allocate_bits(stat, mask_of(want), k, bit_set, avg, bits, ws)
                b = np.full(d_in, B.PROTECTED, np.uint8)
                lo = int(np.floor(avg))
                if avg > lo:
                    n = int(np.floor(avg * d_eff + 1e-9)) - lo * d_eff
                    b[live[:n]], b[live[n:]] = lo + 1, lo
                else:
                    b[live] = lo
                    if lo - 1 in bit_set and lo + 1 in bit_set and d_eff > 0:
                        n = min(int(np.ceil(0.01 * (d_eff - 1) - 1e-12)), d_eff // 2)
                        b[live[:n]], b[live[d_eff - n:]] = lo + 1, lo - 1
                assert np.array_equal(bits.cpu().numpy(), b), (d_in, k, bit_set, avg)
                assert counts == [int((b == w).sum()) for w in bit_set]
                assert bool((around[:3 + offset] == 5).all()) and bool((around[3 + offset + d_in:] == 5).all())


def mask_of(want):
    return torch.from_numpy(want).to(DEV)


@pytest.mark.parametrize("d_in", [300, 8192, 9000])
def test_fewer_free_channels_than_ranks_asked_for(d_in):
    """A mask that protects more channels than `n_protected` says leaves fewer channels than the counts
    of the budget: ranks past the last free channel are not there, whichever kernel ranks (the register
    kernel up to 8192 channels, the other beyond)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    stat = torch.arange(1, d_in + 1, dtype=torch.float32, device=DEV)
    mask = torch.zeros(d_in, dtype=torch.uint8, device=DEV)
    free = d_in // 4
    mask[free:] = 1
    order = np.argsort(-stat.cpu().numpy()[:free], kind="stable")
    for avg in (3.5, 3.0):
        bits = torch.zeros(d_in, dtype=torch.uint8, device=DEV)
        B.allocate_bits(stat, mask, 2, (2, 3, 4), avg, bits, ws)
        want = np.full(d_in, B.PROTECTED, np.uint8)
        n_hi = free if avg > 3 else int(np.ceil(0.01 * (d_in - 2 - 1) - 1e-12))   # counted without the mask
        want[order[:n_hi]] = 4
        want[order[n_hi:]] = 3                                       # the second rank lies past the last
        assert np.array_equal(bits.cpu().numpy(), want), avg
