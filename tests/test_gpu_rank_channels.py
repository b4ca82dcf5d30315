"""O_act and the widths in one call (cmpq_rank_channels) against the two calls it stands for
(cmpq_extract_outliers in channels mode, cmpq_allocate_bits), bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

DEV = "cuda"


@pytest.mark.gpu
@pytest.mark.parametrize("d_in", [1, 2, 9, 100, 1023, 4096, 8185, 8192, 8193, 20000])
def test_one_call_equals_two(d_in):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_in)
    stats = [rng.lognormal(0, 2, d_in + 1).astype(np.float32), np.zeros(d_in + 1, np.float32),
             rng.integers(0, 4, d_in + 1).astype(np.float32), rng.lognormal(0, 60, d_in + 1).astype(np.float32)]
    stats[3][rng.random(d_in + 1) < 0.1] = np.nan
    stats[3][rng.random(d_in + 1) < 0.1] = np.inf
    for s in stats:
        for offset in (0, 1):
            stat = torch.from_numpy(s).to(DEV)[offset:offset + d_in]
            for k in sorted({0, 1, d_in // 200, d_in // 2, d_in}):
                for bit_set, avg in (((2, 3, 4), 2.6), ((2, 3, 4), 3.0), ((3, 4), 4.0), ((1, 2), 1.0), ((1, 2, 3, 4), 2.0),
                                     ((2, 3), 2.0001)):
                    idx = [torch.full((k,), -7, dtype=torch.int32, device=DEV) for _ in range(2)]
                    mask, bits = [[torch.full((d_in + 8,), 5, dtype=torch.uint8, device=DEV) for _ in range(2)] for _ in range(2)]
                    view = lambda t: t[3 + offset:3 + offset + d_in]  # noqa: E731
                    B.extract_channel_outliers(stat, k, idx[0], view(mask[0]), ws)
                    counts = B.allocate_bits(stat, view(mask[0]), k, bit_set, avg, view(bits[0]), ws)
                    assert B.rank_channels(stat, k, bit_set, avg, idx[1], view(mask[1]), view(bits[1])) == counts
                    for a, b in (idx, mask, bits):
                        assert torch.equal(a, b), (d_in, k, bit_set, avg)


def test_what_the_two_calls_refuse_is_refused():
    from paper_2410_13056_amd import binding as B
    L = B.lib()
    fake, bs = ctypes.c_void_p(256), (ctypes.c_int32 * 3)(2, 3, 4)
    cnt = (ctypes.c_int64 * 3)()
    call = lambda s, d, k, n, avg, idx, mask, bits: L.cmpq_rank_channels(s, d, k, bs, n, ctypes.c_double(avg), idx, mask, bits, cnt, None)  # noqa: E731
    assert call(fake, 16, 17, 3, 3.0, fake, fake, fake) == -4          # more than there are
    assert call(fake, 16, 2, 3, 4.5, fake, fake, fake) == -3           # budget
    assert call(fake, 16, 2, 0, 3.0, fake, fake, fake) == -3
    assert call(None, 16, 2, 3, 3.0, fake, fake, fake) == -1
    assert call(fake, 16, 2, 3, 3.0, None, fake, fake) == -1
    assert call(fake, 16, -1, 3, 3.0, fake, fake, fake) == -1
    assert call(fake, 0, 0, 3, 3.0, None, fake, fake) == 0             # nothing to do
