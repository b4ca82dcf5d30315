"""The rows that channels get in the stored format and the slices of O_q, at the sizes where the counting of
widths steps from wavefront to wavefront and from step to step, against a plain count."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d_in", [1, 63, 64, 65, 1023, 1024, 1025, 3000, 8191, 8192, 8193, 17000])
def test_rows_of_each_width(d_in):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    rng = np.random.default_rng(d_in)
    bit_set, d_out = (1, 2, 3, 4), 32
    for kinds in ((1, 2, 3, 4, B.PROTECTED), (2, 4), (3,), (B.PROTECTED,)):
        bits = rng.choice(np.array(kinds, np.uint8), d_in)
        codes = rng.integers(0, 16, (d_in, d_out)).astype(np.uint8)
        codes &= np.where(bits <= 4, (1 << np.minimum(bits, 4).astype(np.int32)) - 1, 0).astype(np.uint8)[:, None]
        counts = [int((bits == b).sum()) for b in bit_set]
        packed = [torch.full((c, b), -1, dtype=torch.int32, device=DEV) if c else None for b, c in zip(bit_set, counts)]
        chan = [torch.full((c,), -1, dtype=torch.int32, device=DEV) if c else None for c in counts]
        lut = [torch.empty((c, 1 << b), dtype=torch.float16, device=DEV) if c else None for b, c in zip(bit_set, counts)]
        cent = torch.zeros((d_in, 16), device=DEV)
        B.pack(torch.from_numpy(codes).to(DEV), torch.from_numpy(bits).to(DEV), cent, bit_set, counts, packed, chan, lut,
               B.Workspace(DEV))
        for b, c, p, ch in zip(bit_set, counts, packed, chan):
            rows = np.flatnonzero(bits == b)
            if c:
                assert np.array_equal(ch.cpu().numpy(), rows)
                want = ((codes[rows][:, :, None] >> np.arange(b)) & 1).reshape(c, -1)      # bit stream, least bit first
                got = (p.cpu().numpy().view(np.uint32)[:, :, None] >> np.arange(32, dtype=np.uint32) & 1).reshape(c, -1)
                assert np.array_equal(got, want)
