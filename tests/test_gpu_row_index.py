"""The rows that channels get in the stored format, and the slices that an ascending list of entries is cut into, a
channel each, at the sizes where their counting steps from wavefront to wavefront, from one pass of 1024 channels to
the next and (slices: 256 to a workgroup) from workgroup to workgroup, against a plain count."""
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


@pytest.mark.parametrize("d_in", [1, 2, 254, 255, 256, 257, 511, 512, 513, 1023, 1024, 3000])
def test_entries_of_each_channel(d_in):
    """Every entry counts in the error of its own channel: entries in the first and the last channel, in some between,
    in none, in all, and (rows of another length) one a workgroup's worth of channels apart."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    rng = np.random.default_rng(d_in)
    bit_set, d_out = (2, 3), 44
    bits = rng.choice(np.array(bit_set, np.uint8), d_in)
    codes = (rng.integers(0, 8, (d_in, d_out)) & ((1 << bits) - 1)[:, None]).astype(np.uint8)
    cent = np.full((d_in, 16), np.inf, np.float32)
    cent[:, :8] = rng.integers(-64, 65, (d_in, 8)) / 64.0
    cent[bits == 2, 4:] = np.inf
    W = (rng.integers(-64, 65, (d_in, d_out)) / 64.0).astype(np.float16)
    counts = [int((bits == b).sum()) for b in bit_set]
    off = (W.astype(np.float64) - np.take_along_axis(cent, codes.astype(np.int64), 1)) ** 2       # exact in 64 bits
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    dW, dk, db, dc, ws = dev(W), dev(codes), dev(bits), dev(cent), B.Workspace(DEV)
    sumsq = torch.ones(d_in, device=DEV)
    first, last = np.arange(3), np.arange(3) + (d_in - 1) * d_out + 5
    some = np.flatnonzero(rng.random(d_in * d_out) < 0.05)
    for lin in (first, last, np.union1d(first, last), some, np.arange(d_in * d_out), np.arange(0, d_in * d_out, 256 * d_out),
                np.arange(min(d_in * d_out, 255 * d_out + 1))):
        packed = [torch.empty((c, -(-d_out * b // 32)), dtype=torch.int32, device=DEV) if c else None
                  for b, c in zip(bit_set, counts)]
        chan = [torch.empty(c, dtype=torch.int32, device=DEV) if c else None for c in counts]
        lut = [torch.empty((c, 1 << b), dtype=torch.float16, device=DEV) if c else None for b, c in zip(bit_set, counts)]
        err, total = torch.full((d_in,), -1.0, dtype=torch.float64, device=DEV), torch.empty(2, dtype=torch.float64, device=DEV)
        B.pack_with_error(dW, dk, db, dc, bit_set, counts, packed, chan, lut, dev(lin.astype(np.int32)), len(lin), sumsq, err,
                          total, ws)
        want = off.copy()
        want.ravel()[lin] = 0.0                              # kept in FP16, as W is
        assert np.array_equal(err.cpu().numpy(), want.sum(1))
        for c, ch, b in zip(counts, chan, bit_set):
            assert c == 0 or np.array_equal(ch.cpu().numpy(), np.flatnonzero(bits == b))
