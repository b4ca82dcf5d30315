"""K-means on FP16 rows that are no whole number of groups of 4 weights or do not start on 8 bytes:
the histogram kernel against the general one (CMPQ_KMEANS_DIRECT takes such rows there), with the
stored format and the error asked for and without.

Bar: levels, codes and packed words identical (both sum exactly); fp64 errors within 1e-12, the
order of their additions."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    B.lib()
    return dict(B=B, ws=B.Workspace(DEV))


def _run(env, W, bits, out_idx, algorithm, format_too, status, start=None):
    B, ws = env["B"], env["ws"]
    d_in, d_out = W.shape
    cent = torch.zeros((d_in, 16), device=DEV) if start is None else start.clone()
    init = B.INIT_QUANTILE if start is None else B.INIT_GIVEN
    # codes inside a larger buffer: what lies around them has to stay
    around = torch.full((d_in * d_out + 64,), 99, dtype=torch.uint8, device=DEV)
    codes = around[33:33 + d_in * d_out].view(d_in, d_out)
    n_out = int(out_idx.numel())
    if not format_too:
        B.kmeans_quantize(W, bits, out_idx, n_out, None, 7, cent, codes, ws, status, init=init, algorithm=algorithm)
        assert bool((around[:33] == 99).all()) and bool((around[33 + d_in * d_out:] == 99).all())
        return [cent, codes]
    bit_set = (1, 2, 3, 4)
    counts = [int((bits == b).sum()) for b in bit_set]
    packed = [torch.full((c, (d_out * b + 31) // 32), -1, dtype=torch.int32, device=DEV) for b, c in zip(bit_set, counts)]
    chan = [torch.empty(c, dtype=torch.int32, device=DEV) for c in counts]
    lut = [torch.empty((c, 1 << b), dtype=torch.float16, device=DEV) for b, c in zip(bit_set, counts)]
    err_ch, err = torch.empty(d_in, dtype=torch.float64, device=DEV), torch.empty(2, dtype=torch.float64, device=DEV)
    sumsq = torch.rand(d_in, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    B.kmeans_quantize_pack(W, bits, out_idx, n_out, 7, cent, codes, bit_set, counts, packed, chan, lut, sumsq, err_ch,
                           err, ws, status, init=init, algorithm=algorithm)
    assert bool((around[:33] == 99).all()) and bool((around[33 + d_in * d_out:] == 99).all())
    return [cent, codes, *packed, *chan, *lut, err_ch, err]


# lengths around a group, a lane's share and each launch shape; rows that start on 2 bytes
@pytest.mark.parametrize("d_out", [1, 2, 3, 5, 30, 31, 257, 511, 1026, 2049, 4099, 8191, 8194, 16387, 28671, 32767])
@pytest.mark.parametrize("offset", [0, 1])
def test_ragged_rows_against_the_general_kernel(env, d_out, offset):
    B = env["B"]
    rng = np.random.default_rng(d_out)
    d_in = 9
    wide = rng.normal(0, 0.02, (d_in, d_out + 3)).astype(np.float16)
    wide[rng.random(wide.shape) < 0.02] *= np.float16(20)
    wide[rng.random(wide.shape) < 0.05] = 0
    wide[rng.random(wide.shape) < 0.02] = np.float16(-0.0)
    W = torch.from_numpy(wide).to(DEV)[:, offset:offset + d_out]
    if offset == 0:
        W = W.contiguous()
    bits = torch.tensor([1, 2, 3, 4, 16, 4, 3, 2, 4], dtype=torch.uint8, device=DEV)
    live = np.flatnonzero(np.repeat(bits.cpu().numpy() != 16, d_out))
    some = np.sort(rng.choice(live, len(live) // 50, replace=False))
    last = [i * d_out + d_out - 1 for i in (0, 3) if d_out > 1]          # the last weight of a row among them
    out_idx = torch.tensor(np.union1d(some, last).astype(np.int32), device=DEV)
    start = torch.randn((d_in, 16), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV) * 0.03
    for idx in (out_idx, out_idx[:0]):
        for first in (None, start):
            st = torch.zeros(2, dtype=torch.int32, device=DEV)
            for fmt in (False, True):
                a = _run(env, W, bits, idx, B.KMEANS_HISTOGRAM, fmt, st[:1], first)
                b = _run(env, W, bits, idx, B.KMEANS_DIRECT, fmt, st[1:], first)
                for x, y in zip(a, b):
                    if x.dtype == torch.float64:
                        assert torch.allclose(x, y, rtol=1e-12, atol=0)
                    else:
                        assert torch.equal(x, y)
            assert not st.any()


def test_ragged_rows_flag_nonfinite_weights_and_keep_their_refusals(env):
    B, ws = env["B"], env["ws"]
    W = torch.randn((4, 37), device=DEV).to(torch.float16)
    W[2, 36] = float("inf")
    bits = torch.full((4,), 3, dtype=torch.uint8, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    cent, codes = _run(env, W, bits, torch.empty(0, dtype=torch.int32, device=DEV), B.KMEANS_HISTOGRAM, False, st)
    assert st.item() == B.STATUS_NONFINITE and int(codes.max()) < 8
    with pytest.raises(B.CmpqError):                                     # no codes: only for aligned groups of 4
        B.kmeans_quantize(W, bits, None, 0, None, 3, cent, None, ws)
    assert B.arrangement_bytes(4, 37) == 0
