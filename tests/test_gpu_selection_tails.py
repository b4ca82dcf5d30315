"""O_q selection where the list's histogram ends: the k-th key far above the guess read off the
sample (then the passes over the whole layer answer), on it, and below it; rows of any length and
alignment; against the oracle's sort, entry by entry."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("dtype,d_in,d_out,skip", [
    (np.float16, 1536, 8193, 0), (np.float16, 1536, 8200, 1), (np.float16, 64, 515, 3), (np.float32, 700, 4099, 1)])
def test_selection_around_the_guess(dtype, d_in, d_out, skip):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as orc
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_in + d_out)
    W = rng.normal(0, 0.02, (d_in, d_out)).astype(dtype)
    W.flat[rng.integers(0, W.size, 40)] = dtype(30.0)            # tied, far above four times any guess
    W.flat[rng.integers(0, W.size, 5)] = dtype(-60000.0)
    bits = rng.integers(2, 5, d_in).astype(np.uint8)
    bits[[0, d_in - 1]] = 16
    cent = np.full((d_in, 16), np.inf, np.float32)
    for i in range(d_in):
        if bits[i] <= 4:
            cent[i, :1 << bits[i]] = np.sort(rng.normal(0, 0.02, 1 << bits[i])).astype(np.float32)
    raw = torch.empty(W.size + skip, dtype=torch.from_numpy(W).dtype, device=DEV)
    Wd = raw[skip:].view(d_in, d_out)                            # skip: the base off its 16-byte line
    Wd.copy_(torch.from_numpy(W))
    cd, bd = torch.from_numpy(cent).to(DEV), torch.from_numpy(bits).to(DEV)
    live = int((bits <= 4).sum()) * d_out
    for k in (1, 4, 20, 44, 300, live // 100, live // 3):
        idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
        val = torch.zeros(k, dtype=torch.float16, device=DEV)
        B.extract_weight_outliers(Wd, cd, None, bd, k, idx, val, ws)
        oidx, oval = orc.weight_outliers(W, cent, None, bits, k)
        assert np.array_equal(idx.cpu().numpy().astype(np.int64), oidx), k
        assert np.array_equal(val.cpu().numpy().view(np.uint16), oval), k


@pytest.mark.parametrize("score", ["magnitude", "residual"])
@pytest.mark.parametrize("share_nan", [1.0, 0.97, 0.6, 0.3])
def test_selection_among_nans(score, share_nan):
    """A guess that falls among NaN keys: every entry asked for comes, NaNs of larger pattern first
    (the residual without codes ranks a NaN weight as infinity)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(0)
    d_in, d_out = 64, 515
    h = (0x7c01 + rng.integers(0, 1023, (d_in, d_out))).astype(np.uint16)     # NaNs of many patterns
    h ^= (rng.integers(0, 2, h.shape) << 15).astype(np.uint16)
    plain = rng.random(h.shape) >= share_nan
    h[plain] = rng.normal(0, 1, int(plain.sum())).astype(np.float16).view(np.uint16)
    W = torch.from_numpy(h.view(np.float16)).to(DEV)
    bits = torch.full((d_in,), 3, dtype=torch.uint8, device=DEV)
    cent = torch.full((d_in, 16), float("inf"), device=DEV)
    cent[:, :8] = 0.0                                                          # the residual is the magnitude
    a = (h & 0x7fff).astype(np.int64).ravel()
    key = np.where(a > 0x7c00, (a | 0x200) if score == "magnitude" else 0x7c00, a)   # order of the keys
    for k in (20, int(0.3 * a.size), int(0.5 * a.size), int(0.6 * a.size), int(0.8 * a.size), a.size):
        idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
        val = torch.zeros(k, dtype=torch.float16, device=DEV)
        B.extract_weight_outliers(W, cent, None, bits, k, idx, val, ws,
                                  score=B.SCORE_MAGNITUDE if score == "magnitude" else B.SCORE_RESIDUAL)
        want = np.sort(np.argsort(-key, kind="stable")[:k])
        assert np.array_equal(idx.cpu().numpy(), want), k
        taken = h.ravel()[want]
        exact = (taken & 0x7fff) <= 0x7c00
        assert np.array_equal(val.cpu().numpy().view(np.uint16)[exact], taken[exact]), k
