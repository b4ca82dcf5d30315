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


@pytest.mark.parametrize("dtype,d_in,d_out,codes", [(np.float16, 512, 2048, False), (np.float16, 300, 1027, True),
                                                    (np.float32, 200, 1000, False)])
@pytest.mark.parametrize("far", [1.5, 3.0, 20.0, 1e4])
def test_selection_at_a_cliff(dtype, d_in, d_out, codes, far):
    """As many far weights as are asked for, a few more and a few less: the k-th key lies on the cliff
    or below it, `far` times the sampled guess (the list's histogram has fine bins up to twice the
    guess and coarse ones beyond); the far weights are spread over a binary octave or all but tied."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as orc
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_in)
    n = d_in * d_out
    n_far = n // 100
    W = rng.uniform(-0.02, 0.02, n)
    at = rng.choice(n, n_far, replace=False)
    for spread in (1.0, 0.001):
        W[at] = np.sign(W[at]) * 0.02 * far * (1 + spread * rng.random(n_far))
        Wt = W.astype(dtype).reshape(d_in, d_out)
        bits = np.full(d_in, 2, np.uint8)
        cent = np.full((d_in, 16), np.inf, np.float32)
        cent[:, :4] = [-0.01, 0.0, 0.01, 1e-3]
        code = np.abs(Wt[..., None].astype(np.float32) - cent[:, None, :4]).argmin(-1).astype(np.uint8) if codes else None
        Wd, cd, bd = (torch.from_numpy(x).to(DEV) for x in (Wt, cent, bits))
        kd = torch.from_numpy(code).to(DEV) if codes else None
        for k in (n_far - 50, n_far - n_far // 20, n_far, n_far + 7, n_far // 8):
            idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
            val = torch.zeros(k, dtype=torch.float16, device=DEV)
            B.extract_weight_outliers(Wd, cd, kd, bd, k, idx, val, ws)
            oidx, oval = orc.weight_outliers(Wt, cent, code, bits, k)
            assert np.array_equal(idx.cpu().numpy().astype(np.int64), oidx), (spread, k)
            assert np.array_equal(val.cpu().numpy().view(np.uint16), oval), (spread, k)


@pytest.mark.parametrize("d_in,d_out", [(512, 2048), (300, 1027)])
@pytest.mark.parametrize("step", [0.02 / 4, 0.02 / 16])
def test_selection_among_few_values(d_in, d_out, step):
    """Weights on a coarse grid: the k-th key is tied with many others and stands alone in its bin of
    the sample, above an empty one or beside its neighbour on the grid."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_out)
    W = (np.round(rng.normal(0, 0.02, (d_in, d_out)) / step) * step).astype(np.float16)
    bits = torch.full((d_in,), 3, dtype=torch.uint8, device=DEV)
    cent = torch.full((d_in, 16), float("inf"), device=DEV)
    cent[:, :8] = torch.linspace(-0.04, 0.04, 8, device=DEV)
    for score, key in ((B.SCORE_MAGNITUDE, np.abs(W.astype(np.float32))),
                       (B.SCORE_RESIDUAL, np.abs(W.astype(np.float32)[..., None] - cent[0, :8].cpu().numpy()).min(-1))):
        order = np.argsort(-key.ravel(), kind="stable")
        for k in (W.size // 2000, W.size // 200, W.size // 100, W.size // 20):
            idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
            val = torch.zeros(k, dtype=torch.float16, device=DEV)
            B.extract_weight_outliers(torch.from_numpy(W).to(DEV), cent, None, bits, k, idx, val, ws, score=score)
            want = np.sort(order[:k])
            assert np.array_equal(idx.cpu().numpy(), want), k
            assert np.array_equal(val.cpu().numpy(), W.ravel()[want]), k


@pytest.mark.parametrize("d_in,d_out", [(512, 2048), (300, 1027)])
def test_selection_among_bounded_scores(d_in, d_out):
    """Scores that end at a bound, inside the topmost bin of the sample, or thin out quickly above the
    k-th (weights drawn uniformly; clipped, so that many are tied at the bound)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as orc
    from paper_2410_13056_amd import binding as B
    ws = B.Workspace(DEV)
    rng = np.random.default_rng(d_out)
    bits = np.full(d_in, 3, np.uint8)
    for W in (rng.uniform(-0.02, 0.02, (d_in, d_out)), rng.normal(0, 0.02, (d_in, d_out)).clip(-0.05, 0.05)):
        W = W.astype(np.float16)
        cent = np.full((d_in, 16), np.inf, np.float32)
        cent[:, :8] = np.quantile(W.astype(np.float32), np.linspace(0.06, 0.94, 8), axis=1).T
        Wd, cd, bd = (torch.from_numpy(x).to(DEV) for x in (W, cent, bits))
        for k in (3, W.size // 2000, W.size // 200, W.size // 100, W.size // 20):
            idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
            val = torch.zeros(k, dtype=torch.float16, device=DEV)
            B.extract_weight_outliers(Wd, cd, None, bd, k, idx, val, ws)
            oidx, oval = orc.weight_outliers(W, cent, None, bits, k)
            assert np.array_equal(idx.cpu().numpy().astype(np.int64), oidx), k
            assert np.array_equal(val.cpu().numpy().view(np.uint16), oval), k
            B.extract_weight_outliers(Wd, cd, None, bd, k, idx, val, ws, score=B.SCORE_MAGNITUDE)
            want = np.sort(np.argsort(-np.abs(W.astype(np.float32)).ravel(), kind="stable")[:k])
            assert np.array_equal(idx.cpu().numpy(), want), k
