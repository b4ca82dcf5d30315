"""The K-means kernels that build, share and read per-channel tables, at the edges of their forms: counts
that do not fit the packed 32-bit word, buckets longer than one fetch of words, groups of channels that
end in the middle of a wavefront, scratch for a few channels only, tables of another row length."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def env():
    import oracle as orc
    from paper_2410_13056_amd import binding as B
    B.lib()
    return dict(B=B, orc=orc, ws=B.Workspace(DEV))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _np(t):
    return t.detach().cpu().numpy()


def _crowded(rng, d_in, d_out):
    """Rows whose weights share a bucket or a few: around 1, with the highest places alone, one value, zeros
    of both signs, a wide row beside them."""
    W = (1.0 + 0.06 * rng.random((d_in, d_out))).astype(np.float16)
    W[1 % d_in] = np.float16(1.0) + np.float16(2 ** -10) * (60 + rng.integers(0, 4, d_out))
    W[2 % d_in] = np.float16(-0.7)
    W[3 % d_in] = np.where(rng.random(d_out) < 0.5, 0.0, -0.0)
    W[4 % d_in] = rng.normal(0, 0.02, d_out)
    return W.astype(np.float16)


@pytest.mark.parametrize("d_out", [64, 1024, 4096, 4100, 8192, 28672, 32768])
@pytest.mark.parametrize("d_in", [1, 6])
def test_crowded_buckets_match_the_oracle(env, d_out, d_in):
    B, ws, orc = env["B"], env["ws"], env["orc"]
    rng = np.random.default_rng(d_out + d_in)
    W = _crowded(rng, d_in, d_out)
    bits = np.array([4, 4, 3, 2, 3, 16][:d_in], np.uint8)
    excl = np.sort(rng.choice(d_in * d_out, max(1, d_in * d_out // 50), replace=False)).astype(np.int32)
    dW, db, de = _dev(W), _dev(bits), _dev(excl)
    tables = torch.empty(B.arrangement_bytes(d_in, d_out), dtype=torch.uint8, device=DEV)
    cent = torch.empty((d_in, 16), dtype=torch.float32, device=DEV)
    codes = torch.empty((d_in, d_out), dtype=torch.uint8, device=DEV)
    B.kmeans_quantize(dW, db, None, 0, None, 6, cent, codes, ws, arrangement=tables, arrangement_use=B.ARRANGEMENT_KEEP)
    oc, ok = orc.kmeans(W, bits, iters=6)
    assert np.array_equal(_np(cent), oc) and np.array_equal(_np(codes), ok)
    oc, ok = orc.kmeans(W, bits, out_idx=excl.astype(np.int64), iters=6)
    for use in (B.ARRANGEMENT_NONE, B.ARRANGEMENT_REUSE):
        cent.fill_(7.0), codes.fill_(255)
        B.kmeans_quantize(dW, db, de, len(excl), None, 6, cent, codes, ws,
                          arrangement=tables if use else None, arrangement_use=use)
        assert np.array_equal(_np(cent), oc) and np.array_equal(_np(codes), ok)


class _Limited:
    """A workspace of a given size, whatever is asked for."""

    def __init__(self, nbytes):
        self.buf = torch.empty(nbytes, dtype=torch.uint8, device=DEV)

    def get(self, nbytes):
        return self.buf


@pytest.mark.parametrize("d_in,d_out,rooms", [(23, 1024, (0,)), (23, 4098, (0,)), (4200, 132, (0, 5, 2047, 2048, 2049, 4199)),
                                              (3090, 1031, (2049,)), (2300, 8192, (1, 2100))])
def test_scratch_for_a_part_of_the_channels_gives_the_same_bits(env, d_in, d_out, rooms):
    B, ws = env["B"], env["ws"]
    rng = np.random.default_rng(3)
    W = rng.normal(0, 0.02, (d_in, d_out)).astype(np.float16)
    bits = rng.choice(np.array([2, 3, 4, 16], np.uint8), d_in)
    excl = _dev(np.sort(rng.choice(d_in * d_out, d_in * d_out // 80, replace=False)).astype(np.int32))
    dW, db = _dev(W), _dev(bits)
    cent = torch.empty((d_in, 16), dtype=torch.float32, device=DEV)
    codes = torch.empty((d_in, d_out), dtype=torch.uint8, device=DEV)
    B.kmeans_quantize(dW, db, excl, excl.numel(), None, 21, cent, codes, ws)
    full = B.workspace_bytes(B.OP_KMEANS, d_in, d_out)
    one = (B.workspace_bytes(B.OP_KMEANS, 1 << 20, d_out) - B.workspace_bytes(B.OP_KMEANS, 1 << 19, d_out)) >> 19
    for channels in rooms:
        c2, k2 = torch.full_like(cent, 7.0), torch.full_like(codes, 255)
        room = max(full - (d_in - channels) * one + 512, B.workspace_bytes(B.OP_KMEANS, d_in, 0))
        B.kmeans_quantize(dW, db, excl, excl.numel(), None, 21, c2, k2, _Limited(room))
        assert torch.equal(c2, cent) and torch.equal(k2, codes)
    with pytest.raises(B.CmpqError):
        B.kmeans_quantize(dW, db, excl, excl.numel(), None, 21, cent, codes, _Limited(256))


@pytest.mark.parametrize("d_in,d_out", [(1, 4), (3100, 131), (3100, 132), (3080, 1028), (3080, 1999), (3300, 2052), (2800, 4095), (2050, 4099),
                                        (2049, 8192), (1030, 16384), (770, 28672), (800, 32768), (800, 32767)])
def test_the_least_scratch_gives_the_same_bits(env, d_in, d_out):
    """The size that holds for rows of any length (asked for without one): every form of the call, bit for bit what
    it leaves with room for the tables of all channels (too many to stay in LDS there)."""
    B, ws = env["B"], env["ws"]
    rng = np.random.default_rng(d_out)
    W = _crowded(rng, d_in, d_out)
    if d_in > 1:
        W[-1, -1] = np.inf
    bits = np.resize(np.array([4, 3, 2, 16, 1], np.uint8), d_in)
    n_out = d_in * d_out // 40
    excl = torch.randperm(d_in * d_out, device=DEV)[:n_out].sort().values.int() if n_out else None
    dW, db = _dev(W), _dev(bits)
    widths = [b for b in (1, 2, 3, 4) if b in bits]
    counts = [int((bits == b).sum()) for b in widths]
    sumsq = torch.ones(d_in, device=DEV)
    least = B.workspace_bytes(B.OP_KMEANS, d_in, 0)
    assert d_in == 1 or not B.kmeans_build_shape(d_in, d_out)[8]
    whole = d_out % 4 == 0

    def forms(space):
        out = []

        def run(n, codes, init, use, tables):
            cent = torch.linspace(-0.1, 0.1, 16, device=DEV).repeat(d_in, 1)
            st = torch.zeros(1, dtype=torch.int32, device=DEV)
            B.kmeans_quantize(dW, db, excl if n else None, n, None, 21, cent, codes, space(), st, init=init, arrangement=tables,
                              arrangement_use=use)
            out.extend([cent, st] + ([codes] if codes is not None else []))

        codes = lambda: torch.full((d_in, d_out), 255, dtype=torch.uint8, device=DEV)
        for n in {0, n_out}:
            for init in (B.INIT_QUANTILE, B.INIT_GIVEN):
                run(n, codes(), init, B.ARRANGEMENT_NONE, None)
        if whole:
            run(n_out, None, B.INIT_QUANTILE, B.ARRANGEMENT_NONE, None)
            tables = torch.zeros(B.arrangement_bytes(d_in, d_out), dtype=torch.uint8, device=DEV)
            run(0, None, B.INIT_QUANTILE, B.ARRANGEMENT_KEEP, tables)
            run(n_out, codes(), B.INIT_QUANTILE, B.ARRANGEMENT_REUSE, tables)
            tables.zero_()
            run(n_out, codes(), B.INIT_QUANTILE, B.ARRANGEMENT_REUSE, tables)
            assert out[-2].item() & B.STATUS_ARRANGEMENT and not out[-1].any()
        cent, k = torch.empty((d_in, 16), device=DEV), codes()
        packed = [torch.full((c, (d_out * b + 31) // 32), -1, dtype=torch.int32, device=DEV) for b, c in zip(widths, counts)]
        idx = [torch.full((c,), -1, dtype=torch.int32, device=DEV) for c in counts]
        lut = [torch.full((c, 1 << b), 7.0, dtype=torch.float16, device=DEV) for b, c in zip(widths, counts)]
        err, tot = torch.empty(d_in, dtype=torch.float64, device=DEV), torch.empty(2, dtype=torch.float64, device=DEV)
        B.kmeans_quantize_pack(dW, db, excl, n_out, 21, cent, k, widths, counts, packed, idx, lut, sumsq, err, tot, space())
        return out + [cent, k, *packed, *idx, *lut, err.view(torch.int64), tot.view(torch.int64)]

    for a, b in zip(forms(lambda: ws), forms(lambda: _Limited(least))):
        assert torch.equal(a, b)


def test_tables_of_another_row_length_are_flagged(env):
    B, ws = env["B"], env["ws"]
    rng = np.random.default_rng(5)
    W = rng.normal(0, 0.02, (3, 4096)).astype(np.float16)
    db = _dev(np.full(3, 3, np.uint8))
    tables = torch.zeros(B.arrangement_bytes(3, 4096), dtype=torch.uint8, device=DEV)
    cent = torch.empty((3, 16), dtype=torch.float32, device=DEV)
    B.kmeans_quantize(_dev(W), db, None, 0, None, 3, cent, None, ws, arrangement=tables, arrangement_use=B.ARRANGEMENT_KEEP)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    codes = torch.full((3, 2048), 9, dtype=torch.uint8, device=DEV)
    B.kmeans_quantize(_dev(W[:, :2048]), db, None, 0, None, 3, cent, codes, ws, st, arrangement=tables,
                      arrangement_use=B.ARRANGEMENT_REUSE)
    assert st.item() == B.STATUS_ARRANGEMENT and not codes.any() and not cent[:, :8].any()


@pytest.mark.parametrize("iters", [4, 24])
@pytest.mark.parametrize("d_out", [132, 1028, 1999, 2052, 4095, 4100, 8192])
def test_many_channels_get_the_bits_of_few(env, d_out, iters):
    """3300 channels in one call, and the same rows in two calls whose tables stay in LDS; few rounds and many."""
    B, ws = env["B"], env["ws"]
    g = torch.Generator(device=DEV).manual_seed(d_out)
    d_in = 3300
    assert [bool(B.kmeans_build_shape(n, d_out)[8]) for n in (d_in, 2048, d_in - 2048)] == [False, True, True]
    W = (torch.randn(d_in, d_out, generator=g, device=DEV) * 0.02).half()
    bits = torch.randint(1, 5, (d_in,), generator=g, device=DEV).to(torch.uint8)
    excl = torch.arange(0, d_in * d_out, 97, dtype=torch.int32, device=DEV)

    def run(lo, hi, out_idx, use, tables):
        cent = torch.full((hi - lo, 16), 7.0, device=DEV)
        codes = torch.full((hi - lo, d_out), 255, dtype=torch.uint8, device=DEV)
        B.kmeans_quantize(W[lo:hi], bits[lo:hi], out_idx, out_idx.numel() if out_idx is not None else 0, None, iters, cent, codes,
                          ws, arrangement=tables, arrangement_use=use)
        return cent, codes

    def both(lo, hi):
        e = excl[(excl >= lo * d_out) & (excl < hi * d_out)] - lo * d_out
        n = B.arrangement_bytes(hi - lo, d_out) if d_out % 4 == 0 else 0
        tables = torch.empty(n, dtype=torch.uint8, device=DEV) if n else None
        first = run(lo, hi, None, B.ARRANGEMENT_KEEP if n else B.ARRANGEMENT_NONE, tables)
        final = run(lo, hi, e, B.ARRANGEMENT_REUSE if n else B.ARRANGEMENT_NONE, tables)
        return first + final + run(lo, hi, e, B.ARRANGEMENT_NONE, None)

    whole, head, tail = both(0, d_in), both(0, 2048), both(2048, d_in)
    for w, h, t in zip(whole, head, tail):
        assert torch.equal(w, torch.cat([h, t]))


@pytest.mark.parametrize("d_out", [2053, 2068, 2101, 2304, 2541, 2543, 2544, 2548, 4095, 4099, 8191, 8196, 28671])
def test_counts_that_run_over_with_entries_removed(env, d_out):
    """Rows of one value with the highest place of its bucket, so that the bucket's sum of places leaves its part
    of the 32-bit word wherever it can; some entries are removed, and rows of no whole number of groups of 4 are
    filled up."""
    B, ws, orc = env["B"], env["ws"], env["orc"]
    rng = np.random.default_rng(d_out)
    d_in = 5
    W = np.empty((d_in, d_out), np.float16)
    W[0] = np.uint16(0x3C7F).view(np.float16)
    W[1] = -0.0
    W[2] = np.uint16(0xBC80).view(np.float16)  # of negative values the smallest magnitude has the highest place
    W[3] = np.where(rng.random(d_out) < 0.97, W[0], rng.normal(0, 0.02, d_out).astype(np.float16))
    W[4] = rng.normal(0, 0.02, d_out)
    far = rng.choice(d_out, 12, replace=False)
    W[:3, far] = np.float16(-7.5)              # few enough for the sum to run over, far enough to move the levels
    bits = np.array([2, 3, 4, 4, 1], np.uint8)
    excl = np.sort((np.arange(d_in)[:, None] * d_out + far[None, :9]).ravel()).astype(np.int32)
    dW, db, de = _dev(W), _dev(bits), _dev(excl)
    for out_idx in (None, de):
        cent = torch.full((d_in, 16), 7.0, device=DEV)
        codes = torch.full((d_in, d_out), 255, dtype=torch.uint8, device=DEV)
        B.kmeans_quantize(dW, db, out_idx, 0 if out_idx is None else len(excl), None, 6, cent, codes, ws)
        oc, ok = orc.kmeans(W, bits, out_idx=None if out_idx is None else excl.astype(np.int64), iters=6)
        assert np.array_equal(_np(cent), oc) and np.array_equal(_np(codes), ok)


def test_calls_without_tables_ask_for_no_room_for_them(env):
    """fp32 weights, importance weights and the direct algorithm run on kernels that keep no tables."""
    B = env["B"]

    class Asked(B.Workspace):
        def get(self, nbytes):
            self.asked = nbytes
            return super().get(nbytes)

    d_in, d_out = 3100, 1024
    W = torch.randn(d_in, d_out, device=DEV)
    bits = torch.full((d_in,), 2, dtype=torch.uint8, device=DEV)
    cent, codes = torch.empty((d_in, 16), device=DEV), torch.empty((d_in, d_out), dtype=torch.uint8, device=DEV)
    ws = Asked(DEV)

    def asked(Wx, **kw):
        B.kmeans_quantize(Wx, bits, None, 0, kw.pop("elem_weight", None), 2, cent, codes, ws, **kw)
        return ws.asked

    least, tables = B.workspace_bytes(B.OP_KMEANS, d_in, 0), B.workspace_bytes(B.OP_KMEANS, d_in, d_out)
    assert least < 64 * d_in < tables
    assert asked(W) == asked(W.half(), elem_weight=torch.ones_like(W)) == asked(W.half(), algorithm=B.KMEANS_DIRECT) == least
    assert asked(W.half()) == tables
    cent.copy_(torch.linspace(-1, 1, 16, device=DEV).repeat(d_in, 1))
    assert asked(W.half(), algorithm=B.KMEANS_DIRECT, init=B.INIT_GIVEN) == tables


def _level_pairs(rng, n):
    """Two different levels: neighbours of FP16 values, sums that meet an FP16 value exactly, subnormals, both sides
    of zero, means of a few weights, far outside FP16."""
    half = rng.integers(0, 0x7800, n).astype(np.uint16).view(np.float16).astype(np.float64) * rng.choice([-1.0, 1.0], n)
    step = np.spacing(half.astype(np.float16)).astype(np.float64)
    k = rng.integers(0, 8, n)
    lo = half.copy()
    hi = np.select([k == 0, k == 1, k == 2, k == 3, k == 4, k == 5, k == 6],
                   [half + step,                                                  # half way between neighbours
                    half + step * rng.integers(1, 40, n),                         # meets a value or the middle of two
                    half + step * rng.integers(1, 4000, n) / 1024,                # close together
                    -half * rng.integers(0, 5, n) / 4,                            # the other side of zero, or zero
                    rng.integers(-2000, 2000, n) * 2.0 ** -24 / rng.integers(1, 9, n),  # about the smallest values
                    half * rng.uniform(1.0, 3.0, n),
                    rng.normal(0, 1, n) * 10.0 ** rng.integers(-8, 8, n)], rng.normal(0, 3e5, n))
    lo = np.where(k == 4, rng.integers(-2000, 2000, n) * 2.0 ** -24 / rng.integers(1, 9, n), lo)
    lo, hi = lo.astype(np.float32), hi.astype(np.float32)
    hi = np.where(lo == hi, np.nextafter(hi, np.float32(np.inf), dtype=np.float32), hi)
    swap = rng.random(n) < 0.5                                                    # either may have the smaller index
    return np.where(swap, hi, lo), np.where(swap, lo, hi)


@pytest.mark.parametrize("d_in", [2048, 40000])
def test_boundaries_lie_at_the_exact_middle(env, d_in):
    """No rounds from two given levels: the codes of the FP16 values about their middle tell where the boundary lies.
    The reference compares 2 w with the levels' sum, exact in fp64 (pairs whose sum is not are left out)."""
    B, ws = env["B"], env["ws"]
    rng = np.random.default_rng(d_in)
    c0, c1 = _level_pairs(rng, d_in)
    a, b = c0.astype(np.float64), c1.astype(np.float64)
    total = a + b
    part = total - a
    exact = (a - (total - part)) + (b - part) == 0.0
    assert exact.mean() > 0.9
    mid = np.clip(total / 2, -65504, 65504).astype(np.float16).view(np.uint16).astype(np.int32)
    key = np.where(mid & 0x8000, 0x8000 - (mid & 0x7fff), 0x8000 + mid)           # value order
    near = np.clip(key[:, None] + np.arange(-12, 12)[None, :], 0x8000 - 0x7bff, 0x8000 + 0x7bff)
    near = np.where(near >= 0x8000, near - 0x8000, 0x8000 | (0x8000 - near)).astype(np.uint16)
    W = np.concatenate([near.view(np.float16), rng.normal(0, 1, (d_in, 4)).astype(np.float16),
                        np.tile(np.array([0.0, -0.0, 65504.0, -65504.0], np.float16), (d_in, 1))], axis=1)
    start = torch.full((d_in, 16), 9.0, device=DEV)
    start[:, 0], start[:, 1] = _dev(c0), _dev(c1)
    codes = torch.empty(W.shape, dtype=torch.uint8, device=DEV)
    B.kmeans_quantize(_dev(W), _dev(np.ones(d_in, np.uint8)), None, 0, None, 0, start, codes, ws, init=B.INIT_GIVEN)
    twice = 2.0 * W.astype(np.float64) - total[:, None]
    upper = np.where(b > a, 1, 0).astype(np.uint8)[:, None]                       # index of the larger level
    want = np.where(twice > 0, upper, np.where(twice < 0, 1 - upper, 0))
    got = _np(codes)
    assert np.array_equal(got[exact], want[exact])
    assert (twice[exact] == 0).any(1).mean() > 0.1                                # ties are among them
