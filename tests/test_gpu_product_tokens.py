"""The product with several tokens (cmpq_lut_matvec with m > 1 on the matrix cores) at the sizes
where its tiles, steps and token groups begin and end, through the C ABI.

Bar: per output and token, the fp32 rounding of the sums - 2e-6 of the sum of the terms'
magnitudes, as for the single-token product - against the product in 64 bits with the weight
rebuilt from W, levels, codes and outlier indices."""
import numpy as np
import pytest
import torch

from test_gpu_deploy import DEV, _dev, _np, _what, env  # noqa: F401

pytestmark = pytest.mark.gpu


def _layer(env, seed, d_in, d_out, bit_set, avg, rho_act=20000, rho_q=10000):
    P, ws = env["P"], env["ws"]
    rng = np.random.default_rng(seed)
    W = rng.normal(0, 0.02, (d_in, d_out)).astype(np.float16)
    far = rng.random(W.shape) < 0.01
    W[far] *= np.float16(12)
    sumsq = rng.lognormal(0, 1, d_in).astype(np.float32)
    r = P.quantize_layer(_dev(W), _dev(sumsq), bit_set, avg, rho_act, rho_q, 3, ws, transposed=True)
    What = _what(W, _np(r.centroids), _np(r.codes), _np(r.bits), _np(r.out_idx).astype(np.int64))
    return P.prepare_deployment(r, ws), _dev(np.asarray(What, dtype=np.float64))


def _check(Y, X, What):
    ref = X.double() @ What
    bar = 2e-6 * (X.double().abs() @ What.abs()) + 1e-30
    assert bool(((Y.double() - ref).abs() <= bar).all())


# channels: one step, a step and one row, many; outputs: one, a tile of 256 and its neighbours,
# unaligned rows; every width; no outliers of either kind
LAYERS = [(32, 1, (2, 3), 2.5, 0, 0), (33, 16, (1, 2, 3, 4), 2.5, 30000, 20000), (31, 257, (3, 4), 3.5, 0, 10000),
          (200, 255, (1, 2), 1.5, 20000, 0), (300, 256, (2, 3, 4), 3.0, 20000, 10000),
          (1000, 513, (2, 3, 4), 3.3, 10000, 10000), (1300, 2056, (2, 3, 4), 2.4, 10000, 5000)]


@pytest.mark.parametrize("m", [2, 4, 5, 8, 9, 16, 17, 32, 33, 70])
def test_tokens_at_the_edges_of_tiles(env, m):
    P, B, ws = env["P"], env["B"], env["ws"]
    gen = torch.Generator(device=DEV).manual_seed(m)
    layers = [_layer(env, 10 + i, *spec) for i, spec in enumerate(LAYERS)]
    deps = [d for d, _ in layers]
    Xs = [torch.randn((m, d.d_in), generator=gen, device=DEV).to(torch.float16) for d in deps]
    Ys = [torch.full((m, d.d_out), float("nan"), device=DEV) for d in deps]
    P.group_products(deps)(Xs, Ys, ws)                       # also: layers of both ways in one call
    for (dep, What), X, Y in zip(layers, Xs, Ys):
        _check(Y, X, What)
        assert torch.equal(Y, P.lut_matvec(dep, X, ws))      # a layer's bits do not depend on its group
    # rows of X and Y inside wider arrays, unaligned
    dep, What = layers[5]
    X, Y = torch.zeros((m, dep.d_in + 3), dtype=torch.float16, device=DEV), torch.zeros((m, dep.d_out + 5), device=DEV)
    X[:, 1:dep.d_in + 1] = Xs[5]
    dep.matvec_into(X[:, 1:dep.d_in + 1], Y[:, 3:dep.d_out + 3], ws)
    assert torch.equal(Y[:, 3:dep.d_out + 3], Ys[5]) and not Y[:, :3].any() and not Y[:, dep.d_out + 3:].any()


@pytest.mark.parametrize("m,d_in,d_out", [(513, 4100, 4099), (520, 2048, 8200), (1100, 1500, 6000)])
def test_many_tokens_decoded_once(env, m, d_in, d_out):
    """Sizes at which the weight is decoded into memory first: partial tiles of outputs and tokens,
    every entry of O_q put in its place, inputs and levels down to subnormals."""
    dep, What = _layer(env, m, d_in, d_out, (2, 3, 4), 3.1, 10000, 10000)
    gen = torch.Generator(device=DEV).manual_seed(m)
    X = torch.randn((m, d_in), generator=gen, device=DEV)
    X[:, ::7] *= 1e-6                                        # subnormal in FP16
    X = X.to(torch.float16)
    Y = env["P"].lut_matvec(dep, X, env["ws"])
    _check(Y, X, What)
    assert torch.equal(Y, env["P"].lut_matvec(dep, X, env["ws"]))


def test_a_workspace_for_single_tokens_only_still_serves(env):
    """The scratch that the token-by-token launch needs, less than cmpq_workspace_bytes asks for, is
    accepted as before; one byte less is refused."""
    B = env["B"]
    dep, What = _layer(env, 3, 96, 64, (2, 3), 2.5)
    X = torch.randn((3, 96), device=DEV).to(torch.float16)
    slabs = sum(-(-c // 32) for c in dep.counts) + -(-int(dep.act_idx.numel()) // 32)
    need = -(-3 * slabs * 64 * 4 // 256) * 256
    assert need < B.workspace_bytes(B.OP_LUT_MATVEC, 96, 64, 3)
    call, buf = dep.call(), torch.empty(need, dtype=torch.uint8, device=DEV)
    for size, rc in ((need, 0), (need - 1, -5)):
        Y = torch.zeros((3, 64), device=DEV)
        assert call._fn(X.data_ptr(), 3, 96, 96, *call._head, Y.data_ptr(), 64, buf.data_ptr(), size, B._stream()) == rc
        torch.cuda.synchronize()
        if rc == 0:
            _check(Y, X, What)


@pytest.mark.parametrize("d_in,m,wide", [(959, 8, 2050), (960, 8, 2050), (500, 8, 8380), (500, 8, 8400),
                                         (1820, 9, 2050), (1821, 9, 2050), (1023, 16, 2050), (1024, 16, 2050),
                                         (1445, 17, 2050), (1446, 17, 2050), (511, 48, 2050), (512, 48, 2050),
                                         (64, 384, 2050)])
def test_both_sides_of_the_lines_to_the_matrix_cores(env, d_in, m, wide):
    """Layers of one input, narrow and wide, at the lines from which tokens are multiplied together: right
    on both sides, in a group as alone, and up to 8 tokens the same however many come together."""
    P, ws = env["P"], env["ws"]
    layers = [_layer(env, d_in + o, d_in, o, (2, 3, 4), 3.0) for o in (1, 40, 257, wide)]
    deps = [d for d, _ in layers]
    X = torch.randn((m, d_in), generator=torch.Generator(device=DEV).manual_seed(m), device=DEV).to(torch.float16)
    Ys = [torch.full((m, d.d_out), float("nan"), device=DEV) for d in deps]
    P.group_products(deps)([X] * len(deps), Ys, ws)
    for (dep, What), Y in zip(layers, Ys):
        _check(Y, X, What)
        assert torch.equal(Y, P.lut_matvec(dep, X, ws))
        if m <= 8 and d_in >= 960:
            assert torch.equal(Y[:2], P.lut_matvec(dep, X[:2], ws))


@pytest.mark.parametrize("m", [95, 96, 520])
def test_layers_of_every_plan_in_one_group(env, m):
    """One call with layers that are decoded once (two of them; one without entries of O_q, one without
    outliers of either kind), one too small for that, one that is not stored whole and one that goes token
    by token: each right, and the same as alone.  95 and 96 tokens: the line to decoding once (from 96
    tokens and 8 * 2^30 products on; the wide layer passes it at 96)."""
    P, B, ws = env["P"], env["B"], env["ws"]
    wide = (8192, 11008) if m < 520 else (4096, 4100)
    specs = [(*wide, 10000, 10000), (*wide, 10000, 0), (4096, 4360, 0, 0), (1000, 700, 10000, 10000),
             (4096, 4099, 20000, 5000), (40, 33, 30000, 10000)]
    layers = [_layer(env, 70 + i, d_in, d_out, (2, 3, 4), 3.1, a, q) for i, (d_in, d_out, a, q) in enumerate(specs)]
    gen = torch.Generator(device=DEV).manual_seed(m)
    Xs = [torch.randn((m, d.d_in), generator=gen, device=DEV).to(torch.float16) for d, _ in layers]
    part = layers[4][0]
    Xs[4][:, part.act_idx.long()] = 0                             # the rows of O_act that the call leaves out
    calls = [d.call() for d, _ in layers]
    calls[4] = B.LutMatvecCall(part.d_in, part.d_out, part.bit_set, part.counts, part.packed, part.chan_idx, part.lut,
                               None, None, part.colptr, part.row_idx, part.delta)
    Ys = [torch.full((m, d.d_out), float("nan"), device=DEV) for d, _ in layers]
    B.LutMatvecGroupCall(calls)(Xs, Ys, ws)
    for call, (_, What), X, Y in zip(calls, layers, Xs, Ys):
        _check(Y, X, What)
        alone = torch.empty_like(Y)
        call(X, alone, ws)
        assert torch.equal(Y, alone)


@pytest.mark.parametrize("m,d_in,d_out", [(3, 1000, 300), (20, 1300, 513), (40, 2048, 700), (513, 4100, 4099)])
def test_infinities_and_nans_stay_with_their_token(env, m, d_in, d_out):
    """An infinity or NaN in one token's inputs reaches all its outputs (no weight of the layer is zero
    for certain, so: none of them is finite where the 64-bit product is not) and no other token's."""
    dep, What = _layer(env, d_in, d_in, d_out, (2, 3, 4), 3.1, 10000, 10000)
    gen = torch.Generator(device=DEV).manual_seed(m)
    X = torch.randn((m, d_in), generator=gen, device=DEV).to(torch.float16)
    bad = X.clone()
    bad[m // 2, d_in // 3], bad[m - 1, d_in - 1] = float("inf"), float("nan")
    Y, Z = env["P"].lut_matvec(dep, X, env["ws"]), env["P"].lut_matvec(dep, bad, env["ws"])
    rows = torch.ones(m, dtype=torch.bool, device=DEV)
    rows[[m // 2, m - 1]] = False
    assert torch.equal(Y[rows], Z[rows])
    ref = bad[~rows].double() @ What
    assert not Z[~rows][~torch.isfinite(ref)].isfinite().any()
    _check(Y, X, What)
