"""The product with one token (cmpq_lut_matvec_group, m = 1, and few tokens of short inputs) at the sizes
where its parts, pairs of rows and tiles of outputs begin and end, through the C ABI.

Bar: per output and token, the fp32 rounding of the sums - 2e-6 of the sum of the terms' magnitudes -
against the product in 64 bits with the weight rebuilt from W, levels, codes and outlier indices."""
import pytest
import torch

from test_gpu_deploy import DEV, env  # noqa: F401
from test_gpu_product_tokens import _check, _layer

pytestmark = pytest.mark.gpu


# channels: one row, part of a group of rows, a whole one and one more, odd pairs, more than a wavefront's
# rows; outputs: one, a lane's 32, a tile of 2048, its neighbours; every width; no outliers of either kind
@pytest.mark.parametrize("bit_set,avg", [((1, 2), 1.5), ((2, 3), 2.4), ((3, 4), 3.5), ((1, 2, 3, 4), 2.6)])
@pytest.mark.parametrize("d_in,d_out,act,oq", [(1, 33, 0, 0), (7, 1, 0, 20000), (9, 32, 0, 10000), (17, 2047, 60000, 10000),
                                               (33, 2049, 0, 0), (130, 2048, 20000, 5000), (517, 4100, 10000, 10000)])
def test_one_token_at_the_edges_of_parts(env, bit_set, avg, d_in, d_out, act, oq):
    P, ws = env["P"], env["ws"]
    dep, What = _layer(env, d_in + d_out, d_in, d_out, bit_set, avg, act, oq)
    gen = torch.Generator(device=DEV).manual_seed(d_in)
    X = torch.randn((3, d_in), generator=gen, device=DEV).to(torch.float16)
    X[1, ::3] *= 1e-6                                        # subnormal in FP16
    for m in (1, 3):
        Y = P.lut_matvec(dep, X[:m], ws)
        _check(Y, X[:m], What)
        assert torch.equal(Y, P.lut_matvec(dep, X[:m], ws))


def test_one_token_layers_of_all_sizes_in_one_group(env):
    """Layers with many parts, few, and none of some widths, and one without any row: each as alone."""
    P, B, ws = env["P"], env["B"], env["ws"]
    layers = [_layer(env, 20 + i, *s, (2, 3, 4), avg, 10000, 10000)
              for i, (s, avg) in enumerate([((3000, 5000), 3.5), ((40, 9), 2.0), ((2100, 2048), 4.0), ((700, 70), 2.7)])]
    calls = [d.call() for d, _ in layers]
    d0 = layers[1][0]
    calls.insert(2, B.LutMatvecCall(d0.d_in, d0.d_out, d0.bit_set, [0, 0, 0], [None] * 3, [None] * 3, [None] * 3, None, None,
                                    None, None, None))
    gen = torch.Generator(device=DEV).manual_seed(5)
    Xs = [torch.randn((1, c.d_in), generator=gen, device=DEV).to(torch.float16) for c in calls]
    Ys = [torch.full((1, c.d_out), float("nan"), device=DEV) for c in calls]
    B.LutMatvecGroupCall(calls)(Xs, Ys, ws)
    assert not Ys[2].any()
    for i, (dep, What) in enumerate(layers):
        j = i + (i >= 2)
        _check(Ys[j], Xs[j], What)
        assert torch.equal(Ys[j], P.lut_matvec(dep, Xs[j], ws))


def test_infinite_levels_and_inputs_stay_where_they_are(env):
    """A level of infinity (FP16 tables overflow) in the last row of a part, next to rows that are not there,
    makes the outputs that use it infinite and leaves the others finite."""
    P, ws = env["P"], env["ws"]
    dep, _ = _layer(env, 9, 45, 300, (3, 4), 3.5, 0, 0)
    X = torch.ones((1, 45), dtype=torch.float16, device=DEV)
    ref = P.lut_matvec(dep, X, ws)
    for j, rows in enumerate(dep.counts):
        if rows:
            dep.lut[j][rows - 1, 0] = float("inf")
    Y = P.lut_matvec(dep, X, ws)
    assert not Y.isnan().any() and Y.isinf().any() and Y.isfinite().any()
    assert torch.equal(Y[Y.isfinite()], ref[Y.isfinite()])
