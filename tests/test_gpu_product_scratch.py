"""The workspace of products: what cmpq_workspace_bytes asks for is enough and nothing outside it is
written, for every plan (multiplying while decoding, in one go and in parts; decoding once; token by
token; FP16 sums in parts), and a smaller one still serves where it did.

Bar: products as in test_gpu_product_tokens (2e-6 of the sum of the terms' magnitudes against 64
bits); everything that may not depend on the workspace is compared bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_deploy import DEV, env  # noqa: F401
from test_gpu_product_tokens import _check, _layer

pytestmark = pytest.mark.gpu

GUARD = 4096


class _Buffer:
    """Stands in for a Workspace: exactly `size` bytes (or what is asked for), a guard behind them."""

    def __init__(self, size=None):
        self.size = size

    def get(self, need):
        n = need if self.size is None else self.size
        self.raw = torch.full((n + GUARD,), 0xa5, dtype=torch.uint8, device=DEV)
        self.n = n
        return self.raw[:n]

    def untouched(self):
        return bool((self.raw[self.n:] == 0xa5).all())


def _x(m, d_in, seed):
    return torch.randn((m, d_in), generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(torch.float16)


def _without_act(env, dep):
    """The layer with the rows of O_act left out: not every channel is stored."""
    from paper_2410_13056_amd import binding as B
    return B.LutMatvecCall(dep.d_in, dep.d_out, dep.bit_set, dep.counts, dep.packed, dep.chan_idx, dep.lut, None, None,
                           dep.colptr, dep.row_idx, dep.delta)


@pytest.mark.parametrize("d_in,d_out,m", [(96, 64, 2), (33, 17, 9), (1000, 513, 24), (2048, 2048, 33), (700, 4099, 8),
                                          (2048, 4200, 97), (1500, 6000, 960), (1500, 6000, 1100), (64, 40, 700)])
def test_the_workspace_asked_for_is_enough_and_kept_to(env, d_in, d_out, m):
    P = env["P"]
    dep, What = _layer(env, m, d_in, d_out, (2, 3, 4), 3.0)
    X, Y = _x(m, d_in, m), torch.full((m, d_out), float("nan"), device=DEV)
    buf = _Buffer()
    dep.call()(X, Y, buf)
    _check(Y, X, What)
    assert buf.untouched()
    # FP16 sums in the same workspace, and one token at a time: the same numbers
    half = P.group_products([dep], fp16acc=True)
    Ya, Yb = torch.empty_like(Y), torch.empty_like(Y)
    half([X], [Ya], buf)
    assert buf.untouched()
    half([X], [Yb], _Buffer(1 << 30))
    assert torch.equal(Ya, Yb)
    # a layer whose rows of O_act are not there: never decoded once, in parts where the tokens are many
    part = _without_act(env, dep)
    X[:, dep.act_idx.long()] = 0
    Y.fill_(float("nan"))
    part(X, Y, buf)
    _check(Y, X, What)
    assert buf.untouched()


def test_a_few_tokens_run_together_in_the_workspace_of_old(env):
    """The rows per slab and token that were asked for before tokens were multiplied together hold the
    plan for a few tokens: the same bits as with ample room, and not those of one token at a time."""
    dep, What = _layer(env, 5, 2048, 4096, (2, 3, 4), 3.0)
    for m in (4, 16):
        X = _x(m, 2048, m)
        Ys = [torch.empty((m, 4096), device=DEV) for _ in range(3)]
        dep.call()(X, Ys[0], _Buffer(1 << 30))
        dep.call()(X, Ys[1], _Buffer(m * (2048 // 32 + 6) * 4096 * 4))
        for t in range(m):
            dep.call()(X[t:t + 1], Ys[2][t:t + 1], _Buffer())
        assert torch.equal(Ys[0], Ys[1]) and not torch.equal(Ys[0], Ys[2])
        _check(Ys[0], X, What)


def test_a_short_workspace_changes_no_layer_for_its_group(env):
    """Less than is asked for, but enough for the token-by-token launch: the layers whose plan does not
    fit go that way, each as in a call of its own with the same workspace; too little for either launch is
    refused."""
    P, B = env["P"], env["B"]
    layers = [_layer(env, 40 + i, *s, (2, 3, 4), 3.0) for i, s in enumerate([(96, 64), (2048, 1024), (1000, 300)])]
    deps = [d for d, _ in layers]
    group = P.group_products(deps)
    m = 3
    rows = lambda d: sum(-(-c // 32) for c in d.counts) + -(-int(d.act_idx.numel()) // 32)
    least = sum(-(-m * rows(d) * d.d_out * 4 // 256) * 256 for d in deps)
    Xs = [_x(m, d.d_in, i) for i, d in enumerate(deps)]
    for size in (least, least + 4096, 1 << 20, 1 << 30):
        Ys = [torch.full((m, d.d_out), float("nan"), device=DEV) for d in deps]
        buf = _Buffer(size)
        group(Xs, Ys, buf)
        assert buf.untouched()
        for (dep, What), X, Y in zip(layers, Xs, Ys):
            _check(Y, X, What)
            alone = torch.empty_like(Y)
            dep.call()(X, alone, _Buffer(size))
            assert torch.equal(Y, alone), size
    with pytest.raises(B.CmpqError):
        group(Xs, Ys, _Buffer(1 << 14))
    # FP16 sums: one token's rows are the least
    half = P.group_products(deps[:1], fp16acc=True)
    one = -(-rows(deps[0]) * 64 * 4 // 256) * 256
    half(Xs[:1], Ys[:1], _Buffer(one))
    with pytest.raises(B.CmpqError):
        half(Xs[:1], Ys[:1], _Buffer(one - 256))
