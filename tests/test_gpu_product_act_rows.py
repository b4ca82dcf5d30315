"""The rows of O_act in the product with the deployed weight, at row lengths where the last tile of outputs ends
inside a lane's eight outputs, for rows at any even address, through the C ABI.

Bar: per output and token, the fp32 rounding of the sums - 2e-6 of the sum of the terms' magnitudes -
against the product in 64 bits with the weight rebuilt from W, levels, codes and outlier indices."""
import pytest
import torch

from test_gpu_deploy import DEV, env  # noqa: F401
from test_gpu_product_tokens import _check, _layer

pytestmark = pytest.mark.gpu


# 39 rows of O_act, the last one alone in its pair; 1 token token by token, 4 and 20 on the matrix cores
@pytest.mark.parametrize("d_out", [1, 7, 8, 13, 40, 250, 256, 263, 2047, 2052, 2304])
@pytest.mark.parametrize("m", [1, 4, 20])
def test_rows_of_any_length_and_address(env, m, d_out):
    P, B, ws = env["P"], env["B"], env["ws"]
    dep, What = _layer(env, d_out, 1300, d_out, (2, 3), 2.4, 30000, 5000)
    assert dep.act_idx.numel() == 39
    X = torch.randn((m, 1300), generator=torch.Generator(device=DEV).manual_seed(m), device=DEV).to(torch.float16)
    Y = P.lut_matvec(dep, X, ws)
    _check(Y, X, What)
    # the same rows further apart, from an odd element on, infinities between them and behind the last
    for ld, first in ((d_out + 3, 1), (-(-d_out // 8) * 8, 0)):
        room = torch.full((first + 39 * ld + 8,), float("inf"), dtype=torch.float16, device=DEV)
        rows = room[first:first + 39 * ld].view(39, ld)[:, :d_out]
        rows.copy_(dep.W_act)
        call = B.LutMatvecCall(dep.d_in, d_out, dep.bit_set, dep.counts, dep.packed, dep.chan_idx, dep.lut, dep.act_idx,
                               rows, dep.colptr, dep.row_idx, dep.delta)
        Z = torch.full_like(Y, float("nan"))
        call(X, Z, ws)
        assert torch.equal(Y, Z)
        rows[38, d_out // 2] = float("inf")                  # an infinite weight stays with its output
        call(X, Z, ws)
        there = torch.arange(d_out, device=DEV) != d_out // 2
        assert torch.equal(Y[:, there], Z[:, there])
        assert torch.equal(Z[:, d_out // 2], torch.sign(X[:, dep.act_idx[38].long()]).float() * float("inf"))
