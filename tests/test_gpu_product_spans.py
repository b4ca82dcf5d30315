"""Products of 9 to 32 tokens around the lines up to which workgroups keep the inputs of their rows in LDS, and in
layers whose fullest workgroups have more rows than LDS could hold them of (tests/test_product_plan.py has the rule
itself on the host).

Bar: per output and token, the fp32 rounding of the sums - 2e-6 of the sum of the terms' magnitudes -
against the product in 64 bits with the weight rebuilt from W, levels, codes and outlier indices."""
import pytest
import torch

from test_gpu_deploy import DEV, env  # noqa: F401
from test_gpu_product_tokens import _check, _layer

pytestmark = pytest.mark.gpu


# the inputs of the fullest workgroup's rows would just fit into LDS (2064, 8528), are 1 step too many, 5 too many (one step
# is 32 rows); tokens times channels at the line and past it; thin layers of 15 and 17 steps, whose parts are cut otherwise,
# with as many outputs as their line and one more
@pytest.mark.parametrize("d_in,d_out,bit_set,avg,m", [
    (2064, 256, (2, 3), 2.75, 32), (4096, 512, (2, 3), 2.5, 32), (5696, 512, (2, 3), 2.5, 32),
    (5120, 640, (2, 3, 4), 2.75, 32), (8528, 256, (2, 3), 2.5, 16), (9824, 256, (2, 3), 2.8, 16),
    (2560, 1000, (2, 3), 2.5, 16), (2561, 1700, (2, 3), 2.5, 16), (1536, 300, (2, 3, 4), 3.0, 17),
    (440, 8200, (2, 3), 2.5, 16), (480, 8192, (2, 3), 2.5, 32), (440, 8192, (2, 3), 2.5, 32), (440, 8193, (2, 3), 2.5, 32)])
def test_inputs_of_full_workgroups(env, d_in, d_out, bit_set, avg, m):
    P, ws = env["P"], env["ws"]
    dep, What = _layer(env, d_in, d_in, d_out, bit_set, avg, 4500)
    wide, _ = _layer(env, d_out, d_in, 8500, bit_set, avg, 4500)      # too large for inputs straight from X
    X = torch.randn((m, d_in), generator=torch.Generator(device=DEV).manual_seed(m), device=DEV).to(torch.float16)
    Y = P.lut_matvec(dep, X, ws)
    _check(Y, X, What)
    for n in (m, m - 1, m // 2 + 1):
        Ys = [torch.full((n, d.d_out), float("nan"), device=DEV) for d in (wide, dep)]
        P.group_products([wide, dep])([X[:n], X[:n]], Ys, ws)
        assert torch.equal(Ys[1], P.lut_matvec(dep, X[:n], ws))
        _check(Ys[1], X[:n], What)


@pytest.mark.parametrize("b", [3, 4])
def test_rows_whose_product_with_the_parts_passes_32_bits(env, b):
    B, ws, n, d_out = env["B"], env["ws"], 900001, 8
    gen = torch.Generator(device=DEV).manual_seed(b)
    codes = torch.randint(0, 1 << b, (n, d_out), generator=gen, device=DEV)
    packed = (codes << (b * torch.arange(d_out, device=DEV))).sum(1, keepdim=True)
    packed = torch.where(packed >= 1 << 31, packed - (1 << 32), packed).to(torch.int32)
    lut = torch.randn((n, 1 << b), generator=gen, device=DEV).to(torch.float16)
    X = torch.randn((1, n), generator=gen, device=DEV).to(torch.float16)
    call = B.LutMatvecCall(n, d_out, (b,), [n], [packed], [torch.arange(n, dtype=torch.int32, device=DEV)], [lut],
                           None, None, None, None, None)
    Y = torch.full((1, d_out), float("nan"), device=DEV)
    call(X, Y, ws)
    _check(Y, X, lut.gather(1, codes).double())
