"""How far the product with one token at a time is from 64 bits, against what the order of its sums gives.

Model: an addition in fp32 is off by 2^-23 * 0.2124 of its result in the root mean square (uniform in a last place that
is 2^-23 to 2^-24 of a result spread evenly over its logarithm), independently of the others, and a sum of n of the
products, which have random signs, is the square root of n in size.  The order: the parts of the plan row by
row (width 4) or pair by pair, four parts of a workgroup in pairs, then the workgroups in 16 runs, eight at a time, and
the runs in pairs."""
import math

import pytest
import torch

from test_gpu_deploy import DEV, env  # noqa: F401
from test_gpu_product_tokens import _layer

pytestmark = pytest.mark.gpu


def _pairs(sizes):
    """(size of the sum, squared sizes of all results) of adding up in pairs; a zero costs nothing."""
    cost = 0
    while len(sizes) > 1:
        sums = [sum(sizes[i:i + 2]) for i in range(0, len(sizes), 2)]
        cost += sum(s for s, i in zip(sums, range(0, len(sizes), 2)) if 0 < sizes[i] < s)
        sizes = sums
    return sizes[0], cost


def _model(parts, rows):
    cost, slabs = 0, []
    for k in range(0, len(parts), 4):
        for width, _, n in parts[k:k + 4]:
            step = 1 if width == 4 else 2
            cost += (step - 1) * n + sum(min(i, n) for i in range(2 * step, n + step, step))
        size, c = _pairs([n for _, _, n in parts[k:k + 4]])
        slabs.append(size)
        cost += c
    per, runs = -(-len(slabs) // 16), []
    for r in range(0, 16 * per, per):
        total = 0
        for e in range(r, r + per, 8):
            size, c = _pairs(slabs[e:min(e + 8, r + per)] or [0])
            cost += c + (total + size if total and size else 0)
            total += size
        runs.append(total)
    cost += _pairs(runs)[1]
    return 2.0 ** -23 * 0.2124 * math.sqrt(cost / rows)


@pytest.mark.parametrize("d_in,d_out,m,bit_set,avg", [(1000, 1000, 16, (3, 4), 3.5), (506, 700, 9, (1, 2), 1.62),
                                                      (900, 2100, 4, (2, 3), 2.5), (5000, 2100, 1, (3, 4), 3.5)])
def test_error_is_that_of_the_order_of_the_sums(env, d_in, d_out, m, bit_set, avg):
    P, B, ws = env["P"], env["B"], env["ws"]
    dep, What = _layer(env, d_in, d_in, d_out, bit_set, avg, 0, 0)
    (way, _, _, n, _, _), parts = B.lut_matvec_shape(d_in, d_out, bit_set, dep.counts, 0, m)
    assert way == 0 and n == len(parts)
    gen = torch.Generator(device=DEV).manual_seed(d_out)
    off = size = 0.0
    for _ in range(max(1, 32 // m)):
        X = torch.randn((m, d_in), generator=gen, device=DEV).to(torch.float16)
        ref = X.double() @ What
        off += float(((P.lut_matvec(dep, X, ws).double() - ref) ** 2).sum())
        size += float((ref ** 2).sum())
    got, want = math.sqrt(off / size), _model(parts, d_in)
    # (the products differ in size, and 32 tokens sample the mean to some 2 %)
    assert got <= 1.08 * want
