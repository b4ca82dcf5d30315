"""A new average width from kept runs where only the levels are taken from them (large layers): the same results, bit
for bit, as with the kept codes."""
import numpy as np
import pytest
import torch

from test_gpu_retarget import DEV, _np, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,d_out,bit_set", [(300, 1024, (2, 3, 4)), (96, 4104, (1, 2)), (65, 516, (3, 4))])
def test_levels_alone_give_the_results_of_levels_and_codes(env, monkeypatch, d_in, d_out, bit_set):
    P, B, ws = env["P"], env["B"], env["ws"]
    rng = np.random.default_rng(d_out)
    W = torch.from_numpy((rng.standard_t(4, size=(d_in, d_out)) * 0.02).astype(np.float16)).to(DEV)
    sumsq = torch.from_numpy(rng.lognormal(0, 1, d_in).astype(np.float32)).to(DEV)
    cache = P.build_width_cache(W, bit_set, 6, ws, transposed=True)
    for avg, rho_q, score in [(bit_set[0] + 0.4, 5000, B.SCORE_RESIDUAL), (bit_set[0] + 1.0, 20000, B.SCORE_RESIDUAL),
                              (bit_set[-1] - 0.3, 0, B.SCORE_RESIDUAL), (bit_set[0] + 0.7, 5000, B.SCORE_MAGNITUDE)]:
        both = []
        for line in (0, 1 << 40):
            monkeypatch.setattr(P, "LEVELS_ONLY", line)
            both.append(P.quantize_layer_from_cache(cache, sumsq, avg, 10000, rho_q, ws, score=score, with_error=True))
        a, b = both
        assert a.counts == b.counts
        for x, y in zip([a.bits, a.act_idx, a.out_idx, a.out_val, a.centroids, a.codes, a.err_ch, a.err_total, *a.packed],
                        [b.bits, b.act_idx, b.out_idx, b.out_val, b.centroids, b.codes, b.err_ch, b.err_total, *b.packed]):
            assert (x is None) == (y is None) and (x is None or np.array_equal(_np(x), _np(y)))
