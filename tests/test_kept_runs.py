"""What the choice among kept K-means runs refuses, with the codes and without (no GPU needed: both look before they
call the library)."""
import pytest
import torch

from paper_2410_13056_amd import binding as B

D_IN, D_OUT = 6, 40


def _runs():
    return [torch.zeros(D_IN, 16) for _ in range(2)], [torch.zeros(D_IN, D_OUT, dtype=torch.uint8) for _ in range(2)]


@pytest.mark.parametrize("spoil", [
    lambda c, k: k.__setitem__(1, torch.zeros(D_IN, D_OUT + 1, dtype=torch.uint8)),
    lambda c, k: k.__setitem__(0, torch.zeros(D_IN - 1, D_OUT, dtype=torch.uint8)),
    lambda c, k: k.__setitem__(0, torch.zeros(D_IN, D_OUT, dtype=torch.int8)),
    lambda c, k: k.__setitem__(1, torch.zeros(D_OUT, D_IN, dtype=torch.uint8).t()),
    lambda c, k: c.__setitem__(0, torch.zeros(D_IN, 15)),
    lambda c, k: c.__setitem__(1, torch.zeros(D_IN, 16, dtype=torch.float64)),
    lambda c, k: c.__setitem__(1, torch.zeros(16, D_IN).t())])
def test_kept_runs_of_another_shape_or_type_are_refused(spoil):
    bits, out = torch.full((D_IN,), 2, dtype=torch.uint8), torch.zeros(D_IN, 16)
    cents, codes = _runs()
    spoil(cents, codes)
    with pytest.raises(ValueError, match="kept runs"):
        B.select_by_width(bits, (2, 3), cents, codes, out, torch.zeros(D_IN, D_OUT, dtype=torch.uint8))
    with pytest.raises(ValueError, match="kept runs"):
        B.select_levels_by_width(bits, (2, 3), cents, codes, out, D_OUT)
