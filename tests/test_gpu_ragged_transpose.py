"""The orientation copy and the statistics at the edges of their pieces: rows of any length and alignment, bit
for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 5), (4, 7), (63, 65), (64, 66), (129, 67), (257, 1031), (1030, 259),
                                       (40, 70001), (3331, 3363)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_orientation_of_any_rows(rows, cols, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_13056_amd import binding as B
    bits = torch.int16 if dtype == torch.float16 else torch.int32
    gen = torch.Generator(device=DEV).manual_seed(rows)
    for off in (0, 1, 2, 3):
        wide = torch.randint(-30000, 30000, (rows, cols + 5), dtype=bits, generator=gen, device=DEV)
        src = wide[:, off:off + cols]
        around = torch.full((cols, rows + 7), 77, dtype=bits, device=DEV)
        B.transpose(src.view(dtype), around[:, 3 - off:3 - off + rows].view(dtype))
        assert torch.equal(around[:, 3 - off:3 - off + rows], src.t())
        assert bool((around[:, :3 - off] == 77).all()) and bool((around[:, 3 - off + rows:] == 77).all())


@pytest.mark.parametrize("n,d_in", [(1, 3), (15, 1), (16, 257), (17, 5), (33, 301), (1031, 999)])
def test_statistics_of_any_rows(n, d_in):
    """Sums of squares of small whole numbers, which no order of adding changes."""
    from paper_2410_13056_amd import binding as B, pipeline as P
    gen = torch.Generator(device=DEV).manual_seed(n)
    wide = torch.randint(-40, 40, (n, d_in + 2), generator=gen, device=DEV).to(torch.float16)
    X = wide[:, 1:d_in + 1]
    acc, sumsq = P.activation_stats(X, B.Workspace(DEV))
    want = (X.double() ** 2).sum(0)
    assert torch.equal(acc, want) and torch.equal(sumsq, want.float())
