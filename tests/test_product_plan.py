"""How the product with the deployed weight cuts up a layer (`cmpq_lut_matvec_shape`), on the host: for any
sizes and counts per width what a launch assumes of its parts has to hold before it is launched."""
import random

from paper_2410_13056_amd import binding as B


def _widths(d_in, bit_set, avg, k_act):
    """Channels per width that average `avg`, of two neighbouring widths."""
    n, lo = d_in - k_act, max(b for b in bit_set if b <= avg)
    hi = int(avg * n + 1e-9) - lo * n
    return [hi if b == lo + 1 else (n - hi if b == lo else 0) for b in bit_set]


def _layers(seed, n):
    """Sizes and counts: the widths of a bit budget, and counts that a caller chose freely."""
    rng = random.Random(seed)
    for d_in, d_out, m, bit_set, avg in [(5696, 512, 32, (2, 3), 2.5), (5056, 512, 32, (2, 3), 2.8),
                                         (5120, 640, 32, (2, 3, 4), 2.75), (9824, 256, 16, (2, 3), 2.8),
                                         (4096, 1024, 32, (2, 3), 2.5), (4096, 512, 32, (2, 3), 2.5)]:
        k_act = B.count_ppm(4500, d_in)
        yield d_in, d_out, m, bit_set, _widths(d_in, bit_set, avg, k_act), k_act
    for _ in range(n):
        d_in, d_out = int(2 ** rng.uniform(5, 15)), int(2 ** rng.uniform(0, 14))
        m, k_act = rng.randint(2, 32), rng.choice([0, d_in // 200, d_in // 20])
        if rng.random() < 0.5:
            bit_set = rng.choice([(1, 2), (2, 3), (2, 3, 4), (3, 4)])
            yield d_in, d_out, m, bit_set, _widths(d_in, bit_set, rng.uniform(bit_set[0], bit_set[-1]), k_act), k_act
        else:
            cuts = sorted(rng.randint(0, d_in - k_act) for _ in range(3))
            yield d_in, d_out, m, (1, 2, 3, 4), [b - a for a, b in zip([0] + cuts, cuts + [d_in - k_act])], k_act


def test_inputs_of_the_fullest_workgroup_fit_into_lds():
    """Up to 32 tokens a workgroup may keep the inputs of all its rows in LDS: a row of 16-bit inputs a token, 8
    more between tokens, behind the tables of levels.  Its rows are those of four neighbouring parts, and parts
    are of even cost, not of even length."""
    taken = {4: 0, 8: 0, 16: 0, 32: 0}
    for d_in, d_out, m, bit_set, counts, k_act in _layers(1, 12000):
        (way, _, groups, n, used, there), parts = B.lut_matvec_shape(d_in, d_out, bit_set, counts, k_act, m)
        if way != 1 or not used:
            continue
        tokens = next(t for t in taken if m <= t)
        steps = [-(-rows // 32) for _, _, rows in parts]
        assert groups == -(-n // 4)
        most = max(sum(steps[i:i + 4]) for i in range(0, n, 4))
        assert tokens * (32 * most + 8) * 2 == used <= there, (d_in, d_out, m, bit_set, counts, k_act, most)
        taken[tokens] += 1
    assert min(taken.values()) > 50, taken                      # (the rule still takes layers)


def test_parts_cover_every_row_once():
    """For one token and for several: the parts of a width follow each other without gap or overlap, none is longer
    than the sums of one wavefront may run, and their partial results fit the workspace.  Up to row counts at which
    rows times parts leaves 32 bits."""
    large = [(n, 8, m, (1, 2, 3, 4), counts, 0) for n in (741441, 800000, 8000000) for m in (1, 2)
             for counts in ([0, 0, 0, n], [0, 0, n, 0], [0, n, 0, 0], [n // 2, 0, 0, n // 2])]
    some = list(_layers(2, 400))
    for d_in, d_out, m, bit_set, counts, k_act in large + some + [(*c[:2], 1, *c[3:]) for c in some]:
        case = (d_in, d_out, m, bit_set, counts, k_act)
        (way, tokens, groups, n, _, _), parts = B.lut_matvec_shape(*case[:2], bit_set, counts, k_act, m)
        assert way < 2 and tokens == m and groups == -(-n // 4), case
        assert groups * m * d_out * 4 <= B.workspace_bytes(B.OP_LUT_MATVEC, d_in, d_out, m), case
        most = {b: 256 if way else (64 if b <= 4 else 8) for b in (1, 2, 3, 4, 16)}
        left = dict(zip(bit_set, counts))
        left[16] = k_act
        at = dict.fromkeys(left, 0)
        for width, row, rows in parts:
            assert row == at[width] and 0 < rows <= most[width], (case, width, row, rows)
            at[width] += rows
        assert at == left, case


def test_parts_of_few_tokens_are_short():
    """Up to 8 tokens a part of width 3 or 4 has at most 4 steps of 32 rows, or as few more as the workspace takes, though
    fewer workgroups than the chip has places for would do: long parts are chains of latencies."""
    for d_in, d_out, most in [(4096, 11008, 4), (5248, 10496, 4), (8192, 10240, 6), (7936, 10821, 6), (5535, 12608, 5)]:
        for m in (2, 4, 5, 8):
            k_act = B.count_ppm(4500, d_in)
            _, parts = B.lut_matvec_shape(d_in, d_out, (3, 4), _widths(d_in, (3, 4), 3.3, k_act), k_act, m)
            assert max(rows for width, _, rows in parts if width <= 4) <= 32 * most, (d_in, d_out, m)
