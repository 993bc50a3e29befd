"""Host check of the register exchanges of the one-wave-per-row and 4-residue
column passes (no GPU): the exchanges of register bits with lane bits put, in
every round, the points into the registers that the round's butterflies take
(base + k 2^sh), from the layout the pass is entered with to the one it leaves,
and back for the inverse; only the first column exchange crosses waves."""
import pytest


def lane_swap(x, lb, pairs):
    """x[wave][lane][reg]: registers a, b of each pair with lane bit lb."""
    for w in x:
        old = [list(r) for r in w]
        for lane in range(64):
            for a, b in pairs:
                p = lane ^ (1 << lb)
                if lane >> lb & 1:
                    w[lane][a] = old[p][b]
                else:
                    w[lane][b] = old[p][a]


def exchange(x, lb):
    lane_swap(x, lb + 1, [(0, 2), (1, 3)])
    lane_swap(x, lb, [(0, 1), (2, 3)])


def rename(x):
    for w in x:
        for r in w:
            r[1], r[2] = r[2], r[1]


def points(log1, sh, waves):
    """[wave][lane] -> the four (point, column) of a round with shift sh (-1: 4t + k)."""
    c_log = 10 - log1 if waves == 4 else 0
    out = []
    for w in range(waves):
        rows = []
        for lane in range(64):
            tid = 64 * w + lane
            c, t = tid & ((1 << c_log) - 1), tid >> c_log
            if sh < 0:
                base, step = 4 * t, 1
            else:
                base, step = ((t >> sh) << (sh + 2)) | (t & ((1 << sh) - 1)), 1 << sh
            rows.append([(base + k * step, c) for k in range(4)])
        out.append(rows)
    return out


def test_row_pass():
    x = points(8, 6, 1)
    for sh, lb in ((4, 4), (2, 2), (0, 0)):
        exchange(x, lb)
        assert x == points(8, sh, 1)
    for sh, lb in ((2, 0), (4, 2), (6, 4)):
        exchange(x, lb)
        assert x == points(8, sh, 1)


@pytest.mark.parametrize("log1", [5, 6, 7, 8])
def test_column_pass(log1):
    n4, odd = log1 // 2, log1 & 1
    shs = [log1 - 2 - 2 * j for j in range(n4)] + ([-1] if odd else [])
    x = points(log1, shs[1], 4)  # after the exchange through LDS
    for j in range(2, len(shs)):
        if shs[j] >= 0:
            exchange(x, 4 if j == 2 else 2)
        else:
            lane_swap(x, 5 if log1 == 5 else 3, [(0, 2), (1, 3)])
            rename(x)
        assert x == points(log1, shs[j], 4)
    for j in range(len(shs) - 1, 1, -1):
        if shs[j] >= 0:
            exchange(x, 4 if j == 2 else 2)
        else:
            rename(x)
            lane_swap(x, 5 if log1 == 5 else 3, [(0, 2), (1, 3)])
        assert x == points(log1, shs[j - 1], 4)
