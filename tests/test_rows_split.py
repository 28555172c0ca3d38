"""How the rows of more than 8192 columns are cut into shares (csrc/cada_rows_split.h), on the host: every row belongs to
exactly one share, the sums of every pair (share, worker) have a slot of their own inside the buffer, and k_rows_sum finds a worker's."""
import pytest

from common_split import SHARED_WORKERS, compile_split


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    return compile_split(tmp_path_factory.mktemp("split"))


SHAPES = [(M, B, p) for p in (8193, 14336, 14337, 20480) for M, B in
          [(1, 1), (1, 2), (1, 4096), (2, 4095), (3, 33), (37, 75), (64, 64), (65, 1), (100, 100), (100, 256), (129, 13), (255, 3), (256, 1),
           (257, 1), (257, 5), (300, 4096), (600, 2), (1000, 7), (5000, 1)]]


@pytest.mark.parametrize("M,B,p", SHAPES)
def test_shares_cover_the_rows(split, M, B, p):
    w = split(M, B, p)
    assert 1 <= w.rows <= 2048 and w.shares >= 1
    assert w.per == 0 or w.shares == M * w.per
    first = [w.first(c) for c in range(w.shares + 1)]
    assert first[0] == 0 and first[-1] == M * B
    taken = {}
    for c in range(w.shares):
        f0, f1 = first[c], first[c + 1]
        assert 1 <= f1 - f0 <= w.rows
        assert w.share(f0) == c == w.share(f1 - 1)
        assert w.per == 0 or f0 // B == (f1 - 1) // B
        for m in range(f0 // B, (f1 - 1) // B + 1):
            slot = w.slot(c, m)
            assert 0 <= slot < w.slots and slot not in taken
            taken[slot] = (c, m)
    for m in range(M):           # a worker's slots follow each other from its first share on
        c0, c1 = w.share(m * B), w.share((m + 1) * B - 1)
        assert [taken[w.slot(c0, m) + i] for i in range(c1 - c0 + 1)] == [(c, m) for c in range(c0, c1 + 1)]


@pytest.mark.parametrize("p,M,B,rule", SHARED_WORKERS)
def test_shapes_whose_shares_meet_several_workers(split, p, M, B, rule):
    """The shapes that test_gpu_logreg_rows.py runs for it: cut evenly, with shares of more than one worker, and ends of a
    worker's rows inside a share after an odd as well as an even number of batches."""
    w = split(M, B, p)
    assert w.per == 0
    batch = 1 if p > 12288 else 2            # rows that k_rows_wide works on together
    pieces = set()
    for c in range(w.shares):
        f, f1 = w.first(c), w.first(c + 1)
        while f // B < (f1 - 1) // B:        # the rows of all workers but the share's last
            n = (f // B + 1) * B - f
            pieces.add((n + batch - 1) // batch % 2)
            f += n
    assert 1 in pieces and (0 in pieces or B < 2 * batch)


@pytest.mark.parametrize("M,B,p,low,high", [(16, 64, 20479, 8, 12), (4, 64, 20479, 12, 24), (64, 16, 20479, 2, 4), (16, 16, 20479, 4, 6), (37, 75, 20001, 6, 6),
                                            (1, 1024, 20479, 32, 32)])
def test_shares_per_worker_near_the_best_measured(split, M, B, p, low, high):
    """Counts within 4 % of the best of 1, 2, 4, 6, 8, 12, 16, 24, 32 shares per worker on the hardware."""
    assert low <= split(M, B, p).per <= high
