"""How rows are cut into shares and which shapes take that path (csrc/cada_rows_split.h), on the host: every row belongs to
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


@pytest.mark.parametrize("p", [4, 54, 257, 1024, 1025, 4096, 4097, 8192])
def test_shares_of_narrow_rows(split, p):
    for M in (1, 2, 3, 31, 32, 33, 64, 255, 256, 257, 1000, 65535):
        for B in (1, 9, 10, 11, 23, 24, 25, 64, 100, 255, 4095, 4096):
            shares, rows = split.narrow(M, B, p)
            assert 1 <= shares <= 8 and (shares - 1) * rows < B <= shares * rows
            assert shares == 1 or M * shares <= 256
            # offsets and labels, then the sums: what the kernel asks for of the 150 KB of LDS it is allowed
            assert (rows + 3) // 4 * 4 * 12 + (8 if p <= 1024 else 1) * 2 * ((p + 3) // 4 * 4) * 4 <= 150 * 1024


@pytest.mark.parametrize("p,M,B,vec,rows", [
    (784, 256, 1, 4, True), (784, 257, 31, 4, False), (784, 257, 32, 4, True), (1024, 300, 8, 4, False), (1025, 300, 8, 1, True),
    (3000, 512, 1, 4, True), (3000, 513, 7, 4, False), (3000, 513, 8, 4, True),
    (4096, 1, 64, 4, True), (4100, 1, 64, 4, False), (4100, 4, 10, 4, True), (4100, 4, 11, 4, False), (6000, 12, 65, 4, True), (6000, 8, 65, 4, False),
    (8191, 1, 128, 1, True), (8191, 1, 129, 1, False), (8191, 2, 256, 1, True), (8191, 2, 257, 1, False), (8192, 1, 4096, 4, True),
    (8196, 512, 1, 4, True), (8196, 513, 15, 4, False), (8196, 513, 16, 4, True), (8197, 4096, 1, 1, True)])
def test_route(split, p, M, B, vec, rows):
    assert split.preferred(M, B, p, vec) == rows


@pytest.mark.parametrize("M,B,p,low,high", [(16, 64, 20479, 8, 12), (4, 64, 20479, 12, 24), (64, 16, 20479, 2, 4), (16, 16, 20479, 4, 6), (37, 75, 20001, 6, 6),
                                            (1, 1024, 20479, 32, 32)])
def test_shares_per_worker_near_the_best_measured(split, M, B, p, low, high):
    """Counts within 4 % of the best of 1, 2, 4, 6, 8, 12, 16, 24, 32 shares per worker on the hardware."""
    assert low <= split(M, B, p).per <= high
