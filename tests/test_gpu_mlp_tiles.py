"""The MLP's contraction kernels at the edges of their tiles, through the C ABI against the fp64 oracle: a worker's rows cut into
steps of 16 and 32 (one row, a whole step, one more, more than a row tile), matrices that end inside a tile, just past one, and at no multiple of the
8 values that leave in one access; fewer steps than the operand ring holds, and more weight-gradient tiles than the 512 workgroups."""
import numpy as np
import pytest

from cada_synth import configs, generators

from common import check_protocol, to_dev, upload, run_library, oracle_run, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [          # layer sizes, workers, rows per worker
    ((33, 40, 5), 1, 1),
    ((65, 33, 40, 3), 2, 16),
    ((130, 135, 36, 4), 3, 17),
    ((129, 257, 130, 6), 2, 129),
    ((600, 140, 33, 4), 48, 48),
    ((48, 700, 45, 4), 60, 31),
]
# 5 x 3 x 64 = 960 tiles in the first layer, ragged on both sides: workgroups go on to a second tile after one step of 16 rows, two, three and five (the
# loads of up to three of a tile's steps have landed before the last tile's way out)
MANY_TILES = [((601, 301, 35, 4), 64, B) for B in (12, 20, 40, 70)]
RULES = {"cada1": configs.RULE_CADA1, "cada2": configs.RULE_CADA2, "always": configs.RULE_ALWAYS}


def _config(shape, rule):
    dims, M, B = shape
    return configs.CFG5.scaled(name="tiles", layer_dims=dims, M=M, N_m=max(B, 40), B=B, K=5, D=3, c=20.0, rule=RULES[rule])


@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("shape", SHAPES + MANY_TILES, ids=lambda s: "-".join(map(str, s[0])) + "_M%d_B%d" % s[1:])
def test_gradients_and_left_hand_sides(shape, rule):
    cfg = _config(shape, rule)
    prob = generators.make_problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    # Step 0: the stored gradients are the fresh ones.  Split bf16 operands carry 2^-16 per product, three products to a sum, two to four
    # contractions in a row: 4 x 3 x 2^-16 = 1.8e-4 of a worker's block if nothing averaged out.  A pre-activation within 2^-16 of zero may fall on
    # either side: one (unit, sample) pair in 2^16, so in few of the workers, whose gradient then lacks a term of one of its B samples or has
    # one too many (an eighth would be one of the 64 largest terms; a block in a wrong place differs by its whole norm).
    o, _ = oracle_run(cfg, prob, sched[:1])
    out = run_library(cfg, dev, sched[:1])
    assert out["error_flags"][0] == 0
    off = 0
    for a, b in zip(cfg.layer_dims, cfg.layer_dims[1:]):
        for n in (a * b, b):
            got, want = out["stored"][:, off:off + n], np.asarray(o.G)[:, off:off + n]
            errs = [rel_l2(got[m], want[m]) for m in range(cfg.M)]
            assert np.median(errs) < 1.8e-4 and max(errs) < 0.125, (a, b, n)
            off += n
    # later steps: innovations against stored ones (CADA1) and per-worker reference points (CADA2).  Differences are single bf16 products
    # (2^-8 on their norm, so 2^-7 on the squared norm, where a unit's sign is the same on both sides)
    stats, o, tr, rep = check_protocol(cfg, prob, dev, sched, 2e-2, lhs_rtol=None, own_mask_exact=False, free_margin=None)
    # The always-upload rule records the left-hand side of stored gradients.  In no worker may the bulk be off: a unit on the other side of zero in one sample
    # moves it by up to some 1 / 32 (one sample of few), a tile or an edge that is left out, counted twice or another worker's by its share in most of the steps.
    big = tr["lhs"] > 1e-9 * tr["lhs"].max()
    rel = np.abs(rep["trace_lhs"] - tr["lhs"]) / np.maximum(tr["lhs"], 1e-300)
    assert float(np.median(rel[big])) < 2.0 ** -7 and float(np.quantile(rel[big], 0.99)) < 0.2
    assert all(float(np.median(rel[big[:, m], m])) < 0.05 for m in range(cfg.M) if big[:, m].any())
    assert stats["own_disagreements"] <= max(2, 0.03 * tr["mask"].size)


def _exact_network(dims, rows, rng):
    """Small integers (times powers of two) throughout: every activation and logit is exact in any order of summation.  Row 0 of X is zero, and no
    hidden unit is active there."""
    X = rng.integers(0, 4, size=(rows + 1, dims[0])).astype(np.float32)
    X[0] = 0.0
    theta = []
    for l, (a, b) in enumerate(zip(dims, dims[1:])):
        theta.append(rng.integers(-2, 3, size=a * b) * 2.0 ** (-2 - l))
        theta.append(np.full(b, -0.5 if l + 2 < len(dims) else 0.0))
    return X, rng.integers(0, dims[-1], size=rows + 1).astype(np.int32), np.concatenate(theta).astype(np.float32)


@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("shape", SHAPES + MANY_TILES, ids=lambda s: "-".join(map(str, s[0])) + "_M%d_B%d" % s[1:])
def test_every_column_of_every_workers_gradients(shape, rule):
    """Where no unit can fall on the other side of zero (pre-activations are exact), the bound above holds for every worker, and in it for every unit's
    column and bias (relative to the column, or to the block's average column where that is larger)."""
    dims, M, B = shape
    cfg = _config(shape, rule)
    X, y, theta = _exact_network(dims, M * cfg.N_m, np.random.default_rng(7))
    prob = generators.make_problem(cfg)
    prob.X, prob.y, prob.theta0 = X[1:], y[1:], theta
    sched = generators.make_schedule(cfg)[:1]
    o, _ = oracle_run(cfg, prob, sched)
    out = run_library(cfg, upload(prob), sched)
    assert out["error_flags"][0] == 0
    off = 0
    for a, b in zip(dims, dims[1:]):
        for rows in (a, 1):                      # the weights, the biases
            got, want = (np.asarray(v)[:, off:off + rows * b].reshape(M, rows, b) for v in (out["stored"], o.G))
            norm = np.linalg.norm(want, axis=1)
            scale = np.maximum(norm, np.sqrt((norm ** 2).mean(axis=1, keepdims=True)))
            err = np.linalg.norm(got - want, axis=1) / scale
            assert scale.min() > 0 and err.max() < 1.8e-4, (a, b, rows, err.max(), np.argwhere(err >= 1.8e-4)[:5].tolist())
            off += rows * b


# 1200 to 1300 forward blocks of 32 x 32: row blocks that are a multiple of eight and not, rows that fit an XCD's L2 and do not
@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("shape", [((100, 130, 5), 40, 200), ((100, 130, 5), 36, 200), ((100, 130, 5), 37, 200), ((700, 65, 10), 40, 320)], ids=lambda s: "-".join(map(str, s[0])) + "_M%d_B%d" % s[1:])
def test_forward_blocks_in_and_past_the_l2(shape, rule):
    test_every_column_of_every_workers_gradients(shape, rule)


@pytest.mark.parametrize("rule", ["cada2", "always"])
@pytest.mark.parametrize("dims", [(24, 45, 7), (24, 20, 5), (24, 150, 40, 5)], ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("B", [7, 33, 64, 100, 192, 224, 300, 513])
def test_order_of_the_bias_gradients_sums(B, dims, rule):
    """A hidden bias gradient is the sum of its signals over the rows in one order, whichever launch forms the signals: bands of 64 rows, in a band the rows with
    row / 4 even one after the other, then the others, then the two sums; the bands one after the other.  float32 sums in that
    order give the result bit for bit.  The signals come from workers that have one such row and otherwise rows on which no unit is active: zeros, which
    leave a sum as it is."""
    rng = np.random.default_rng(B)
    X, y, theta = _exact_network(dims, B, rng)

    def stored(M, n, X, y, sched):
        cfg = configs.CFG4.scaled(name="bias_order", layer_dims=dims, M=M, N_m=n, B=B, K=1, D=3, rule=RULES[rule])
        out = run_library(cfg, (to_dev(X), to_dev(y), to_dev(theta)), sched)
        assert out["error_flags"][0] == 0 and out["trace_mask"].all()
        return out["stored"]

    pairs = np.stack([np.arange(1, B + 1), np.zeros(B, dtype=np.int64)], axis=1).reshape(-1)      # worker m: row m + 1, the zero row
    one = np.ones((1, B, B), dtype=np.int32)
    one[0, np.arange(B), np.arange(B)] = 0
    single = stored(B, 2, X[pairs], y[pairs], one)
    got = stored(1, B, X[1:], y[1:], np.arange(B, dtype=np.int32).reshape(1, 1, B))[0]

    off = dims[0] * dims[1]
    for a, b, c in zip(dims, dims[1:], dims[2:]):
        x = single[:, off:off + b].astype(np.float32)
        want, other = np.zeros(b, np.float32), np.zeros(b, np.float32)
        for r0 in range(0, B, 64):
            half = np.zeros((2, b), np.float32)
            for r in range(r0, min(r0 + 64, B)):
                half[(r >> 2) & 1] += x[r]
            want += half[0] + half[1]
        for r in range(B):
            other += x[r]
        assert np.abs(x).max() > 0 and (B < 33 or not np.array_equal(want, other)), "the case must tell orders apart"
        assert np.array_equal(got[off:off + b], want), (b, np.abs(got[off:off + b] - want).max(), int((got[off:off + b] != want).sum()))
        off += b + b * c


@pytest.mark.parametrize("dims,B", [((100, 1024, 1000, 5), 90), ((100, 1021, 1003, 5), 180)], ids=["even", "odd"])
def test_gradients_past_the_caches(dims, B):
    """With 64 workers these 290 MB of gradients go past the caches (rules without a second gradient), with three they do not: another kernel, which adds the same
    products up in the same order.  Forward products, whose order depends on the number of workers, are exact (see above)."""
    M, some = 64, [0, 29, 63]
    rng = np.random.default_rng(B)
    X, y, theta = _exact_network(dims, M * B, rng)
    X, y = X[1:].reshape(M, B, -1), y[1:].reshape(M, B)

    def stored(X, y):
        cfg = configs.CFG4.scaled(name="past_caches", layer_dims=dims, M=len(X), N_m=B, B=B, K=1, D=3, rule=configs.RULE_ALWAYS)
        sched = np.tile(np.arange(B, dtype=np.int32), (1, len(X), 1))
        out = run_library(cfg, (to_dev(X.reshape(-1, dims[0])), to_dev(y.reshape(-1)), to_dev(theta)), sched)
        assert out["error_flags"][0] == 0
        return out["stored"]

    many, few = stored(X, y), stored(X[some], y[some])
    assert np.isfinite(many).all() and all(np.abs(few[i]).max() > 0 for i in range(len(some)))
    for i, m in enumerate(some):
        assert np.array_equal(many[m], few[i]), (m, rel_l2(many[m], few[i]), int((many[m] != few[i]).sum()))
