"""The MLP's contraction kernels at the edges of their tiles, through the C ABI against the fp64 oracle: a worker's rows cut into
steps of 16 and 32 (one row, a whole step, one more, more than a row tile), matrices that end inside a tile, just past one, and at no multiple of the
8 values that leave in one access; fewer steps than the operand ring holds, and several tiles per workgroup."""
import numpy as np
import pytest

from cada_synth import configs, generators

from common import check_protocol, upload, run_library, oracle_run, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [          # layer sizes, workers, rows per worker
    ((33, 40, 5), 1, 1),
    ((65, 33, 40, 3), 2, 16),
    ((130, 135, 36, 4), 3, 17),
    ((129, 257, 130, 6), 2, 129),
    ((600, 140, 33, 4), 48, 48),
    ((48, 700, 45, 4), 60, 31),
]
RULES = {"cada1": configs.RULE_CADA1, "cada2": configs.RULE_CADA2, "always": configs.RULE_ALWAYS}


def _config(shape, rule):
    dims, M, B = shape
    return configs.CFG5.scaled(name="tiles", layer_dims=dims, M=M, N_m=max(B, 40), B=B, K=5, D=3, c=20.0, rule=RULES[rule])


@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s[0])) + "_M%d_B%d" % s[1:])
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
    if rule == "always":
        return
    big = tr["lhs"] > 1e-9 * tr["lhs"].max()
    rel = np.abs(rep["trace_lhs"] - tr["lhs"])[big] / tr["lhs"][big]
    assert float(np.median(rel)) < 2.0 ** -7
