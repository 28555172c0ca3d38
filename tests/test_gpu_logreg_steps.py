"""Whole iterations with the rows in registers (cada_logreg_steps.hip): every variant at the edges of its columns and rows, the numbers of workers at which the exchange asks for its rows
in other batches, all rules, single steps against launches of several, the route of cada_logreg_rows.hip; and gradients that look like the mark of one that has not come yet."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from oracle.driver import oracle_for

from common import check_protocol, inject_oracle_state, rel_l2, run_library, to_dev, upload

pytestmark = pytest.mark.gpu


def _cfg(p, M, B, rule, **kw):
    kw = {"K": 12, "D": 4, **kw}
    return configs.CFG1.scaled(name="steps", layer_dims=(p,), M=M, N_m=B + 40, B=B, rule=rule, server=1 if rule == configs.RULE_LAG else 0, c=0.5 if p < 100 else 2e-3, **kw)


def _problem(cfg):
    prob = generators.make_problem(cfg)
    prob.X *= np.float32(1.0 / np.sqrt(cfg.layer_dims[0]))
    return prob


# one quad per lane up to 256 columns, two up to 512, four up to 1024; a quad that ends with the row; two, four and eight rows per wavefront; 8, 16, 24 and 32 gradients at a time
SHAPES = [(4, 1, 1), (5, 3, 8), (63, 8, 9), (255, 9, 16), (256, 16, 17), (257, 17, 32), (54, 24, 33), (256, 25, 64), (300, 32, 40), (510, 33, 16), (512, 3, 64), (511, 65, 24), (513, 4, 16),
          (784, 20, 32), (1021, 2, 17), (1024, 33, 8)]


@pytest.mark.parametrize("rule", [configs.RULE_ALWAYS, configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_LAG], ids=["always", "cada1", "cada2", "lag"])
@pytest.mark.parametrize("p,M,B", SHAPES)
def test_against_the_oracle(p, M, B, rule):
    cfg = _cfg(p, M, B, rule)
    prob = _problem(cfg)
    # (bounds of the other logistic kernels' tests: float32 sums of up to 64 rows, theta from twelve updates)
    check_protocol(cfg, prob, upload(prob), generators.make_schedule(cfg), 1e-4, lhs_rtol=1e-4, free_margin=1e-3, path=binding.PATH_WHOLE_STEPS, expect_phase="logreg_whole_steps")


@pytest.mark.parametrize("rule", [configs.RULE_ALWAYS, configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_LAG], ids=["always", "cada1", "cada2", "lag"])
# (511 columns and 10 rows, 1021 and 5: wavefronts that have columns and no rows; 5, 65, 260, 513 and 650 columns with more than 56 workers, whose selectors do not travel with the count of a single step: wavefronts
# with columns for fewer than 16 lanes)
@pytest.mark.parametrize("p,M,B", [(5, 3, 8), (54, 57, 10), (256, 25, 64), (511, 33, 24), (511, 33, 10), (784, 20, 32), (1021, 2, 17), (1021, 24, 5), (5, 58, 9), (65, 57, 8), (260, 60, 17), (513, 64, 9),
                                   (650, 130, 8), (1021, 61, 8)])
def test_single_steps_end_where_a_launch_of_several_does(p, M, B, rule):
    cfg = _cfg(p, M, B, rule)
    prob = _problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    want = run_library(cfg, dev, sched, path=binding.PATH_WHOLE_STEPS)
    eng = binding.Cada.from_config(cfg, *dev, trace_steps=cfg.K, path=binding.PATH_WHOLE_STEPS)
    idx = to_dev(sched.astype(np.int32))
    for a, b in ((0, 1), (1, 2), (2, 7), (7, 8), (8, 10), (10, 12)):      # (turns of the exchange that do not start at the first)
        eng.step(idx[a]) if b == a + 1 else eng.run(idx[a:b].contiguous())
    st = eng.state()
    for name in ("theta", "theta_lo", "h", "v", "vhat", "nabla", "tau", "mask", "lhs", "ring", "trace_mask", "trace_lhs", "trace_rhs", "trace_tau", "uploads_total", "error_flags"):
        assert np.array_equal(st[name].cpu().numpy(), want[name]), name
    assert np.array_equal(eng.stored_gradients().cpu().numpy(), want["stored"])
    eng.close()


# the route of cada_logreg_rows.hip: two batches of rows, at both edges of what is taken and just beyond
@pytest.mark.parametrize("rule", [configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_LAG], ids=["cada1", "cada2", "lag"])
@pytest.mark.parametrize("p,M,B", [(4, 3, 65), (22, 10, 92), (256, 32, 128), (255, 5, 129), (257, 4, 65), (600, 3, 64), (784, 10, 60), (1024, 16, 49), (1021, 5, 65)])
def test_rows_of_two_batches(p, M, B, rule):
    cfg = _cfg(p, M, B, rule)
    prob = _problem(cfg)
    check_protocol(cfg, prob, upload(prob), generators.make_schedule(cfg), 1e-4, lhs_rtol=1e-4, free_margin=1e-3, expect_phase="logreg_rows")


@pytest.mark.parametrize("steps", [1, 6])
def test_gradients_that_are_no_numbers(steps):
    """All bits set is the mark of a gradient that has not come yet, and a NaN of that pattern among the features may come out as such a gradient: it is passed on as another NaN, and no
    wait hangs on it."""
    cfg = _cfg(54, 10, 10, configs.RULE_ALWAYS, K=6)
    prob = _problem(cfg)
    X = prob.X.copy()
    X.view(np.uint32)[:, 7] = 0xffffffff
    eng = binding.Cada.from_config(cfg, to_dev(X), to_dev(prob.y), to_dev(prob.theta0), path=binding.PATH_WHOLE_STEPS)
    idx = to_dev(generators.make_schedule(cfg).astype(np.int32))
    for a in range(0, 6, steps):
        eng.step(idx[a]) if steps == 1 else eng.run(idx)
    st = eng.state()
    torch.cuda.synchronize()
    assert int(st["error_flags"][0]) == 0 and bool(torch.isnan(st["theta"]).all())
    eng.close()


def test_a_state_handed_over_between_launches():
    """A loaded checkpoint continues as the run that it was taken of, whatever turn of the exchange the context was at."""
    cfg = _cfg(200, 12, 20, configs.RULE_CADA2, K=10)
    prob = _problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    idx = to_dev(sched.astype(np.int32))
    eng = binding.Cada.from_config(cfg, *dev, path=binding.PATH_WHOLE_STEPS)
    eng.run(idx[:5].contiguous())
    block = eng.checkpoint()
    eng.run(idx[5:].contiguous())
    want = eng.state()["theta"].clone()
    for before in (0, 2, 3):
        other = binding.Cada.from_config(cfg, *dev, path=binding.PATH_WHOLE_STEPS)
        if before:
            other.run(idx[:before].contiguous())
        other.restore(block)
        other.run(idx[5:].contiguous())
        assert torch.equal(other.state()["theta"], want)
        other.close()
    eng.close()


def _leave_gradients_behind(eng):
    """The exchange's rows, which lie at the end of the workspace, as a launch that gave up waiting could leave them: gradients that nobody has read."""
    nbytes = 4 * eng.M * ((eng.p + 3) // 4 * 4) * 4
    end = eng._ws_off + eng.cfg.workspace_bytes
    rows = eng.workspace[end - (nbytes + 255) // 256 * 256:][:nbytes].view(torch.float32)
    assert int(rows.view(torch.int32).eq(-1).sum()) >= rows.numel() // 2      # (the rows of the next two steps are marked as not there)
    rows.fill_(0.25)


@pytest.mark.parametrize("before", [0, 1, 2, 3])
def test_the_exchange_starts_afresh(before):
    """cada_set_state and a loaded checkpoint: whatever was on its way before is not taken for a gradient of the steps to come."""
    cfg = _cfg(203, 12, 20, configs.RULE_CADA2, K=10)
    prob = _problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    idx = to_dev(sched.astype(np.int32))
    o = oracle_for(cfg, prob).run(sched[:5])
    want = {}
    for poisoned in (False, True):
        eng = binding.Cada.from_config(cfg, *dev, path=binding.PATH_WHOLE_STEPS)
        if before:
            eng.run(idx[:before].contiguous())
        if poisoned:
            _leave_gradients_behind(eng)
        inject_oracle_state(eng, o)
        block = eng.checkpoint()
        eng.run(idx[5:].contiguous())
        if poisoned:
            assert torch.equal(eng.state()["theta"], want["theta"])
            other = binding.Cada.from_config(cfg, *dev, path=binding.PATH_WHOLE_STEPS)
            if before:
                other.run(idx[:before].contiguous())
            _leave_gradients_behind(other)
            other.restore(block)
            other.run(idx[5:].contiguous())
            assert torch.equal(other.state()["theta"], want["theta"]) and int(other.state()["error_flags"][0]) == 0
            other.close()
        else:
            want["theta"] = eng.state()["theta"].clone()
        eng.close()


@pytest.mark.parametrize("D", [1, 3])
@pytest.mark.parametrize("p,M,B", [(54, 10, 10), (300, 9, 24), (600, 3, 8)])
def test_replay_beyond_the_retained_iterates(p, M, B, D):
    """A replay mask that keeps a CADA2 worker silent for more than D iterations: the oldest retained iterate stands for its reference point, here as in the two passes over the rows."""
    cfg = _cfg(p, M, B, configs.RULE_CADA2, D=D)
    prob = _problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    replay = (np.random.default_rng(3).random((cfg.K, M)) < 0.25).astype(np.uint8)
    replay[0], replay[1:, 0] = 1, 0                       # (one worker says nothing after the first step)
    want = run_library(cfg, dev, sched, replay=replay, path=binding.PATH_TWO_PASS)
    got = run_library(cfg, dev, sched, replay=replay, path=binding.PATH_WHOLE_STEPS, expect_phase="logreg_whole_steps")
    eng = binding.Cada.from_config(cfg, *dev, trace_steps=cfg.K, path=binding.PATH_WHOLE_STEPS)
    idx, mask = to_dev(sched.astype(np.int32)), to_dev(replay)
    for k in range(cfg.K):
        eng.step(idx[k], mask[k].contiguous())
    assert np.array_equal(eng.state()["theta"].cpu().numpy(), got["theta"]) and np.array_equal(eng.state()["trace_lhs"].cpu().numpy(), got["trace_lhs"])
    eng.close()
    assert want["error_flags"][0] == got["error_flags"][0] == 8
    assert np.array_equal(got["trace_tau"], want["trace_tau"]) and got["trace_tau"].max() > D
    # (bounds of the comparisons with the oracle above)
    assert rel_l2(got["theta64"], want["theta64"]) < 1e-4
    big = want["trace_lhs"] > 1e-9 * want["trace_lhs"].max()
    assert big[2:, 0].any()                               # (the silent worker's left-hand sides are among them)
    np.testing.assert_allclose(got["trace_lhs"][big], want["trace_lhs"][big], rtol=1e-4)
