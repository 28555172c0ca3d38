"""The differences to the workers' reference points (CADA2, k_stage): groups of blocks that share a list of the distinct ones out (up to 256 workers, a table of up to 4160
delays), against blocks that find out for themselves whether an earlier worker has the same delay.  D decides which of the two runs and, with the masks given,
changes nothing else: every result agrees bit for bit."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from common import upload

pytestmark = pytest.mark.gpu
TABLE = 4160


def _run(cfg, dev, sched, masks):
    eng = binding.Cada.from_config(cfg, *dev, trace_steps=cfg.K)
    eng.run(torch.from_numpy(sched.astype(np.int32)).cuda(), torch.from_numpy(masks).cuda())
    out = {name: t.cpu().numpy().copy() for name, t in eng.state().items() if name in ("theta", "theta_lo", "h", "vhat", "nabla", "trace_lhs", "trace_tau", "error_flags")}
    out["trace_tau"] = out["trace_tau"][1:]      # (the first iteration's delays are D)
    out["stored"] = eng.stored_gradients().cpu().numpy()
    eng.close()
    return out


# one worker, the last ones with a word of 64 to themselves, all 256; one tile and more tiles than make one group a worker (784-300-10: 70, 30 groups of up to 44 points);
# D at both ends of the table
@pytest.mark.parametrize("dims,M,D", [((20, 9, 3), 1, 60), ((40, 40, 5), 64, 60), ((40, 40, 5), 65, 60), ((40, 70, 5), 129, TABLE - 1), ((100, 32, 10), 256, 60),
                                      ((70, 130, 66, 4), 100, 60), ((784, 300, 10), 100, 60)])
@pytest.mark.parametrize("masks", ["all", "apart", "mixed"])
def test_list_and_search_agree(dims, M, D, masks):
    cfg = configs.CFG5.scaled(name="reference", layer_dims=dims, M=M, N_m=30, B=4, K=45, D=D, rule=configs.RULE_CADA2)
    k, m = np.arange(cfg.K)[:, None], np.arange(M)[None, :]
    up = (k == 0) | {"all": k >= 0, "apart": k % 45 == m % 45, "mixed": np.random.default_rng(M).random((cfg.K, M)) < 0.1}[masks] | np.zeros((cfg.K, M), bool)
    dev, sched = upload(generators.make_problem(cfg)), generators.make_schedule(cfg)
    a, b = (_run(c, dev, sched, up.astype(np.uint8)) for c in (cfg, cfg.scaled(D=TABLE)))
    assert a["error_flags"][0] == b["error_flags"][0] == 0
    if masks == "apart":
        assert len(np.unique(a["trace_tau"][-1])) == min(M, 44)      # (worker 44 and its like have uploaded with all at first)
    for name in a:
        assert np.array_equal(a[name], b[name]), name
