"""cada_step of the small logistic workloads: one launch whose last workgroup runs the server phase.  It must end
where the same iteration inside a longer cada_run launch ends, bit for bit, alone and mixed with runs."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators

from common import run_library, to_dev, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(base=configs.CFG2, K=24, N_m=200, D=5),                                           # 16-byte rows, CADA1, snapshots
    dict(base=configs.CFG1, K=24, M=1, B=1, N_m=50, D=5),                                   # one workgroup
    dict(base=configs.CFG1, K=16, M=64, B=64, N_m=90, D=4, c=0.05),                         # the most workers and rows
    dict(base=configs.CFG1, K=16, M=7, layer_dims=(257,), B=9, rule=configs.RULE_LAG, server=configs.SERVER_SGD),
    dict(base=configs.CFG1, K=16, M=5, layer_dims=(1,), B=3, rule=configs.RULE_ALWAYS),
])
def test_single_steps_equal_a_run(kw):
    from paper_2012_15469_amd.binding import Cada, cada_profile_phase_names
    kw = dict(kw)
    cfg = kw.pop("base").scaled(**kw)
    prob = generators.make_problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    replay = np.full((cfg.K, cfg.M), 255, dtype=np.uint8)
    replay[3] = 0
    ref = run_library(cfg, dev, sched, replay=replay, expect_phase="logreg_whole_steps")
    for pieces in ([1] * cfg.K, [1, 5, 1, 1, 2, cfg.K - 10]):
        eng = Cada.from_config(cfg, *dev, trace_steps=cfg.K)
        assert cada_profile_phase_names(eng.ctx) == ["logreg_whole_steps"]
        idx, rp = to_dev(sched), to_dev(replay)
        k = 0
        for n in pieces:
            if n == 1:
                eng.step(idx[k], rp[k])
            else:
                eng.run(idx[k:k + n].contiguous(), rp[k:k + n].contiguous())
            k += n
        torch.cuda.synchronize()
        st = eng.state()
        torch.cuda.synchronize()
        assert k == cfg.K
        for name in ("theta", "theta_lo", "h", "v", "vhat", "nabla", "tau", "mask", "lhs", "uploads_total", "error_flags", "ring",
                     "trace_mask", "trace_own_mask", "trace_lhs", "trace_rhs", "trace_tau"):
            assert np.array_equal(st[name].cpu().numpy(), ref[name]), name
        assert np.array_equal(eng.stored_gradients().cpu().numpy(), ref["stored"])
        eng.close()
