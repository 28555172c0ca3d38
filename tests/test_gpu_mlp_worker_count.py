"""A worker's gradients do not depend on how many others there are: bit for bit the same on both sides of the line where the small forward products take four wavefronts per workgroup
in place of eight (more than 512 blocks of 32 x 32, inner dimensions up to 512), for inner dimensions of one tile step and of many, whole and ragged, in the first layer and in the second."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from common import to_dev

pytestmark = pytest.mark.gpu


def _after_a_step(cfg, prob, sched, M):
    """Stored gradients and left-hand sides after one step from a state with reference points beside the iterate; everybody uploads."""
    n, p = M * cfg.N_m, cfg.p
    eng = binding.Cada.from_config(cfg.scaled(M=M), to_dev(prob.X[:n]), to_dev(prob.y[:n]), to_dev(prob.theta0), trace_steps=8)
    rng = np.random.default_rng(5)
    away = lambda s: (prob.theta0 + s * rng.standard_normal(p)).astype(np.float32)
    theta, ref = away(1e-2), away(1e-2)
    zeros = np.zeros((M, p), np.float32)
    kw = {}
    if cfg.rule == configs.RULE_CADA1:
        kw = {"reference": to_dev(ref), "stored_innovations": to_dev(zeros)}
    elif cfg.rule == configs.RULE_CADA2:
        kw = {"reference": to_dev(np.broadcast_to(ref, (M, p)))}
    eng.set_state(k=3, theta=to_dev(theta), h=to_dev(zeros[0]), vhat=to_dev(zeros[0]), stored_gradients=to_dev(zeros), tau=torch.ones(M, dtype=torch.int32, device="cuda"),
                  ring=torch.full((cfg.d_max,), 1e-6, device="cuda"), **kw)
    eng.step(to_dev(np.ascontiguousarray(sched[0, :M]).astype(np.int32)), torch.ones(M, dtype=torch.uint8, device="cuda"))
    st = eng.state()
    out = eng.stored_gradients().cpu().numpy(), st["lhs"].cpu().numpy().copy(), int(st["error_flags"][0])
    eng.close()
    return out


# layer sizes, the workers that make 512 blocks or just fewer, rows per worker
@pytest.mark.parametrize("dims,M,B", [((20, 512, 4), 32, 12), ((96, 512, 4), 32, 12), ((129, 512, 4), 32, 12), ((256, 500, 4), 32, 32), ((500, 257, 10), 56, 7), ((512, 130, 6), 34, 70), ((317, 301, 150, 26), 12, 100),
                                      ((40, 150, 301, 26), 12, 100)])
@pytest.mark.parametrize("rule", [configs.RULE_ALWAYS, configs.RULE_CADA1, configs.RULE_CADA2], ids=["always", "cada1", "cada2"])
def test_four_wavefronts_add_up_as_eight_do(dims, M, B, rule):
    more = M + max(1, M // 12)                    # (of two hidden layers only the larger one changes sides)
    blocks = (B + 31) // 32 * ((max(dims[1:-1]) + 31) // 32)
    assert M * blocks <= 512 < more * blocks <= 1024 and max(dims[:-2]) <= 512
    cfg = configs.CFG5.scaled(name="count", layer_dims=dims, M=more, N_m=B + 20, B=B, K=1, D=3, c=20.0, rule=rule)
    prob, sched = generators.make_problem(cfg), generators.make_schedule(cfg)
    (few, few_lhs, e0), (many, many_lhs, e1) = _after_a_step(cfg, prob, sched, M), _after_a_step(cfg, prob, sched, more)
    assert e0 == 0 and e1 == 0 and np.isfinite(few).all() and np.abs(few).max() > 0 and np.abs(few_lhs).max() > 0
    assert np.array_equal(few, many[:M])
    assert np.array_equal(few_lhs, many_lhs[:M])
