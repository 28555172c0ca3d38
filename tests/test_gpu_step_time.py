"""Steps of one workload against each other on one device, where a serial walk on the device once made one of them several times as long as the other.  The shortest of
seven runs of 200 steps each, in turn; the bounds lie half way (as a ratio) between what the walk cost and what is measured without it."""
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from common import upload

pytestmark = pytest.mark.gpu
STEPS = 200


def _shortest(engines, sched, masks):
    """us per step of each engine"""
    best = [float("inf")] * len(engines)
    for eng, mask in zip(engines, masks):
        for _ in range(2):
            eng.run(sched, mask)
    for _ in range(7):
        for i, (eng, mask) in enumerate(zip(engines, masks)):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            eng.run(sched, mask)
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1000 / STEPS)
    for eng in engines:
        eng.close()
    return best


def test_distinct_reference_points():
    """200 workers with 200 delays against all with one: 48 and 55 us per step (with a walk over the workers and the points in every block: 127 and 55)."""
    cfg = configs.CFG5.scaled(name="time", layer_dims=(100, 32, 10), M=200, N_m=40, B=8, D=STEPS + 10, K=STEPS, rule=configs.RULE_CADA2)
    dev, sched = upload(generators.make_problem(cfg)), torch.from_numpy(generators.make_schedule(cfg).astype("int32")).cuda()
    k, m = torch.arange(STEPS, device="cuda")[:, None], torch.arange(cfg.M, device="cuda")[None, :]
    apart, all_ = ((k - m) % STEPS == 0).to(torch.uint8).contiguous(), torch.ones(STEPS, cfg.M, dtype=torch.uint8, device="cuda")
    t = _shortest([binding.Cada.from_config(cfg, *dev) for _ in range(2)], sched, [apart, all_])
    print(t)
    assert t[0] < 1.4 * t[1], t


@pytest.mark.parametrize("dims,M,B", [((8193,), 4, 64), ((100, 60, 5), 8, 12)])
def test_long_ring(dims, M, B):
    """A ring of 1024 squared steps against one of 64: 22 and 22, 44 and 44 us per step (added up by one thread: 95 and 23, 114 and 45)."""
    base = configs.CFG5.scaled(name="time", layer_dims=dims, rule=configs.RULE_CADA1) if len(dims) > 1 else configs.CFG1.scaled(name="time", layer_dims=dims)
    cfg = base.scaled(M=M, N_m=80, B=B, K=STEPS)
    dev, sched = upload(generators.make_problem(cfg)), torch.from_numpy(generators.make_schedule(cfg).astype("int32")).cuda()
    t = _shortest([binding.Cada.from_config(cfg.scaled(d_max=d), *dev) for d in (1024, 64)], sched, [None, None])
    print(t)
    assert t[0] < 1.6 * t[1], t
