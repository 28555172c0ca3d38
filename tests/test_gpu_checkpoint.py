"""Checkpoint / resume through the C ABI: a run continued from a saved block, in the same
context or in a fresh one, is bitwise the run that was never interrupted."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd.binding import Cada, CadaError

from common import upload, to_dev

pytestmark = pytest.mark.gpu


def _final(eng):
    torch.cuda.synchronize()
    st = eng.state()
    torch.cuda.synchronize()
    return {k: (v.cpu().numpy().copy() if torch.is_tensor(v) else v) for k, v in st.items()}, eng.stored_gradients().cpu().numpy()


@pytest.mark.parametrize("cfg", [
    configs.CFG1.scaled(K=60),
    configs.CFG2.scaled(K=40, N_m=200),
    configs.CFG4.scaled(name="mlp2_small", layer_dims=(40, 24, 10), M=4, N_m=100, B=16, K=24, D=6),
], ids=lambda c: c.name)
def test_resume_is_bitwise_the_uninterrupted_run(cfg):
    prob = generators.make_problem(cfg)
    X, y, th0 = upload(prob)
    sched = to_dev(generators.make_schedule(cfg).astype(np.int32))
    K, K1 = cfg.K, cfg.K // 3
    ref = Cada.from_config(cfg, X, y, th0, trace_steps=K)
    for k in range(K):
        ref.step(sched[k])
    want, want_g = _final(ref)

    a = Cada.from_config(cfg, X, y, th0, trace_steps=K)
    for k in range(K1):
        a.step(sched[k])
    block = a.checkpoint()
    for k in range(K1, K1 + 5):          # run on, then rewind the same context
        a.step(sched[k])
    a.restore(block)
    assert a.k == K1
    for k in range(K1, K):
        a.step(sched[k])
    b = Cada.from_config(cfg, X, y, th0, trace_steps=K)      # and a fresh context
    b.restore(block)
    for k in range(K1, K):
        b.step(sched[k])
    for eng in (a, b):
        got, got_g = _final(eng)
        assert got["k"] == want["k"] == K
        for name in ("theta", "theta_lo", "h", "vhat", "tau", "ring", "uploads_total", "trace_mask", "trace_lhs"):
            assert np.array_equal(got[name], want[name]), name
        assert np.array_equal(got_g, want_g)


def test_block_of_another_configuration_is_refused():
    cfg = configs.CFG1.scaled(K=4)
    prob = generators.make_problem(cfg)
    X, y, th0 = upload(prob)
    a = Cada.from_config(cfg, X, y, th0)
    block = a.checkpoint()
    # d_max changes a few bytes inside one 256-byte piece of the workspace: same size, other header
    b = Cada.from_config(cfg.scaled(d_max=cfg.d_max - 1), X, y, th0)
    if b.checkpoint().numel() == block.numel():
        with pytest.raises(CadaError):
            b.restore(block)
    with pytest.raises(CadaError):
        a.restore(torch.zeros_like(block))
    a.restore(block)            # a valid block still loads afterwards


@pytest.mark.parametrize("M,B", [(3, 20), (24, 20), (3, 1)])
@pytest.mark.parametrize("save,load", [(a, b) for a in ("two_pass", "rows", "whole") for b in ("two_pass", "rows", "whole") if a != b])
def test_block_of_another_path(save, load, M, B):
    """The path is no part of a block.  The newest squared step is kept in parts that each path cuts in its own way (p = 784 are four
    server blocks; M = 3 is fewer, M = 24 more, and too much state for a server inside the rows kernel): a run that goes on on
    another path forms the right-hand sides that the saving context forms, and both report the same ring."""
    from paper_2012_15469_amd import binding
    from paper_2012_15469_amd.binding import cada_profile_phase_names
    paths = {"two_pass": (binding.PATH_TWO_PASS, "logreg_two_pass"), "rows": (binding.PATH_SINGLE_PASS, "logreg_rows"),
             "whole": (binding.PATH_WHOLE_STEPS, "logreg_whole_steps")}      # (a single pass starts at 8192 columns: the rows kernel before that)
    cfg = configs.CFG2.scaled(K=14, N_m=50, M=M, B=B, D=5)
    K1, prob = 6, generators.make_problem(cfg)
    X, y, th0 = upload(prob)
    sched = to_dev(generators.make_schedule(cfg).astype(np.int32))
    engines = {}
    for name in (save, load):
        engines[name] = Cada.from_config(cfg, X, y, th0, trace_steps=cfg.K, path=paths[name][0])
        assert paths[name][1] in cada_profile_phase_names(engines[name].ctx)
    for k in range(K1):
        engines[save].step(sched[k])
    engines[load].restore(engines[save].checkpoint())
    want, _ = _final(engines[save])
    got, _ = _final(engines[load])
    assert np.array_equal(got["ring"], want["ring"])      # the same parts, added up by the same kernel
    for k in range(K1, cfg.K):
        for name in (save, load):
            engines[name].step(sched[k], torch.ones(M, dtype=torch.uint8, device="cuda"))
    want, _ = _final(engines[save])
    got, _ = _final(engines[load])
    # (float32 sums of 784 terms in another order, over eight steps: 1e-6; a missing part is a quarter of the newest term)
    assert np.allclose(got["trace_rhs"], want["trace_rhs"], rtol=1e-5, atol=0)
    assert np.allclose(got["ring"], want["ring"], rtol=1e-5, atol=0)
