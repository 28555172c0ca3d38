"""The logistic step of one or two launches (cada_logreg_rows.hip) against the oracle, at the edges of its variants:
pieces per lane and wavefronts per row change at 256, 512, 1024, 2048 and 4096 columns, the last quad of a row may overlap
its neighbour, a worker's rows are split into shares from 64 rows and 256 KB on, and small states take the
server update into the launch."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from common import check_protocol, to_dev, upload
from common_split import SHARED_WORKERS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,M,B,rule", [
    (4, 3, 70, 2), (5, 70, 9, 1), (22, 10, 92, 3), (255, 3, 65, 2), (256, 66, 8, 1), (257, 3, 129, 2), (513, 5, 66, 1),
    (784, 10, 60, 2), (1024, 4, 300, 2), (1025, 4, 300, 1), (1027, 3, 67, 0), (2048, 40, 40, 1), (2049, 3, 130, 2), (4097, 9, 64, 1),
    (8191, 5, 150, 2), (8192, 3, 33, 1)])
def test_rows_path(p, M, B, rule, K=24, spare=40):
    lag = rule == configs.RULE_LAG
    cfg = configs.CFG1.scaled(name="rows", layer_dims=(p,), M=M, N_m=B + spare, B=B, K=K, D=6, rule=rule, c=0.5 if p < 100 else 2e-3,
                              alpha=0.005, server=1 if lag else 0)
    prob = generators.make_problem(cfg)
    prob.X *= np.float32(1.0 / np.sqrt(p))           # (rows of norm about one, so that the decisions mix)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    stats, o, tr, rep = check_protocol(cfg, prob, dev, sched, 1e-4, lhs_rtol=1e-4, expect_phase="logreg_rows")
    print(p, M, B, rule, stats, tr["mask"].mean())
    assert stats["stored_rel_l2"] < 1e-5


# more than 8192 columns: five to ten quads per lane, the last ones with theta - theta_ref in LDS; shares of one row and of many
@pytest.mark.parametrize("p,M,B,rule", [
    (8193, 3, 33, 1), (8196, 5, 64, 2), (10240, 2, 7, 2), (10243, 4, 50, 1), (12290, 3, 40, 3), (14336, 70, 6, 2), (14337, 3, 61, 2),
    (16385, 9, 30, 1), (18433, 3, 45, 0), (20001, 6, 75, 1), (20478, 3, 100, 2), (20480, 2, 1, 1)])
def test_wide_rows_path(p, M, B, rule):
    test_rows_path(p, M, B, rule)


@pytest.mark.parametrize("p,M,B,rule", SHARED_WORKERS)
def test_wide_rows_path_shares_of_several_workers(p, M, B, rule):
    # (LAG: samples enough that no minibatch is drawn twice running.  Its left-hand side |g - g_stored|^2 has no digits where both gradients
    # are over the same rows: 5e-14 for |g|^2 = 0.25 is a difference of 5e-7 |g| between float32 vectors of 6e-8 |g| rounding each.)
    test_rows_path(p, M, B, rule, K=8, spare=40 if rule == configs.RULE_LAG else 3)


# the rule in the server's launch up to 256 workers (or, with the server, in the last workgroup), in the last workgroup up to 512, in a launch of its own for more; more than 8192
# columns: in the server's launch up to 256, in a launch of its own for more
@pytest.mark.parametrize("p,M,B,rule", [(54, 512, 33, 2), (54, 513, 33, 1), (257, 530, 40, 3), (1025, 513, 8, 2), (2050, 513, 9, 0), (8193, 32, 5, 1), (8200, 33, 5, 2),
                                        (10241, 40, 9, 0)])
def test_rows_path_many_workers(p, M, B, rule):
    test_rows_path(p, M, B, rule, K=8, spare=40 if rule == configs.RULE_LAG else 3)


@pytest.mark.parametrize("p,M,B,path,phase", [
    (784, 257, 8, binding.PATH_AUTO, "logreg_two_pass"), (784, 257, 8, binding.PATH_SINGLE_PASS, "logreg_two_pass"), (784, 257, 32, binding.PATH_AUTO, "logreg_rows"),
    (6000, 2, 40, binding.PATH_AUTO, "logreg_two_pass"), (6000, 2, 10, binding.PATH_AUTO, "logreg_rows"), (8196, 513, 4, binding.PATH_AUTO, "logreg_single_pass"),
    (8197, 513, 4, binding.PATH_AUTO, "logreg_rows"), (8196, 3, 8, binding.PATH_AUTO, "logreg_rows"), (8196, 3, 8, binding.PATH_SINGLE_PASS, "logreg_single_pass"),
    (8196, 3, 8, binding.PATH_WHOLE_STEPS, "logreg_rows"), (8196, 3, 8, binding.PATH_TWO_PASS, "logreg_two_pass"), (54, 3, 8, binding.PATH_WHOLE_STEPS, "logreg_whole_steps")])
def test_routes(p, M, B, path, phase):
    """Which kernels a shape and a request take; a request that the shape does not allow takes what it would take by itself."""
    cfg = configs.CFG1.scaled(name="route", layer_dims=(p,), M=M, N_m=B, B=B, K=2)
    prob = generators.make_problem(cfg)
    eng = binding.Cada.from_config(cfg, *upload(prob), path=path)
    assert phase in binding.cada_profile_phase_names(eng.ctx)
    eng.step(to_dev(generators.make_schedule(cfg)[0].astype(np.int32)))
    torch.cuda.synchronize()
    eng.close()


def test_rows_path_flags_and_repeats():
    """An index out of range is clamped and flagged; two runs agree bit for bit."""
    from common import run_library
    cfg = configs.CFG1.scaled(name="rows", layer_dims=(300,), M=3, N_m=200, B=100, K=6)
    prob = generators.make_problem(cfg)
    dev, sched = upload(prob), generators.make_schedule(cfg)
    bad = sched.copy(); bad[3, 2, 70] = cfg.N_m + 5
    fixed = sched.copy(); fixed[3, 2, 70] = cfg.N_m - 1
    out, ref = run_library(cfg, dev, bad, expect_phase="logreg_rows"), run_library(cfg, dev, fixed)
    assert out["error_flags"][0] == 1 and ref["error_flags"][0] == 0
    for name in ("theta", "h", "vhat", "stored", "trace_lhs"):
        assert np.array_equal(out[name], ref[name]), name


@pytest.mark.parametrize("p,M", [(8192, 3), (1024, 1)])
def test_sums_of_the_rule_keep_small_terms(p, M):
    """The rule compares sums of squares in double.  All values here are powers of two: every gradient, and with alpha = 1 every step of the SGD
    server, is exact; a float32 sum that meets a large square first and then small ones of half a unit in the last place loses these.
    8192 columns: the left-hand side, four squares of 1 and then twelve of 2^-22 in each lane.  1024 columns and one worker: the
    server runs in the same launch, and the squared step is 1 in the first and 2^-24 in each other wavefront's columns."""
    B = 128
    x = torch.zeros(p, device="cuda")
    if p == 8192:
        x[:] = 2.0 ** -10
        x[:2048] = 2.0
    else:
        x[64:512:64] = 2.0 ** -11
        x[0] = 2.0
    squares = float(((0.5 * x.double()) ** 2).sum())
    X = x.repeat(M * B, 1).contiguous()
    eng = binding.Cada(model="logreg", layer_dims=[p], M=M, B=B, n_samples=[B] * M, X=X, y=torch.ones(M * B, device="cuda"),
                       theta0=torch.zeros(p, device="cuda"), rule=3, D=50, d_max=10, c=0.5, alpha=1.0, beta1=0.9, beta2=0.999, eps=1e-8, lam=0.0,
                       gemm_dtype="fp32", server=1, trace_steps=1)
    assert "logreg_rows" in binding.cada_profile_phase_names(eng.ctx)
    eng.step(torch.arange(B, dtype=torch.int32, device="cuda").repeat(M, 1).contiguous())
    st = eng.state()
    torch.cuda.synchronize()
    want = np.float32(squares)
    assert want == (2048 + 6144 * 2.0 ** -22 if p == 8192 else 1 + 8 * 2.0 ** -24)
    assert (st["trace_lhs"].cpu().numpy().ravel() == want).all()
    assert st["lhs"].cpu().numpy().tolist() == [want] * M
    assert st["ring"].cpu().numpy()[0] == want
    eng.close()


@pytest.mark.parametrize("p,M,path,phase", [(784, 10, binding.PATH_AUTO, "logreg_rows"), (1025, 4, binding.PATH_AUTO, "logreg_rows"), (54, 300, binding.PATH_AUTO, "logreg_rows"),
                                            (8192, 3, binding.PATH_AUTO, "logreg_rows"), (8193, 3, binding.PATH_AUTO, "logreg_rows"), (1025, 4, binding.PATH_TWO_PASS, "logreg_two_pass")])
def test_left_hand_side_past_float32(p, M, path, phase):
    """A left-hand side past float32's range is infinite, which is more than any right-hand side: the worker uploads.  (Not a number, and the worker silent, where what
    infinity is rounded by was added to it.)"""
    B = 70
    X = torch.full((2 * M * B, p), 1e20, device="cuda")
    y = torch.ones(2, B, device="cuda")
    y[1] = -1.0
    eng = binding.Cada(model="logreg", layer_dims=[p], M=M, B=B, n_samples=[2 * B] * M, X=X, y=y.reshape(-1).repeat(M).contiguous(), theta0=torch.zeros(p, device="cuda"),
                       rule=configs.RULE_LAG, D=50, d_max=10, c=0.5, alpha=1e-30, beta1=0.9, beta2=0.999, eps=1e-8, server=1, trace_steps=2, path=path)
    assert phase in binding.cada_profile_phase_names(eng.ctx)
    rows = torch.arange(2 * B, dtype=torch.int32, device="cuda").view(2, 1, B).repeat(1, M, 1).contiguous()      # a gradient, then its opposite
    eng.run(rows)
    st = {name: t.cpu().numpy().copy() for name, t in eng.state().items() if name.startswith("trace")}
    eng.close()
    assert np.isposinf(st["trace_lhs"]).all() and np.isfinite(st["trace_rhs"]).all(), (st["trace_lhs"], st["trace_rhs"])
    assert st["trace_own_mask"].all() and st["trace_mask"].all()
