"""The rule in the server's launch (cada_server.hip): which shapes take it, its sums over few and many parts of the left-hand sides at the edges of
their groups of workers, the decisions and the books, and more coordinates than its workgroups take in one turn; against the oracle."""
import numpy as np
import pytest
import torch

from cada_synth import configs, generators
from paper_2012_15469_amd import binding

from common import check_protocol, to_dev, upload

pytestmark = pytest.mark.gpu
TOGETHER, APART = "rule_and_server_update", "server_update"


def _check(cfg, phase, tol, lhs_rtol):
    prob = generators.make_problem(cfg)
    if cfg.model == "logreg":
        prob.X *= np.float32(1.0 / np.sqrt(cfg.layer_dims[0]))
    dev, sched = upload(prob), generators.make_schedule(cfg)
    stats, o, tr, rep = check_protocol(cfg, prob, dev, sched, tol, lhs_rtol=lhs_rtol, own_mask_exact=lhs_rtol is not None,
                                       free_margin=None if lhs_rtol is None else 1e-3, expect_phase=phase)
    # The decisions follow from the recorded sides (float32 of the doubles that are compared: 2^-24 each), and the books agree with the trace.
    lhs, rhs, tau = rep["trace_lhs"].astype(np.float64), rep["trace_rhs"].astype(np.float64)[:, None], rep["trace_tau"]
    own = (lhs > rhs) | (tau >= cfg.D) | (cfg.rule == configs.RULE_ALWAYS)
    clear = (abs(lhs - rhs) > 2.0 ** -22 * rhs) | (tau >= cfg.D)
    assert np.array_equal(rep["trace_own_mask"][clear].astype(bool), own[clear])
    assert np.array_equal(rep["lhs"], rep["trace_lhs"][-1]) and np.array_equal(rep["mask"], rep["trace_mask"][-1])
    assert rep["uploads_total"][0] == rep["trace_mask"].sum()
    # the right-hand side: squared steps of float32 updates whose gradients carry the path's own error (a step of Adam moves less than its gradient)
    ok = tr["rhs"] > 0
    assert ok.any() and (abs(rep["trace_rhs"] - tr["rhs"])[ok] <= 2e-2 * tr["rhs"][ok]).all()


# layer sizes, workers, where the rule runs: 10 parts per worker (each thread adds its own worker's up), 28 parts (a wavefront takes eight workers; up to 8 and 16 of
# them share their parts among four and two wavefronts), 180 parts and 498 thousand coordinates (two turns of 1792 workgroups)
NETWORKS = [((100, 60, 5), 3, TOGETHER), ((100, 60, 5), 256, TOGETHER), ((100, 60, 5), 257, APART), ((130, 129, 5), 5, TOGETHER), ((130, 129, 5), 8, TOGETHER),
            ((130, 129, 5), 9, TOGETHER), ((130, 129, 5), 16, TOGETHER), ((130, 129, 5), 17, TOGETHER), ((130, 129, 5), 32, TOGETHER), ((130, 129, 5), 33, APART),
            ((700, 700, 10), 3, TOGETHER)]


@pytest.mark.parametrize("rule", [configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_ALWAYS], ids=["cada1", "cada2", "always"])
@pytest.mark.parametrize("dims,M,phase", NETWORKS)
def test_networks(dims, M, phase, rule):
    if rule == configs.RULE_ALWAYS and M <= 256:      # (a part per 4096 coordinates: few)
        phase = TOGETHER
    _check(configs.CFG5.scaled(name="rule", layer_dims=dims, M=M, N_m=30, B=6, K=6, D=3, c=20.0, rule=rule), phase, 2e-2, None)


# networks without a second gradient, whose parts are two per 4096 coordinates: 10 parts up to 128 workers, 4 up to 256
@pytest.mark.parametrize("dims,M,phase", [((130, 129, 5), 128, TOGETHER), ((130, 129, 5), 129, APART), ((100, 60, 5), 256, TOGETHER), ((100, 60, 5), 257, APART)])
def test_networks_with_one_gradient(dims, M, phase):
    _check(configs.CFG5.scaled(name="rule", layer_dims=dims, M=M, N_m=60, B=6, K=6, D=3, rule=configs.RULE_LAG, c=20.0, server=1), phase, 2e-2, None)


# The sums of 28 and 180 parts above, and of 765, 770 and 924, which four wavefronts take in one round of 192, in two of which the last holds one part, and in two; against the
# oracle's left-hand sides, so that no part is left out, counted twice or another worker's.  (Bounds as in test_gpu_mlp_tiles.)
@pytest.mark.parametrize("rule", [configs.RULE_CADA1, configs.RULE_CADA2], ids=["cada1", "cada2"])
@pytest.mark.parametrize("dims,M", [(d, m) for d, m, phase in NETWORKS if phase == TOGETHER] + [((12032, 200, 10), 3), ((24448, 40, 10), 3), ((24448, 40, 10), 1), ((1800, 1700, 10), 2)])
def test_left_hand_sides_of_networks(dims, M, rule):
    cfg = configs.CFG5.scaled(name="rule", layer_dims=dims, M=M, N_m=30, B=6, K=5, D=3, c=20.0, rule=rule)
    prob = generators.make_problem(cfg)
    stats, o, tr, rep = check_protocol(cfg, prob, upload(prob), generators.make_schedule(cfg), 2e-2, lhs_rtol=None, own_mask_exact=False, free_margin=None, expect_phase=TOGETHER)
    big = tr["lhs"] > 1e-9 * tr["lhs"].max()
    rel = np.abs(rep["trace_lhs"] - tr["lhs"]) / np.maximum(tr["lhs"], 1e-300)
    assert float(np.median(rel[big])) < 2.0 ** -7 and float(np.quantile(rel[big], 0.99)) < 0.2
    assert all(float(np.median(rel[big[:, m], m])) < 0.05 for m in range(M) if big[:, m].any())


# rows of more than 8192 columns: 9, 10 and 20 parts; widths that are no multiple of four
@pytest.mark.parametrize("p,M,phase", [(8193, 1, TOGETHER), (20479, 5, TOGETHER), (8193, 33, TOGETHER), (9300, 256, TOGETHER), (8196, 257, APART)])
def test_wide_rows(p, M, phase):
    _check(configs.CFG1.scaled(name="rule", layer_dims=(p,), M=M, N_m=12, B=4, K=6, D=4, rule=configs.RULE_CADA2, c=2e-3), phase, 1e-4, 1e-4)


# rows of up to 8192 columns whose server has a launch of its own: every variant, a share per worker and several, up to 256 workers; above, the last workgroup runs the rule
@pytest.mark.parametrize("rule", [configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_LAG], ids=["cada1", "cada2", "lag"])
@pytest.mark.parametrize("p,M,B,phase", [(54, 33, 130, TOGETHER), (256, 256, 65, TOGETHER), (300, 64, 130, TOGETHER), (512, 65, 130, TOGETHER), (512, 255, 33, TOGETHER), (784, 33, 130, TOGETHER),
                                         (784, 256, 40, TOGETHER), (1024, 64, 66, TOGETHER), (1024, 256, 33, TOGETHER), (1025, 256, 12, TOGETHER), (2049, 255, 12, TOGETHER), (4100, 256, 10, TOGETHER),
                                         (54, 257, 65, APART), (300, 512, 33, APART), (784, 257, 40, APART), (1025, 257, 12, APART), (2049, 512, 12, APART), (8191, 257, 10, APART)])
def test_rows(p, M, B, phase, rule):
    cfg = configs.CFG1.scaled(name="rule", layer_dims=(p,), M=M, N_m=B + 40, B=B, K=6, D=4, rule=rule, c=0.5 if p < 100 else 2e-3, server=1 if rule == configs.RULE_LAG else 0)
    prob = generators.make_problem(cfg)
    eng = binding.Cada.from_config(cfg, *upload(prob))
    assert binding.cada_profile_phase_names(eng.ctx) == ["logreg_rows", phase]
    eng.close()
    _check(cfg, phase, 1e-4, 1e-4)


def test_phase_names():
    """Whole steps and the paths whose gradient launches run the rule keep the phases that they had."""
    cfg = configs.CFG1.scaled(name="rule", layer_dims=(8192,), M=257, N_m=4, B=4, K=1)
    eng = binding.Cada.from_config(cfg, *upload(generators.make_problem(cfg)))
    assert binding.cada_profile_phase_names(eng.ctx) == ["logreg_rows", "server_update"]
    eng.close()


# the LAG rule's left-hand side in a launch of its own: blocks of 4096 coordinates read 16 bytes at a time, rows that end inside a block, an access, or in the first
@pytest.mark.parametrize("p,M,rule", [(1, 3, 3), (3, 2, 3), (7, 5, 0), (1023, 3, 3), (4095, 2, 3), (4096, 2, 0), (4099, 3, 3), (12290, 4, 3)])
def test_lag_left_hand_sides(p, M, rule):
    cfg = configs.CFG1.scaled(name="rule", layer_dims=(p,), M=M, N_m=60, B=9, K=8, D=4, rule=rule, c=0.5 if p < 100 else 2e-3, server=1 if rule == configs.RULE_LAG else 0)
    prob = generators.make_problem(cfg)
    prob.X *= np.float32(1.0 / np.sqrt(p))
    dev, sched = upload(prob), generators.make_schedule(cfg)
    check_protocol(cfg, prob, dev, sched, 1e-4, lhs_rtol=1e-4, path=binding.PATH_TWO_PASS, expect_phase="logreg_two_pass")


def test_lag_sums_keep_small_terms():
    """The rule compares sums of squares in double, and so are they added up inside a block of 4096 coordinates and handed on: two blocks of 1024 + 2^-14 (a float32 sum
    loses what it adds to a square of 1, and a float32 part half a unit in its last place) and one of 2^-14.  All values are powers of two, every gradient is exact."""
    p, M, B = 12288, 3, 128
    x = torch.zeros(p, device="cuda")
    x[:1024] = x[4096:5120] = 2.0
    x[1024:2048] = x[5120:6144] = x[8192:9216] = 2.0 ** -11
    eng = binding.Cada(model="logreg", layer_dims=[p], M=M, B=B, n_samples=[B] * M, X=x.repeat(M * B, 1).contiguous(), y=torch.ones(M * B, device="cuda"),
                       theta0=torch.zeros(p, device="cuda"), rule=configs.RULE_LAG, D=50, d_max=10, c=0.5, alpha=1.0, beta1=0.9, beta2=0.999, eps=1e-8, server=1,
                       trace_steps=1, path=binding.PATH_TWO_PASS)
    assert "logreg_two_pass" in binding.cada_profile_phase_names(eng.ctx)
    eng.step(torch.arange(B, dtype=torch.int32, device="cuda").repeat(M, 1).contiguous())
    lhs = eng.state()["trace_lhs"].cpu().numpy().ravel()
    eng.close()
    assert (lhs == np.float32(2048 + 3 * 2.0 ** -14)).all()


@pytest.mark.parametrize("dims,rule,store", [((617, 301, 150, 26), configs.RULE_LAG, 0), ((617, 301, 150, 26), configs.RULE_ALWAYS, 1), ((20, 33, 3), configs.RULE_LAG, 0),
                                             ((5, 3, 2), configs.RULE_ALWAYS, 1), ((200, 181, 7), configs.RULE_LAG, 0)])
def test_lag_left_hand_sides_of_networks(dims, rule, store):
    """Everybody uploads at every step: a left-hand side is then |gradient now - gradient of the step before|^2 of the stored rows, and float32 of a sum in double."""
    cfg = configs.CFG5.scaled(name="lag", layer_dims=dims, M=24, N_m=60, B=10, K=8, D=50, rule=rule, server=1 if rule == configs.RULE_LAG else 0)
    eng = binding.Cada.from_config(cfg, *upload(generators.make_problem(cfg)), trace_steps=cfg.K, gradient_store=store)
    everybody, before = torch.ones(cfg.M, dtype=torch.uint8, device="cuda"), np.zeros((cfg.M, cfg.p), np.float32)
    for k, idx in enumerate(generators.make_schedule(cfg)):
        eng.step(to_dev(idx.astype(np.int32)), everybody)
        now = eng.stored_gradients().cpu().numpy()
        got = eng.state()["trace_lhs"][k].cpu().numpy()
        want = ((now - before).astype(np.float64) ** 2).sum(axis=1)      # (the differences are float32, as in the kernel)
        # two sums in double of up to 240 thousand terms, and a pair of float32 per block: 2^-40 covers them
        assert ((got == np.float32(want * (1 - 2.0 ** -40))) | (got == np.float32(want * (1 + 2.0 ** -40)))).all(), (k, got, want)
        before = now
    eng.close()


# the right-hand side over rings that a wavefront takes in one round, in two, and in sixteen, before and after they have gone round
@pytest.mark.parametrize("dims,d_max,K", [((8193,), 1, 8), ((8193,), 64, 70), ((8196,), 65, 70), ((8193,), 1024, 20), ((60, 40, 5), 1, 6), ((60, 40, 5), 65, 70)])
def test_ring_lengths(dims, d_max, K):
    if len(dims) > 1:
        _check(configs.CFG5.scaled(name="ring", layer_dims=dims, M=3, N_m=30, B=6, K=K, D=9, d_max=d_max, c=20.0, rule=configs.RULE_CADA2), TOGETHER, 2e-2, None)
    else:
        _check(configs.CFG1.scaled(name="ring", layer_dims=dims, M=2, N_m=12, B=4, K=K, D=9, d_max=d_max, rule=configs.RULE_CADA2, c=2e-3), TOGETHER, 1e-4, 1e-4)
