"""Networks whose loss and last weight gradient share a launch (at most 32 rows per worker, at most 256 workgroups of 32 units, one more per worker), at both sides of both lines, and hidden
layers whose small forward products take four wavefronts per workgroup (more than 512 blocks of 32 x 32, at most 512 inputs), against the oracle."""
import numpy as np
import pytest

from cada_synth import configs, generators

from common import check_protocol, upload

pytestmark = pytest.mark.gpu

# 1, 31, 32 and 33 rows; one unit and no multiple of 32 of them; 255 workgroups (51 workers), 256 and 264 (193 and 224 units), 288 and 297; 512 blocks of the forward product and 544, 1024 inputs and 1025
SHAPES = [((40, 33, 5), 3, 1), ((50, 1, 2), 4, 31), ((60, 70, 32), 5, 32), ((60, 70, 32), 5, 33), ((30, 97, 6), 51, 9), ((30, 225, 3), 32, 9), ((30, 225, 3), 33, 9), ((30, 193, 3), 32, 9), ((30, 224, 3), 32, 9), ((30, 224, 3), 33, 9), ((40, 50, 65, 7), 8, 20),
          ((64, 512, 4), 32, 12), ((64, 513, 4), 32, 12), ((1024, 256, 4), 65, 8), ((1025, 256, 4), 65, 8)]


@pytest.mark.parametrize("rule", [configs.RULE_CADA1, configs.RULE_CADA2, configs.RULE_ALWAYS], ids=["cada1", "cada2", "always"])
@pytest.mark.parametrize("dims,M,B", SHAPES)
def test_against_the_oracle(dims, M, B, rule):
    cfg = configs.CFG5.scaled(name="loss", layer_dims=dims, M=M, N_m=B + 20, B=B, K=5, D=3, c=20.0, rule=rule)
    prob = generators.make_problem(cfg)
    # (bounds of test_gpu_rule_in_server: split bf16 products, left-hand sides of single bf16 ones)
    stats, o, tr, rep = check_protocol(cfg, prob, upload(prob), generators.make_schedule(cfg), 2e-2, lhs_rtol=None, own_mask_exact=False, free_margin=None)
    if rule != configs.RULE_ALWAYS:
        big = tr["lhs"] > 1e-9 * tr["lhs"].max()
        rel = np.abs(rep["trace_lhs"] - tr["lhs"]) / np.maximum(tr["lhs"], 1e-300)
        assert float(np.median(rel[big])) < 2.0 ** -7 and float(np.quantile(rel[big], 0.99)) < 0.2
