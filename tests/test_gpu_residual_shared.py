"""Residual layers whose dense branch shares the launch of the experts' second product in the few-weights kernel, its sums combined
unrounded: tiles of 16, 32 and 64 rows on either side, one expert and all of them without rows for some, one and two choices, inner
dimensions of whole and ragged 32-deep blocks, plain and packed weights, and both sides of each bound of the rule -- through moe_layer_forward against the oracle."""
import pytest

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# T, d, f, E, top_k, capacity, shared on plain, on packed weights
CASES = [(1, 128, 256, 2, 1, 1, True, True), (2, 256, 512, 8, 2, 1, True, True), (16, 136, 264, 4, 1, 8, True, True), (17, 128, 1024, 4, 2, 17, False, True),
         (33, 256, 520, 16, 1, 3, True, True), (64, 512, 2048, 8, 1, 16, True, True), (65, 128, 512, 4, 2, 16, False, True), (100, 264, 1032, 32, 1, 1, False, True),
         (256, 128, 1024, 16, 1, 16, False, True),
         (1, 1040, 4096, 8, 2, 1, True, True), (4, 1040, 4096, 8, 1, 1, False, False), (9, 1040, 4096, 8, 1, 2, False, True),
         (16, 1040, 2048, 8, 1, 2, False, False), (120, 1040, 4096, 12, 1, 12, False, True), (129, 1040, 4096, 12, 1, 12, False, False),
         (200, 1024, 4096, 16, 1, 16, False, True), (215, 1024, 4096, 16, 1, 16, False, False), (40, 2056, 8192, 4, 1, 10, False, True),
         (128, 1024, 1024, 16, 1, 16, False, True), (129, 1024, 1024, 16, 1, 16, False, False), (1, 2048, 2040, 2, 1, 1, False, False), (1, 2048, 2048, 2, 1, 1, True, False)]


@pytest.mark.parametrize("T,d,f,E,k,C,plain,packed", CASES)
def test_shared_second_products(T, d, f, E, k, C, plain, packed):
    print(f"case T={T} d={d} f={f} E={E} k={k} C={C}", flush=True)
    assert [plan(T, d, f, E, k, C, True, p)[0][3] < 0 for p in (False, True)] == [plain, packed]
    cfg = CONFIGS["c3a"].scaled(name="shared", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=True, seed=13)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)
