"""The few-weights bf16 kernel (decode steps, dense branches) at the edges of its tiles: 16, 32 and 64 rows, 16, 32 and
64 columns per work-group, ragged K and N, K of less than a block per wave, plain and packed weights, shared launches,
through moe_layer_forward against the oracle."""
import pytest

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# capacity, T, d, f, E, top_k, residual
CASES = [
    (1, 1, 8, 8, 1, 1, False), (1, 1, 1024, 4096, 3, 1, False), (2, 3, 40, 136, 4, 2, False), (16, 16, 512, 2056, 2, 1, True),
    (15, 17, 296, 1160, 3, 1, True), (8, 8, 256, 2048, 8, 1, False), (16, 33, 264, 520, 4, 2, True), (5, 64, 128, 10248, 16, 1, True),
    (17, 40, 96, 8192, 3, 1, True), (33, 65, 136, 8200, 2, 1, True), (64, 130, 72, 4104, 3, 2, True), (64, 200, 1024, 640, 4, 1, True),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", CASES)
def test_few_weights_layer(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c4"].scaled(name="rows", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=6)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)
