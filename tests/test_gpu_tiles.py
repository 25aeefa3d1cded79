"""The tiled kernel at the edges of its tiles (rows, columns, an inner dimension that ends inside a stage), one product and two
in a launch, through moe_layer_forward against the oracle, plain and packed weights.  Which tile shape a case gets is the
dispatch's business here; test_gpu_tile_choice.py takes every shape with every epilogue."""
import pytest

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# capacity, T, d, f, E, top_k, residual
CASES = [
    (65, 150, 128, 256, 3, 1, False), (127, 300, 96, 136, 2, 2, False), (128, 300, 160, 264, 4, 1, True), (129, 400, 128, 1032, 3, 1, False),
    (257, 1100, 64, 520, 4, 1, False), (383, 1500, 96, 128, 3, 2, False), (120, 2300, 1024, 64, 16, 1, True),
    (200, 3000, 128, 4096, 16, 1, False),          # 256 x 256 tiles, one round, and 128 x 128 ones
    (313, 4000, 64, 8200, 12, 1, False), (320, 2600, 128, 8192, 6, 1, True), (256, 1300, 64, 4104, 4, 1, True),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", CASES)
def test_tiled_layer(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c3a"].scaled(name="tiles", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=7)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


# the inner dimension ends inside a 32-deep stage, in the first product (d) or the second (f)
RAGGED = [(70, 200, 8, 72, 3, 1, False), (130, 300, 40, 104, 3, 1, True), (300, 700, 1000, 264, 3, 2, False),
          (256, 1100, 72, 1000, 5, 1, True), (200, 3000, 120, 4104, 16, 1, False), (100, 500, 200, 3016, 8, 2, True)]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", RAGGED)
def test_tiled_layer_ragged_k(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c3a"].scaled(name="tiles", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=8)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)
