"""fp32 layers at the edges of the fp32 kernels' tiles: 16, 32 and 64 rows, 64 and 128 columns, 16- and 32-deep blocks
of K, one row more or less, through moe_layer_forward (gather, GELU, scatter / combine epilogues) against the oracle."""
import pytest

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# capacity (selects the kernel), T, d, f, E, top_k, residual
CASES = [
    (1, 1, 4, 4, 1, 1, False), (3, 9, 20, 68, 4, 2, False), (16, 40, 64, 60, 3, 1, False), (17, 40, 132, 128, 3, 1, True),
    (32, 70, 48, 196, 2, 2, True), (33, 70, 64, 64, 2, 1, False), (64, 200, 36, 132, 3, 2, False), (65, 140, 100, 256, 2, 1, True),
    (129, 300, 60, 124, 2, 1, False), (300, 700, 256, 516, 3, 2, True),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", CASES)
def test_f32_layer(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c1"].scaled(name="f32", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=5)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


# the same with more than 512 tiles of 32 x 64 in one or both expert products, or in the dense branch's (fewer of them are
# another kernel's): 64- and 128-row tiles, one row more or less, and the last launch of the few (512 tiles)
MANY_TILES = [
    (33, 400, 64, 516, 32, 1, False), (65, 900, 60, 772, 14, 2, True), (129, 2600, 196, 132, 26, 1, False),
    (65, 5000, 64, 68, 180, 1, False), (1030, 4100, 196, 132, 4, 1, True), (128, 500, 132, 256, 4, 1, False),
    (512, 1500, 64, 512, 4, 1, False),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", MANY_TILES)
def test_f32_layer_many_tiles(C, T, d, f, E, k, residual):
    test_f32_layer(C, T, d, f, E, k, residual)
