"""fp32 layers with d_model up to 64 and d_ffn up to 256, whose two products are one launch: the edges of its row tiles, of 32 columns per
wave and of 16-deep blocks of K; the last shapes that it takes, the first ones beyond, and what those go to."""
import pytest

from tests import gpu_util as U
from tests.test_gpu_nonfinite import test_infinity_in_the_last_weight_row as infinity_in_the_last_weight_row
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# capacity, T, d, f, E, top_k, residual
CASES = [
    (1, 1, 64, 256, 8, 1, False), (16, 60, 64, 252, 3, 2, True), (17, 60, 60, 256, 3, 1, True), (31, 100, 52, 36, 4, 1, False),
    (32, 100, 16, 32, 4, 2, False), (33, 100, 12, 28, 3, 1, False), (65, 300, 64, 196, 5, 2, True), (1024, 2500, 64, 228, 32, 1, False),
    (1025, 2500, 64, 228, 32, 1, False), (40, 100, 68, 256, 3, 1, True), (40, 100, 64, 260, 3, 1, True), (65, 6000, 64, 260, 180, 1, False),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", CASES)
def test_f32_narrow_layer(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c1"].scaled(name="f32", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=6)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


@pytest.mark.parametrize("C,d,f", [(12, 64, 252), (40, 52, 36), (12, 68, 264), (16, 84, 72), (30, 100, 132), (60, 68, 100)])
@pytest.mark.parametrize("second", [False, True])
def test_infinity_in_the_last_weight_row(C, d, f, second):
    infinity_in_the_last_weight_row("f32", C, d, f, second)
