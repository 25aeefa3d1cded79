"""Tiled kernel: every tile shape with every epilogue that it can have in a layer, plain and packed weights, whole and ragged
inner dimensions, one product and two in a launch -- each case says which kernel it is there for, and the dispatch is asked
whether it takes it -- through moe_layer_forward against the oracle."""
import pytest

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu
T256, T256N, T128, T128X2, T128N = 256256, 256128, 128256, 128257, 128128
GEMM1, GEMM2, DENSE1, DENSE2 = range(4)

# capacity, T, d, f, E, top_k, residual, product, kernel, two products in the launch
CASES = [
    (257, 2056, 64, 1000, 16, 1, False, GEMM1, T256N, False), (257, 2056, 1000, 64, 16, 1, False, GEMM2, T256N, False),
    (257, 1028, 1000, 64, 16, 2, False, GEMM2, T256N, False), (150, 4500, 40, 1000, 32, 1, False, GEMM1, T256N, False),
    (160, 4500, 1000, 40, 32, 1, False, GEMM2, T256N, False), (130, 2000, 1000, 72, 32, 2, False, GEMM2, T256N, False),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual,product,kernel,shared", CASES)
def test_tile_choice(C, T, d, f, E, k, residual, product, kernel, shared):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    for packed in (False, True):
        kernels, both = plan(T, d, f, E, k, C, residual, packed)
        assert kernels[product] == kernel and bool(both[product % 2]) == shared
    cfg = CONFIGS["c3a"].scaled(name="choice", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=10)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)
