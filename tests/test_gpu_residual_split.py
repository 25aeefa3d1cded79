"""Residual layers of 33 (packed weights: 41) to 192 tokens whose dense branch's second product runs on the streaming kernel with K split, the combine adding its
sums up: tiles of 64 rows whole and ragged, columns off 128, an inner dimension off 32, one and two choices, with and without
biases, plain and packed weights -- through moe_layer_forward against the oracle; and the first lengths on either side."""
import pytest

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# T, d, f, E, top_k, capacity, dense second product split on plain, on packed weights
CASES = [(32, 128, 8192, 2, 2, 32, False, False), (33, 128, 8192, 2, 2, 33, True, False), (40, 128, 8192, 2, 2, 40, True, False),
         (41, 128, 8192, 2, 2, 41, True, True), (33, 128, 4096, 2, 2, 33, True, False),
         (48, 136, 8200, 1, 1, 40, True, True), (49, 128, 4096, 2, 2, 49, True, True), (64, 264, 4104, 2, 2, 64, True, True),
         (65, 128, 4096, 4, 2, 40, True, True), (129, 200, 4096, 2, 2, 64, True, True), (190, 128, 5000, 8, 1, 64, True, True),
         (192, 256, 4096, 4, 2, 64, True, True), (193, 128, 4096, 8, 1, 64, False, False), (40, 128, 4088, 2, 2, 40, False, False)]


@pytest.mark.parametrize("bias", [0.05, None])
@pytest.mark.parametrize("T,d,f,E,k,C,plain,packed", CASES)
def test_split_dense_product(T, d, f, E, k, C, plain, packed, bias):
    print(f"case T={T} d={d} f={f} E={E} k={k} C={C} bias={bias}", flush=True)
    kernels = [plan(T, d, f, E, k, C, True, p)[0][3] for p in (False, True)]
    assert [c >= 200 and c % 100 in (32, 64) for c in kernels] == [plain, packed]
    cfg = CONFIGS["c3a"].scaled(name="split", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=True, seed=14)
    inp = make_inputs(cfg, "cuda", bias_std=bias or 0.0)
    if bias is None:
        inp.bd2 = None
    U.check_layer(inp, capacity=C)
