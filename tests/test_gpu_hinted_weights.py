"""Weights of more than 128 MB on the four-wave tile kernel, which reads them with the non-temporal hint where one row tile needs
them: every epilogue that has the hint (GELU, scatter, store), tiles of 128 and of 256 rows, inner dimensions of whole 64-deep
chunks, of half of one and ragged, all groups with the hint or each as its rows ask for (groups on both sides of 256 rows), and
pairs with a dense branch, through moe_layer_forward against the oracle."""
import pytest

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu
H128, H256, GROUP = 128259, 256259, 256260
WHOLE, HALF, RAGGED = (1024, 1088), (1056, 1056), (1032, 1032)

# (d, f), capacity, T, E, top_k, residual, first and second product
CASES = [(K, C, T, 64, k, False, kernel, kernel) for K in (WHOLE, RAGGED)
         for C, T, k, kernel in ((100, 4000, 1, H128), (100, 2000, 2, H128), (200, 9000, 1, H256), (200, 4500, 2, H256),
                                 (300, 16768, 1, GROUP), (300, 8384, 2, GROUP))]
CASES += [(HALF, 100, 4000, 64, 1, False, H128, H128), (HALF, 200, 4500, 64, 2, False, H256, H256),
          (HALF, 300, 16768, 64, 1, False, GROUP, GROUP),
          (WHOLE, 100, 9000, 64, 1, True, GROUP, GROUP), (WHOLE, 300, 8384, 64, 2, True, GROUP, GROUP),
          ((1032, 520), 24, 2400, 128, 1, False, H128, H128), ((1024, 528), 40, 2200, 128, 2, False, H128, H128)]


@pytest.mark.parametrize("K,C,T,E,k,residual,first,second", CASES)
def test_hinted_layer(K, C, T, E, k, residual, first, second):
    (d, f) = K
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    assert plan(T, d, f, E, k, C, residual, packed=True)[0][:2] == [first, second]
    cfg = CONFIGS["c3a"].scaled(name="hint", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=12)
    inp = make_inputs(cfg, "cuda", bias_std=0.05)
    U.check_layer(inp, capacity=C, lazy_experts=True)
