"""The decode block where sums that were launches of their own are part of another kernel: the projection's split-K sums in the
LayerNorm (from 33 tokens on; rows of one and of two pieces per thread), and the residual add in the last kernel of the MoE layer -- the
scatter of the expert kernels (few-weights, streaming with split K, tiled), dropped tokens, the top-2 combine, the dense branch's
combine in its product (100 tokens) and behind products that share a launch in the few-weights kernel, and the pair of tiled products that
keeps its add -- against the oracle."""
import pytest

from tests.plan_util import plan
from tests.test_gpu_block import DEV, _check_block
from workloads import CONFIGS, make_block_inputs

pytestmark = pytest.mark.gpu

# T, d, f, E, top_k, capacity factor, residual, heads, room for positions
CASES = [
    (3, 128, 256, 4, 1, 0.5, False, 2, 70), (40, 128, 256, 4, 1, 0.5, False, 1, 300), (64, 256, 2048, 4, 1, 1.0, False, 2, 256),
    (200, 128, 256, 2, 1, 1.5, False, 2, 40), (90, 2176, 256, 2, 1, 1.0, False, 17, 20), (33, 256, 512, 4, 2, 1.0, False, 4, 257),
    (1, 128, 256, 2, 1, 1.0, True, 1, 9), (33, 128, 512, 4, 1, 1.0, True, 2, 33), (100, 256, 512, 4, 2, 0.5, True, 2, 33),
    (140, 256, 512, 2, 1, 1.0, True, 2, 16),
]


@pytest.mark.parametrize("T,d,f,E,k,cf,residual,heads,room", CASES)
def test_block(T, d, f, E, k, cf, residual, heads, room):
    print(f"case T={T} d={d} f={f} E={E} k={k} cf={cf} residual={residual}", flush=True)
    cfg = CONFIGS["c4"].scaled(name="b-sums", T=T, d_model=d, d_ffn=f, E=E, top_k=k, capacity_factor=cf, residual=residual, seed=6)
    kernels, shared = plan(T, d, f, E, k, cfg.capacity, residual)
    assert bool(shared[1] or kernels[3] < 0) == (residual and T != 100)     # second products in one launch
    print(_check_block(make_block_inputs(cfg, heads, room, DEV)), flush=True)
