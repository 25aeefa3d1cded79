"""The decode block where sums that were launches of their own are part of another kernel: the projection's split-K sums in the
LayerNorm (from 33 tokens on; rows of one and of two pieces per thread), and the residual add in the last kernel of the MoE layer -- the
scatter of the expert kernels (few-weights, streaming, whole and with split K), dropped tokens, the top-2 combine, the dense branch's
combine in its product, behind products that share a launch in the few-weights kernel and behind a product with split K -- and the tiled
products, alone and as a pair, that keep their add -- against the oracle."""
import pytest

from tests.plan_util import plan
from tests.test_gpu_block import DEV, _check_block
from workloads import CONFIGS, make_block_inputs

pytestmark = pytest.mark.gpu

# T, d, f, E, top_k, capacity factor, residual, heads, room for positions; second products of experts and dense branch, plain / packed weights
CASES = [
    (3, 128, 256, 4, 1, 0.5, False, 2, 70, "rows", "rows"), (40, 128, 256, 4, 1, 0.5, False, 1, 300, "rows", "rows"),
    (64, 256, 2048, 4, 1, 1.0, False, 2, 256, "rows", "rows"), (200, 128, 256, 2, 1, 1.5, False, 2, 40, "tiled", "tiled"),
    (90, 2176, 256, 2, 1, 1.0, False, 17, 20, "split", "rows"), (100, 256, 2048, 4, 1, 0.8, False, 2, 20, "split", "split"),
    (64, 2048, 128, 96, 1, 1.0, False, 16, 40, "whole", "whole"), (33, 256, 512, 4, 2, 1.0, False, 4, 257, "split", "rows"),
    (1, 128, 256, 2, 1, 1.0, True, 1, 9, "rows+sums", "rows+sums"), (33, 128, 512, 4, 1, 1.0, True, 2, 33, "rows+sums", "rows+sums"),
    (100, 256, 512, 4, 2, 0.5, True, 2, 33, "split+rows", "split+rows"), (140, 256, 512, 2, 1, 1.0, True, 2, 16, "pair", "pair"),
    (100, 256, 4096, 4, 1, 0.8, True, 2, 33, "split+split", "split+split"), (64, 128, 4096, 2, 2, 0.7, True, 1, 20, "split+split", "split+split"),
]


def second_products(cfg, packed):
    kernels, shared = plan(cfg.T, cfg.d_model, cfg.d_ffn, cfg.E, cfg.top_k, cfg.capacity, cfg.residual, packed)
    if shared[1]:
        return "pair"
    names = ["sums" if c < 0 else "rows" if c < 100 else "whole" if c < 200 else "split" if c < 1000 else "tiled" for c in kernels]
    return names[1] + ("+" + names[3] if cfg.residual else "")


@pytest.mark.parametrize("T,d,f,E,k,cf,residual,heads,room,plain,packed", CASES)
def test_block(T, d, f, E, k, cf, residual, heads, room, plain, packed):
    print(f"case T={T} d={d} f={f} E={E} k={k} cf={cf} residual={residual}", flush=True)
    cfg = CONFIGS["c4"].scaled(name="b-sums", T=T, d_model=d, d_ffn=f, E=E, top_k=k, capacity_factor=cf, residual=residual, seed=6)
    assert [second_products(cfg, p) for p in (False, True)] == [plain, packed]
    bi = make_block_inputs(cfg, heads, room, DEV)
    stats = _check_block(bi)
    print(stats, flush=True)
    if cf < 1.0 and k == 1:
        assert stats["kept"] < T                                  # tokens without an expert: their rows are x1 (and the dense branch)
