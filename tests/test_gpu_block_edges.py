"""The decode block where its kernels change path: more than eight attention chunks, rows of 1152, 2176 and 4224 elements
(one, two and too many pieces per thread of the LayerNorm), and caches whose unused rows hold NaN."""
import pytest
import torch

from tests.test_gpu_block import DEV, _check_block, _run_block
from workloads import CONFIGS, make_block_inputs

pytestmark = pytest.mark.gpu

CASES = {
    "chunks": (CONFIGS["c4"].scaled(name="b-chunks", T=12, d_model=128, d_ffn=256, E=4, capacity_factor=4.0), 2, 2500),
    "d1152": (CONFIGS["c4"].scaled(name="b-1152", T=5, d_model=1152, d_ffn=256, E=4, capacity_factor=4.0), 9, 130),
    "d2176": (CONFIGS["c4"].scaled(name="b-2176", T=3, d_model=2176, d_ffn=256, E=2, capacity_factor=2.0), 17, 66),
    "d4224": (CONFIGS["c4"].scaled(name="b-4224", T=3, d_model=4224, d_ffn=256, E=2, capacity_factor=2.0), 33, 33),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_decode_block_edges(name):
    cfg, heads, max_len = CASES[name]
    print(name, _check_block(make_block_inputs(cfg, heads, max_len, DEV)), flush=True)


def test_unused_cache_rows_are_never_used():
    cfg, heads, max_len = CASES["chunks"]
    bi = make_block_inputs(cfg, heads, max_len, DEV)
    assert int(bi.pos.min()) == 0                     # a sequence without any cached position is among them
    ref = _run_block(bi, False)
    rows = torch.arange(max_len, device=DEV)[None, None, :, None] >= bi.pos[:, None, None, None]
    for cache in (bi.k_cache, bi.v_cache):
        cache.masked_fill_(rows, float("nan"))
    res = _run_block(bi, False)
    assert torch.equal(ref["out"], res["out"]) and torch.equal(ref["x1"], res["x1"])


def test_decode_block_large_cache():
    """Caches of more than 256 MB together are read with the non-temporal hint; here with 64 elements per head."""
    cfg = CONFIGS["c4"].scaled(name="b-large", T=33, d_model=1024, d_ffn=256, E=4, capacity_factor=4.0)
    print(_check_block(make_block_inputs(cfg, 16, 2200, DEV), packed_too=False), flush=True)
