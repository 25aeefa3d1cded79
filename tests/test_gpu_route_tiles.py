"""Routing of more than 256 tokens: the histograms of the tiles before a block's own are summed sixteen rows at a time and what is left in
powers of two -- numbers of tiles with each of these, all and none of them, with a ragged last one and a row group less --
tables equal to the oracle's."""
import pytest
import torch

from oracle import moe_oracle as orc
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


# 256 columns: four row groups of tiles of 32 tokens
@pytest.mark.parametrize("tiles", [9, 12, 16, 21, 32, 33, 63, 64, 65, 95, 96, 127, 128, 190])
def test_sums_over_tiles(tiles):
    T, E, k = 32 * tiles - 5, 128, 2
    print(f"case T={T} tiles={tiles}", flush=True)
    logits = torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(tiles), device="cuda")
    logits += torch.linspace(0.0, 2.0, E, device="cuda")
    U.assert_routing_equal(U.gpu_route(logits, k, T // 64), orc.gate(logits.cpu().numpy(), k, T // 64))
