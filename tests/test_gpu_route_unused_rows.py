"""Routing of at most 256 tokens: the rows of slot_token without a token, on both sides of the number of experts from which an expert's rows
are a wave's work -- one row per expert, fewer and more than a wave has lanes, off powers of two -- tables equal to the oracle's."""
import pytest
import torch

from oracle import moe_oracle as orc
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 127, 128, 129, 300, 512, 1000, 1024])
@pytest.mark.parametrize("T,k,C", [(1, 1, 1), (200, 2, 3), (256, 1, 64), (77, 2, 77), (256, 2, 300)])
def test_unused_rows(E, T, k, C):
    k = min(k, E)
    print(f"case T={T} E={E} k={k} C={C}", flush=True)
    logits = torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(E + T), device="cuda")
    U.assert_routing_equal(U.gpu_route(logits, k, C), orc.gate(logits.cpu().numpy(), k, C))
