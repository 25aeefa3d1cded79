"""Routing of many tokens from given logits, on both sides of the size from which tiles hold 256 tokens: tables equal to the
oracle's, with a last tile that is full, nearly empty or of an odd size, experts below and above what fits in registers."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k", [(32767, 64, 2), (32768, 128, 2), (32769, 16, 1), (33000, 200, 2), (40001, 1024, 1), (131072 + 77, 7, 2),
                                   (70000, 31, 1), (36864, 1024, 2)])
def test_routing_of_many_tokens(T, E, k):
    print(f"case T={T} E={E} k={k}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + E)
    logits = torch.randn((T, E), generator=gen, device="cuda")
    logits[::5] = logits[::5].round()                       # ties
    C = max(1, (T * k) // E)
    U.assert_routing_equal(U.gpu_route(logits, k, C), orc.gate(logits.cpu().numpy(), k, C))
