"""Routing from logits that hold -inf (masked experts) and NaN: every table entry stays inside the experts and tokens."""
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,E,T", [(2, 8, 40), (2, 20, 300), (1, 128, 256), (2, 128, 700), (2, 200, 90)])
def test_masked_and_nan_logits(k, E, T):
    print(f"case k={k} E={E} T={T}", flush=True)
    g = torch.Generator().manual_seed(E + T)
    logits = torch.full((T, E), float("-inf"))
    only = torch.randint(1, E, (T,), generator=g)
    logits[torch.arange(T), only] = torch.randn((T,), generator=g)      # one expert left: the second choice is the lowest other
    logits[3] = float("nan")
    logits[4] = float("-inf")
    res = U.gpu_route(logits.cuda(), k, T)
    idx, slot, rows = (res[n].cpu() for n in ("expert_idx", "slot_idx", "expert_rows"))
    live = torch.ones(T, dtype=torch.bool)
    live[3:5] = False
    assert torch.equal(idx[live, 0].long(), only[live])
    assert torch.equal(res["gate_w"].cpu()[live, 0], torch.ones(int(live.sum())))
    assert idx[4].tolist() == list(range(k))
    if k == 2:
        assert (idx[live, 1] == 0).all() and (res["gate_w"].cpu()[live, 1] == 0).all()
    assert ((idx >= 0) & (idx < E)).all()
    assert torch.equal(torch.bincount(idx.reshape(-1).long(), minlength=E), rows.long())
    pairs = idx.long() * T + slot.long()                                # nothing dropped: all (expert, slot) pairs differ
    assert (slot >= 0).all() and pairs.unique().numel() == T * k
