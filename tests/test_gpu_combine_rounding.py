"""Residual layers with experts of few rows: the gate-weighted expert rows are added to the dense branch's fp32 sums, which are
rounded to bf16 once.  All operands are chosen so that every value before that rounding is exact (first halves with zero weights
and a bias of 32, where GELU is the identity; multiples of 1/32 as second weights; gate weights of 1 or 1/2), so the result is
the exact sum rounded once; sums that were rounded before the addition differ in a large share of the elements."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan

CASES = [   # capacity, T, d, f, E, top_k: packed weights put the experts on tiles in one or both products, or not
    (33, 1000, 2048, 128, 64, 1), (3, 129, 1024, 128, 128, 2), (32, 1030, 1024, 160, 130, 1), (16, 1030, 1000, 72, 130, 2),
    (64, 700, 256, 128, 16, 1), (2, 100, 512, 64, 64, 1), (40, 256, 2048, 64, 64, 2),
]


@pytest.mark.parametrize("C,T,d,f,E,k", CASES)
def test_second_halves_stay_apart(C, T, d, f, E, k):
    """A shared launch of the second halves would leave rounded dense sums to the combine."""
    for packed in (False, True):
        assert not plan(T, d, f, E, k, C, True, packed)[1][1]


@pytest.mark.gpu
@pytest.mark.parametrize("C,T,d,f,E,k", CASES)
def test_one_rounding(C, T, d, f, E, k):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k}", flush=True)
    m, bf = U.amd(), torch.bfloat16
    gen = torch.Generator().manual_seed(C)

    def ints(lim, *shape):
        return torch.randint(-lim, lim + 1, shape, generator=gen, dtype=torch.float32)

    token = torch.arange(T)
    x, Wg = torch.zeros((T, d)), torch.zeros((d, E))
    Wg[torch.arange(E), torch.arange(E)] = 200.0                # all other experts' probabilities vanish in fp32
    for j in range(k):
        x[token, (token + j) % E] = 1.0
    W2 = torch.zeros((E, f, d))
    W2[:, :4] = ints(60, E, 4, d) / 32                          # expert outputs: integers up to 240, exact in bf16
    Wd2, bd2 = ints(120, f, d) / 32, ints(100, d)               # dense sums: integers of some hundreds up to thousands
    one = dict(b1=torch.full((E, f), 32.0), b2=torch.zeros((E, d)), bd1=torch.full((f,), 32.0))
    put = {n: v.to(bf).cuda() for n, v in dict(one, W1=torch.zeros((E, d, f)), W2=W2, Wd1=torch.zeros((d, f)), Wd2=Wd2, bd2=bd2).items()}
    dense, ye = 32 * Wd2.sum(0) + bd2, 32 * W2.sum(1)
    assert ye.abs().max() <= 256 and dense.abs().max() < 2 ** 20
    for packed in (False, True):
        layer = m.MoELayer(T, d, f, E, k, C, "bf16", Wg.cuda(), None, put["W1"], put["b1"], put["W2"], put["b2"], put["Wd1"],
                           put["bd1"], put["Wd2"], put["bd2"], pack_weights=packed)
        out = layer(x.to(bf).cuda()).float().cpu()
        slot, expert = layer.routing["slot_idx"].cpu(), layer.routing["expert_idx"].cpu().long()
        assert torch.equal(layer.routing["gate_w"].cpu(), torch.full((T, k), 1.0 / k))
        kept = (slot >= 0).float() / k
        exact = dense + (kept[:, :, None] * ye[expert]).sum(1)
        once, twice = exact.to(bf).float(), (dense.to(bf).float() + (exact - dense)).to(bf).float()
        assert (once != twice).float().mean() > 0.05            # the inputs tell the two apart
        assert torch.equal(out, once), f"packed={packed}: {(out != once).float().mean().item():.3f} differ"
