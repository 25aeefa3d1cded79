"""Masked experts (bias -inf) and a NaN token through the whole gate from tokens: the decode gate (up to 256 tokens), logits and
routing as kernels of their own, and the fused gate (2048 and more) each have their own publishing and histogram code; every
table entry stays inside the experts and tokens."""
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2])
@pytest.mark.parametrize("T,E", [(40, 8), (256, 128), (17, 20), (700, 64), (2300, 128), (2300, 20), (20000, 33)])
def test_masked_experts_and_nan_tokens(T, E, k):
    print(f"case T={T} E={E} k={k}", flush=True)
    m, d, only = U.amd(), 64, E // 2
    gen = torch.Generator(device="cuda").manual_seed(T + E)
    x = torch.randn((T, d), generator=gen, device="cuda").to(torch.bfloat16)
    x[3], x[T - 1] = float("nan"), float("nan")
    Wg = torch.randn((d, E), generator=gen, device="cuda") * 0.1
    bg = torch.full((E,), float("-inf"), device="cuda")
    bg[only] = 0.5
    shape = m.make_shape(T, d, 8, E, k, T, "bf16")
    i32, f32 = torch.int32, torch.float32
    logits, idx, slot, gw, rows, table = [torch.full(s, -7, dtype=t, device="cuda") for s, t in
                                          (((T, E), f32), ((T, k), i32), ((T, k), i32), ((T, k), f32), ((E,), i32), ((E, T), i32))]
    m.moe_gate(shape, x, Wg, bg, logits, idx, slot, gw, rows, table, m.alloc_workspace(shape, "cuda"))
    torch.cuda.synchronize()
    logits, idx, slot, gw, rows, table = (t.cpu() for t in (logits, idx, slot, gw, rows, table))
    live = torch.ones(T, dtype=torch.bool)
    live[3] = live[T - 1] = False
    assert bool(torch.isnan(logits[~live]).all()) and bool((logits[live][:, torch.arange(E) != only] == float("-inf")).all())
    assert bool((idx[live, 0] == only).all()) and bool((gw[live, 0] == 1).all())
    if k == 2:                                             # nothing else is left: the lowest other expert, with weight 0
        assert bool((idx[live, 1] == (1 if only == 0 else 0)).all()) and bool((gw[live, 1] == 0).all())
    assert bool(((idx >= 0) & (idx < E)).all())
    assert torch.equal(torch.bincount(idx.reshape(-1).long(), minlength=E), rows.long())
    assert bool((slot >= 0).all()) and (idx.long() * T + slot.long()).unique().numel() == T * k
    tokens = torch.arange(T, dtype=torch.int32)[:, None].expand(T, k).reshape(-1)
    assert torch.equal(table[idx.reshape(-1).long(), slot.reshape(-1).long()], tokens)
    assert bool((table[torch.arange(T)[None, :] >= rows[:, None]] == -1).all())
