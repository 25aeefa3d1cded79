"""fp32 layers with d_model up to 64 and d_ffn up to 256, whose two products are one launch: the edges of its row tiles, of 32 columns per
wave and of 16-deep blocks of K; the last shapes that it takes, the first ones beyond, and what those go to."""
import pytest
import torch

from tests import gpu_util as U
from tests.test_gpu_nonfinite import test_infinity_in_the_last_weight_row as infinity_in_the_last_weight_row
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# capacity, T, d, f, E, top_k, residual
CASES = [
    (1, 1, 64, 256, 8, 1, False), (16, 60, 64, 252, 3, 2, True), (17, 60, 60, 256, 3, 1, True), (31, 100, 52, 36, 4, 1, False),
    (32, 100, 16, 32, 4, 2, False), (33, 100, 12, 28, 3, 1, False), (65, 300, 64, 196, 5, 2, True), (1024, 2500, 64, 228, 32, 1, False),
    (1025, 2500, 64, 228, 32, 1, False), (40, 100, 68, 256, 3, 1, True), (40, 100, 64, 260, 3, 1, True), (65, 6000, 64, 260, 180, 1, False),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual", CASES)
def test_f32_narrow_layer(C, T, d, f, E, k, residual):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    cfg = CONFIGS["c1"].scaled(name="f32", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=6)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


@pytest.mark.parametrize("C,d,f", [(12, 64, 252), (40, 52, 36), (12, 68, 264), (16, 84, 72), (30, 100, 132), (60, 68, 100)])
@pytest.mark.parametrize("second", [False, True])
def test_infinity_in_the_last_weight_row(C, d, f, second):
    infinity_in_the_last_weight_row("f32", C, d, f, second)


def _chains(a, b, bias):
    """a b + bias in fp32, K in chains of 16 fused multiply-adds and the chains added in turn."""
    total = None
    for k0 in range(0, a.shape[-1], 16):
        acc = torch.zeros(*a.shape[:-1], b.shape[-1], device=a.device)
        for k in range(k0, min(k0 + 16, a.shape[-1])):
            acc = (acc.double() + a[..., k:k + 1].double() * b[..., k:k + 1, :].double()).float()
        total = acc if total is None else total + acc
    return total + bias


@pytest.mark.parametrize("one_sided", [True, False])
@pytest.mark.parametrize("d,f", [(20, 36), (64, 64), (40, 160), (64, 256)])
def test_rounding_of_both_sums(d, f, one_sided):
    """No further from 64 bits than chains of 16 products.  Rounding adds to a chain's variance with the square of the sum so far: 1 + 2 + .. + n
    for products of either sign, 1 + 4 + .. + n^2 for those of one.  Chains of 32 have 1.9 and 3.8 times that of two chains of 16; in the
    result, beside the first product's errors and the last roundings, 1.12 to 1.40 times the error (f up to 160).  The device's sums of 16
    are in another order than the ones here: 1.05 at most, so the line is at 1.1."""
    print(f"case d={d} f={f} one_sided={one_sided}", flush=True)
    m, E, C = U.amd(), 16, 128
    g = torch.Generator(device="cuda").manual_seed(d + f)
    n = lambda *s, std: torch.empty(s, device="cuda").normal_(0.0, std, generator=g)
    xe, W1, b1, W2, b2 = n(E, C, d, std=1.0), n(E, d, f, std=0.05), n(E, 1, f, std=0.05), n(E, f, d, std=0.05), n(E, 1, d, std=0.05)
    if one_sided:
        xe, W1, W2 = xe.abs(), W1.abs(), W2.abs()
    shape = m.make_shape(C, d, f, E, 1, C, "f32")
    ye = torch.empty_like(xe)
    m.moe_expert_ffn(shape, xe, torch.full((E,), C, dtype=torch.int32, device="cuda"), W1, b1, W2, b2, ye, m.alloc_workspace(shape, "cuda"))
    gelu = lambda z: torch.nn.functional.gelu(z.double(), approximate="tanh")
    ref = gelu(xe.double() @ W1.double() + b1.double()) @ W2.double() + b2.double()
    chains = _chains(gelu(_chains(xe, W1, b1)).float(), W2, b2)
    error, allowed = (ye.double() - ref).norm().item(), (chains.double() - ref).norm().item()
    print(f"  {error / allowed:.3f}", flush=True)
    assert error <= 1.1 * allowed
