"""fp32 layers at the far end of what the entry points take: more row tiles than one grid dimension holds threads for, and
weight rows so long that 32 of them are beyond a 32-bit offset."""
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _normal(*shape, std):
    return torch.empty(shape, device="cuda").normal_(0.0, std, generator=torch.Generator(device="cuda").manual_seed(sum(shape)))


def test_two_to_the_thirty_expert_rows():
    """256 experts with room for 2^22 rows each: the same output as with room for the 64 tokens that there are."""
    m, T, d, E = U.amd(), 64, 4, 256
    x, Wg, W1, W2 = _normal(T, d, std=1.0), _normal(d, E, std=0.5), _normal(E, d, d, std=0.5), _normal(E, d, d, std=0.5)
    outs = []
    for C in (T, 1 << 22):
        print(f"capacity {C}", flush=True)
        shape = m.make_shape(T, d, d, E, 1, C, "f32")
        ws = m.alloc_workspace(shape, "cuda")
        out = torch.full((T, d), float("nan"), device="cuda")
        m.moe_layer_forward(shape, x, Wg, None, W1, None, W2, None, None, None, None, None, out, None, None, None, None, None, None, ws)
        torch.cuda.synchronize()
        outs.append(out)
        del ws
        torch.cuda.empty_cache()
    # another kernel for the larger capacity, so another order of sums: 8 products of up to 4 terms, 2^-24 each
    assert (outs[0] - outs[1]).abs().max() <= 16 * 2.0 ** -24 * outs[0].abs().max()


def test_two_to_the_twenty_five_columns():
    """d_ffn = 2^25 and more than 32 rows: every column of the first product counts in the second."""
    m, T, d, f = U.amd(), 33, 32, 1 << 25
    x, W1, W2 = _normal(1, T, d, std=1.0), _normal(1, d, f, std=0.1), _normal(1, f, d, std=0.1)
    print(f"d={d} f={f}", flush=True)
    shape = m.make_shape(T, d, f, 1, 1, T, "f32")
    ws = m.alloc_workspace(shape, "cuda")
    ye = torch.full((1, T, d), float("nan"), device="cuda")
    m.moe_expert_ffn(shape, x, torch.tensor([T], dtype=torch.int32, device="cuda"), W1, None, W2, None, ye, ws)
    torch.cuda.synchronize()
    ref = torch.zeros((T, d), dtype=torch.float64, device="cuda")
    for c in range(0, f, 1 << 21):                          # 64 bits, a part of the columns at a time
        h = torch.nn.functional.gelu(x[0].double() @ W1[0, :, c:c + (1 << 21)].double(), approximate="tanh")
        ref += h @ W2[0, c:c + (1 << 21)].double()
    # fp32 sums of 2^25 terms, in at most 2^23 steps each of which rounds the sum by 2^-24: random signs, 4 standard deviations
    assert (ye[0].double() - ref).abs().max() <= 4 * 2.0 ** 11.5 * 2.0 ** -24 * ref.abs().max()
