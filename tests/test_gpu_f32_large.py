"""fp32 layers at the far end of what the entry points take: more row tiles than one grid dimension holds threads for."""
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
