"""Experts with room for at most 64 rows on the tiled kernel (packed weights): row counts at the edges of its 16-, 32- and
64-row branches, whole and ragged inner dimensions, scatter, store and combine, dense branches on both sides of 128 tokens,
through moe_layer_forward against the oracle; and the slice entry point, which leaves fp32 partial sums."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu
TILES = (256258, 256259, 256260, 128258, 128259, 128257, 256128, 128128)      # on packed weights

# capacity, T, d, f, E, top_k, residual, first and second product on tiles
CASES = [
    (15, 256, 64, 264, 16, 1, False, False, False), (17, 300, 264, 64, 16, 2, False, True, False), (32, 800, 128, 512, 24, 1, False, True, False),
    (33, 700, 40, 136, 20, 1, False, True, False), (48, 900, 520, 264, 16, 2, False, True, False), (64, 1100, 2048, 72, 17, 1, False, True, False),
    (5, 256, 96, 1288, 64, 1, False, True, False), (40, 2600, 64, 1000, 66, 1, False, True, False), (2, 256, 1024, 128, 128, 1, False, False, True),
    (33, 2100, 1032, 64, 104, 1, False, True, True), (20, 1300, 1032, 72, 104, 2, False, True, True), (16, 1600, 2056, 40, 64, 1, False, False, True),
    (64, 3000, 2048, 96, 64, 2, False, True, True), (49, 1000, 1024, 264, 128, 1, False, False, False),
    (3, 128, 1024, 128, 128, 2, True, False, False), (3, 129, 1024, 128, 128, 2, True, False, True), (16, 1030, 1000, 72, 130, 2, True, False, True),
    (48, 1000, 72, 264, 16, 1, True, True, False),
]

@pytest.mark.parametrize("C,T,d,f,E,k,residual,first,second", CASES)
def test_few_rows_on_tiles(C, T, d, f, E, k, residual, first, second):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    kernels = plan(T, d, f, E, k, C, residual, packed=True)[0][:2]
    assert [x in TILES for x in kernels] == [first, second] and all(x < 1000 for x in plan(T, d, f, E, k, C, residual)[0][:2])
    cfg = CONFIGS["c3a"].scaled(name="few", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=11)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


def test_slice_of_few_rows():
    """One slice on packed weights and the sum of it: the expert FFN's result on plain ones (both bf16 products of the same
    operands; the first product's rounding to bf16 can differ by one unit, 2^-8 of an `h` of order one, among f terms)."""
    m, bf, C, d, f, E = U.amd(), torch.bfloat16, 33, 1032, 72, 104
    gen = torch.Generator(device="cuda").manual_seed(C)
    W1, W2 = (torch.randn(s, generator=gen, device="cuda").mul_(0.1).to(bf) for s in ((E, d, f), (E, f, d)))
    b2, xe = torch.randn((E, d), generator=gen, device="cuda").to(bf), torch.randn((E, C, d), generator=gen, device="cuda").to(bf)
    rows = torch.randint(0, C + 1, (E,), generator=gen, device="cuda", dtype=torch.int32)
    T = C * E
    assert plan(T, d, f, E, 1, C, packed=True)[0][1] in TILES
    plain, packed = m.make_shape(T, d, f, E, 1, C, "bf16"), m.make_shape(T, d, f, E, 1, C, "bf16", False, m.MOE_FLAG_PACKED_WEIGHTS)
    ws = m.alloc_workspace(plain, "cuda")
    part = torch.zeros((1, E, C, d), device="cuda")
    got, ref = torch.zeros((E, C, d), dtype=bf, device="cuda"), torch.zeros((E, C, d), dtype=bf, device="cuda")
    m.moe_expert_ffn_slice(packed, xe, rows, m.moe_pack_weights(W1), None, m.moe_pack_weights(W2), part[0], ws)
    m.moe_expert_ffn_slice_reduce(packed, 1, part, rows, b2, got)
    m.moe_expert_ffn(plain, xe, rows, W1, None, W2, b2, ref, ws)
    live = torch.arange(C, device="cuda")[None, :, None] < rows[:, None, None]
    assert bool((got == 0).masked_select(~live.expand_as(got)).all()) and bool(torch.isfinite(got.float()).all())
    assert (got.float() - ref.float()).abs().max() <= 2.0 ** -7 * ref.float().abs().max()
