"""Tiled kernel: every tile shape with every epilogue that it can have in a layer, plain and packed weights, whole and ragged
inner dimensions, one product and two in a launch -- each case says which kernel it is there for, and the dispatch is asked
whether it takes it -- through moe_layer_forward against the oracle."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu
T256, T256N, T128, T128X2, T128N = 256256, 256128, 128256, 128257, 128128
W256, W256G, W128 = 256258, 256260, 128258                     # packed weights, 256 columns: the four-wave kernel
PACKED = {T256: W256, T256N: T256N, T128: W128, T128X2: T128X2, T128N: T128N}       # K up to 512
GEMM1, GEMM2, DENSE1, DENSE2 = range(4)

# capacity, T, d, f, E, top_k, residual, product, kernel on plain weights (with that on packed ones where PACKED has another), two
# products in the launch
CASES = [
    # GELU epilogue (first product); K = d whole and ragged
    (65, 32, 64, 64, 1, 1, False, GEMM1, T128N, False), (520, 260, 40, 40, 1, 1, False, GEMM1, T128N, False),
    (130, 4290, 64, 200, 66, 1, False, GEMM1, T128, False), (130, 4290, 40, 200, 66, 1, False, GEMM1, T128, False),
    (65, 2145, 64, 1000, 66, 1, False, GEMM1, T128X2, False), (65, 2145, 40, 1000, 66, 1, False, GEMM1, T128X2, False),
    (257, 257, 64, 8192, 2, 1, False, GEMM1, T256N, False), (130, 2080, 40, 1000, 32, 1, False, GEMM1, T256N, False),
    (130, 4290, 64, 264, 66, 1, False, GEMM1, T256, False), (130, 4290, 40, 264, 66, 1, False, GEMM1, T256, False),
    # two first products in a launch
    (65, 130, 64, 64, 2, 1, True, GEMM1, T128N, True), (65, 130, 64, 8192, 4, 1, True, GEMM1, T128, True),
    (65, 260, 64, 8192, 8, 1, True, GEMM1, T128X2, True), (257, 4240, 512, 512, 33, 1, True, GEMM1, T256, True),
    (300, 300, 256, 256, 64, 1, True, GEMM1, T128, True),
    # scatter epilogue (second product, top-1); K = f whole and ragged
    (65, 32, 64, 64, 1, 1, False, GEMM2, T128N, False), (520, 260, 40, 40, 1, 1, False, GEMM2, T128N, False),
    (130, 4290, 200, 64, 66, 1, False, GEMM2, T128, False), (130, 4290, 200, 40, 66, 1, False, GEMM2, T128, False),
    (65, 520, 4104, 64, 16, 1, False, GEMM2, T128X2, False), (65, 520, 4104, 40, 16, 1, False, GEMM2, T128X2, False),
    (257, 2056, 1000, 64, 16, 1, False, GEMM2, T256N, False), (130, 2080, 1000, 40, 32, 1, False, GEMM2, T256N, False),
    (130, 4290, 264, 64, 66, 1, False, GEMM2, T256, False), (130, 4290, 264, 40, 66, 1, False, GEMM2, T256, False),
    # store epilogue (second product, top-2 or beside a dense branch); K = f whole and ragged
    (65, 32, 64, 64, 1, 1, True, GEMM2, T128N, False), (520, 260, 40, 40, 1, 1, True, GEMM2, T128N, False),
    (130, 4290, 200, 64, 66, 2, False, GEMM2, T128, False), (130, 4290, 200, 40, 66, 2, False, GEMM2, T128, False),
    (65, 520, 4104, 64, 16, 2, False, GEMM2, T128X2, False), (65, 520, 4104, 40, 16, 2, False, GEMM2, T128X2, False),
    (257, 1028, 1000, 64, 16, 2, False, GEMM2, T256N, False), (257, 2056, 1000, 64, 16, 1, True, GEMM2, T256N, False),
    (130, 1040, 1000, 40, 32, 2, False, GEMM2, T256N, False),
    (130, 4290, 264, 64, 66, 2, False, GEMM2, T256, False), (130, 4290, 264, 40, 66, 2, False, GEMM2, T256, False),
    # two second products in a launch
    (65, 130, 64, 64, 2, 1, True, GEMM2, T128N, True), (65, 130, 8192, 64, 4, 1, True, GEMM2, T128, True),
    (65, 260, 8192, 64, 8, 1, True, GEMM2, T128X2, True), (257, 257, 8192, 64, 2, 1, True, GEMM2, T256, True),
    (300, 300, 256, 32, 64, 1, True, GEMM2, T128, True),
    # packed weights, two paired tiles per compute unit chosen with K beyond 512: four waves with 128 or 256 rows; and pairs of
    # groups of at most 128 rows with a dense branch, in a round of 128-row tiles and beyond
    (65, 1248, 520, 1032, 64, 1, False, GEMM1, (T128X2, W128), False), (65, 1248, 1032, 520, 64, 1, False, GEMM2, (T128X2, W128), False),
    (600, 11520, 520, 520, 64, 1, False, GEMM1, (T128X2, W128), False), (400, 5760, 576, 2048, 16, 1, True, GEMM1, (T128X2, W256), True),
    (384, 3686, 576, 1024, 32, 1, True, GEMM1, (T128X2, W128), True), (384, 1843, 2048, 1024, 16, 1, True, GEMM2, (T128X2, W128), True),
    (100, 300, 576, 1024, 64, 1, True, GEMM1, (T128X2, W128), True), (100, 300, 1024, 1024, 64, 1, True, GEMM2, (T128X2, W128), True),
    (80, 3000, 576, 2112, 40, 1, True, GEMM1, (T128X2, W256), True), (80, 300, 576, 2112, 64, 1, True, GEMM1, (T128X2, W256G), True),
    (80, 300, 2112, 1024, 64, 1, True, GEMM2, (T128X2, W256G), True),
    # combine epilogue (the dense branch's second product in a launch of its own)
    (128, 256, 4104, 64, 2, 1, True, DENSE2, T128N, False), (128, 256, 4104, 40, 2, 1, True, DENSE2, T128N, False),
    (300, 900, 4104, 64, 3, 1, True, DENSE2, (T128, T128), False), (300, 900, 4104, 40, 3, 1, True, DENSE2, (T128, T128), False),
    (128, 3379, 8192, 64, 33, 1, True, DENSE2, T128X2, False), (128, 3379, 8192, 40, 33, 1, True, DENSE2, T128X2, False),
    (300, 3600, 2056, 64, 12, 1, True, DENSE2, (T256, T256), False), (300, 3600, 2056, 40, 12, 1, True, DENSE2, (T256, T256), False),
]


@pytest.mark.parametrize("C,T,d,f,E,k,residual,product,kernel,shared", CASES)
def test_tile_choice(C, T, d, f, E, k, residual, product, kernel, shared):
    print(f"case C={C} T={T} d={d} f={f} E={E} k={k} residual={residual}", flush=True)
    for packed, want in enumerate(kernel if isinstance(kernel, tuple) else (kernel, PACKED[kernel])):
        kernels, both = plan(T, d, f, E, k, C, residual, bool(packed))
        assert kernels[product] == want and bool(both[product % 2]) == shared
    cfg = CONFIGS["c3a"].scaled(name="choice", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=10)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("C,d,f,E,kernel", [(65, 64, 64, 3, T128N), (130, 200, 40, 66, T128), (70, 4104, 64, 16, T128X2), (257, 1000, 64, 16, T256N),
                                            (144, 1000, 40, 32, T256N), (130, 264, 40, 66, T256)])
def test_slice_on_every_tile(C, d, f, E, kernel, packed):
    """moe_expert_ffn_slice leaves fp32 partial sums: with one slice and the sum of it, the expert FFN's result."""
    print(f"case C={C} d={d} f={f} E={E} packed={packed}", flush=True)
    m, bf = U.amd(), torch.bfloat16
    assert plan(C * E // 2, d, f, E, 1, C, packed=packed)[0][GEMM2] == (PACKED[kernel] if packed else kernel)
    gen = torch.Generator(device="cuda").manual_seed(C)
    W1, W2 = (torch.randn(s, generator=gen, device="cuda").mul_(0.1).to(bf) for s in ((E, d, f), (E, f, d)))
    b2, xe = torch.randn((E, d), generator=gen, device="cuda").to(bf), torch.randn((E, C, d), generator=gen, device="cuda").to(bf)
    rows = torch.randint(0, C + 1, (E,), generator=gen, device="cuda", dtype=torch.int32)
    shape = m.make_shape(C * E // 2, d, f, E, 1, C, "bf16", False, m.MOE_FLAG_PACKED_WEIGHTS if packed else 0)
    if packed:
        W1, W2 = m.moe_pack_weights(W1), m.moe_pack_weights(W2)
    ws = m.alloc_workspace(shape, "cuda")
    part = torch.zeros((1, E, C, d), device="cuda")
    got, ref = torch.zeros((E, C, d), dtype=bf, device="cuda"), torch.zeros((E, C, d), dtype=bf, device="cuda")
    m.moe_expert_ffn_slice(shape, xe, rows, W1, None, W2, part[0], ws)
    m.moe_expert_ffn_slice_reduce(shape, 1, part, rows, b2, got)
    m.moe_expert_ffn(shape, xe, rows, W1, None, W2, b2, ref, ws)
    live = torch.arange(C, device="cuda")[None, :, None] < rows[:, None, None]
    assert bool((got == 0).masked_select(~live.expand_as(got)).all())
    # the same sums rounded to bf16 once: half a unit in the last place each; the four-wave kernel's sums begin with the bias that
    # the reduction adds last, and fp32 sums that differ in their last bits may round to neighbours: one unit, at most 2^-7
    bound = 2.0 ** -7 if packed else 2.0 ** -8
    assert (got.float() - ref.float()).abs().max() <= bound * ref.float().abs().max() and bool(torch.isfinite(got.float()).all())
