"""The fp32 kernels on split operands: 64 x 128 tiles (one and two sets of waves), 32 x 64 tiles of few (four and eight waves), each with every
epilogue (test_layers); the edges of tiles and steps; errors against 64 bits, which a product of pieces left out or a wrong piece would
multiply (test_no_further_from_64_bits_than_fp32); operands that the split does not hold.  tests/test_dispatch.py says which kernel a shape takes."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan_f32
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


def _ffn(E, C, d, f, rows, edit=None, scale=1.0):
    """moe_expert_ffn and the same in 64 bits; h in 64 bits too."""
    m, g = U.amd(), torch.Generator(device="cuda").manual_seed(E * C + d)
    n = lambda *s, std: torch.empty(s, device="cuda").normal_(0.0, std, generator=g)
    xe, W1, W2, b1, b2 = n(E, C, d, std=scale), n(E, d, f, std=0.05 / scale), n(E, f, d, std=0.05), n(E, f, std=0.05), n(E, d, std=0.05)
    if edit:
        edit(xe, W1, W2)
    r = torch.tensor(rows, dtype=torch.int32, device="cuda")
    shape = m.make_shape(C, d, f, E, 1, C, "f32")
    ye = torch.full_like(xe, 12345.0)
    m.moe_expert_ffn(shape, xe, r, W1, b1, W2, b2, ye, m.alloc_workspace(shape, "cuda"))
    torch.cuda.synchronize()
    ref = torch.empty(E, C, d, dtype=torch.float64, device="cuda")
    for e in range(E):
        z = xe[e].double() @ W1[e].double() + b1[e].double()
        ref[e] = torch.nn.functional.gelu(z, approximate="tanh") @ W2[e].double() + b2[e].double()
    return ye, ref


# rows with room for, K and N off the steps (32 and 64 k), half steps and tiles (64 rows, 128 columns); products on either side of the rules
@pytest.mark.parametrize("E,C,d,f,rows", [
    (4, 1100, 132, 260, [1100, 1, 33, 64]), (16, 70, 260, 516, [70, 65, 64, 63, 32, 33, 31, 1, 0] + [70] * 7), (2, 700, 516, 1028, [700, 129]),
    (1, 2100, 148, 1156, [2049]), (8, 600, 196, 132, [600, 97, 96, 577, 0, 128, 300, 16]),
])
def test_edges(E, C, d, f, rows):
    print(f"case E={E} C={C} d={d} f={f}", flush=True)
    ye, ref = _ffn(E, C, d, f, rows)
    for e, r in enumerate(rows):
        if r:   # 6 to 26 units of 2^-24 of the root mean square with either instruction; without one of the six products of pieces 42 on average
                # (2^-18.6 of every product) and about four times that somewhere
            assert (ye[e, :r].double() - ref[e, :r]).abs().max() <= 40 * EPS * ref[e, :r].square().mean().sqrt()
        assert bool((ye[e, r:] == 12345.0).all())


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_values_beyond_the_split(value):
    """In one weight and one activation: what a sum of the same products holds; other rows, columns and tiles as without."""
    print(f"case {value}", flush=True)
    E, C, d, f = 4, 640, 256, 1024

    def edit(xe, W1, W2):
        W2[1, 700, 130] = value
        xe[2, 333, 7] = value
    clean, _ = _ffn(E, C, d, f, [C] * E)
    ye, ref = _ffn(E, C, d, f, [C] * E, edit)
    hit = torch.zeros_like(ye, dtype=torch.bool)
    hit[1, :, 130], hit[2, 333] = True, True
    bad = ~torch.isfinite(ref) | (ref.abs() > 3.4e38)
    assert bool((bad <= hit).all())
    assert bool((torch.isfinite(ye) == ~bad)[hit].all())
    assert torch.equal(torch.isnan(ye), torch.isnan(ref)) or value == 3.4e38     # beyond the range: infinities of either sign may meet
    assert (ye - clean)[~hit].abs().max() <= 4 * f ** 0.5 * EPS * clean.abs().max()


@pytest.mark.parametrize("scale", [2.0 ** -118, 2.0 ** -100, 2.0 ** 100])
def test_far_from_one(scale):
    """Activations whose second and third pieces the matrix instruction would take for zero, under large weights; and the reverse."""
    print(f"case {scale}", flush=True)
    ye, ref = _ffn(4, 640, 256, 1024, [640] * 4, scale=scale)
    assert (ye.double() - ref).abs().max() <= 2 * 1024 ** 0.5 * 2 * EPS * ref.abs().max()


# tiles of 32 x 64 and products next to them: rows around 16 and 32, K and N off the blocks
@pytest.mark.parametrize("E,C,d,f,rows", [
    (2, 17, 132, 260, [17, 1]), (3, 32, 196, 148, [32, 31, 0]), (4, 33, 516, 132, [33, 32, 16, 1]), (16, 32, 260, 2052, [32] * 15 + [5]),
    (1, 300, 132, 1028, [300]), (8, 256, 2052, 516, [256, 255, 1, 0, 97, 96, 64, 33]),
])
def test_few_tiles(E, C, d, f, rows):
    test_edges(E, C, d, f, rows)


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_values_beyond_the_split_few_tiles(value):
    print(f"case {value}", flush=True)

    def edit(xe, W1, W2):
        W2[1, 200, 130] = value
        xe[0, 33, 7] = value
    clean, _ = _ffn(2, 40, 256, 300, [40, 40])
    ye, ref = _ffn(2, 40, 256, 300, [40, 40], edit)
    hit = torch.zeros_like(ye, dtype=torch.bool)
    hit[1, :, 130], hit[0, 33] = True, True
    bad = ~torch.isfinite(ref) | (ref.abs() > 3.4e38)
    assert bool((torch.isfinite(ye) == ~bad)[hit].all())
    assert torch.equal(torch.isnan(ye), torch.isnan(ref)) or value == 3.4e38
    assert (ye - clean)[~hit].abs().max() <= 4 * 300 ** 0.5 * EPS * clean.abs().max()


@pytest.mark.parametrize("scale", [2.0 ** -118, 2.0 ** -100, 2.0 ** 100])
def test_far_from_one_few_tiles(scale):
    print(f"case {scale}", flush=True)
    ye, ref = _ffn(2, 40, 256, 300, [40, 40], scale=scale)
    assert (ye.double() - ref).abs().max() <= 2 * 300 ** 0.5 * 2 * EPS * ref.abs().max()


def _fp32_products(a, b, bias, chains):
    """a b + bias as the fp32 matrix instructions sum it: every 2nd (64 x 128 tiles) or 8th (few tiles) block of 16 k in one chain of fused
    multiply-adds."""
    acc = [torch.zeros(*a.shape[:-1], b.shape[-1], device=a.device) for _ in range(chains)]
    for k in range(a.shape[-1]):
        q = k // 16 % chains
        acc[q] = (acc[q].double() + a[..., k:k + 1].double() * b[..., k:k + 1, :].double()).float()
    return sum(acc[1:], acc[0]) + bias


def _device_gelu(z):
    """The kernels' own gelu, exactly: experts whose rows and second weights are unit matrices, values as their first weights."""
    m, n = U.amd(), 128
    w = z.reshape(-1, n, n)
    eye = torch.eye(n, device="cuda").expand_as(w).contiguous()
    zero = torch.zeros(w.shape[0], n, device="cuda")
    shape = m.make_shape(n, n, n, w.shape[0], 1, n, "f32")
    h = torch.empty_like(w)
    m.moe_expert_ffn(shape, eye, torch.full((w.shape[0],), n, dtype=torch.int32, device="cuda"), w, zero, eye, zero, h, m.alloc_workspace(shape, "cuda"))
    return h.reshape(z.shape)


OPERANDS = ["normal", "one sign", "rectified", "one large column", "one sign, one large column", "mantissas"]


@pytest.mark.parametrize("operands", OPERANDS)
@pytest.mark.parametrize("E,C,d,f,chains", [(32, 640, 512, 128, (2, 2)), (8, 1200, 512, 128, (2, 2)), (8, 1200, 128, 512, (2, 2)),
                                            (32, 64, 132, 128, (8, 8)), (32, 64, 2048, 128, (8, 2)), (64, 96, 2048, 128, (8, 2)),
                                            (64, 96, 128, 1024, (2, 8))])
def test_no_further_from_64_bits_than_fp32(E, C, d, f, chains, operands):
    """Operands of one sign, rectified ones (half of the products zero: no rounding in an fp32 chain), one column 1000 times the others (in
    its group of eight the products are cut to its grid), values whose neglected piece products are the largest (2^-24 of the product)."""
    print(f"case E={E} C={C} d={d} f={f} {operands}", flush=True)
    m, g = U.amd(), torch.Generator(device="cuda").manual_seed(d + f)
    n = lambda *s, std: torch.empty(s, device="cuda").normal_(0.0, std, generator=g)
    xe, W1, W2, b1, b2 = n(E, C, d, std=1.0), n(E, d, f, std=0.05), n(E, f, d, std=0.05), n(E, 1, f, std=0.05), n(E, 1, d, std=0.05)
    if operands.startswith("one sign"):
        xe, W1, W2 = xe.abs(), W1.abs(), W2.abs()
    elif operands == "rectified":
        xe, W1 = xe.clamp_min(0.0), W1 * 16                  # gelu: the second product's rows are rectified, too
    if operands.endswith("one large column"):
        xe[..., d // 2 + 1] *= 1000.0
        W1[..., f // 2 + 1] *= 1000.0
    if operands == "mantissas":
        xe, W1, W2 = [torch.sign(v) * s * (1 + 2.0 ** -8 - 2.0 ** -17) for v, s in ((xe, 1.0), (W1, 0.0625), (W2, 0.0625))]
    shape = m.make_shape(E * C, d, f, E, 1, C, "f32")
    ye = torch.empty_like(xe)
    m.moe_expert_ffn(shape, xe, torch.full((E,), C, dtype=torch.int32, device="cuda"), W1, b1, W2, b2, ye, m.alloc_workspace(shape, "cuda"))
    gelu = lambda z: torch.nn.functional.gelu(z.double(), approximate="tanh")
    ref = gelu(xe.double() @ W1.double() + b1.double()) @ W2.double() + b2.double()
    fp32 = _fp32_products(_device_gelu(_fp32_products(xe, W1, b1, chains[0])), W2, b2, chains[1])
    error, allowed = (ye.double() - ref).norm().item(), (fp32.double() - ref).norm().item()
    print(f"  {error / allowed:.3f}", flush=True)
    assert error <= 1.01 * allowed                           # the fp32 kernels themselves: 0.78 to 1.001 (their order of 16 k)


# one and two sets of waves per tile; eight and four waves per tile of 32 rows
SHAPES = [(32, 640, 512, 128), (8, 1200, 512, 128), (32, 64, 512, 128), (64, 96, 512, 128)]


def _expert_ffn(xe, W1, W2):
    m, (E, C, d), f = U.amd(), xe.shape, W1.shape[2]
    shape = m.make_shape(E * C, d, f, E, 1, C, "f32")
    ye, zero = torch.empty_like(xe), torch.zeros(E, max(d, f), device="cuda")
    m.moe_expert_ffn(shape, xe, torch.full((E,), C, dtype=torch.int32, device="cuda"), W1, zero[:, :f].contiguous(), W2, zero[:, :d].contiguous(), ye,
                     m.alloc_workspace(shape, "cuda"))
    torch.cuda.synchronize()
    return ye


@pytest.mark.parametrize("x,w", [(-130, 0), (-130, 20), (-140, 19), (-140, 30), (-110, 10), (-100, 0), (-60, -50), (-60, 0), (100, -100), (60, -60), (0, 0)])
@pytest.mark.parametrize("E,C,d,f", SHAPES + [(2, 300, 4096, 128)])
def test_magnitudes(E, C, d, f, x, w):
    """Activations around 2^x (below -126 subnormal, below -134 without a bf16 piece) under weights around 2^w, no bias: sums as small as fp32 holds."""
    print(f"case E={E} C={C} d={d} f={f} 2^{x} 2^{w}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + f)
    n = lambda *s, std: torch.empty(s, device="cuda").normal_(0.0, std, generator=g)
    xe, W1, W2 = n(E, C, d, std=2.0 ** x), n(E, d, f, std=2.0 ** (w - 5)), n(E, f, d, std=2.0 ** -min(x + w, 0) if x + w > -120 else 2.0 ** 100)
    ye = _expert_ffn(xe, W1, W2)
    ref = torch.nn.functional.gelu(xe.double() @ W1.double(), approximate="tanh") @ W2.double()
    # subnormal intermediate values: K units of 2^-149 times the second weights
    floor = f * 2.0 ** -149 * W2.abs().max().item() * 4
    assert (ye.double() - ref).abs().max() <= 2 * f ** 0.5 * 2 * EPS * ref.abs().max() + floor
    assert ye.abs().max() > 0


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e38, 3.0 * 2 ** 40, 2.0 ** -135])
@pytest.mark.parametrize("E,C,d,f", SHAPES)
def test_rows_and_columns_do_not_see_each_other(E, C, d, f, value):
    """A row of activations or a column of weights beyond the split changes its own results only: the others stay the same bit by bit."""
    print(f"case E={E} C={C} d={d} f={f} {value}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + f)
    n = lambda *s, std: torch.empty(s, device="cuda").normal_(0.0, std, generator=g)
    xe, W1, W2 = n(E, C, d, std=1.0), n(E, d, f, std=0.05), n(E, f, d, std=0.05)
    clean = _expert_ffn(xe, W1, W2)
    rows, columns = [0, 5, C // 2, C - 1], [3, 64, d - 1]
    for r in rows:
        xe[1, r] = value if abs(value) < 1 else xe[1, r].clone().index_fill_(0, torch.tensor([7], device="cuda"), value)
    ye = _expert_ffn(xe, W1, W2)
    keep = torch.ones(E, C, d, dtype=torch.bool, device="cuda")
    keep[1, rows] = False
    assert torch.equal(ye[keep], clean[keep])
    xe[1, rows] = 1.0
    clean = _expert_ffn(xe, W1, W2)
    W2[1, f // 2, columns] = value
    ye = _expert_ffn(xe, W1, W2)
    keep[1, rows] = True
    keep[1, :, columns] = False
    assert torch.equal(ye[keep], clean[keep])


# every split kernel with every epilogue: the first product gathers, the second one stores (top-2), scatters (top-1, tokens dropped) or combines
# (dense branch); ragged rows, experts without any, K and N off the steps and tiles
LAYERS = [
    (2000, 164, 1092, 8, 1, 270, False, ["split1", "rows_split8"]),
    (1200, 516, 260, 24, 2, 140, False, ["split2", "split2"]),
    (2000, 1028, 196, 16, 1, 130, True, ["rows_split8", "split1", "rows_split8", "split1"]),
    (2000, 1028, 196, 16, 1, 130, False, ["rows_split8", "split1"]),
    (1000, 1028, 196, 16, 2, 130, False, ["rows_split8", "split1"]),
    (1500, 1028, 260, 4, 1, 400, True, ["rows_split8", "split2", "rows_split8", "split2"]),
    (1500, 1028, 260, 4, 1, 400, False, ["rows_split8", "split2"]),
    (600, 516, 516, 31, 1, 30, False, ["rows_split4", "rows_split4"]),
    (60, 516, 580, 31, 2, 30, False, ["rows_split4", "rows_split4"]),
    (100, 516, 516, 5, 1, 30, True, ["rows_split8", "rows_split8", "rows_split8", "rows_split8"]),
    (1000, 516, 516, 5, 2, 60, True, ["rows_split8", "rows_split8", "rows_split4", "rows_split4"]),
]


@pytest.mark.parametrize("T,d,f,E,k,C,residual,kernels", LAYERS)
def test_layers(T, d, f, E, k, C, residual, kernels):
    print(f"case T={T} d={d} f={f} E={E} k={k} C={C} residual={residual}", flush=True)
    assert plan_f32(T, d, f, E, k, C, residual) == kernels
    cfg = CONFIGS["c1"].scaled(name="f32", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=7)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05), capacity=C)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("T,d,f,E,k,C,residual,kernels", [c for c in LAYERS if c[4] == 1])
def test_weights_beyond_the_split(T, d, f, E, k, C, residual, kernels, value):
    """In a column of the second product: that column of the tokens that it concerns, and no other bit, whatever the epilogue."""
    print(f"case T={T} d={d} f={f} E={E} residual={residual} {value}", flush=True)
    cfg = CONFIGS["c1"].scaled(name="f32", T=T, d_model=d, d_ffn=f, E=E, top_k=k, residual=residual, seed=7)
    inp = make_inputs(cfg, "cuda", bias_std=0.05)
    clean = U.gpu_forward(inp, C)
    expert = int(clean["expert_rows"].argmax())
    kept = (clean["expert_idx"][:, 0] == expert) & (clean["slot_idx"][:, 0] >= 0)
    inp.W2[expert, f - 1, 70] = value
    out = U.gpu_forward(inp, C)["out"]
    hit = torch.zeros_like(out, dtype=torch.bool)
    hit[kept, 70] = True
    assert bool((~torch.isfinite(out) == hit).all()) and torch.equal(out[~hit], clean["out"][~hit])
    if not residual:
        return
    inp.W2[expert, f - 1, 70] = 1.0
    clean = U.gpu_forward(inp, C)["out"].clone()
    inp.Wd2[f - 1, 3] = value
    out = U.gpu_forward(inp, C)["out"]
    assert not bool(torch.isfinite(out[:, 3]).any())
    out[:, 3] = clean[:, 3]
    assert torch.equal(out, clean)
