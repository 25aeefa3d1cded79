"""Infinities and NaN that the operands hold: what a sum of the same products holds must come out, from every tile and
remainder, and nothing that takes no part (positions, rows of K past the end) may add to it."""
import pytest
import torch

from tests import gpu_util as U
from tests.test_gpu_block import DEV, _run_block
from workloads import CONFIGS, make_block_inputs, make_inputs

pytestmark = pytest.mark.gpu
NAN, INF = float("nan"), float("inf")

# one sequence per position at which a lane group, a wave or a chunk of the attention kernel ends; ten chunks in all
POS = [1, 3, 65, 64, 255, 256, 257, 1000, 2304, 2499, 0, 2]


def _block(dh):
    cfg = CONFIGS["c4"].scaled(name=f"nonfinite-{dh}", T=len(POS), d_model=2 * dh, d_ffn=256, E=4, capacity_factor=4.0)
    bi = make_block_inputs(cfg, 2, 2500, DEV)
    bi.pos.copy_(torch.tensor(POS, dtype=torch.int32))
    return bi


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("which", ["first", "last"])
def test_nan_in_a_cached_key(dh, which):
    """A NaN score makes its sequence's attention NaN, wherever the position lies, and no other sequence's."""
    print(f"case dh={dh} {which}", flush=True)
    bi = _block(dh)
    ref = _run_block(bi)["x1"]
    assert bool(torch.isfinite(ref.float()).all())
    for b, p in enumerate(POS):
        if p > 0 and b % 2 == 0:
            bi.k_cache[b, 1, 0 if which == "first" else p - 1, 5] = NAN
    got = _run_block(bi)["x1"]
    for b, p in enumerate(POS):
        if p > 0 and b % 2 == 0:
            assert bool(torch.isnan(got[b]).all()), f"NaN key of the sequence with {p} positions is lost"
        else:
            assert torch.equal(got[b], ref[b])


@pytest.mark.parametrize("dh", [64, 128])
def test_nan_in_the_new_key(dh):
    """The new token's key alone: for sequences at 0, 64, 256 and 2304 positions it begins a lane group, a wave, a chunk."""
    print(f"case dh={dh}", flush=True)
    bi = _block(dh)
    bi.bqkv[2 * dh + 7] = NAN
    got = _run_block(bi)["x1"]
    lost = [p for b, p in enumerate(POS) if not bool(torch.isnan(got[b]).all())]
    assert not lost, f"NaN key of the new token is lost at positions {lost}"


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("where", ["first", "last", "new"])
def test_infinity_in_a_value(dh, where):
    """An infinite value with a positive weight: infinite attention output, so x1 is infinite with the signs of Wo's row."""
    print(f"case dh={dh} {where}", flush=True)
    bi = _block(dh)
    ref = _run_block(bi)["x1"]
    if where == "new":
        bi.bqkv[4 * dh + 3] = INF                                   # columns q | k | v of 2 dh each: element 3 of head 0
        hit = set(range(len(POS)))
    else:
        hit = {b for b, p in enumerate(POS) if p > 0 and (b % 2 == 0 or p == 2499)}   # 2499: the last chunk too
        for b in hit:
            bi.k_cache[b, 0] = 0.0                                  # equal scores but the new token's: no weight underflows
            bi.v_cache[b, 0, 0 if where == "first" else POS[b] - 1, 3] = INF
    want = torch.where(bi.Wo[3] > 0, INF, -INF).to(ref.dtype)
    assert bool((bi.Wo[3] != 0).all())
    got = _run_block(bi)["x1"]
    for b, p in enumerate(POS):
        assert torch.equal(got[b], want if b in hit else ref[b]), f"sequence with {p} positions"


# dtype, capacity, d, f: at most 16, 32 and more rows per expert, K (d, then f) of whole blocks, ragged, less than a block
LAST_ROW = [("f32", 1, 4, 4), ("f32", 12, 64, 256), ("f32", 16, 20, 72), ("f32", 30, 36, 132), ("f32", 60, 64, 128), ("f32", 60, 36, 100),
            ("bf16", 1, 8, 8), ("bf16", 12, 40, 136), ("bf16", 16, 72, 264), ("bf16", 9, 1000, 1032)]


@pytest.mark.parametrize("dtype,C,d,f", LAST_ROW)
@pytest.mark.parametrize("second", [False, True])
def test_infinity_in_the_last_weight_row(dtype, C, d, f, second):
    """An infinite weight in the last row of W1 or W2: the sums that it takes part in are infinite, as any order of additions
    gives them, and the others what they were."""
    print(f"case {dtype} C={C} d={d} f={f} second={second}", flush=True)
    cfg = (CONFIGS["c1"] if dtype == "f32" else CONFIGS["c4"]).scaled(name="last-row", T=C, d_model=d, d_ffn=f, E=1, top_k=1, seed=9)
    inp = make_inputs(cfg, DEV, bias_std=0.05)
    inp.x[:, -1] = inp.x[:, -1].abs() + 0.5
    ref = U.gpu_forward(inp, C)["out"].clone()
    if second:                                           # h[:, f - 1] > 0 through its bias: column 2 of the output is -inf
        inp.W1[0, :, -1] = 0.0
        inp.b1[0, -1] = 1.0
        inp.W2[0, -1, 2] = -INF
        got = U.gpu_forward(inp, C)["out"]
        assert bool((got[:, 2] == -INF).all()) and bool(torch.isfinite(got[:, torch.arange(d) != 2].float()).all())
    else:                                                # h[:, 1] = +inf: every output is infinite with W2's sign
        inp.W1[0, -1, 1] = INF
        got = U.gpu_forward(inp, C)["out"]
        assert bool((inp.W2[0, 1] != 0).all())
        assert torch.equal(got, torch.where(inp.W2[0, 1] > 0, INF, -INF).to(got.dtype).expand_as(got))
    assert bool(torch.isfinite(ref.float()).all())
