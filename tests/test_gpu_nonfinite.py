"""Infinities and NaN that the operands hold: what a sum of the same products holds must come out, from every tile and
remainder, and nothing that takes no part (positions, rows of K past the end) may add to it."""
import pytest
import torch

from tests.test_gpu_block import DEV, _run_block
from workloads import CONFIGS, make_block_inputs

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
