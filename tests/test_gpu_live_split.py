"""The second product of an expert FFN on the streaming kernel, whose K is split by the experts that have rows: none, one, few, most and all of
them, inner dimensions in whole chunks and ragged, columns off 128, fewer experts than XCDs, plain and packed weights -- through
moe_expert_ffn against the same product in 32 bits, and rows beyond the counts are left alone.  How many parts K was split into is read
off the workspace, whose last region holds their sums: with equal counts every number of them from two to the plan's own, parts
without a chunk, experts without rows between those with some; the plan's own where the counts are very different.  And the
layer whose sums go straight to the tokens' rows, some of which are dropped."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu

# T, d, f, E, capacity: 1024 waves' tiles of all experts at most
SHAPES = [(1000, 1000, 4000, 40, 48), (300, 128, 520, 70, 9), (200, 264, 4096, 7, 33), (100, 136, 2048, 3, 64), (512, 2048, 1024, 33, 16)]

# the same, experts with rows, parts that K then has (fewer than the plan's own)
REDUCED = [(1000, 1000, 2000, 40, 48, 10, 5),     # sixteen chunks of K, the last one ragged, four in each part: one part has none
           (1000, 1000, 2000, 40, 48, 20, 3), (1000, 1000, 2000, 40, 48, 30, 2), (1000, 1000, 2000, 40, 48, 40, 2),
           (1000, 1000, 760, 40, 48, 10, 5),      # six chunks, two in each: two parts have none
           (200, 2048, 1040, 7, 33, 7, 4),        # fewer experts than XCDs
           (200, 2048, 1040, 7, 33, 5, 5), (512, 2048, 1024, 33, 16, 33, 1)]


def parts_written(ws, shape, room, rows):
    """Parts of K whose sums the call left behind, in a workspace that was all ones before; each for every row or for none."""
    E, C, d = shape.E, shape.capacity, shape.d_model
    n, total = room * E * C * d * 4, U.amd().moe_workspace_bytes(shape)
    start = total - -(-n // 256) * 256
    sums = ws[start:start + n].view(torch.float32).view(room, E, C, d)
    alive = (torch.arange(C)[None, :] < rows.cpu()[:, None]).cuda()
    written = ~torch.isnan(sums[:, alive])
    each = written.flatten(1).all(1)
    assert bool((written.flatten(1).any(1) == each).all()), "a part was written in places"
    n = int(each.sum())
    assert bool(each[:n].all()), "parts after the last"
    return n


def check_ffn(T, d, f, E, C, rows, packed, gen):
    """moe_expert_ffn for these counts against the product in 32 bits; (parts of K that it took, the plan's own)."""
    m, bf = U.amd(), torch.bfloat16
    code = plan(T, d, f, E, 1, C, False, packed)[0][1]
    assert 200 <= code < 1000, "K is not split on the streaming kernel"
    W1, W2 = (torch.randn(s, generator=gen) * s[1] ** -0.5 for s in ((E, d, f), (E, f, d)))
    W1, W2, b2, xe = (t.to(bf).cuda() for t in (W1, W2, torch.randn((E, d), generator=gen), torch.randn((E, C, d), generator=gen)))
    shape = m.make_shape(T, d, f, E, 1, C, "bf16", flags=m.MOE_FLAG_PACKED_WEIGHTS if packed else 0)
    got = torch.full((E, C, d), 7.0, dtype=bf, device="cuda")
    w1, w2 = (m.moe_pack_weights(w) if packed else w for w in (W1, W2))
    ws = m.alloc_workspace(shape, "cuda").fill_(255)
    m.moe_expert_ffn(shape, xe, rows.cuda(), w1, None, w2, b2, got, ws)
    h = torch.nn.functional.gelu(torch.matmul(xe.float(), W1.float()), approximate="tanh").to(bf).float()
    want = torch.matmul(h, W2.float()) + b2.float()[:, None, :]
    alive = (torch.arange(C)[None, :] < rows[:, None]).cuda()[..., None].expand_as(got)
    # the result in bf16 (2^-9 of it), and h in bf16, of which any may round to a neighbour (2^-8) of what it is here; f32 sums are far below
    bound = 2.0 ** -8 * (want.abs() + torch.matmul(h.abs(), W2.float().abs()))
    assert bool(((got.float() - want).abs() <= bound)[alive].all())
    assert bool((got == 7.0)[~alive].all())
    return parts_written(ws, shape, code // 100, rows) if bool((rows > 0).any()) else 0, code // 100


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("live", [0, 1, 2, 5, 0.6, 1.0])
@pytest.mark.parametrize("T,d,f,E,C", SHAPES)
def test_split_by_live_experts(T, d, f, E, C, live, packed):
    n = min(E, live) if isinstance(live, int) else round(E * live)
    print(f"case T={T} d={d} f={f} E={E} C={C} live={n} packed={packed}", flush=True)
    gen = torch.Generator().manual_seed(E + n)
    rows = torch.zeros(E, dtype=torch.int32)
    rows[torch.randperm(E, generator=gen)[:n]] = torch.randint(1, C + 1, (n,), generator=gen).to(torch.int32)
    check_ffn(T, d, f, E, C, rows, packed, gen)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("even", [True, False])
@pytest.mark.parametrize("T,d,f,E,C,live,parts", REDUCED)
def test_fewer_parts_than_planned(T, d, f, E, C, live, parts, even, packed):
    print(f"case T={T} d={d} f={f} E={E} C={C} live={live} even={even} packed={packed}", flush=True)
    gen = torch.Generator().manual_seed(E + live)
    rows = torch.zeros(E, dtype=torch.int32)
    experts = torch.randperm(E, generator=gen)[:live]
    rows[experts] = C - 1
    if not even:
        rows[experts[:(live + 3) // 4]] = C // 4 - 1               # a quarter of them with less than a quarter of the rows
    took, planned = check_ffn(T, d, f, E, C, rows, packed, gen)
    assert parts < planned and took == (parts if even else planned)


# T, d, f, E, capacity, experts with rows: too few rows per expert on average, too few tiles of all experts for another factor
@pytest.mark.parametrize("T,d,f,E,C,live", [(119, 1000, 2000, 40, 17, 40), (23, 4096, 1040, 16, 2, 16), (100, 128, 2048, 4, 40, 4)])
def test_parts_as_planned(T, d, f, E, C, live):
    print(f"case T={T} d={d} f={f} E={E} C={C} live={live}", flush=True)
    gen = torch.Generator().manual_seed(E + live)
    took, planned = check_ffn(T, d, f, E, C, torch.full((E,), C, dtype=torch.int32), False, gen)
    assert took == planned


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("T,d,f,E,C,dead,parts", [(1000, 1000, 1400, 40, 20, 0, 2), (1000, 1000, 1400, 40, 20, 20, 3), (300, 2048, 1040, 7, 33, 2, 5)])
def test_scattered_sums(T, d, f, E, C, dead, parts, packed):
    print(f"case T={T} d={d} f={f} E={E} C={C} dead={dead} packed={packed}", flush=True)
    m = U.amd()
    code = plan(T, d, f, E, 1, C, False, packed)[0][1]
    assert 200 <= code < 1000 and parts < code // 100
    inp = make_inputs(CONFIGS["c4"].scaled(name="scatter", T=T, d_model=d, d_ffn=f, E=E, top_k=1, seed=15), "cuda", bias_std=0.05)
    inp.bg = torch.zeros(E, device="cuda")
    inp.bg[1:1 + 2 * dead:2] = -50.0                              # experts that no token chooses, between those that some do
    stats = U.check_layer(inp, capacity=C)
    assert stats["dropped_tokens"] > 0
    layer = m.MoELayer(T, d, f, E, 1, C, "bf16", inp.Wg, inp.bg, inp.W1, inp.b1, inp.W2, inp.b2, pack_weights=packed)
    layer.ws.fill_(255)
    layer(inp.x)
    rows = layer.routing["expert_rows"].clamp(max=C)
    assert int((rows > 0).sum()) == E - dead and int((4 * rows <= rows.max()).sum()) == dead
    assert parts_written(layer.ws, layer.shape, code // 100, rows) == parts
