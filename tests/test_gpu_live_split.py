"""The second product of an expert FFN on the streaming kernel, whose K is split by the experts that have rows: none, one, few, most and all of
them, inner dimensions in whole chunks and ragged, columns off 128, fewer experts than XCDs, plain and packed weights -- through
moe_expert_ffn against the same product in 32 bits, and rows beyond the counts are left alone."""
import pytest
import torch

from tests import gpu_util as U
from tests.plan_util import plan

pytestmark = pytest.mark.gpu

# T, d, f, E, capacity: 1024 waves' tiles of all experts at most
SHAPES = [(1000, 1000, 4000, 40, 48), (300, 128, 520, 70, 9), (200, 264, 4096, 7, 33), (64, 136, 2048, 3, 64), (512, 2048, 1024, 33, 16)]


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("live", [0, 1, 2, 5, 0.6, 1.0])
@pytest.mark.parametrize("T,d,f,E,C", SHAPES)
def test_split_by_live_experts(T, d, f, E, C, live, packed):
    n = min(E, live) if isinstance(live, int) else round(E * live)
    print(f"case T={T} d={d} f={f} E={E} C={C} live={n} packed={packed}", flush=True)
    m, bf = U.amd(), torch.bfloat16
    code = plan(T, d, f, E, 1, C, False, packed)[0][1]
    assert packed or code >= 200, "K is not split on the streaming kernel"
    gen = torch.Generator().manual_seed(E + n)
    rows = torch.zeros(E, dtype=torch.int32)
    rows[torch.randperm(E, generator=gen)[:n]] = torch.randint(1, C + 1, (n,), generator=gen).to(torch.int32)
    W1, W2 = (torch.randn(s, generator=gen) * s[1] ** -0.5 for s in ((E, d, f), (E, f, d)))
    W1, W2, b2, xe = (t.to(bf).cuda() for t in (W1, W2, torch.randn((E, d), generator=gen), torch.randn((E, C, d), generator=gen)))
    shape = m.make_shape(T, d, f, E, 1, C, "bf16", flags=m.MOE_FLAG_PACKED_WEIGHTS if packed else 0)
    got = torch.full((E, C, d), 7.0, dtype=bf, device="cuda")
    w1, w2 = (m.moe_pack_weights(w) if packed else w for w in (W1, W2))
    m.moe_expert_ffn(shape, xe, rows.cuda(), w1, None, w2, b2, got, m.alloc_workspace(shape, "cuda"))
    h = torch.nn.functional.gelu(torch.matmul(xe.float(), W1.float()), approximate="tanh").to(bf).float()
    want = torch.matmul(h, W2.float()) + b2.float()[:, None, :]
    alive = (torch.arange(C)[None, :] < rows[:, None]).cuda()[..., None].expand_as(got)
    # the result in bf16 (2^-9 of it), and h in bf16, of which any may round to a neighbour (2^-8) of what it is here; f32 sums are far below
    bound = 2.0 ** -8 * (want.abs() + torch.matmul(h.abs(), W2.float().abs()))
    assert bool(((got.float() - want).abs() <= bound)[alive].all())
    assert bool((got == 7.0)[~alive].all())
