"""The launch order of the experts: every expert with rows appears in it once, whatever the counts are -- none, ties, one busy
expert, more experts than a wave has lanes, row counts beyond the keys of 32 bits -- or moe_expert_ffn leaves rows unwritten."""
import pytest
import torch

from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def counts(kind, E, C, gen):
    if kind == "random":
        return torch.randint(0, C + 1, (E,), generator=gen)
    if kind == "ties":
        return torch.randint(0, 3, (E,), generator=gen) * 5
    if kind == "one":
        rows = torch.zeros(E, dtype=torch.int64)
        rows[E // 2] = C
        return rows
    return torch.where(torch.arange(E) % 7 == 0, C, 1) if kind == "skewed" else torch.zeros(E, dtype=torch.int64)


@pytest.mark.parametrize("E,C,kind", [(E, 70, k) for E in (1, 2, 15, 17, 64, 65, 128, 129, 256, 257, 1000, 1024)
                                      for k in ("random", "ties", "one", "skewed", "none")] + [(3, (1 << 20) + 1, "one"), (5, (1 << 20) + 64, "random")])
def test_every_expert_once(E, C, kind):
    print(f"case E={E} C={C} {kind}", flush=True)
    m, bf, d, f = U.amd(), torch.bfloat16, 8, 16
    gen = torch.Generator().manual_seed(E)
    rows = counts(kind, E, C, gen).to(torch.int32)
    W1, W2, b2 = torch.randn((E, d, f), generator=gen), torch.randn((E, f, d), generator=gen), torch.randn((E, d), generator=gen)
    xe = torch.randn((1, C, d), generator=gen).expand(E, C, d).contiguous()
    W1, W2, b2, xe = (t.to(bf).cuda() for t in (W1, W2, b2, xe))
    shape = m.make_shape(16, d, f, E, 1, C, "bf16")
    got = torch.full((E, C, d), 7.0, dtype=bf, device="cuda")
    m.moe_expert_ffn(shape, xe, rows.cuda(), W1, None, W2, b2, got, m.alloc_workspace(shape, "cuda"))
    h = torch.nn.functional.gelu(torch.matmul(xe.float(), W1.float()), approximate="tanh").to(bf).float()
    want = torch.matmul(h, W2.float()) + b2.float()[:, None, :]
    live = torch.arange(C)[None, :] < rows[:, None]
    live = live.cuda()[..., None].expand_as(got)
    # bf16 results (2^-9 of the value) of h rounded to bf16, which may round to a neighbour (2^-8 of one of 16 terms |h W2|)
    bound = 2.0 ** -8 * (want.abs() + torch.matmul(h.abs(), W2.float().abs()))
    assert bool(((got.float() - want).abs() <= bound)[live].all())
    assert bool((got == 7.0)[~live].all())
