"""The decode gate (at most 256 bf16 tokens) on scratch memory full of small whole numbers, such as the counts and indices
that earlier users of the memory leave: same logits and tables as on cleared memory, call after call."""
import pytest
import torch

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k", [(128, 2048, 128, 1), (31, 1024, 64, 2), (256, 256, 100, 2)])
def test_gate_on_used_scratch(T, d, E, k):
    print(f"case T={T} d={d} E={E} k={k}", flush=True)
    m, C = U.amd(), T
    inp = make_inputs(CONFIGS["c4"].scaled(name="scratch", T=T, d_model=d, d_ffn=8, E=E, top_k=k, seed=4), "cuda")
    shape = m.make_shape(T, d, 8, E, k, C, "bf16")
    ws = m.alloc_workspace(shape, "cuda")
    words = ws.view(torch.int32)
    i32, f32 = torch.int32, torch.float32
    outs = [torch.empty(s, dtype=t, device="cuda") for s, t in (((T, E), f32), ((T, k), i32), ((T, k), i32), ((T, k), f32), ((E,), i32), ((E, C), i32))]
    refs = None
    # downwards, two values at a time: a count of calls that goes up would meet them at some call
    for v in [0] + list(range(800, 0, -1)):
        words[0::2] = v
        words[1::2] = v + 1 if v else 0
        for o in outs:
            o.fill_(-7)
        m.moe_gate(shape, inp.x, inp.Wg, inp.bg, *outs, ws)
        if refs is None:
            refs = [o.clone() for o in outs]
        assert all(torch.equal(o, r) for o, r in zip(outs, refs)), f"scratch full of {v}"
