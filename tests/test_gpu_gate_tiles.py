"""Gate of 257 to 2047 bf16 tokens: tiles of 32 and of 64 tokens (those from 1985 tokens of more than 64 experts on), the last tile partly filled,
plain gate weights (split as they are loaded) and packed ones: the same logits bit by bit."""
import pytest
import torch

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E", [(257, 3), (1984, 128), (1985, 65), (2017, 64), (2047, 128)])
def test_gate(T, E):
    print(f"case T={T} E={E}", flush=True)
    inp = make_inputs(CONFIGS["c2"].scaled(name="gate", T=T, d_model=160, d_ffn=32, E=E, seed=T), "cuda", bias_std=0.02)
    U.check_layer(inp)
    m, logits = U.amd(), []
    for packed in (False, True):
        shape = m.make_shape(T, 160, 32, E, 1, 64, "bf16", False, m.MOE_FLAG_PACKED_GATE if packed else 0)
        out, i32 = torch.empty(T, E, device="cuda"), lambda *s: torch.empty(s, dtype=torch.int32, device="cuda")
        m.moe_gate(shape, inp.x, m.moe_pack_gate(inp.Wg) if packed else inp.Wg, inp.bg, out, i32(T, 1), i32(T, 1), torch.empty(T, 1, device="cuda"),
                   i32(E), i32(E, 64), m.alloc_workspace(shape, "cuda"))
        logits.append(out)
    assert torch.equal(*logits)
