"""Gate of 257 to 4096 tokens off the bf16 matrix cores (fp32 tokens, or d_model off 32) with at most 64 experts: logits, top-k and
the ranks of 16 tokens in one launch -- edges of the tiles of 16 and 256 tokens and of the range, experts of one lane, of whole and
ragged 16-lane rows, d_model of whole, ragged and fewer steps than the waves share -- through moe_layer_forward against the oracle."""
import pytest

from tests import gpu_util as U
from workloads import CONFIGS, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,dtype", [
    (257, 64, 8, 1, "f32"), (257, 200, 31, 2, "f32"), (272, 4, 2, 2, "f32"), (511, 512, 64, 1, "f32"), (513, 128, 64, 2, "f32"),
    (1023, 100, 1, 1, "f32"), (1536, 512, 8, 2, "f32"), (4095, 36, 17, 2, "f32"), (4096, 128, 33, 1, "f32"), (4097, 64, 8, 2, "f32"),
    (300, 64, 65, 2, "f32"), (257, 1000, 40, 2, "bf16"), (1000, 40, 16, 1, "bf16"), (4096, 8, 64, 2, "bf16"), (4097, 40, 64, 1, "bf16"),
])
def test_gate(T, d, E, k, dtype):
    print(f"case T={T} d={d} E={E} k={k} {dtype}", flush=True)
    cfg = CONFIGS["c1" if dtype == "f32" else "c3a"].scaled(name="gate", T=T, d_model=d, d_ffn=2 * d, E=E, top_k=k, residual=False, seed=11)
    U.check_layer(make_inputs(cfg, "cuda", bias_std=0.05))
