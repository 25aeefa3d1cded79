"""bench.py: the work of products that share a launch is counted in the stage that was timed."""
import numpy as np
import pytest

import bench
from workloads import CONFIGS

C1, C3B = CONFIGS["c1"], CONFIGS["c3b"]


@pytest.mark.parametrize("cfg,timed,shared", [
    (C1, ["gate_logits", "expert_gemm1"], {"expert_gemm1": "both products"}),
    (C1, ["expert_gemm1", "expert_gemm2"], {}),
    (C1.scaled(residual=True), ["expert_gemm1", "dense_gemm1"], {"expert_gemm1": "both products", "dense_gemm1": "both products"}),
    (C1.scaled(residual=True), ["expert_gemm1", "expert_gemm2", "dense_gemm1"], {"dense_gemm1": "both products"}),
    (C3B, ["expert_gemm1", "expert_gemm2"], {"expert_gemm1": "experts + dense branch", "expert_gemm2": "experts + dense branch"}),
    (C3B, ["expert_gemm1", "expert_gemm2", "dense_gemm1"], {"expert_gemm2": "experts + dense branch"}),
    (C3B, ["expert_gemm1", "expert_gemm2", "dense_gemm1", "dense_gemm2"], {}),
])
def test_work_of_shared_launches(cfg, timed, shared):
    rows = np.full(cfg.E, 4)
    alg, plain = bench.algorithmic_work(cfg, rows), bench.algorithmic_work(cfg, rows)
    assert bench.place_work(cfg, alg, dict.fromkeys(timed, 1.0)) == shared
    for work in ("stage_bytes", "stage_flops"):
        products = [s for s in plain[work] if "gemm" in s and (cfg.residual or "dense" not in s)]
        assert sum(alg[work][s] for s in timed if "gemm" in s) == sum(plain[work][s] for s in products)
