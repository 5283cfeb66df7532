"""The pivots of the fused selection (scores of 1024 sampled keys per landmark
row) in each of their kernels: a row per wave, and sixteen rows per workgroup of
4, 8 and 16 waves. A wrong pivot gives a list that misses the row's top-k or
holds too much: outputs are compared bit for bit with the path over stored scores
(mita.Config full_scores), and the rows that fall back are counted.
"""
from __future__ import annotations

import dataclasses

import pytest
import torch

from paper_2602_01219_amd import mita
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

# 40 landmarks are two blocks of 16 rows and a part of a third. Heads: 3 blocks;
# each side of 64 (63 and 66) and of 128 blocks (126 and 129); fp32 and d = 128
# change kernels at 64.
CASES = [(1, 64, "bf16"), (21, 64, "bf16"), (22, 64, "bf16"), (42, 64, "bf16"), (43, 64, "bf16"), (21, 128, "bf16"),
         (22, 128, "bf16"), (21, 64, "f32"), (22, 64, "f32"), (2, 128, "f32"), (22, 128, "f32")]


@pytest.mark.parametrize("how", ["s1", "s2", "staged"])
@pytest.mark.parametrize("case", CASES, ids=["h%d_d%d_%s" % c for c in CASES])
def test_crowded_rows(case, how):
    """Head 0's keys are one vector u plus noise in the upper half of the
    dimensions. Landmarks 0, 5, 10, ... (one to four of each block of 16 rows)
    have no part there: all their samples tie, far more than the 64 of a bin that
    are ranked, and the whole block finds its pivots by bisection. Those rows
    list every token and fall back; their neighbours, whose samples spread, and
    the other heads do not."""
    H, d, dtype = case
    N, M, k = 2048, 40, 128
    cfg = mita.Config(B=1, H=H, N=N, d=d, grid_h=1, grid_w=N, M=M, lm_h=1, lm_w=M, k=k, dtype=dtype,
                      s=2 if how == "s2" else 1, staged_gather=how == "staged")
    plan = mita.select_plan(cfg)
    assert plan["fused"] and plan["ns"] == 1024 and plan["cap"] < N
    g = torch.Generator("cuda").manual_seed(7 + H)
    dt = cfg.torch_dtype
    q, K, v = ((0.5 * torch.randn((1, H, N, d), device="cuda", generator=g)).to(dt) for _ in range(3))
    q_lm = (0.5 * torch.randn((1, H, M, d), device="cuda", generator=g)).to(dt)
    K[0, 0, :, :d // 2] = K[0, 0, 0, :d // 2]
    q_lm[0, 0, ::5, d // 2:] = 0
    ws = torch.empty(mita.workspace_size(cfg), dtype=torch.uint8, device="cuda")
    o = mita.forward(cfg, q, K, v, ws=ws, q_lm=q_lm)
    n = mita.forward_fallbacks(cfg, ws)
    ref = mita.forward(dataclasses.replace(cfg, full_scores=True, staged_gather=False), q, K, v, q_lm=q_lm)
    log(f"  {n} rows fell back, {int((o != ref).sum())} elements differ")
    assert n == M // 5
    assert torch.isfinite(o).all() and torch.equal(o, ref)
