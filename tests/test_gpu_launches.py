"""The launches of a call, by the kernel names its timer records: which variant
a size takes, at each side of the rules' lines. What the variants compute is
tested elsewhere (test_gpu_forward_paths.py, test_gpu_parity.py)."""
from __future__ import annotations

import dataclasses

import pytest
import torch

from paper_2602_01219_amd import mita

pytestmark = pytest.mark.gpu


def _launches(cfg, backward=False):
    g = torch.Generator("cuda").manual_seed(3)
    q, k, v = ((0.3 * torch.randn((cfg.B, cfg.H, cfg.N, cfg.d), device="cuda", generator=g)).to(cfg.torch_dtype)
               for _ in range(3))
    t = mita.Timer(1)
    o = mita.forward(cfg, q, k, v, timer=None if backward else t)
    if backward:
        mita.backward(cfg, q, k, v, o, q, timer=t)
    names = [n for n, _, _ in t.launches()[0]]
    t.close()
    return names


def _cfg(H, N, M, k, **kw):
    return mita.Config(B=1, H=H, N=N, d=kw.pop("d", 64), grid_h=1, grid_w=N, M=M, lm_h=1, lm_w=M, k=k, **kw)


@pytest.mark.parametrize("s,backward", [(1, False), (2, False), (1, True)])
def test_direct_selection_routes_behind_the_scores(s, backward):
    """N <= 1024 with more scores than the one-launch form takes: sets and
    landmark values first, then the routing, the attention right behind it."""
    names = _launches(_cfg(96, 1024, 49, 49, s=s), backward)
    logits = "route_tops_kernel" if s > 1 else "route_logits_kernel"
    assert names[1:6] == ["sample_pivot_kernel", "scores_kernel", "merge_kernel", logits, "topk_scatter_kernel"]


@pytest.mark.parametrize("s", [1, 2])
def test_listed_selection_routes_before_the_scores(s):
    names = _launches(_cfg(4, 1025, 16, 49, s=s))
    logits = names.index("route_tops_kernel" if s > 1 else "pivots_logits_kernel")
    assert logits < names.index("scores_kernel") < names.index("topk_scatter_kernel")


@pytest.mark.parametrize("N,H,finish", [(1100, 64, "finalize_kernel"), (1100, 65, "finalize_wave_kernel"),
                                        (4096, 96, "finalize_kernel"), (4096, 97, "finalize_wave_kernel")])
def test_few_rows_finish_by_workgroups(N, H, finish):
    """Sixteen landmarks per head: 1024 and 1040 rows, 1536 and 1552."""
    assert finish in _launches(_cfg(H, N, 16, 40))


def test_launches_by_name():
    """Every kernel of a call under its own name."""
    assert _launches(_cfg(6, 196, 16, 49)) == ["pool_small_kernel", "direct_kernel", "attend16_kernel"]
    assert _launches(_cfg(2, 4096, 16, 300, d=128)) == ["pool_kernel", "pivots_logits_kernel", "scores16_kernel",
                                                        "finalize_kernel", "topk_scatter_kernel", "attend16_kernel"]
    assert _launches(_cfg(2, 2048, 16, 100, s=2, dtype="f32")) == [
        "pool_kernel", "route_tops_kernel", "sample_pivot_kernel", "scores_kernel", "finalize_kernel",
        "topk_scatter_kernel", "attend_kernel", "combine_kernel"]
