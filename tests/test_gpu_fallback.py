"""Rows of the fused selection that fall back, where several experts per query
or the backward pass use their sets: the default path against the one over
stored scores (mita.Config full_scores), which selects every set from a stored
score row.

Forward outputs are equal bit for bit (scores, sets, routing and the order of
every merge are the same). Gradients are sums of the same products in an order
that varies from run to run: an element moves by at most the rounding of its
fp32 sums and one rounding to the io type, 2^-8 of its value in bf16 and, of
the tensor's norm, 1e-6 in fp32.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

from paper_2602_01219_amd import mita, synth
from tests.gpu_helpers import inputs_to_dev, log

pytestmark = pytest.mark.gpu

SAMPLE = 1024  # keys the forward samples per landmark row for its top-k pivot

# N with and without a factor of four (the selection's loads), landmarks in one
# block, in several and (1000: 2000 groups at s > 1) in more than 1024 groups
# N, landmark rows and columns, k, d, dtype, H, clusters
SHAPES = [(2048, 8, 8, 128, 64, "bf16", 2, 12), (1601, 1, 17, 40, 64, "bf16", 3, 5), (4098, 5, 13, 100, 128, "bf16", 1, 20),
          (3000, 20, 50, 33, 64, "bf16", 1, 64), (2050, 3, 7, 64, 64, "f32", 2, 6), (17000, 4, 8, 700, 64, "bf16", 1, 9)]
IDS = ["n%d_m%d_k%d_d%d_%s" % (c[0], c[1] * c[2], c[3], c[4], c[5]) for c in SHAPES]


def _case(shape, s=1):
    N, lh, lw, k, d, dtype, H, clusters = shape
    g = next(g for g in range(int(N ** 0.5), 0, -1) if N % g == 0)
    if lh > g:
        g, lh, lw = 1, 1, lh * lw
    wl = synth.Workload(name="fallback", B=1, H=H, grid_h=g, grid_w=N // g, d=d, lm_h=lh, lm_w=lw, k=k, dtype=dtype,
                        clusters=clusters, std=0.5, cluster_map="iid", seed=N + k)
    cfg = dataclasses.replace(mita.Config.from_workload(wl), s=s)
    plan = mita.select_plan(cfg)
    assert plan["fused"] and plan["ns"] < N
    return cfg, inputs_to_dev(synth.generate(wl))


def _keys(kind, K, N):
    """Head 0's keys such that its rows' lists miss: all alike (every score
    ties, beyond the list) or large at exactly the sampled positions (the
    pivot lies above the k-th score)."""
    K = K.clone()
    if kind == "zero":
        K[0, 0] = 0
    else:
        pos = ((2 * np.arange(SAMPLE) + 1) * N) // (2 * SAMPLE)
        K[0, 0, torch.from_numpy(pos).cuda()] *= 8
    return K


@pytest.mark.parametrize("kind", ["zero", "sample"])
@pytest.mark.parametrize("s", [1, 2, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_forward(shape, s, kind):
    cfg, (q, k, v) = _case(shape, s)
    K = _keys(kind, k, cfg.N)
    ws = torch.empty(mita.workspace_size(cfg), dtype=torch.uint8, device="cuda")
    ref = mita.forward(dataclasses.replace(cfg, full_scores=True), q, K, v)
    for staged in (False, True):
        c = dataclasses.replace(cfg, staged_gather=staged)
        ws = torch.empty(mita.workspace_size(c), dtype=torch.uint8, device="cuda")
        o = mita.forward(c, q, K, v, ws=ws)
        n = mita.forward_fallbacks(c, ws)
        log(f"  staged {staged}: {n} rows of {cfg.H * cfg.M} fell back, {int((o != ref).sum())} elements differ")
        # (a pivot rank of k leaves at least k sampled tokens above the pivot)
        assert n == cfg.M if kind == "zero" else n >= 1 or mita.select_plan(cfg)["rank"] >= cfg.k
        assert torch.isfinite(o).all() and torch.equal(o, ref)


@pytest.mark.parametrize("kind", ["zero", "sample"])
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_backward(shape, kind):
    cfg, (q, k, v) = _case(shape)
    K = _keys(kind, k, cfg.N)
    o = mita.forward(cfg, q, K, v)
    dO = torch.randn(q.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(5)).to(q.dtype)
    got = mita.backward(cfg, q, K, v, o, dO)
    ref = mita.backward(dataclasses.replace(cfg, full_scores=True), q, K, v, o, dO)
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        err = float((a.double() - b.double()).norm() / b.double().norm())
        log(f"  {name}: {err:.1e}")
        assert torch.isfinite(a.float()).all() and err <= (2.0 ** -8 if cfg.dtype == "bf16" else 1e-6), name


@pytest.mark.parametrize("s", [1, 2])
def test_rows_of_experts_without_queries_are_not_rescored(s):
    """Every row falls back (zero keys in all heads) and is listed, but only
    those of experts with queries are scored: the score rows of the others keep
    the bits the workspace held on entry."""
    cfg, (q, k, v) = _case((2048, 8, 16, 64, 64, "bf16", 2, 7), s)
    K = torch.zeros_like(k)
    ws = torch.full((mita.workspace_size(cfg),), 0xFF, dtype=torch.uint8, device="cuda")
    o = mita.forward(cfg, q, K, v, ws=ws)
    assert mita.forward_fallbacks(cfg, ws) == cfg.H * cfg.M
    assert torch.equal(o, mita.forward(dataclasses.replace(cfg, full_scores=True), q, K, v))
    # the workspace begins with q_lm, v_lm (bf16 [H, M, d], 256-byte aligned) and S (fp32 [H, M, N])
    lm = cfg.H * cfg.M * cfg.d * 2
    assert lm % 256 == 0
    S = ws[2 * lm:2 * lm + cfg.H * cfg.M * cfg.N * 4].view(torch.int32).view(cfg.H, cfg.M, cfg.N)
    expert = mita.route(cfg, q, mita.landmarks(cfg, q))[0].view(cfg.H, -1).long()
    live = torch.zeros((cfg.H, cfg.M), dtype=torch.bool, device="cuda").scatter_(1, expert, True)
    log(f"  {int(live.sum())} of {cfg.H * cfg.M} experts have queries")
    assert 0 < int(live.sum()) < cfg.H * cfg.M
    assert torch.equal((S != -1).all(-1), live) and torch.equal((S != -1).any(-1), live)


def _us(f, n=5):
    f()
    best = float("inf")
    for _ in range(3):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(n):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / n * 1e3)
    return best


@pytest.mark.parametrize("what", ["s1", "s2", "backward"])
def test_fallback_rows_use_the_whole_chip(what):
    """Every row of 12 heads falls back (padded or repeated tokens do this):
    the call may take longer than with stored scores, whose pass forms 64
    landmarks' scores at once and not one row's, but not by an order of
    magnitude. Measured: 2.9 (s = 1), 2.1 (s = 2) and 1.4 times (backward); 24,
    15 and 5 with the rows on 64 workgroups."""
    shape = (16384, 8, 16, 512, 64, "bf16", 12, 32)
    cfg, (q, k, v) = _case(shape, 2 if what == "s2" else 1)
    K = torch.zeros_like(k)
    full = dataclasses.replace(cfg, full_scores=True)
    t = []
    for c in (cfg, full):
        ws = torch.empty(mita.workspace_size(c), dtype=torch.uint8, device="cuda")
        o = mita.forward(c, q, K, v, ws=ws)
        if what == "backward":
            wb = torch.empty(mita.workspace_size(c, mita.WS_BACKWARD), dtype=torch.uint8, device="cuda")
            out = [torch.empty_like(q) for _ in range(3)]
            dO = torch.ones_like(q)
            t.append(_us(lambda: mita.backward(c, q, K, v, o, dO, *out, ws=wb)))
        else:
            t.append(_us(lambda: mita.forward(c, q, K, v, o=o, ws=ws)))
    log(f"  {what}: {t[0]:.0f} us, with stored scores {t[1]:.0f} us")
    assert t[0] <= 4.0 * t[1]
