"""GPU parity of the bf16 backward's key passes and dQ pass at the sizes where
their blocks can go wrong, against the oracle's backward_slice (the method and
tolerance of test_gpu_backward.py).

The tolerance is that file's bf16 bound: weights and their gradients enter the
products rounded to bf16 (relative 2^-9 each), sums are fp32; neither changes
with the blocks.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mita_oracle as O
from paper_2602_01219_amd import mita, synth
from tests.gpu_helpers import from_dev, log, maxrel, to_dev
from tests.test_gpu_backward import TOL, _check_backward, _upstream

pytestmark = pytest.mark.gpu

# grid, landmark grid, k, d, clusters: one key past a block (65 of 64 or 128
# keys per block) and past the landmarks' two-wave block, exactly one block of
# each, a single key and a single query stage, long experts (several stages
# of 64 queries, with a remainder), a block of at most 64 keys by four waves (32
# queries per expert) and by two (fewer), more slots per token block than the kernel
# keeps in LDS (k = N: every token in every expert's set), d = 128.
# (The keys of an expert must not be all alike: dq sums dZ_j k_j with sum dZ_j =
# 0, so the rounding of D = dO . o to bf16's o comes back times the keys' mean.)
CASES = [(29, 37, 5, 13, 65, 64, 4), (16, 16, 8, 8, 64, 64, 4), (16, 24, 8, 16, 128, 64, 4), (1, 130, 1, 2, 1, 64, 2),
         (40, 50, 2, 2, 129, 64, 64), (16, 40, 4, 5, 64, 64, 4), (16, 40, 3, 7, 37, 64, 4), (12, 12, 3, 3, 144, 64, 3), (20, 21, 4, 5, 200, 128, 4), (9, 15, 3, 3, 135, 128, 3)]


def _workload(case):
    gh, gw, lh, lw, k, d, clusters = case
    return synth.Workload(name="bwd_keys", B=1, H=2, grid_h=gh, grid_w=gw, d=d, lm_h=lh, lm_w=lw, k=k, dtype="bf16",
                          clusters=clusters, std=0.5, cluster_map="voronoi" if gh > 1 and clusters < 64 else "iid", seed=7 + gh * gw + k)


@pytest.mark.parametrize("case", CASES, ids=["%dx%d_m%d_k%d_d%d" % (c[0], c[1], c[2] * c[3], c[4], c[5]) for c in CASES])
def test_key_blocks(case):
    wl = _workload(case)
    _check_backward(mita.Config.from_workload(wl), synth.generate(wl), [(0, 0), (0, 1)])


@pytest.mark.parametrize("d", [64, 128])
def test_scores_far_above_the_first_tile(d):
    """Every routed key's score exceeds the first key tile's maximum (the
    landmarks come first) by more than 2^7 (log2 units), so the one-sweep dQ
    pass overflows and runs again with each query's own log-sum-exp. Dim 0
    lifts the scores: 4 in the queries, so in the landmarks too, and 40 sqrt(d)
    in the keys. dq is compared without it: there the keys' common part comes
    back times the rounding of D = dO . o (o is bf16)."""
    wl = _workload((20, 21, 6, 6, 70, d, 64))
    inp = synth.generate(wl)
    q, k, v, dO = (synth.bf16_bits_to_f32(t) for t in (inp.q, inp.k, inp.v, _upstream(wl)))
    q[..., 0], k[..., 0] = 4.0, 40.0 * np.sqrt(d)
    cfg = mita.Config.from_workload(wl)
    t = [to_dev(synth.f32_to_bf16_bits(y), "bf16") for y in (q, k, v, dO)]
    o = mita.forward(cfg, *t[:3])
    got = [from_dev(y) for y in mita.backward(cfg, *t[:3], o, t[3])]
    q_lm = mita.landmarks(cfg, t[0])
    idx = mita.topk(cfg, mita.scores(cfg, q_lm, t[1], want_v_lm=False)[0]).cpu().numpy().astype(np.int64)
    expert = mita.route(cfg, t[0], q_lm)[0].cpu().numpy().astype(np.int64)
    for h in range(wl.H):
        x = [from_dev(y)[0, h].astype(np.float64) for y in t]
        ref = O.backward_slice(*x, cfg.grid_h, cfg.grid_w, cfg.lm_h, cfg.lm_w, cfg.k, None, 1, 1,
                               force_idx=idx[0, h], force_expert=expert[0, h])
        errs = [maxrel(got[0][0, h][:, 1:], ref.dq[:, 1:]), maxrel(got[1][0, h], ref.dk), maxrel(got[2][0, h], ref.dv)]
        log(f"  head {h}: max-rel dq {errs[0]:.3e} dk {errs[1]:.3e} dv {errs[2]:.3e}")
        assert max(errs) <= TOL["bf16"], errs
