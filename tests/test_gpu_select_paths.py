"""Score passes and selection at the sizes and score distributions where their
paths change.

  rows    score_stream (at most 64 score rows: one, 32, 33 and 64) and the
          one-barrier double buffer of score_pass (65 rows and more), 64 and 128
          wide, with candidates that end inside a 16-key tile, at a chunk and one
          past it, prompts shorter than the window, both normalisers and pools
  scores  select_threshold: every score equal (more than its list holds), a tie
          at the threshold, scores more than 64 octaves below the largest (the
          lowest histogram bin), spread out and all within one part of it

Bounds are those of the selection and score checks of every compression test.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2511_03092_amd as snap
import synth
from snaphelp import GpuCache, check_compress, gpu_compress, oracle_params, params_of, run_case, TOL

pytestmark = pytest.mark.gpu

_WL = synth.Workload("select-paths", 16, 8, 2, 64, 64, False, 4, 32, 200, 32, 7, "bf16", "bf16", layers=1, batch=2,
                     length=None, length_range=(10, 3000), decode_steps=4, rope=True, plant_frac=0.01)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,w,norm,pool", [
    (1, 1, synth.NORM_CAND, synth.POOL_MAX),
    (2, 16, synth.NORM_ROW, synth.POOL_MAX),
    (3, 11, synth.NORM_CAND, synth.POOL_AVG),
    (2, 32, synth.NORM_CAND, synth.POOL_MAX),
    (5, 13, synth.NORM_ROW, synth.POOL_AVG),
])
def test_score_rows(d, heads, w, norm, pool):
    wl = synth.small(_WL, n_q_heads=2 * heads, d_qk=d, d_v=d, obs_window=w, norm=norm, pool=pool)
    p = params_of(wl)
    ends = p.sink + p.recent
    # 256 keys: the shortest chunk; 16: a tile of a wave
    lengths = [10, ends + 1, ends + 241, ends + 256, ends + 257, ends + 2 * 1024 + 17]
    print(f"\n[case] {heads * w} rows of {d}, norm {norm}, pool {pool}, lengths {lengths}", flush=True)
    run_case(wl, p, lengths, list(range(6)), 6, 2, torch.float32, TOL["bf16"])


def _k_of_logits(z, q0):
    """Keys [n, 64] whose logit with the query q0 * e0 is z (rounded to bf16)."""
    k = torch.zeros((len(z), 64))
    k[:, 0] = torch.as_tensor(z, dtype=torch.float32) * math.sqrt(64) / q0
    return k.to(torch.bfloat16)


@pytest.mark.parametrize("name", ["equal", "tie", "deep", "deep-narrow"])
@pytest.mark.parametrize("pool", [synth.POOL_MAX, synth.POOL_AVG])
def test_score_distributions(name, pool):
    wl = synth.small(_WL, n_q_heads=2, n_kv_heads=1, obs_window=8, topk=700, pool=pool, rope=False)
    p = params_of(wl)
    L, g = 5100, np.random.default_rng(7)
    z = np.zeros(L)
    if name == "tie":
        z[g.choice(np.arange(200, L - 200), 60, replace=False)] = 3.0
    elif name.startswith("deep"):
        z = g.normal(0.0, 1.0 if name == "deep" else 0.02, L)
        z[g.choice(np.arange(200, L - 200), 20, replace=False)] = 60.0
    q0 = 8.0
    q = torch.zeros((1, 2, 8, 64))
    q[..., 0] = q0
    q = q.to(torch.bfloat16)
    k = _k_of_logits(z, q0)[None, None]
    v = torch.from_numpy(g.normal(size=(1, 1, L, 64))).to(torch.bfloat16)
    print(f"\n[case] scores {name}, pool {pool}: {L - p.sink - p.recent} candidates, {p.topk} kept", flush=True)
    cache = GpuCache(p, 1)
    sel, pooled = gpu_compress(p, cache, q, k, v, [L], [0])
    check_compress(p, cache, q, k, v, [L], [0], sel, pooled)
    if name in ("equal", "tie") and pool == synth.POOL_MAX:
        # equal scores: the lowest tokens
        P = oracle.compress(oracle_params(p), [L], q, k, v).groups[0][0].P
        assert sel[0, 0].tolist() == list(oracle.topk(L, p.sink, p.recent, p.topk, P))
