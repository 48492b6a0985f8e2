"""snap_decode_step (append + attend for one layer in one call) against the two
calls it replaces, snap_cache_append then snap_decode_attn: outputs and cache
bytes must be identical bit for bit at every step, and the fused outputs match
the fp64 oracle.  Cases cover the fused kernels (bf16 and fp8, MFMA rows of 64
and 128 and latent) and the two-launch one (fp32), a prompt shorter than the
sinks (new tokens land in sink rows), the ring wrapping, and an invalid slot id.

Every case prints what names it before touching the GPU.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_03092_amd as snap
import synth
from snaphelp import TOL, GpuCache, decode_steps, gpu_compress, params_of, run_case

pytestmark = pytest.mark.gpu

GQA = synth.Workload("step-gqa", 12, 8, 2, 128, 128, False, 4, 16, 300, 32, 7, "bf16", "bf16", layers=1, batch=3,
                     length=None, length_range=(700, 3000), decode_steps=40, rope=True, plant_frac=0.01)


def _announce(msg):
    print(f"\n[case] {msg}", flush=True)


def _clone(cache: GpuCache) -> GpuCache:
    c2 = GpuCache.__new__(GpuCache)
    c2.p, c2.n_slots = cache.p, cache.n_slots
    c2.k = cache.k.clone()
    c2.v = None if cache.v is None else cache.v.clone()
    c2.k_scale = None if cache.k_scale is None else cache.k_scale.clone()
    c2.v_scale = None if cache.v_scale is None else cache.v_scale.clone()
    c2.pos = cache.pos.clone()
    c2.n_topk = cache.n_topk.clone()
    return c2


def _fused_vs_two_calls(wl, p, lengths, slots, n_slots, steps, out_dtype, invalid_slot=False):
    q, k, v = synth.prefill_batch(wl, 0, lengths)
    a = GpuCache(p, n_slots)
    if a.k_scale is not None:
        a.k_scale.fill_(0.05)
        if a.v_scale is not None:
            a.v_scale.fill_(0.05)
    gpu_compress(p, a, q, k, v, lengths, slots, debug=False)
    b = _clone(a)
    call_slots = list(slots) + ([-1] if invalid_slot else [])
    sl = torch.tensor(call_slots, dtype=torch.int32, device="cuda")
    n = len(call_slots)
    ws_a = snap.workspace(snap.snap_decode_workspace(p, n))
    ws_b = snap.workspace(snap.snap_decode_workspace(p, n))
    out_a = torch.zeros((n, p.n_q_heads, p.d_v), dtype=out_dtype, device="cuda")
    out_b = torch.zeros_like(out_a)
    for step in range(steps):
        positions = [int(x) for x in a.pos[sl.clamp_min(0).long()].cpu()]
        qd, kn, vn = synth.decode_inputs(wl, 0, step, positions, device="cuda")
        vn_ = None if vn is None else vn
        snap.snap_cache_append(p, a.c(), a.pos, sl, kn, vn_)
        snap.snap_decode_attn(p, a.c(), a.pos, a.n_topk, sl, qd, out_a, ws_a)
        snap.snap_advance(a.pos, sl)
        snap.snap_decode_step(p, b.c(), b.pos, b.n_topk, sl, qd, kn, vn_, out_b, ws_b)
        snap.snap_advance(b.pos, sl)
        torch.cuda.synchronize()
        nv = len(slots)  # the invalid slot's output row is never written by either path
        assert torch.equal(out_a[:nv].view(torch.int16 if out_dtype == torch.bfloat16 else torch.int32),
                           out_b[:nv].view(torch.int16 if out_dtype == torch.bfloat16 else torch.int32)), step
        assert torch.equal(a.k.view(torch.uint8), b.k.view(torch.uint8)), step
        if a.v is not None:
            assert torch.equal(a.v.view(torch.uint8), b.v.view(torch.uint8)), step
        assert torch.equal(a.pos, b.pos)
    return b


def test_step_gqa_bf16_fused_kernel():
    wl = GQA
    p = params_of(wl)
    lengths = [2900, 2, 1200]
    _announce(f"decode_step bf16 GQA (fused MFMA kernel): lengths {lengths}, ring 16 wraps, one prompt < sinks")
    b = _fused_vs_two_calls(wl, p, lengths, [2, 0, 1], 4, 40, torch.bfloat16, invalid_slot=True)
    # the fused path also matches the oracle from this state on
    err = decode_steps(p, wl, b, [2, 0, 1], 6, torch.bfloat16, TOL["bf16"], salt=7, fused=True)
    print(f"  fused decode max abs err vs oracle: {err:.3e}", flush=True)


def test_step_latent_bf16_fused_kernel():
    wl = synth.small(synth.WORKLOADS["mla-8head-61layer-b16-128k"], recent=64, topk=1000)
    p = params_of(wl)
    lengths = [3000, 3, 1500]
    _announce(f"decode_step bf16 latent (fused LDS kernel): lengths {lengths}, ring 64 wraps")
    b = _fused_vs_two_calls(wl, p, lengths, [0, 1, 2], 3, 80, torch.bfloat16, invalid_slot=True)
    err = decode_steps(p, wl, b, [0, 1, 2], 4, torch.bfloat16, TOL["bf16"], salt=7, fused=True)
    print(f"  fused decode max abs err vs oracle: {err:.3e}", flush=True)


@pytest.mark.parametrize("hq,recent,topk,lengths", [
    (8, 64, 1000, [3000, 3, 1500]),    # the ring wraps over a block boundary; a prompt shorter than the sinks
    (16, 60, 64, [200, 1, 127]),       # one or two 64-row blocks, most workgroups with none
    (3, 192, 700, [70, 900, 255]),     # the new row in the ragged last block
])
def test_step_latent_fp8_fused_kernel(hq, recent, topk, lengths):
    wl = synth.small(synth.WORKLOADS["mla-8head-61layer-b16-128k"], n_q_heads=hq, recent=recent, topk=topk,
                     obs_window=8, kv_dtype="fp8")
    for hint in (snap.SNAP_KV_KEEP, snap.SNAP_KV_STREAM):
        p = params_of(wl, kv_reuse=hint)
        _announce(f"decode_step fp8 latent (fused LDS kernel), {hq} heads, hint {hint}: lengths {lengths}, ring {recent}")
        b = _fused_vs_two_calls(wl, p, lengths, [0, 1, 2], 3, 70, torch.bfloat16, invalid_slot=True)
        err = decode_steps(p, wl, b, [0, 1, 2], 4, torch.float32, TOL["fp8"], salt=7, fused="alt")
        print(f"  max abs err vs oracle: {err:.3e}", flush=True)


@pytest.mark.parametrize("lengths", [[11, 700], [1, 63], [64, 65]])
def test_step_latent_fp8_new_row_is_the_last(lengths):
    """No kept rows: the new token's row is the last valid one and what follows it in its 64-row block must not reach the
    output (cache rows that no token filled are NaN codes)."""
    wl = synth.small(synth.WORKLOADS["mla-8head-61layer-b16-128k"], sink=6, recent=162, topk=0, kv_dtype="fp8")
    p = params_of(wl)
    _announce(f"decode_step fp8 latent, the new row the last one: lengths {lengths}")
    run_case(wl, p, lengths, [1, 0], 2, 4, torch.float32, TOL["fp8"], fp8_scales=True, fused="alt")


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_step_latent_of_two_kv_heads(kv):
    """576-wide latent rows of more than one KV head (decode_generic)."""
    wl = synth.small(synth.WORKLOADS["mla-8head-61layer-b16-128k"], n_kv_heads=2, recent=64, topk=300, obs_window=8,
                     kv_dtype=kv)
    p = params_of(wl)
    lengths = [900, 211]
    _announce(f"decode_step {kv} latent, 2 KV heads: lengths {lengths}")
    run_case(wl, p, lengths, [1, 0], 2, 6, torch.float32, TOL[kv], fp8_scales=kv == "fp8", fused="alt")


def test_step_fp8_fused_and_fp32_two_launch_paths():
    wl = synth.small(GQA, kv_dtype="fp8")
    p = params_of(wl)
    lengths = [2000, 900, 3]
    _announce(f"decode_step fp8 GQA (fused kernel, new row quantised in LDS): lengths {lengths}, one prompt < sinks")
    _fused_vs_two_calls(wl, p, lengths, [1, 0, 2], 3, 24, torch.bfloat16, invalid_slot=True)
    wl = synth.WORKLOADS["tiny-fp32"]
    p = params_of(wl)
    _announce("decode_step fp32 tiny (generic kernel, two launches)")
    _fused_vs_two_calls(wl, p, [wl.length], [0], 1, 24, torch.float32)


@pytest.mark.parametrize("kv_reuse", [snap.SNAP_KV_AUTO, snap.SNAP_KV_STREAM])
def test_fp8_query_products(kv_reuse):
    """snap_params.fp8_qk = 1 over a GQA fp8 cache: the query is quantised per
    head and Q K^T runs on the fp8 MFMA.  Checked against the oracle attending
    with the same quantised query (oracle.fp8_scale / quantize), to the fp8
    tolerance; the deviation from the exact query is reported beside it.  The
    fused step (new row quantised in LDS) and the two-call path both run, with
    ordinary loads (the default at this size) and with streaming loads."""
    from snaphelp import fp8_query
    wl = synth.small(GQA, kv_dtype="fp8")
    p = params_of(wl, fp8_qk=1, kv_reuse=kv_reuse)
    lengths = [2000, 900, 3]
    _announce(f"fp8 query products (fp8_qk=1, kv_reuse {kv_reuse}): lengths {lengths}, fused step then two calls")
    q, k, v = synth.prefill_batch(wl, 0, lengths)
    c = GpuCache(p, 3)
    c.k_scale.fill_(0.05)
    c.v_scale.fill_(0.05)
    gpu_compress(p, c, q, k, v, lengths, [0, 1, 2], debug=False)
    stats = {}
    err = decode_steps(p, wl, c, [0, 1, 2], 6, torch.bfloat16, TOL["fp8"], salt=3, fused=True, q_oracle=fp8_query,
                       stats=stats)
    err2 = decode_steps(p, wl, c, [0, 1, 2], 3, torch.bfloat16, TOL["fp8"], salt=4, fused=False, q_oracle=fp8_query,
                        stats=stats)
    print(f"  max abs err vs oracle with the fp8 query: {max(err, err2):.3e}; "
          f"deviation from the exact query: {stats['exact_query_dev']:.3e}", flush=True)


@pytest.mark.parametrize("kind", ["gqa-bf16", "gqa-fp8", "latent-bf16", "latent-fp8"])
def test_load_hint_keeps_results(kind):
    """snap_params.kv_reuse only changes how the cache rows are loaded: the
    same decode call with ordinary (SNAP_KV_KEEP) and streaming
    (SNAP_KV_STREAM) loads gives the same bits, except the bf16 GQA kernel,
    which adds the dot products' pieces in another order under streaming
    loads (outputs then agree to a few bf16 ulps)."""
    if kind.startswith("gqa"):
        wl = synth.small(GQA, kv_dtype="fp8") if kind == "gqa-fp8" else GQA
        lengths = [2900, 40, 1200]
    else:
        wl = synth.small(synth.WORKLOADS["mla-8head-61layer-b16-128k"], recent=64, topk=1000,
                         kv_dtype="fp8" if kind == "latent-fp8" else "bf16")
        lengths = [3000, 70, 1500]
    p = params_of(wl)
    _announce(f"load hint keep vs stream: {kind}, lengths {lengths}")
    q, k, v = synth.prefill_batch(wl, 0, lengths)
    c = GpuCache(p, 3)
    if c.k_scale is not None:
        c.k_scale.fill_(0.05)
        if c.v_scale is not None:
            c.v_scale.fill_(0.05)
    gpu_compress(p, c, q, k, v, lengths, [0, 1, 2], debug=False)
    sl = torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda")
    positions = [int(x) for x in c.pos.cpu()]
    qd, _, _ = synth.decode_inputs(wl, 0, 0, positions, device="cuda")
    outs = {}
    for hint in (snap.SNAP_KV_KEEP, snap.SNAP_KV_STREAM):
        ph = params_of(wl, kv_reuse=hint)
        out = torch.zeros((3, p.n_q_heads, p.d_v), dtype=torch.float32, device="cuda")
        ws = snap.workspace(snap.snap_decode_workspace(ph, 3))
        snap.snap_decode_attn(ph, c.c(), c.pos, c.n_topk, sl, qd, out, ws)
        torch.cuda.synchronize()
        outs[hint] = out
    a, b = outs[snap.SNAP_KV_KEEP], outs[snap.SNAP_KV_STREAM]
    assert torch.isfinite(a).all()
    if kind == "gqa-bf16":
        diff = float((a - b).abs().max())
        print(f"  max abs difference: {diff:.3e}", flush=True)
        assert diff <= 1e-4 * max(1.0, float(a.abs().max()))
    else:
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# 64-wide rows and caches whose values are the key rows keep 32-bit
# probabilities (split into three bf16 parts for the value product), so with
# fp32 outputs they are held to the fp32 bound.
@pytest.mark.parametrize("d,v_in_k,kv,hq,hkv,stream", [
    (64, False, "bf16", 8, 2, False),
    (64, False, "bf16", 16, 1, True),   # 16 heads fill the matrix instruction's columns
    (64, False, "fp8", 6, 2, True),
    (64, False, "fp8", 2, 2, False),
    (64, True, "bf16", 3, 1, False),
    (64, True, "fp8", 8, 2, True),
    (128, True, "bf16", 8, 2, True),
    (128, True, "fp8", 4, 4, False),
])
def test_step_with_32_bit_probabilities(d, v_in_k, kv, hq, hkv, stream):
    wl = synth.small(GQA, name="step-32bit", n_q_heads=hq, n_kv_heads=hkv, d_qk=d, d_v=d, v_in_k=v_in_k, kv_dtype=kv,
                     topk=301, obs_window=8, rope=not v_in_k, plant_frac=None if v_in_k else 0.01)
    p = params_of(wl, kv_reuse=snap.SNAP_KV_STREAM if stream else snap.SNAP_KV_KEEP)
    lengths = [2900, 2, 333]
    _announce(f"decode_step d {d} v_in_k {int(v_in_k)} cache {kv} heads {hq}/{hkv} stream {int(stream)}: {lengths}")
    b = _fused_vs_two_calls(wl, p, lengths, [2, 0, 1], 4, 24, torch.bfloat16, invalid_slot=True)
    err = decode_steps(p, wl, b, [2, 0, 1], 4, torch.float32, TOL["f32"], salt=7, fused="alt")
    print(f"  max abs err vs oracle: {err:.3e}", flush=True)


@pytest.mark.parametrize("kv_reuse", [snap.SNAP_KV_KEEP, snap.SNAP_KV_STREAM])
def test_infinite_value_stays_infinite(kv_reuse):
    """A value row holding +inf and -inf (bf16 overflow) makes those output
    dims infinite of that sign, whatever the later parts of its split
    probability are, and leaves the others finite."""
    wl = synth.small(GQA, name="step-inf", d_qk=64, d_v=64, plant_frac=None)
    p = params_of(wl, kv_reuse=kv_reuse)
    _announce(f"infinite values, d 64, kv_reuse {kv_reuse}")
    q, k, v = synth.prefill_batch(wl, 0, [700])
    c = GpuCache(p, 1)
    gpu_compress(p, c, q, k, v, [700], [0], debug=False)
    c.v[0, :, 7, 5] = float("inf")
    c.v[0, :, 40, 9] = float("-inf")
    sl = torch.tensor([0], dtype=torch.int32, device="cuda")
    qd, kn, vn = synth.decode_inputs(wl, 0, 0, [700], device="cuda")
    qd[0, 0] = 0  # equal logits: every probability is 1, its later parts are zero
    out = torch.zeros((1, p.n_q_heads, p.d_v), dtype=torch.float32, device="cuda")
    snap.snap_decode_step(p, c.c(), c.pos, c.n_topk, sl, qd, kn, vn, out, snap.workspace(snap.snap_decode_workspace(p, 1)))
    torch.cuda.synchronize()
    assert (out[0, :, 5] == float("inf")).all() and (out[0, :, 9] == float("-inf")).all()
    assert torch.isfinite(out[0, :, [d for d in range(64) if d not in (5, 9)]]).all()


def _latent_in_32_row_blocks(q, rows, scale, n_chunks):
    """Attention of q [G][576] over latent rows [nv][576] (values: the first 512
    dims) as a split-K wave takes it: one run of rows per chunk (a multiple of 32
    of them), 32 rows at a time, a head's reference moved only when a block's
    largest logit passes it by more than 8 (log2 units), probabilities against
    that reference rounded to bf16 for the value product and summed unrounded."""
    nv = rows.shape[0]
    per = (-(-nv // n_chunks) + 31) & ~31
    x = (q.astype(np.float64) @ rows.T.astype(np.float64) * (scale * np.log2(np.e))).astype(np.float32)
    part = []
    for v0 in range(0, nv, per):
        m = np.full(q.shape[0], -np.inf, np.float32)
        l, acc = np.zeros(q.shape[0]), np.zeros((q.shape[0], 512))
        for vb in range(v0, min(v0 + per, nv), 32):
            end = min(vb + 32, v0 + per, nv)
            bm = x[:, vb:end].max(1)
            mn = np.where(bm > m + 8, bm, m)
            alpha = np.exp2((m - mn).astype(np.float64))
            m = mn
            pe = np.exp2((x[:, vb:end] - m[:, None]).astype(np.float64)).astype(np.float32)
            pb = torch.from_numpy(pe).to(torch.bfloat16).double().numpy()
            l = l * alpha + pe.sum(1, dtype=np.float64)
            acc = acc * alpha[:, None] + pb @ rows[vb:end, :512].astype(np.float64)
        part.append((m.astype(np.float64), l, acc))
    top = np.max([m for m, _, _ in part], axis=0)
    num = sum(np.exp2(m - top)[:, None] * acc for m, _, acc in part)
    return num / sum(np.exp2(m - top) * l for m, l, _ in part)[:, None]


@pytest.mark.parametrize("hq,n_topk", [(8, 444), (8, 301), (16, 20), (3, 0)])
def test_fp8_latent_rounding_order(hq, n_topk):
    """Which probabilities an fp8 latent decode rounds to which bf16 values: the
    reference moves per 32 rows of one run of rows per chunk.  Rows taken in
    another order or grouping (64 at a time, interleaved over the chunks) are as
    near the exact attention, 1.7e-3, but differ from this order by 0.8e-3 to
    2.6e-3.  What is left between equal orders is a logit's fp32 rounding (about
    2e-6 in log2 units), which moves at most about 1e-3 of the probabilities over
    a bf16 rounding edge (2^-8 of each): 2^-8 * sqrt(1e-3) = 1.2e-4, held to 3e-4
    (measured 2e-7 to 3e-5).
    n_topk 301: the second chunk starts at row 192; 20 and 0: a last block of
    fewer than 32 rows."""
    sink, recent, topk, n = 4, 64, 444, 2
    p = snap.Params(n_q_heads=hq, n_kv_heads=1, d_qk=576, d_v=512, sink=sink, recent=recent, topk=topk, obs_window=8,
                    pool_kernel=7, v_in_k=True, kv_dtype=snap.SNAP_FP8_E4M3)
    _announce(f"fp8 latent, rounding order: {hq} heads, n_topk {n_topk}")
    gen = torch.Generator().manual_seed(hq + n_topk)
    codes = (torch.randn((n, 1, p.budget, 576), generator=gen) * 40).to(torch.float8_e4m3fn)
    q = torch.randn((n, hq, 576), generator=gen).to(torch.bfloat16)
    c = GpuCache(p, n)
    c.k.copy_(codes.view(torch.uint8))
    c.k_scale.fill_(0.0625)
    c.pos.fill_(1000)
    c.n_topk.fill_(n_topk)
    sl = torch.arange(n, dtype=torch.int32, device="cuda")
    out = torch.zeros((n, hq, 512), dtype=torch.float32, device="cuda")
    snap.snap_decode_attn(p, c.c(), c.pos, c.n_topk, sl, q.to("cuda"), out, snap.workspace(snap.snap_decode_workspace(p, n)))
    torch.cuda.synchronize()
    table = np.array([oracle.e4m3_value(i) for i in range(256)])
    for b in range(n):
        rows = table[codes[b, 0, :sink + recent + n_topk].view(torch.uint8).numpy()] * 0.0625
        # 512 rows of two sequences make two chunks of at least 256
        exp = _latent_in_32_row_blocks(q[b].double().numpy(), rows, 576 ** -0.5, 2)
        got = out[b].double().cpu().numpy()
        err = float(np.linalg.norm(got - exp) / np.linalg.norm(exp))
        print(f"  sequence {b}: {err:.2e}", flush=True)
        assert err <= 3e-4
