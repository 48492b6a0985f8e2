"""The orders in which the attention's workgroups go over the KV heads: 8 and more that keep to one XCD each, the rest
of them spread over all, and batches that are spread as a whole (snap_prefill against the fp64 oracle)."""
import pytest

import synth
from snaphelp import params_of
from test_gpu_prefill import GQA, _announce, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,lengths", [
    (1, [515]),            # one group, its blocks on all XCDs
    (3, [260]),
    (9, [130]),            # 8 on an XCD each, 1 spread
    (12, [200, 65]),       # a batch of 24, spread as a whole
    (12, [140]),           # 8 and 4
    (6, [300, 40, 129]),   # 18 spread: turns of 4
    (2, [64, 450, 1, 200]),  # 8 spread: turns of 1
    (4, [450, 1, 200, 64, 130, 300, 90, 513]),  # 32 spread: 9 places a turn
])
def test_prefill_group_orders(hkv, lengths):
    wl = synth.small(GQA, n_q_heads=2 * hkv, n_kv_heads=hkv, d_qk=64, d_v=64, obs_window=8, recent=16, topk=40)
    p = params_of(wl)
    _announce(f"snap_prefill {len(lengths)} x {hkv} KV heads: lengths {lengths}")
    _run(wl, p, lengths)
