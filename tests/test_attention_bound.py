"""The bound that the GPU attention tests hold a layer's output to (gpu_util.attention_reference)
is passed by an emulation of the device's roundings and failed by an output that leaves out a
single key, also where that key is one of many."""
import numpy as np
import pytest

import kvp_inputs as ki
from oracle import attention as oat

from gpu_util import attention_reference, oracle_weights, small_workload


@pytest.mark.parametrize("S,key", [(65, 64), (193, 192), (385, 320), (900, 832)])
def test_one_key_left_out_breaks_the_bound(S, key):
    a, g = 3, 1
    w = small_workload("split-keys", 1, a * 128, a, g, [0])
    lw = oracle_weights(w)[0]
    x = ki.prefill_x(w, [0], np.arange(S))[0]
    _, k, v = oat.project_qkv(x.astype(np.float64), np.arange(S), lw, a, g, 128, w.rope_base)
    rnd = lambda t: ki.round_to_bf16(t.astype(np.float32)).astype(np.float64)  # noqa: E731
    k, v = rnd(k), rnd(v)
    ref, bound = attention_reference(x, lw, k, v, a, w.rope_base)
    wrong, _ = attention_reference(x, lw, k, v, a, w.rope_base, drop=[key])
    assert (np.abs(wrong - ref) / bound).max() > 1.5
    # Weights rounded to bf16 against the row's maximum, the sum of the unrounded ones, output rounded.
    q, _, _ = oat.project_qkv(x.astype(np.float64), np.arange(S), lw, a, g, 128, w.rope_base, kv=False)
    s = rnd(q) @ k[0].T / np.sqrt(128)
    s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    o = rnd(rnd(p) @ v[0] / p.sum(-1, keepdims=True)).transpose(1, 0, 2).reshape(S, -1)
    assert (np.abs(o - ref) / bound).max() <= 0.75
