"""Scores that are not finite: a NaN key reaches every query that sees it and no other."""
import math

import numpy as np
import pytest
import torch

import kvp_inputs as ki
from paper_2608_15943_amd import binding as kb

from gpu_util import DEV, build_device_model, say, small_workload, tdtype, to_np, workspace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kb.lib()


def _consumer(dm, x, B, S):
    """Layer 1 of a [0, 0] stack on x: it reads layer 0's slot as it is."""
    o, y = torch.zeros_like(x), torch.zeros_like(x)
    ws, n = workspace(dm, kb.KVP_PHASE_PREFILL, B, S)
    dm.model.kvp_layer_forward(1, x.data_ptr(), o.data_ptr(), y.data_ptr(), B, S, ws.data_ptr(), n,
                               torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return o, y


@pytest.mark.parametrize("key", [0, 16, 17, 32, 48, 79])
def test_fp32_nan_key_reaches_the_queries_that_see_it(key):
    """fp32 attention in tiles of 16 keys, every fourth tile to a wave: the first key of a tile
    is all that its first query sees of it."""
    S = 80
    w = small_workload("nan-key", 2, 64, 4, 2, [0, 0], dtype="fp32", d_h=16, seed=41)
    say(f"[nan key] {key}")
    dm = build_device_model(w, 1, S, S, fill_cache_npos=S)
    x = torch.from_numpy(np.ascontiguousarray(ki.prefill_x(w, [0], np.arange(S)))).to(tdtype(w)).to(DEV)
    clean, _ = _consumer(dm, x, 1, S)
    assert torch.isfinite(clean).all()
    dm.slots[0][0][:, :, key] = math.nan
    o, y = _consumer(dm, x, 1, S)
    assert torch.equal(o[0, :key], clean[0, :key])
    assert torch.isnan(o[0, key:]).all() and torch.isnan(y[0, key:]).all()


def test_fp32_nan_key_reaches_the_gradients():
    """The log-sum-exp of a row that sees a NaN score is NaN, also where the score is all that
    one wave sees of the row: dK and dV of every key that the row sees gather it."""
    S, key = 17, 16
    w = small_workload("nan-key-bwd", 2, 64, 4, 2, [0, 0], dtype="fp32", d_h=16, seed=43)
    dm = build_device_model(w, 1, S, S)
    st = torch.cuda.current_stream().cuda_stream
    x = torch.from_numpy(np.ascontiguousarray(ki.prefill_x(w, [0], np.arange(S)))).to(tdtype(w)).to(DEV)
    dy = torch.from_numpy(np.ascontiguousarray(ki.prefill_dy(w, [0], np.arange(S)))).to(tdtype(w)).to(DEV)
    dx, y = torch.zeros_like(x), torch.zeros_like(x)
    ws, n = workspace(dm, kb.KVP_PHASE_PREFILL, 1, S)
    nsv = dm.model.kvp_train_saved_size(1, S)
    saved = torch.zeros(nsv, dtype=torch.uint8, device=DEV)
    wsb, nb = workspace(dm, kb.KVP_PHASE_BACKWARD, 1, S)
    keep = []
    for l in range(2):
        g = [torch.zeros_like(dm.tensors[f"{k}{l}"]) if f"{k}{l}" in dm.tensors else None
             for k in ("wq", "wk", "wv", "wo")]
        keep.append(g)
        dm.model.kvp_set_layer_grads(l, *[t.data_ptr() if t is not None else 0 for t in g])
    dm.model.kvp_train_forward(x.data_ptr(), y.data_ptr(), 1, S, saved.data_ptr(), nsv, ws.data_ptr(), n, st)
    dm.slots[0][0][:, :, key] = math.nan
    dm.model.kvp_backward(x.data_ptr(), dy.data_ptr(), dx.data_ptr(), 1, S, saved.data_ptr(), nsv, wsb.data_ptr(), nb,
                          st)
    torch.cuda.synchronize()
    assert torch.isnan(dx).all()
