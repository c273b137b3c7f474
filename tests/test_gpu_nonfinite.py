"""Scores that are not finite.  A NaN key reaches every query that sees it and no other; keys
whose scores are -inf (a product past the fp32 range) weigh nothing, wherever they lie in the
runs of keys that the attention kernels sum separately."""
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


def _hidden_reference(x, wq, K, V, hidden, heads, S):
    """Attention of x over K, V [S][128] without the hidden keys, in 64 bits; rows that see no
    other key are NaN."""
    d = 128
    ang = np.arange(S)[:, None] * 10000.0 ** (-2.0 * np.arange(d // 2) / d)[None]
    out = []
    for j in range(heads):
        q = x @ wq[j * d:(j + 1) * d].T
        a, b = q[:, : d // 2], q[:, d // 2:]
        q = np.concatenate([a * np.cos(ang) - b * np.sin(ang), b * np.cos(ang) + a * np.sin(ang)], 1)
        s = q @ K.T / math.sqrt(d)
        see = np.tril(np.ones((S, S), bool)) & ~hidden[None]
        s = np.where(see, s, -np.inf)
        with np.errstate(invalid="ignore"):
            p = np.exp(s - s.max(1, keepdims=True))
            out.append(p @ V / p.sum(1, keepdims=True))
    return np.concatenate(out, 1)


@pytest.mark.parametrize("lo,hi", [(0, 64), (64, 128), (0, 128), (128, 192)])
@pytest.mark.parametrize("B", [1, 200])
def test_flash_keys_with_scores_of_minus_infinity(lo, hi, B):
    """Keys [lo, hi) score -inf for every query.  B 1 splits the keys of a tile between wave
    groups, so a group's first 64 keys can all be such; B 200 does not."""
    S, a = 260, 2
    w = small_workload("inf-keys", 2, a * 128, a, 1, [0, 0], seed=47)
    say(f"[-inf keys] {lo}..{hi} B={B}")
    dm = build_device_model(w, B, S, 320, fill_cache_npos=S)
    # Dimension 63 of every query is about 8 (it turns by 1.2e-4 a position), and of the hidden
    # keys -3e38: the product leaves the fp32 range.
    wq = dm.tensors["wq1"]
    for j in range(a):
        wq[128 * j + 63] = 0
        wq[128 * j + 63, 0] = 8
        wq[128 * j + 127] = 0
    x = torch.from_numpy(np.ascontiguousarray(ki.prefill_x(w, [0], np.arange(S)))).to(tdtype(w))
    x[:, :, 0] = 1
    x = x.expand(B, S, w.h).contiguous().to(DEV)
    K, V = dm.slots[0]
    K.copy_(K[:1].expand_as(K).clone())
    V.copy_(V[:1].expand_as(V).clone())
    K[:, :, :, 63] = 0
    K[:, :, lo:hi, 63] = -3e38
    o, _ = _consumer(dm, x, B, S)
    hidden = np.zeros(S, bool)
    hidden[lo:hi] = True
    k64 = to_np(K[0, 0, :S])
    k64[hidden] = 0
    ref = _hidden_reference(to_np(x[0]), to_np(wq), k64, to_np(V[0, 0, :, :S]).T, hidden, a, S)
    for b in {0, B - 1}:
        got = to_np(o[b])
        none = np.isnan(ref).any(1)                     # rows that see hidden keys only
        assert none.sum() == (hi if lo == 0 else 0)
        assert np.isnan(got[none]).all()
        err = np.abs(got[~none] - ref[~none]).max()
        assert err <= 2e-2 * np.abs(ref[~none]).max(), err


@pytest.mark.parametrize("tiles", [(0,), (1,), (1, 2, 700)])
def test_decode_tiles_with_scores_of_minus_infinity(tiles):
    """A context of 1500 tiles of 64 positions over 1024 waves: some waves have one tile, some
    two, so hidden tiles start, end and fill the pieces."""
    n = 1500 * 64 - 1
    w = small_workload("inf-decode", 1, 128, 1, 1, [0], seed=53)
    say(f"[-inf decode] {tiles}")
    dm = build_device_model(w, 1, 1, 1500 * 64, fill_cache_npos=n)
    x = torch.from_numpy(np.ascontiguousarray(ki.decode_x(w, [0]))).to(tdtype(w)).to(DEV)
    x64, wq = to_np(x[0]), to_np(dm.tensors["wq0"])
    q = wq @ x64
    ang = n * 10000.0 ** (-2.0 * np.arange(64) / 128)
    q = np.concatenate([q[:64] * np.cos(ang) - q[64:] * np.sin(ang), q[64:] * np.cos(ang) + q[:64] * np.sin(ang)])
    assert np.abs(q).sum() > 8                          # times 3e38: past the fp32 range
    K, V = dm.slots[0]
    hidden = np.zeros(n + 1, bool)
    for t in tiles:
        hidden[64 * t:64 * t + 64] = True
        K[0, 0, 64 * t:64 * t + 64] = torch.from_numpy(-3e38 * np.sign(q)).to(K)
    y = torch.zeros_like(x)
    ws, nb = workspace(dm, kb.KVP_PHASE_DECODE, 1)
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    dm.model.kvp_decode_step(x.data_ptr(), lens.data_ptr(), n, y.data_ptr(), 1, ws.data_ptr(), nb,
                             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    s = to_np(K[0, 0])[~hidden] @ q / math.sqrt(128)
    p = np.exp(s - s.max())
    ref = x64 + to_np(dm.tensors["wo0"]) @ ((p / p.sum()) @ to_np(V[0, 0]).T[~hidden])
    assert np.abs(to_np(y[0]) - ref).max() <= 2e-2 * np.abs(ref).max()
