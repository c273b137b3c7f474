"""The projection GEMMs choose a tile size from the product's sizes.  Layer forwards at sizes
that take each tile, with row and column remainders of it (rows that fill no tile, an odd
number of heads so that the last column tile is half empty), against the fp64 oracle at the
bf16 tolerance; and, since every tile sums K in the same order, the same sequence alone and
inside a large batch gives the same bits, but for the attention, which splits the keys of a
small grid: its outputs are held to the roundings of each row, and the rest is compared
through them."""
import numpy as np
import pytest
import torch

import kvp_inputs as ki
from kvp_inputs import device as kd
from oracle import attention as oat
from paper_2608_15943_amd import binding as kb

from gpu_util import (DEV, attention_reference, build_device_model, oracle_weights, rel_err, run_prefill, say,
                      small_workload, to_np, tol, workspace)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kb.lib()


def _forward(dm, B, S):
    w = dm.w
    x = torch.empty((B, S, w.h), dtype=torch.bfloat16, device=DEV)
    kd.fill_prefill_x(w, x.data_ptr(), B, S)
    y, o = torch.empty_like(x), torch.empty_like(x)
    ws, n = workspace(dm, kb.KVP_PHASE_PREFILL, B, S)
    dm.model.kvp_layer_forward(0, x.data_ptr(), o.data_ptr(), y.data_ptr(), B, S, ws.data_ptr(), n,
                               torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return y, o


def assert_attention(o, w, b, K, V, S):
    """Attention output o [S][a * 128] of sequence b against the oracle over the device's own K
    and V of that sequence, within the roundings of each row's weights and of the output."""
    ref, bound = attention_reference(ki.prefill_x(w, [b], np.arange(S))[0], oracle_weights(w)[0], to_np(K[b, :, :S]),
                                     to_np(V[b, :, :, :S]).transpose(0, 2, 1), w.a, w.rope_base)
    e = np.abs(to_np(o) - ref) / bound
    say(f"  attention of sequence {b}: {e.max():.3f} of its bound")
    assert e.max() <= 1, e.max()


@pytest.mark.parametrize("a,g,B,S", [
    (1, 1, 1, 1),        # one row, 64-wide tiles
    (3, 1, 1, 63),
    (3, 1, 1, 65),
    (3, 3, 3, 43),       # 129 rows, positions not a multiple of 8
    (3, 1, 40, 67),
    (3, 1, 300, 67),     # 20100 rows: 256-wide tiles, 132 rows in the last, half of a column tile
    (16, 8, 12, 127),    # 1524 rows at width 2048: 128 x 256 tiles, then 128 x 128
    (33, 3, 9, 127),     # 1143 rows at width 4224: 128 x 256 tiles, the last column tile half empty
    (16, 8, 33, 127),    # 4191 rows at width 2048: 256-wide tiles, 95 rows in the last
    (33, 3, 245, 67),    # 16415 rows at width 4224: 256-wide tiles, the last column tile half empty
])
def test_layer_forward_over_the_tile_sizes(a, g, B, S):
    w = small_workload(f"tiles-a{a}-g{g}", 1, a * 128, a, g, [0])
    say(f"[gemm tiles] h={w.h} g={g} B={B} S={S}")
    cap = (S + 63) // 64 * 64
    dm = build_device_model(w, B, S, cap)
    y, o = _forward(dm, B, S)
    K, V = dm.slots[0]
    K, V = K.clone(), V.clone()
    ow = oracle_weights(w)
    for b in sorted({0, B - 1}):
        ref, _, _, caches = oat.stack_prefill(ki.prefill_x(w, [b], np.arange(S))[0], ow, w.tau, w.a, w.g, w.d_h,
                                              w.rope_base)
        assert rel_err(to_np(y[b]), ref) <= tol(w), b
        assert rel_err(to_np(K[b, :, :S]), caches[0][0]) <= tol(w), b
        assert rel_err(to_np(V[b, :, :, :S]).transpose(0, 2, 1), caches[0][1]) <= tol(w), b
        assert_attention(o[b], w, b, K, V, S)
    assert torch.isfinite(y.float()).all() and torch.isfinite(o.float()).all()
    y1, o1 = _forward(dm, 1, S)
    assert_attention(o1[0], w, 0, K, V, S)
    same = (o1[0] == o[0]).all(1)
    assert same[:64].all()   # queries that see no key of a second half
    assert torch.equal(y1[0][same], y[0][same])
    # Elsewhere y differs by what o does, and the two roundings of y to bf16 (8 bits: 2^-8 each).
    do = (o1[0].double() - o[0].double()).abs().cpu()
    bound = do @ torch.from_numpy(np.abs(np.asarray(ow[0].wo, dtype=np.float64))).T + 2.0**-7 * y[0].double().abs().cpu()
    assert ((y1[0].double() - y[0].double()).abs().cpu() <= 1.01 * bound + 1e-5).all()
    assert torch.equal(dm.slots[0][0][0], K[0]) and torch.equal(dm.slots[0][1][0], V[0])


@pytest.mark.parametrize("S", [64, 65, 128, 129, 191, 193, 256, 385, 900])
def test_attention_with_split_keys(S):
    """Lengths around the halves of a key tile and around a workgroup's 128 queries: the first
    sequence alone (keys split) and in a batch large enough for unsplit workgroups, against the
    oracle."""
    a, g = 3, 1
    B = 512 // (a * ((S + 127) // 128)) + 1
    w = small_workload("split-keys", 1, a * 128, a, g, [0])
    say(f"[split keys] S={S} B={B}")
    dm = build_device_model(w, B, S, (S + 63) // 64 * 64)
    _, o1 = _forward(dm, 1, S)
    K, V = dm.slots[0]
    assert_attention(o1[0], w, 0, K, V, S)
    _, o = _forward(dm, B, S)
    assert_attention(o[0], w, 0, K, V, S)


@pytest.mark.parametrize("B,S", [
    (12, 127),    # 1524 rows: layer 0's Q|K|V on 128 x 256 tiles, the rest on 128 x 128
    (3, 1000),    # 3000 rows: Q|K|V on 256 x 256, the consumer's Q and both outputs on 128 x 256
    (33, 127),    # 4191 rows: 256 x 256
])
def test_fp32_residual_over_the_tile_sizes(B, S):
    """A producer and its consumer at width 2048: the second layer's output product updates the
    fp32 residual stream, on each of the larger tiles, with a row remainder."""
    w = small_workload("tiles-2L", 2, 2048, 16, 8, [0, 0], seed=3)
    say(f"[fp32 residual] B={B} S={S}")
    dm = build_device_model(w, B, S, (S + 63) // 64 * 64)
    _, y = run_prefill(dm, B, S)
    ow = oracle_weights(w)
    for b in sorted({0, B - 1}):
        ref, _, _, _ = oat.stack_prefill(ki.prefill_x(w, [b], np.arange(S))[0], ow, w.tau, w.a, w.g, w.d_h, w.rope_base)
        assert rel_err(to_np(y[b]), ref) <= tol(w), b
