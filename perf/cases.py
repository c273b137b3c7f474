"""The work whose speed this library is judged by, as cases that a measuring program runs.

A case is one pass through the public entry points (``paper_2608_15943_amd.binding``): a decode
step, a prefill, a single layer, or a training step (forward that keeps activations, then the
backward).  The listed cases span the smallest calls to the largest, odd and ragged sizes, slots
and paged storage, bf16 and fp32 models; ``draw`` gives more of the same ranges.  Widths and head
counts are those of the library's own workloads (GQA 16/8 at 2048, 32/8 at 4096, 64/8 at 8192, the
four-layer fp32 stack at 256) and neighbours of them.

Fields of a case:
  kind      "decode", "layer" (one layer of a prefill), "prefill", "train"
  dtype     "bf16" or "fp32"
  L, h, a, g   layers, width, query heads, KV heads
  share     every how many layers one owns K/V (2: layers 1, 3, ... read layers 0, 2, ...)
  B, S      sequences and tokens each (prefill, layer, train)
  lo, hi    shortest and longest cached context (decode)
  paged     K/V in 64-position pages (decode, prefill)
  noalloc   decode through the entry point that takes no workspace
  consumer  layer: run the layer that reads another layer's K/V
"""
import math

import torch

from paper_2608_15943_amd import binding as kb

PAGE = 64
# Total bytes of K/V above which a decode step's caches (its inputs but for one row a sequence)
# are not returned beside its output.
RETURN_KV = 160 << 20


def _case(name, kind, h, a, g, L=1, dtype="bf16", share=2, B=1, S=0, lo=0, hi=0, paged=False, noalloc=False,
          consumer=False):
    return dict(name=name, kind=kind, dtype=dtype, L=L, h=h, a=a, g=g, share=share, B=B, S=S, lo=lo, hi=hi,
                paged=paged, noalloc=noalloc, consumer=consumer)


def listed():
    return [
        # One user's chat turn: one sequence, a short context; weights and launches count.
        _case("decode-1", "decode", 4096, 32, 8, L=2, B=1, lo=977, hi=977),
        # A small serving batch at a few thousand tokens each.
        _case("decode-8-4k", "decode", 4096, 32, 8, L=2, B=8, lo=2500, hi=5700),
        # A batch above 16 sequences of mixed lengths, none of them a round number.
        _case("decode-37-ragged", "decode", 4096, 32, 8, L=2, B=37, lo=301, hi=9001),
        # The long-context serving batch of the benchmark (64 sequences of 32K), two of its layers.
        _case("decode-64-32k", "decode", 4096, 32, 8, L=2, B=64, lo=32768, hi=32768),
        # Capacity-driven serving: paged storage and more sequences than one kernel launch takes.
        _case("decode-paged-96", "decode", 4096, 32, 8, L=2, B=96, lo=4000, hi=12000, paged=True),
        # A short prompt, alone: the first layer of it.
        _case("layer-200", "layer", 4096, 32, 8, B=1, S=200),
        # A few prompts of an odd length, a producer and its consumer.
        _case("prefill-3x1000", "prefill", 2048, 16, 8, L=2, B=3, S=1000),
        # The benchmark's pipeline-stage share: eight layers, four sequences of 4096 tokens.
        _case("prefill-stage", "prefill", 2048, 16, 8, L=8, share=0, B=4, S=4096),
        # One layer of the 70B-shaped stage over a long prompt.
        _case("layer-8k-wide", "layer", 8192, 64, 8, B=1, S=8192),
        # Two layers of the stage's training step.
        _case("train-4x4096", "train", 2048, 16, 8, L=2, B=4, S=4096),
        # A training step on sequences of an odd length (no power of two divides the tokens).
        _case("train-2x777", "train", 2048, 16, 8, L=2, B=2, S=777),
        # The small full-precision stack, trained: what a numerics check or a small model runs.
        _case("train-fp32", "train", 256, 4, 4, L=4, dtype="fp32", B=1, S=128),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges, costing no more than the largest of them."""
    limit = max(_cost(c) for c in listed()) * 0.9
    while True:
        c = _draw(rng)
        if _cost(c) <= limit:
            return c


def _draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "layer", "prefill", "prefill", "train", "train"])
    if rng.random() < 0.15:
        d, a = rng.choice([32, 64, 128]), rng.choice([2, 4, 8])
        g = rng.choice([x for x in (1, 2, 4, 8) if a % x == 0])
        kind = rng.choice(["train", "prefill", "decode"])
        c = _case("", kind, a * d, a, g, L=rng.choice([2, 4]), dtype="fp32", B=_loguniform(rng, 1, 4),
                  S=_loguniform(rng, 5, 200))
        if kind == "decode":
            c["S"], c["lo"], c["hi"] = 0, 3, _loguniform(rng, 20, 600)
    else:
        h, a, g = rng.choice([(1024, 8, 4), (2048, 16, 8), (2048, 16, 16), (4096, 32, 8), (4096, 32, 8), (5120, 40, 8),
                              (8192, 64, 8)])
        c = _case("", kind, h, a, g, L=rng.choice([1, 2, 2]), paged=rng.random() < 0.3)
        if kind == "decode":
            c["B"] = _loguniform(rng, 1, 100)
            c["hi"] = _loguniform(rng, 60, 40000)
            c["lo"] = max(1, int(c["hi"] * rng.choice([0.1, 0.5, 1.0])))
            c["noalloc"] = not c["paged"] and c["B"] <= 64 and rng.random() < 0.3
        else:
            c["S"] = _loguniform(rng, 24, 8000)
            if rng.random() < 0.3:
                c["S"] = max(64, c["S"] // 64 * 64)
            c["B"] = _loguniform(rng, 1, 6)
            if kind == "layer":
                c["L"], c["consumer"] = 1, rng.random() < 0.5
            c["paged"] = c["paged"] and kind == "prefill"
    del c["name"]
    return c


def _cost(c):
    """Rough microseconds of a pass, for keeping drawn cases below the largest listed one."""
    w = work(c)
    if c["dtype"] == "fp32":
        # A token's work over its keys is a serial chain in the small full-precision kernels.
        return 100.0 + w["flops"] * 3e-7 + (c["S"] * _dh(c) * (c["a"] // c["g"]) if c["kind"] == "train" else 0)
    return 30.0 + w["flops"] / 8e8 + w["bytes"] / 5e6


def _dh(c):
    return c["h"] // c["a"]


def _tau(c):
    if c["share"] == 0:          # the stage's own map: four full layers, then two sharing pairs
        return [0, 1, 2, 3, 4, 4, 6, 6]
    if c["kind"] == "layer":
        return [0, 0] if c["consumer"] else [0]
    return [l - l % c["share"] for l in range(c["L"])]


def _lens(c, seed=0):
    """Cached lengths: evenly spread over [lo, hi], in an order that the seed gives."""
    B = c["B"]
    xs = [c["lo"] + (c["hi"] - c["lo"]) * i // max(1, B - 1) for i in range(B)]
    order = torch.randperm(B, generator=torch.Generator().manual_seed(seed)).tolist()
    return [xs[i] for i in order]


def _cap(c):
    n = c["hi"] + 1 if c["kind"] == "decode" else c["S"]
    return (n + PAGE - 1) // PAGE * PAGE


def work(case):
    """Bytes: weights, activations in and out, K/V written, and in decode each layer's cache read
    once by that layer.  FLOPs: the matrix products, causal pairs only."""
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    d, h = _dh(c), c["h"]
    nq, nkv = c["a"] * d, c["g"] * d
    tau = _tau(c)
    layers = [len(tau) - 1] if c["kind"] == "layer" else range(len(tau))
    by = fl = 0
    if c["kind"] == "decode":
        rows, kept = c["B"], sum(_lens(c)) + c["B"]
        pairs = kept
    else:
        rows, kept = c["B"] * c["S"], c["B"] * c["S"]
        pairs = c["B"] * c["S"] * (c["S"] + 1) // 2
    by += 2 * rows * h * e
    for l in layers:
        prod = tau[l] == l
        n = nq + (2 * nkv if prod else 0)
        proj = 2 * rows * h * (n + nq)
        attn = 4 * d * c["a"] * pairs
        wb = (n + nq) * h * e
        by += wb + (2 * rows * nkv * e if prod else 0)
        if c["kind"] == "decode":
            by += 2 * kept * nkv * e
        elif c["kind"] == "layer":
            by += rows * nq * e + (0 if prod else 2 * rows * nkv * e)
        fl += proj + attn
        if c["kind"] == "train":
            # Backward: twice the projections, and five products per pair for the forward's two.
            fl += 2 * proj + attn * 5 // 2
            by += wb + (n + nq) * h * 4 + 2 * rows * (2 * nq + h) * e
    if c["kind"] == "train":
        by += 2 * rows * h * 4
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # Relative errors between two correct implementations of the same precision: about four times
    # what the results are off from 64 bits.  bf16: Q, K, V, the softmax weights and the attention
    # output are rounded to 8 bits, and so are the gradients between the backward's products
    # (measured: 0.0017 for the output of a decode step or of two layers, 0.0025 for eight layers,
    # 0.005 for weight gradients, 0.006 for a layer's attention output).  fp32: 7e-7, and sums in
    # another order.
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 8e-3 if case["kind"] in ("decode", "prefill") and case["L"] <= 2 else 2e-2}


def prepare(case, seed):
    c = case
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    d, h, B, S = _dh(c), c["h"], c["B"], c["S"]
    tau, cap = _tau(c), _cap(c)
    L = len(tau)
    nq, nkv = c["a"] * d, c["g"] * d

    def normal(*shape, std=1.0, dtype=dt):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, std, generator=gen)

    m = kb.Model(L, h, c["a"], c["g"], d, kb.KVP_DTYPE_BF16 if dt is torch.bfloat16 else kb.KVP_DTYPE_FP32, tau,
                 max_batch=B, max_seq=max(S, 1), kv_capacity=cap)
    s = {"case": c, "m": m, "w": [], "kv": {}, "tau": tau}
    decode = c["kind"] == "decode"
    if decode:
        s["lens_host"] = _lens(c, int(seed))
        s["lens"] = torch.tensor(s["lens_host"], dtype=torch.int32, device=dev)
    if c["paged"]:
        need = [(n + PAGE) // PAGE for n in s["lens_host"]] if decode else [(S + PAGE - 1) // PAGE] * B
        n_pages, stride = sum(need) + 8, max(need)
        pager = kb.Pager(n_pages, B, stride)
        for upto in range(1, stride + 16, 16):      # sequences grow in turns, so their pages interleave
            for b in range(B):
                pager.reserve(b, PAGE * min(upto, need[b]))
        rows = pager.rows(list(range(B)))
        s["pages"], s["stride"], s["pager"] = torch.from_numpy(rows).to(dev), stride, pager
    for l in range(L):
        prod = tau[l] == l
        w = {"wq": normal(nq, h, std=0.02), "wo": normal(h, nq, std=0.02)}
        if prod:
            w["wk"], w["wv"] = normal(nkv, h, std=0.02), normal(nkv, h, std=0.02)
        s["w"].append(w)
        m.kvp_set_layer(l, w["wq"].data_ptr(), w["wk"].data_ptr() if prod else 0, w["wv"].data_ptr() if prod else 0,
                        w["wo"].data_ptr())
        if not prod:
            continue
        shk, shv = ((c["g"], n_pages, PAGE, d), (c["g"], n_pages, d, PAGE)) if c["paged"] else \
            ((B, c["g"], cap, d), (B, c["g"], d, cap))
        filled = decode or c["consumer"]
        k = normal(*shk) if filled else torch.zeros(shk, dtype=dt, device=dev)
        v = normal(*shv) if filled else torch.zeros(shv, dtype=dt, device=dev)
        s["kv"][l] = (k, v)
        if c["paged"]:
            m.kvp_set_kv_pool(l, k.data_ptr(), v.data_ptr(), n_pages)
        else:
            m.kvp_set_kv_slot(l, k.data_ptr(), v.data_ptr())
    s["x"] = normal(B, h) if decode else normal(B, S, h)
    s["y"] = torch.zeros_like(s["x"])
    s["n"] = m.kvp_workspace_size(kb.KVP_PHASE_DECODE if decode else kb.KVP_PHASE_PREFILL, B, max(S, 1))
    s["ws"] = torch.empty(s["n"], dtype=torch.uint8, device=dev)
    if c["kind"] == "layer":
        s["o"] = torch.zeros((B, S, nq), dtype=dt, device=dev)
    if c["kind"] == "train":
        s["dy"] = normal(B, S, h, dtype=torch.float32)
        s["dx"] = torch.zeros_like(s["dy"])
        s["nsaved"] = m.kvp_train_saved_size(B, S)
        s["saved"] = torch.empty(s["nsaved"], dtype=torch.uint8, device=dev)
        s["nb"] = m.kvp_workspace_size(kb.KVP_PHASE_BACKWARD, B, S)
        s["wsb"] = torch.empty(s["nb"], dtype=torch.uint8, device=dev)
        s["dw"] = []
        for l in range(L):
            gr = {"d" + k: torch.zeros(t.shape, dtype=torch.float32, device=dev) for k, t in s["w"][l].items()}
            s["dw"].append(gr)
            m.kvp_set_layer_grads(l, gr["dwq"].data_ptr(), gr["dwk"].data_ptr() if "dwk" in gr else 0,
                                  gr["dwv"].data_ptr() if "dwv" in gr else 0, gr["dwo"].data_ptr())
    return s


def _returns_kv(c):
    if c["kind"] == "layer" and c["consumer"]:
        return False
    if c["kind"] != "decode":
        return True
    tau, e = _tau(c), 2 if c["dtype"] == "bf16" else 4
    return 2 * (sum(_lens(c)) + PAGE * c["B"]) * c["g"] * _dh(c) * e * sum(t == l for l, t in enumerate(tau)) <= RETURN_KV


def run(state):
    s = state
    c, m = s["case"], s["m"]
    st = torch.cuda.current_stream().cuda_stream
    x, y, ws, n, B, S = s["x"].data_ptr(), s["y"].data_ptr(), s["ws"].data_ptr(), s["n"], c["B"], c["S"]
    out = {"y": s["y"]}
    if c["kind"] == "decode":
        if c["paged"]:
            m.kvp_decode_step_paged(x, s["lens"].data_ptr(), c["hi"], s["pages"].data_ptr(), s["stride"], y, B, ws, n, st)
        elif c["noalloc"]:
            m.kvp_decode_step_noalloc(x, s["lens"].data_ptr(), c["hi"], y, B, st)
        else:
            m.kvp_decode_step(x, s["lens"].data_ptr(), c["hi"], y, B, ws, n, st)
    elif c["kind"] == "layer":
        m.kvp_layer_forward(len(s["tau"]) - 1, x, s["o"].data_ptr(), y, B, S, ws, n, st)
        out["o"] = s["o"]
    elif c["kind"] == "prefill":
        if c["paged"]:
            m.kvp_prefill_paged(x, y, B, S, s["pages"].data_ptr(), s["stride"], ws, n, st)
        else:
            m.kvp_prefill(x, y, B, S, ws, n, st)
    else:
        m.kvp_train_forward(x, y, B, S, s["saved"].data_ptr(), s["nsaved"], ws, n, st)
        m.kvp_backward(x, s["dy"].data_ptr(), s["dx"].data_ptr(), B, S, s["saved"].data_ptr(), s["nsaved"],
                       s["wsb"].data_ptr(), s["nb"], st)
        out["dx"] = s["dx"]
        out["dw"] = s["dw"]
    if _returns_kv(c):
        out["kv"] = {str(l): kv for l, kv in s["kv"].items()}
    return out


# ---- the same in 64 bits, plain torch ---------------------------------------------------------

def _rope(x, pos, transpose=False):
    """x [..., positions, d]: rotate-half by pos * 10000^(-2i/d)."""
    d = x.shape[-1]
    th = 10000.0 ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    ang = pos.to(torch.float64)[:, None] * th[None, :]
    co, si = ang.cos(), ang.sin()
    x1, x2 = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([x1 * co - x2 * si, x2 * co + x1 * si], dim=-1)


def _heads(t, n):
    return t.reshape(t.shape[0], n, -1).transpose(0, 1).contiguous()


def _causal(q, k, v):
    """q [a, S, d], k, v [g, S, d] of one sequence -> [S, a * d]; a KV head's queries at a time."""
    a, S, d = q.shape
    g = k.shape[0]
    hidden = torch.ones(S, S, dtype=torch.bool, device=q.device).triu(1)
    os_ = []
    for j in range(a):
        p = (q[j] @ k[j * g // a].T) / math.sqrt(d)
        p = torch.softmax(p.masked_fill(hidden, -math.inf), dim=-1)
        os_.append(p @ v[j * g // a])
    return torch.stack(os_, 1).reshape(S, a * d)


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    d, B, S, tau = _dh(c), c["B"], c["S"], s["tau"]
    a, g = c["a"], c["g"]
    f = lambda t: t.to(torch.float64)  # noqa: E731
    w = [{k: f(t) for k, t in ws.items()} for ws in s["w"]]
    if c["kind"] == "decode":
        return _exact_decode(s, w)
    train = c["kind"] == "train"
    if train:
        for ws in w:
            for t in ws.values():
                t.requires_grad_(True)
    pos = torch.arange(S, device="cuda")
    layers = [len(tau) - 1] if c["kind"] == "layer" else range(len(tau))
    kv64 = {l: (torch.zeros(k.shape, dtype=torch.float64, device="cuda"),
                torch.zeros(v.shape, dtype=torch.float64, device="cuda")) for l, (k, v) in s["kv"].items()} \
        if _returns_kv(c) else {}
    ys, os_, dxs = [], [], []
    for b in range(B):
        x = f(s["x"][b])
        if train:
            x.requires_grad_(True)
        cur, kv = x, {}
        for l in layers:
            if tau[l] == l:
                kv[l] = (_rope(_heads(cur @ w[l]["wk"].T, g), pos), _heads(cur @ w[l]["wv"].T, g))
            elif c["kind"] == "layer":
                k, v = s["kv"][0]
                kv[0] = (f(k[b, :, :S]), f(v[b, :, :, :S]).transpose(1, 2).contiguous())
            q = _rope(_heads(cur @ w[l]["wq"].T, a), pos)
            o = _causal(q, *kv[tau[l]])
            cur = cur + o @ w[l]["wo"].T
        if train:
            (cur * f(s["dy"][b])).sum().backward()
            dxs.append(x.grad)
        ys.append(cur.detach())
        if c["kind"] == "layer":
            os_.append(o)
        for l, (k64, v64) in kv64.items():
            k, v = kv[l][0].detach(), kv[l][1].detach().transpose(1, 2)
            if c["paged"]:
                for i, p in enumerate(s["pages"][b].tolist()[: (S + PAGE - 1) // PAGE]):
                    n = min(PAGE, S - PAGE * i)
                    k64[:, p, :n] = k[:, PAGE * i: PAGE * i + n]
                    v64[:, p, :, :n] = v[:, :, PAGE * i: PAGE * i + n]
            else:
                k64[b, :, :S] = k
                v64[b, :, :, :S] = v
        del cur, kv
    out = {"y": torch.stack(ys)}
    if c["kind"] == "layer":
        out["o"] = torch.stack(os_)
    if train:
        out["dx"] = torch.stack(dxs)
        out["dw"] = [{"d" + k: t.grad for k, t in ws.items()} for ws in w]
    if kv64:
        out["kv"] = {str(l): t for l, t in kv64.items()}
    return out


def _exact_decode(s, w):
    c = s["case"]
    d, a, g, tau, B = _dh(c), c["a"], c["g"], s["tau"], c["B"]
    f = lambda t: t.to(torch.float64)  # noqa: E731
    keep = _returns_kv(c)
    kv64 = {l: (f(k), f(v)) for l, (k, v) in s["kv"].items()} if keep else {}
    x = f(s["x"])
    cur = x
    new = {}
    for l in range(len(tau)):
        if tau[l] == l:
            new[l] = (cur @ w[l]["wk"].T, cur @ w[l]["wv"].T)
        q = cur @ w[l]["wq"].T
        k, v = s["kv"][tau[l]]
        os_ = []
        for b in range(B):
            n = s["lens_host"][b]
            at = torch.tensor([n], device="cuda")
            if c["paged"]:
                rows = s["pages"][b, : n // PAGE + 1].long()
                kb_ = k[:, rows].reshape(g, -1, d)[:, :n]
                vb_ = v[:, rows].transpose(2, 3).reshape(g, -1, d)[:, :n]
            else:
                kb_, vb_ = k[b, :, :n], v[b, :, :, :n].transpose(1, 2)
            kn = _rope(new[tau[l]][0][b].reshape(g, 1, d), at)
            vn = new[tau[l]][1][b].reshape(g, 1, d)
            if keep and tau[l] == l:
                if c["paged"]:
                    p, r = int(s["pages"][b, n // PAGE]), n % PAGE
                    kv64[l][0][:, p, r], kv64[l][1][:, p, :, r] = kn[:, 0], vn[:, 0]
                else:
                    kv64[l][0][b, :, n], kv64[l][1][b, :, :, n] = kn[:, 0], vn[:, 0]
            kk, vv = torch.cat([f(kb_), kn], 1), torch.cat([f(vb_), vn], 1)
            qq = _rope(q[b].reshape(a, 1, d), at).reshape(g, a // g, d)
            p = torch.softmax(torch.matmul(qq, kk.transpose(1, 2).contiguous()) / math.sqrt(d), dim=-1)
            os_.append(torch.matmul(p, vv.contiguous()).reshape(a * d))
        cur = cur + torch.stack(os_) @ w[l]["wo"].T
    out = {"y": cur}
    if keep:
        out["kv"] = {str(l): t for l, t in kv64.items()}
    return out
