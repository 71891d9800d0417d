"""Performance cases: the calls a user of the library makes, over the sizes it is used at.

A case is a dict of plain values.  ``listed()`` names the standing ones, ``draw(rng)`` makes
more of the same ranges, ``prepare`` builds what a program holds before the call (a model
with its weights laid out, a session with resident cells, the tokens), ``run`` is one call
through the public binding, ``work`` its unavoidable bytes and operations, ``exact`` the same
result in 64-bit torch and ``tolerance`` how far another correct implementation may be off.

The models are this repository's own shapes (synth/: the fp32 tiny model, the 8B, 32B and
MXFP4 70B shapes, the small bf16 model of the session tests), cut to a few layers: every
layer is alike, and each layer's weights and cells are larger than a cache.  Weights are
N(0, 0.02), norm gains 1 + N(0, 0.02), resident cells N(0, 1) and tokens uniform, as in the
repository's synthetic workloads.
"""
import math

import numpy as np
import torch

import paper_2606_29565_amd as spp

# d_model, query heads, kv heads, head_dim, ffn_dim, vocab, rope base, storage
MODELS = {
    "tiny-f32": (256, 4, 4, 64, 1024, 4096, 1.0e4, "f32"),
    "small": (256, 4, 2, 64, 512, 2048, 1.0e4, "bf16"),
    "8b": (4096, 32, 8, 128, 14336, 128256, 5.0e5, "bf16"),
    "32b": (5120, 64, 8, 128, 27648, 152064, 1.0e6, "bf16"),
    "70b-mxfp4": (8192, 64, 8, 128, 28672, 128256, 5.0e5, "mxfp4"),
}
EPS = 1e-5
PROJ = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")
KINDS = (spp.SPP_W_Q, spp.SPP_W_K, spp.SPP_W_V, spp.SPP_W_O, spp.SPP_W_GATE, spp.SPP_W_UP,
         spp.SPP_W_DOWN)
E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
DEV = "cuda"


def listed():
    return [
        # serve time: one request against one cached distribution of the 8B vocabulary
        {"name": "gate_one", "call": "gate", "vocab": 128256, "n": 1},
        # serve time: a tick over 64 sessions' cached distributions
        {"name": "gate_64", "call": "gate", "vocab": 128256, "n": 64},
        # the fp32 model of the smoke and parity tests: launches and latency
        {"name": "entry_tiny_f32", "call": "preposition", "model": "tiny-f32", "layers": 2,
         "past": 512, "rows": 16},
        # one decode step after a fall-through
        {"name": "decode_8b", "call": "resume", "model": "8b", "layers": 4, "past": 8192, "rows": 1},
        # the streaming entry: 24 data tokens and an 8-token header
        {"name": "stream_8b", "call": "preposition", "model": "8b", "layers": 4, "past": 8192,
         "rows": 32},
        # the agentic envelope: 128 tokens against a long history
        {"name": "agentic_8b", "call": "preposition", "model": "8b", "layers": 4, "past": 32768,
         "rows": 128},
        # a tool result of odd length committed to the history
        {"name": "append_8b", "call": "append", "model": "8b", "layers": 4, "past": 5001, "rows": 203},
        # the headline entry, with the LM-head bias of that workload
        {"name": "entry_32b", "call": "preposition", "model": "32b", "layers": 4, "past": 16384,
         "rows": 32, "bias": True},
        # the 4-bit model's entry
        {"name": "entry_70b", "call": "preposition", "model": "70b-mxfp4", "layers": 4, "past": 8192,
         "rows": 32},
        # the 4-bit model takes in a document
        {"name": "append_70b", "call": "append", "model": "70b-mxfp4", "layers": 3, "past": 1000,
         "rows": 700},
        # 64 sessions of unequal lengths pre-positioned in one pass
        {"name": "batch_8b", "call": "batch", "model": "8b", "layers": 2, "past": 8192, "rows": 64,
         "n": 64},
        # the sliding window drops its oldest cells
        {"name": "shift_8b", "call": "shift", "model": "8b", "layers": 4, "past": 8192, "delta": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(("gate", "preposition", "preposition", "idle", "resume", "append", "batch", "shift"))
    if call == "gate":
        return {"call": call, "vocab": _log(rng, 2000, 160000), "n": _log(rng, 1, 64)}
    model = rng.choice(("tiny-f32", "small", "8b", "8b", "32b", "70b-mxfp4"))
    big = model in ("32b", "70b-mxfp4")
    if call == "batch" and big:
        model, big = "8b", False
    case = {"call": call, "model": model, "layers": rng.randint(1, 3 if big else 4),
            "past": _log(rng, 64, 16384)}
    if call == "shift":
        case["delta"] = min(case["past"] - 1, _log(rng, 1, 4096))
    elif call == "batch":
        case.update(layers=min(case["layers"], 2), past=min(case["past"], 8192),
                    rows=_log(rng, 2, 64), n=_log(rng, 2, 64))
    elif call == "resume":
        case["rows"] = _log(rng, 1, 64)
    elif call == "append":
        case["rows"] = _log(rng, 16, 640 if big else 2000)
    else:
        case["rows"] = _log(rng, 4, 256)
        case["bias"] = rng.random() < 0.3
    return case


# ---- inputs -------------------------------------------------------------------------------


def _gen(seed, stream=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + stream)
    return g


def _shapes(model):
    d, nq, nkv, dh, F, V, _, _ = MODELS[model]
    return {"wq": (nq * dh, d), "wk": (nkv * dh, d), "wv": (nkv * dh, d), "wo": (d, nq * dh),
            "w_gate": (F, d), "w_up": (F, d), "w_down": (d, F)}


def _weights(case, seed):
    """Row-major weights on the GPU, in the binding's names."""
    d, _, _, _, _, V, _, fmt = MODELS[case["model"]]
    dt = torch.float32 if fmt == "f32" else torch.bfloat16
    g = _gen(seed, 1)

    def normal(shape, mean, sigma):
        return torch.empty(shape, dtype=dt, device=DEV).normal_(mean, sigma, generator=g)

    w = {"embed": normal((V, d), 0.0, 0.02), "final_norm": normal((d,), 1.0, 0.02),
         "lm_head": normal((V, d), 0.0, 0.02)}
    for k in ("attn_norm", "mlp_norm"):
        w[k] = [normal((d,), 1.0, 0.02) for _ in range(case["layers"])]
    if fmt == "mxfp4":
        w["scales"] = {}
    for k, (rows, cols) in _shapes(case["model"]).items():
        if fmt == "mxfp4":
            w[k] = [torch.randint(0, 256, (rows, cols // 2), dtype=torch.uint8, device=DEV, generator=g)
                    for _ in range(case["layers"])]
            w["scales"][k] = [torch.randint(119, 122, (rows, cols // 32), dtype=torch.uint8, device=DEV,
                                            generator=g) for _ in range(case["layers"])]
        else:
            w[k] = [normal((rows, cols), 0.0, 0.02) for _ in range(case["layers"])]
    if case.get("bias"):
        # the planted bias that makes most decisions clear the gap
        w["lm_bias"] = torch.zeros(V, dtype=torch.float32, device=DEV)
        w["lm_bias"][V // 3] = 10.1
    return w


def _sessions(case, seed):
    """(resident cells, entry tokens) of each session; the tokens are from the seed, the
    lengths of a batch from the case."""
    V = MODELS[case["model"]][5]
    r = np.random.RandomState((7919 * seed + 13) % (1 << 31))
    if case["call"] != "batch":
        return [(case["past"], r.randint(0, V, case.get("rows", 0)).tolist())]
    lens = np.random.RandomState(case["past"] + 31 * case["rows"] + 1009 * case["n"])
    past = lens.randint(max(1, case["past"] // 8), case["past"] + 1, case["n"])
    rows = lens.randint(max(1, case["rows"] // 8), case["rows"] + 1, case["n"])
    return [(int(p), r.randint(0, V, m).tolist()) for p, m in zip(past, rows)]


def _kv_dtype(case):
    return torch.float32 if MODELS[case["model"]][7] == "f32" else torch.bfloat16


def _cap(past, rows):
    return past + rows + 40


def _kv_elems(case, cap):
    _, _, nkv, dh, _, _, _, _ = MODELS[case["model"]]
    return case["layers"] * 2 * nkv * dh * ((cap + 63) // 64 * 64)


def _fill_kv(case, seed, i, t):
    t.normal_(0.0, 1.0, generator=_gen(seed, 100 + i))


def _model(case, seed, max_tokens, max_sessions=1):
    """The model with its projections already in the library's tiled layout, as a serving
    program keeps them (one copy of the weights)."""
    d, nq, nkv, dh, F, V, base, fmt = MODELS[case["model"]]
    w = _weights(case, seed)
    mx = fmt == "mxfp4"
    cfg = spp.model_config(case["layers"], d, nq, nkv, dh, F, V, base, fmt != "f32", rms_eps=EPS,
                           max_tokens=max_tokens, max_sessions=max_sessions, weights_packed=True,
                           mxfp4=mx)
    for k, which in zip(PROJ, KINDS):
        for l in range(case["layers"]):
            dst = torch.empty_like(w[k][l])
            if mx:
                sc = torch.empty_like(w["scales"][k][l])
                spp.pack_weight_mxfp4(cfg, which, w[k][l], w["scales"][k][l], dst, sc)
                w["scales"][k][l] = sc
            else:
                spp.pack_weight(cfg, which, w[k][l], dst)
            w[k][l] = dst
    torch.cuda.synchronize()
    return spp.Model(case["layers"], d, nq, nkv, dh, F, V, base, fmt != "f32", w, rms_eps=EPS,
                     max_tokens=max_tokens, max_sessions=max_sessions, weights_packed=True, mxfp4=mx)


def _gate_logits(case, seed):
    """Distributions as a model leaves them: N(0, 1.3) logits with one raised token, its
    margin spread over both sides of the threshold."""
    g = _gen(seed, 2)
    n, V = case["n"], case["vocab"]
    x = torch.empty((n, V), dtype=torch.float32, device=DEV).normal_(0.0, 1.3, generator=g)
    hot = torch.randint(0, V, (n,), device=DEV, generator=g)
    x[torch.arange(n, device=DEV), hot] = 6.0 + 3.0 * torch.rand(n, device=DEV, generator=g)
    bits = torch.randint(-2 ** 31, 2 ** 31, ((V + 31) // 32,), device=DEV, generator=g).to(torch.int32)
    return x, bits


TAU = 2.0


def _prepare_gate(case, seed):
    # a small model carries the sessions; the distributions are what the gate reads
    V, n = case["vocab"], case["n"]
    V16 = V // 16 * 16  # a batched model takes vocabularies that are multiples of 16
    MODELS["gate"] = (256, 4, 4, 64, 512, V if n == 1 else V16, 1.0e4, "f32")
    c = {"call": "preposition", "model": "gate", "layers": 1, "past": 8, "rows": 2}
    m = _model(c, seed, 16, 1 if n == 1 else 64)
    x, bits = _gate_logits(dict(case, vocab=V if n == 1 else V16), seed)
    kvs, sessions, readies = [], [], []
    for i in range(n):
        kv = torch.empty(_kv_elems(c, 16), dtype=torch.float32, device=DEV)
        _fill_kv(c, seed, i, kv)
        s = spp.Session(m, 16, kv=kv)
        s.restore(8)
        scratch = torch.empty_like(x[i])
        scratch.copy_(x[i])
        readies.append(s.preposition([1, 2], x[i]))
        spp.ready_summary(readies[-1])
        x[i].copy_(scratch)
        kvs.append(kv)
        sessions.append(s)
    torch.cuda.synchronize()
    state = {"call": "gate", "n": n, "keep": (m, sessions, kvs, x), "readies": readies, "bits": bits}
    if n > 1:  # a serving loop keeps the batch's arguments marshalled
        state["gate"] = spp.GateCall(readies, [TAU] * n, [bits] * n)
    return state


def _cells(case, kv, cap, past, rows):
    """The cells an entry of `rows` tokens wrote: K [layer][head][row][dim], V^T
    [layer][head][dim][row] (views of the session's buffer)."""
    _, _, nkv, dh, _, _, _, _ = MODELS[case["model"]]
    cs = (cap + 63) // 64 * 64
    t = kv.view(case["layers"], 2, nkv * cs * dh)
    k = t[:, 0].view(case["layers"], nkv, cs, dh)[:, :, past:past + rows]
    v = t[:, 1].view(case["layers"], nkv, dh, cs)[:, :, :, past:past + rows]
    return k, v


def prepare(case, seed):
    call = case["call"]
    if call == "gate":
        return _prepare_gate(case, seed)
    V = MODELS[case["model"]][5]
    spec = _sessions(case, seed)
    total = max(1, sum(len(t) for _, t in spec))
    m = _model(case, seed, total, max(1, case.get("n", 1)))
    caps = [_cap(p, len(t)) for p, t in spec]
    pool = torch.empty(sum(_kv_elems(case, c) for c in caps), dtype=_kv_dtype(case), device=DEV)
    _fill_kv(case, seed, 0, pool)
    sessions, at = [], 0
    for (past, _), cap in zip(spec, caps):
        n = _kv_elems(case, cap)
        s = spp.Session(m, cap, kv=pool[at:at + n])
        s.restore(past)
        sessions.append(s)
        at += n
    st = {"call": call, "model": m, "sessions": sessions, "pool": pool,
          "past": [p for p, _ in spec], "entries": [t for _, t in spec]}
    if call == "shift":
        st["delta"] = case["delta"]
        return st
    if call == "batch":
        st["dist"] = torch.empty((len(spec), V), dtype=torch.float32, device=DEV)
        st["dists"] = list(st["dist"])
        return st
    st["cells"] = _cells(case, pool, caps[0], spec[0][0], len(spec[0][1]))
    st["dist"] = torch.empty(V, dtype=torch.float32, device=DEV)
    if call == "idle":
        st["flag"] = spp.YieldFlag()
    return st


def run(st):
    call = st["call"]
    if call == "gate":
        if st["n"] == 1:
            outcome, token, s = spp.gate(st["readies"][0], TAU, st["bits"])
            return {"outcome": outcome, "token": token, "argmax": s.argmax, "top1": s.top1,
                    "top2": s.top2, "gap": s.gap}
        st["gate"]()
        return {"served": np.array(st["gate"].outcomes(), dtype=np.int32)}
    if call == "batch":
        spp.preposition_batch(st["sessions"], st["entries"], st["dists"])
        return {"dist": st["dist"], "pool": st["pool"]}
    s = st["sessions"][0]
    if call == "preposition":
        s.preposition(st["entries"][0], st["dist"])
    elif call == "idle":
        s.preposition_idle(st["entries"][0], st["dist"], st["flag"])
    else:
        # back to the committed cells (a restore is metadata only), then the call itself
        s.restore(st["past"][0])
        if call == "resume":
            s.resume(st["entries"][0], st["dist"])
        elif call == "append":
            s.append_delta(st["entries"][0])
            return {"k": st["cells"][0], "v": st["cells"][1]}
        else:
            s.shift(st["delta"])
            return {"pool": st["pool"]}
    return {"dist": st["dist"], "k": st["cells"][0], "v": st["cells"][1]}


# ---- cost and result ----------------------------------------------------------------------


def work(case):
    call = case["call"]
    if call == "gate":
        return {"bytes": 4.0 * case["vocab"] * case["n"], "flops": 0.0}
    d, nq, nkv, dh, F, V, _, fmt = MODELS[case["model"]]
    eb = 4 if fmt == "f32" else 2
    cell = 2.0 * nkv * dh * eb  # bytes of one cell of one layer (K and V)
    L = case["layers"]
    if call == "shift":
        moved = case["past"] - case["delta"]
        return {"bytes": 2.0 * moved * cell * L, "flops": 3.0 * moved * nkv * dh * L}
    # (a batch's lengths are uniform in [1/8, 1] of the largest)
    f = 9.0 / 16.0 if call == "batch" else 1.0
    n = case.get("n", 1)
    rows, past = f * case["rows"], f * case["past"]
    wb = 17.0 / 32.0 if fmt == "mxfp4" else float(eb)
    qkv, rest = d * (nq + 2.0 * nkv) * dh, nq * dh * d + 3.0 * d * F
    logits = call != "append"
    # the last layer: its cells need every row, what follows only the decision rows
    full, tail = rows * n, float(n) if logits else 0.0
    attn = 4.0 * nq * dh * (past + rows / 2)
    flops = 2.0 * full * (qkv * L + rest * (L - 1)) + attn * full * (L - 1)
    flops += (2.0 * rest + attn) * tail
    layers = L if logits else L - 1
    nbytes = wb * (qkv * L + rest * layers) + n * (past * layers + rows * L) * cell + full * d * eb
    if logits:
        flops += 2.0 * n * V * d
        nbytes += float(V) * d * eb + 4.0 * n * V
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Four times the distance from exact() measured over the listed cases (2-norm).  fp32
    # model: 7e-7 for the sums' order, more over long histories.  bf16 and MXFP4 models:
    # 1.7e-3 to 2.0e-3, the rounding of a cell to bf16.  shift: 1.1e-3 over the whole buffer,
    # one bf16 rounding of the turned keys.
    call = case["call"]
    if call == "gate":
        return "exact"
    if MODELS[case["model"]][7] == "f32":
        return {"rel": 5e-6, "max": 1e-4}
    if call == "shift":
        return {"rel": 4.5e-3, "max": 3e-2}
    return {"rel": 8e-3, "max": 4e-2}


def _dense(case, w, k, l):
    if MODELS[case["model"]][7] != "mxfp4":
        return w[k][l].double()
    codes, sc = w[k][l], w["scales"][k][l]
    table = torch.tensor(E2M1 + tuple(-v for v in E2M1), dtype=torch.float64, device=DEV)
    both = torch.stack((codes & 15, codes >> 4), dim=-1).reshape(codes.shape[0], -1)
    scale = torch.exp2(sc.double() - 127.0)
    out = torch.empty(both.shape, dtype=torch.float64, device=DEV)
    for a in range(0, both.shape[0], 4096):
        b = both[a:a + 4096].long()
        out[a:a + 4096] = table[b] * scale[a:a + 4096].repeat_interleave(32, dim=1)
    return out


def _turn(x, pos, base):
    """Rotate-half RoPE of x [..., rows, dh] at the positions pos [rows]."""
    half = x.shape[-1] // 2
    th = pos[:, None].double() * base ** (-2.0 * torch.arange(half, device=DEV).double() / x.shape[-1])
    c, s = th.cos(), th.sin()
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * c - b * s, a * s + b * c), dim=-1)


def _rms(x, g):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g.double()


def _exact_forward(case, seed):
    d, nq, nkv, dh, F, V, base, _ = MODELS[case["model"]]
    G, L = nq // nkv, case["layers"]
    w = _weights(case, seed)
    spec = _sessions(case, seed)
    caps = [_cap(p, len(t)) for p, t in spec]
    pool = torch.empty(sum(_kv_elems(case, c) for c in caps), dtype=_kv_dtype(case), device=DEV)
    _fill_kv(case, seed, 0, pool)
    x = torch.cat([w["embed"][torch.tensor(t, device=DEV)] for _, t in spec]).double()
    pos = torch.cat([torch.arange(p, p + len(t), device=DEV) for p, t in spec])
    ks, vs = [], []
    for l in range(L):
        h = _rms(x, w["attn_norm"][l])
        M = h.shape[0]
        q = (h @ _dense(case, w, "wq", l).T).view(M, nq, dh).transpose(0, 1)
        k = (h @ _dense(case, w, "wk", l).T).view(M, nkv, dh).transpose(0, 1)
        v = (h @ _dense(case, w, "wv", l).T).view(M, nkv, dh).transpose(0, 1)
        q, k = _turn(q, pos, base), _turn(k, pos, base)
        ks.append(k)
        vs.append(v.transpose(1, 2))
        o = torch.empty((M, nq, dh), dtype=torch.float64, device=DEV)
        r0 = at = 0
        for (past, tok), cap in zip(spec, caps):
            m, cs, n = len(tok), (cap + 63) // 64 * 64, _kv_elems(case, cap)
            t = pool[at:at + n].view(L, 2, nkv * cs * dh)[l]
            rk, rv = t[0].view(nkv, cs, dh), t[1].view(nkv, dh, cs)
            see = torch.arange(past + m, device=DEV)[None] <= pos[r0:r0 + m, None]
            for j in range(nkv):
                # the cells are stored in the cache's type, the entry's own among them
                kk = torch.cat((rk[j, :past], k[j, r0:r0 + m].to(pool.dtype))).double()
                vv = torch.cat((rv[j, :, :past].T, v[j, r0:r0 + m].to(pool.dtype))).double()
                for a in range(j * G, j * G + G):
                    s = (q[a, r0:r0 + m] @ kk.T) / math.sqrt(dh)
                    p = torch.softmax(s.masked_fill(~see, -math.inf), dim=-1)
                    o[r0:r0 + m, a] = p @ vv
            r0 += m
            at += n
        x = x + o.reshape(M, nq * dh) @ _dense(case, w, "wo", l).T
        h = _rms(x, w["mlp_norm"][l])
        gate = torch.nn.functional.silu(h @ _dense(case, w, "w_gate", l).T)
        gate *= h @ _dense(case, w, "w_up", l).T
        x = x + gate @ _dense(case, w, "w_down", l).T
    ends = torch.tensor(np.cumsum([len(t) for _, t in spec]) - 1, device=DEV)
    z = _rms(x[ends], w["final_norm"])
    dist = torch.cat([z @ w["lm_head"][a:a + 16384].double().T for a in range(0, V, 16384)], dim=1)
    if "lm_bias" in w:
        dist = dist + w["lm_bias"].double()
    return dist, torch.stack(ks), torch.stack(vs)


def exact(case, seed):
    call = case["call"]
    if call == "gate":
        V = case["vocab"] if case["n"] == 1 else case["vocab"] // 16 * 16
        x, bits = _gate_logits(dict(case, vocab=V), seed)
        top = x.double().topk(2, dim=1)
        served, words = [], bits.cpu().numpy().astype(np.uint32)
        for i in range(case["n"]):
            # the lowest index of the largest value
            t = int((x[i] == x[i].max()).nonzero()[0])
            gap = float(top.values[i, 0] - top.values[i, 1])
            member = (int(words[t >> 5]) >> (t & 31)) & 1
            out = spp.SPP_FALL_GAP if not gap > TAU else (spp.SPP_SERVED if member else spp.SPP_FALL_NOT_IN_SET)
            served.append((out, t if out == spp.SPP_SERVED else -1, t))
        if case["n"] > 1:
            return {"served": np.array([s[:2] for s in served], dtype=np.int32)}
        a, b = float(top.values[0, 0]), float(top.values[0, 1])
        return {"outcome": served[0][0], "token": served[0][1], "argmax": served[0][2], "top1": a,
                "top2": b, "gap": a - b}
    if call == "shift":
        _, _, nkv, dh, _, _, base, _ = MODELS[case["model"]]
        cap, n, delta = _cap(case["past"], 0), case["past"], case["delta"]
        pool = torch.empty(_kv_elems(case, cap), dtype=_kv_dtype(case), device=DEV)
        _fill_kv(case, seed, 0, pool)
        cs, L = (cap + 63) // 64 * 64, case["layers"]
        out = pool.double().view(L, 2, nkv * cs * dh)
        k, v = out[:, 0].view(L, nkv, cs, dh), out[:, 1].view(L, nkv, dh, cs)
        back = torch.full((n - delta,), -delta, device=DEV)
        k[:, :, :n - delta] = _turn(k[:, :, delta:n].clone(), back, base)
        v[:, :, :, :n - delta] = v[:, :, :, delta:n].clone()
        return {"pool": out.reshape(-1)}
    dist, k, v = _exact_forward(case, seed)
    if call == "batch":
        return {"dist": dist, "pool": None}
    if call == "append":
        return {"k": k, "v": v}
    return {"dist": dist[0], "k": k, "v": v}
