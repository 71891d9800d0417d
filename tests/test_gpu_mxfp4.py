"""4-bit weight-only variant (MXFP4 projections) on the GPU.

The headline model of Sec. 4 is a 70B-class model at 4-bit precision.  The library
streams its projections as MXFP4 (e2m1 codes, one power-of-two scale per 32 weights along
K) and dequantizes them exactly to bf16 in registers.  The oracle dequantizes the same
generated bytes itself (``oracle.dequant_mxfp4``) and runs its plain forward pass; the
GPU logits must match within the pre-position bar."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build_model, fill_synthetic_kv, log, max_abs, oracle_logits, read_kv

pytestmark = pytest.mark.gpu

TOL = 5e-2
SMALL = synth.Shape("fp4small", 2, 256, 4, 2, 64, 512, 2048, 1e4, "bf16", wfmt="mxfp4")


def test_generator_bytes_match_cpu():
    import torch
    n = 4099
    for kind, cpu in ((0, synth.cpu_fp4_bytes), (1, synth.cpu_e8m0_bytes)):
        t = torch.empty(n, dtype=torch.uint8, device="cuda")
        synth.gpu_fill_bytes(t.data_ptr(), kind, n, 77, 12345, lbase=1001)
        torch.cuda.synchronize()
        assert np.array_equal(t.cpu().numpy(), cpu(n, 77, 12345, lbase=1001))


def test_pack_layout_follows_the_documented_tiles():
    """Code block (row block cb, step ks) at time-major position p holds, for lane
    l = 16 g + r, the source dwords of row 16 cb + r at bytes 64 ks + 16 c + 4 g
    (c = 0..3); the scale block holds each row's four scale bytes of the step."""
    import torch
    import paper_2606_29565_amd as spp
    shape = synth.Shape("fp4pack", 1, 512, 4, 2, 128, 1024, 256, 1e4, "bf16", wfmt="mxfp4")
    cfg = spp.model_config(1, shape.d_model, shape.n_q, shape.n_kv, shape.head_dim, shape.ffn,
                           shape.vocab, shape.rope_base, True, max_tokens=32, mxfp4=True)
    w = synth.gpu_weights(shape, 3)
    rows, cols = shape.weight_shape(synth.WD)       # [512][1024]: 8 steps per row
    codes, scales = w["w_down"][0], w["scales"]["w_down"][0]
    cd, sd = torch.empty_like(codes), torch.empty_like(scales)
    spp.pack_weight_mxfp4(cfg, spp.SPP_W_DOWN, codes, scales, cd, sd)
    torch.cuda.synchronize()
    src = codes.cpu().numpy().reshape(rows, cols // 2)
    ssrc = scales.cpu().numpy().reshape(rows, cols // 32)
    dst = cd.cpu().numpy().reshape(-1, 1024)
    sdst = sd.cpu().numpy().reshape(-1, 64)
    KS, nblk = cols // 128, rows // 16
    # find the slab T: the position of (cb=0, ks=1) is (1 % T) * (KS / T) + 1 / T blocks in
    lane0_step1 = np.concatenate([src[0, 64 + 16 * c: 64 + 16 * c + 4] for c in range(4)])
    hits = [T for T in range(1, KS + 1) if KS % T == 0 and
            np.array_equal(dst[((1 % T) * (KS // T) + 1 // T) * nblk, :16], lane0_step1)]
    assert len(hits) >= 1
    T = hits[0]
    log(f"mxfp4 pack: {KS} steps per row, slab {T}")
    rng = np.random.default_rng(0)
    for _ in range(40):
        cb, ks = int(rng.integers(nblk)), int(rng.integers(KS))
        pos = ((ks % T) * (KS // T) + ks // T) * nblk + cb
        for lane in (0, 5, 17, 38, 63):
            r, g = lane % 16, lane // 16
            want = np.concatenate([src[16 * cb + r, 64 * ks + 16 * c + 4 * g: 64 * ks + 16 * c + 4 * g + 4]
                                   for c in range(4)])
            assert np.array_equal(dst[pos, 16 * lane: 16 * lane + 16], want)
        for r in range(16):
            assert np.array_equal(sdst[pos, 4 * r: 4 * r + 4], ssrc[16 * cb + r, 4 * ks: 4 * ks + 4])


@pytest.mark.parametrize("packed", [False, True])
def test_small_mxfp4_model_matches_oracle(packed):
    import torch
    import paper_2606_29565_amd as spp
    seed = 69   # oracle gap 0.307 > 0.1: the argmax is compared too
    b = build_model(SMALL, seed, max_tokens=64, packed=packed)
    n_past, L = 40, 24
    toks = synth.cpu_tokens(n_past + L, seed, 0, SMALL.vocab).tolist()
    sess = spp.Session(b.model, 96)
    sess.append_delta(toks[:n_past])
    dist = torch.empty(SMALL.vocab, dtype=torch.float32, device="cuda")
    r = sess.preposition(toks[n_past:], dist)
    torch.cuda.synchronize()
    kvs = []
    ref = oracle_logits(SMALL, seed, n_past, toks[n_past:], prefill=toks[:n_past], kv_out=kvs)
    got = dist.cpu().numpy()
    err = max_abs(got, ref)
    s_ref = oracle.summary(ref)
    log(f"mxfp4 small (packed={packed}): max|dlogit| {err:.2e}, oracle gap {s_ref.gap:.3f}")
    assert err <= TOL
    assert s_ref.gap > 0.1 and spp.ready_summary(r).argmax == s_ref.argmax
    for layer in range(SMALL.n_layers):
        K, V = read_kv(b, sess, layer, n_past + L)
        Kr, Vr = kvs[0].layer(layer)
        assert np.allclose(K, np.asarray(Kr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)
        assert np.allclose(V, np.asarray(Vr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)


@pytest.mark.timeout(600)
def test_70b_mxfp4_layer_full_width_matches_oracle():
    """The headline model's real widths (d 8192, 64/8 heads x 128, F 28672, V 128256) on
    one layer over 1024 synthetic resident cells, 32 entry tokens: every logit."""
    import torch
    import paper_2606_29565_amd as spp
    wl = synth.WORKLOADS["stream70b_mxfp4"]
    shape = wl.shape.with_layers(1)
    n_past = 1024
    entry = synth.entry_tokens(wl, 0).tolist()
    b = build_model(shape, wl.seed, max_tokens=32)
    sess = spp.Session(b.model, n_past + 32)
    fill_synthetic_kv(b, sess, 0, n_past)
    sess.restore(n_past)
    dist = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    r = sess.preposition(entry, dist)
    torch.cuda.synchronize()
    got = dist.cpu().numpy()
    log("70b-mxfp4 layer: GPU done, running the oracle")
    ref = oracle_logits(shape, wl.seed, n_past, entry, kv_synth=True, last_only=True)
    err = max_abs(got, ref)
    s_ref = oracle.summary(ref)
    log(f"70b-mxfp4 layer: max|dlogit| {err:.2e}, logit std {np.std(ref):.3f}, "
        f"oracle gap {s_ref.gap:.3f}")
    assert err <= TOL
    if s_ref.gap > 0.1:
        assert spp.ready_summary(r).argmax == s_ref.argmax


@pytest.mark.parametrize("n_past,L", [(100, 3), (70, 65), (33, 1)])
def test_mxfp4_row_counts_of_every_launch_shape(n_past, L):
    """Prefill rows of 100 / 70 / 33 and entries of 3, 65 and 1 rows (the streaming kernel with
    16, 64 and 128 rows) against the oracle, logits and every cache cell."""
    import torch
    import paper_2606_29565_amd as spp
    seed = 71
    b = build_model(SMALL, seed, max_tokens=128)
    toks = synth.cpu_tokens(n_past + L, seed, 0, SMALL.vocab).tolist()
    sess = spp.Session(b.model, n_past + L + 8)
    sess.append_delta(toks[:n_past])
    dist = torch.empty(SMALL.vocab, dtype=torch.float32, device="cuda")
    sess.preposition(toks[n_past:], dist)
    torch.cuda.synchronize()
    kvs = []
    ref = oracle_logits(SMALL, seed, n_past, toks[n_past:], prefill=toks[:n_past], kv_out=kvs)
    err = max_abs(dist.cpu().numpy(), ref)
    log(f"mxfp4 small, prefill {n_past} + entry {L}: max|dlogit| {err:.2e}")
    assert err <= TOL
    for layer in range(SMALL.n_layers):
        K, V = read_kv(b, sess, layer, n_past + L)
        Kr, Vr = kvs[0].layer(layer)
        assert np.allclose(K, np.asarray(Kr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)
        assert np.allclose(V, np.asarray(Vr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)


@pytest.mark.parametrize("packed", [False, True])
def test_mxfp4_wide_mlp_four_column_blocks(packed):
    """A 4-bit MLP as wide as 2 x 16384 outputs: four column blocks per wave at up to 64 rows
    (then the separate SwiGLU), two at 65-128, the tile kernel with the SwiGLU fused at 150.
    All against the oracle, logits and every cache cell, with the library packing its own
    copies or handed tiled ones."""
    import torch
    import paper_2606_29565_amd as spp
    shape = synth.Shape("fp4wide", 1, 256, 4, 2, 64, 16384, 2048, 1e4, "bf16", wfmt="mxfp4")
    seed = 73
    b = build_model(shape, seed, max_tokens=150, packed=packed)
    for n_past, L in ((40, 24), (30, 12), (20, 60), (10, 100), (20, 150)):
        toks = synth.cpu_tokens(n_past + L, seed, n_past, shape.vocab).tolist()
        sess = spp.Session(b.model, n_past + L + 8)
        sess.append_delta(toks[:n_past])
        dist = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
        sess.preposition(toks[n_past:], dist)
        torch.cuda.synchronize()
        kvs = []
        ref = oracle_logits(shape, seed, n_past, toks[n_past:], prefill=toks[:n_past], kv_out=kvs)
        err = max_abs(dist.cpu().numpy(), ref)
        log(f"mxfp4 wide MLP (packed={packed}), prefill {n_past} + entry {L}: max|dlogit| {err:.2e}")
        assert err <= TOL
        K, V = read_kv(b, sess, 0, n_past + L)
        Kr, Vr = kvs[0].layer(0)
        assert np.allclose(K, np.asarray(Kr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)
        assert np.allclose(V, np.asarray(Vr)[:, :n_past + L], atol=4e-2, rtol=2.0 ** -7)
        sess.close()
    b.model.close()


# layers, d, query heads, kv heads, head_dim, F.  "small": an odd number of K-steps (F = 384: 3 of
# 128), matrices narrower than a workgroup's columns, heads of 64 dims.  "long": 15 and 13 steps, so
# K-splits of unequal ranges that begin inside a slab (3 steps, for O) and turn the tile kernel's
# buffers many times.  "fused": past 128 rows the SwiGLU fused over 15 steps.
EDGE_SHAPES = {"small": (2, 256, 4, 2, 64, 384), "long": (1, 1920, 15, 1, 128, 1664),
               "fused": (1, 1920, 15, 1, 128, 8320)}


@pytest.mark.parametrize("name,rows",
                         [("small", r) for r in (1, 16, 17, 32, 33, 64, 65, 127, 128, 129, 272, 1100)] +
                         [("long", r) for r in (1, 24, 48, 65, 129, 300)] + [("fused", r) for r in (129, 300)])
def test_mxfp4_rows_at_the_edges_of_the_projection_tiles(name, rows):
    """Every edge of the row tiles (16, 32, 64 and 128 rows of the streaming kernel, 128 of the
    tile kernel, whose second band begins at 1025 rows): logits and cells against the oracle."""
    import torch
    import paper_2606_29565_amd as spp
    layers, d, n_q, n_kv, dh, F = EDGE_SHAPES[name]
    shape = synth.Shape("fp4edge", layers, d, n_q, n_kv, dh, F, 2048, 1e4, "bf16", wfmt="mxfp4")
    seed = 77
    b = build_model(shape, seed, max_tokens=rows)
    toks = synth.cpu_tokens(20 + rows, seed, 0, shape.vocab).tolist()
    sess = spp.Session(b.model, 20 + rows + 8)
    for i in range(0, 20, rows):
        sess.append_delta(toks[i:min(i + rows, 20)])
    dist = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    sess.preposition(toks[20:], dist)
    torch.cuda.synchronize()
    kvs = []
    ref = oracle_logits(shape, seed, 20, toks[20:], prefill=toks[:20], kv_out=kvs)
    err = max_abs(dist.cpu().numpy(), ref)
    log(f"mxfp4 edges, {name}, {rows} rows: max|dlogit| {err:.2e}")
    assert err <= TOL
    for l in range(shape.n_layers):
        K, V = read_kv(b, sess, l, 20 + rows)
        Ko, Vo = kvs[0].layer(l)
        # one bf16 rounding of the cell apart, and the slack of the other cell comparisons
        for got, want in ((K, Ko[:, :20 + rows]), (V, Vo[:, :20 + rows])):
            assert np.all(np.abs(got - want) <= 2.0 ** -7 * np.maximum(np.abs(got), np.abs(want)) + 8e-3)


@pytest.mark.parametrize("rows", [4, 70])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_mxfp4_activations_that_are_not_finite_are_never_served(rows, bad):
    """An embedding with an infinity or a NaN: the distribution is flagged as it is with bf16
    weights."""
    import torch
    import paper_2606_29565_amd as spp
    b = build_model(SMALL, 5, max_tokens=128)
    toks = synth.cpu_tokens(rows, 5, 0, SMALL.vocab).tolist()
    b.weights["embed"].view(SMALL.vocab, SMALL.d_model)[toks[-1], 37] = bad
    sess = spp.Session(b.model, rows + 8)
    dist = torch.empty(SMALL.vocab, dtype=torch.float32, device="cuda")
    r = sess.preposition(toks, dist)
    torch.cuda.synchronize()
    assert not torch.isfinite(dist).any()
    bitmap = torch.full(((SMALL.vocab + 31) // 32,), -1, dtype=torch.int32, device="cuda")
    assert spp.gate(r, 0.0, bitmap)[0] == spp.SPP_FALL_NONFINITE


# ---- the activations' precision, element by element
#
# A model whose matrices are rows of unit vectors (code 2 is 1.0, scale byte 127 is 2^0), so
# that every projection copies single elements of its input and the logits (an identity LM
# head) are the residual stream times the final 1/RMS: what an activation lost on its way
# into a projection shows in one logit.  One channel in 32 carries a norm gain of `ratio`, as
# the outlier channels of trained models do; the others share its 32-element block.
UNIT = synth.Shape("fp4unit", 1, 256, 4, 2, 64, 256, 256, 1e4, "bf16", wfmt="mxfp4")


def _unit_rows(rows, cols, pick):
    codes = np.zeros((rows, cols // 2), np.uint8)
    for r, k in enumerate(pick):
        codes[r, k // 2] |= 2 << (4 * (k & 1))
    return codes


def _unit_model(rows, gains, mats):
    """UNIT with the given norm gains and the unit-vector picks of `mats` (other matrices 0)."""
    import torch
    b_w = synth.gpu_weights(UNIT, 1)
    d = UNIT.d_model
    rng = np.random.default_rng(11)
    embed = torch.from_numpy(rng.standard_normal((UNIT.vocab, d)).astype(np.float32)).bfloat16().cuda()
    b_w["embed"] = embed.reshape(-1).contiguous()
    b_w["final_norm"] = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    b_w["lm_head"] = torch.eye(UNIT.vocab, d, dtype=torch.bfloat16, device="cuda").reshape(-1).contiguous()
    for key in ("attn_norm", "mlp_norm"):
        g = gains.get(key, np.ones(d, np.float32))
        b_w[key] = [torch.from_numpy(g).bfloat16().cuda()]
    kinds = {"wq": synth.WQ, "wk": synth.WK, "wv": synth.WV, "wo": synth.WO, "w_gate": synth.WG,
             "w_up": synth.WU, "w_down": synth.WD}
    for key, kind in kinds.items():
        n, k = UNIT.weight_shape(kind)
        pick = mats.get(key)
        codes = _unit_rows(n, k, pick) if pick is not None else np.zeros((n, k // 2), np.uint8)
        b_w[key] = [torch.from_numpy(codes).reshape(-1).cuda()]
        b_w["scales"][key] = [torch.full((n * k // 32,), 127, dtype=torch.uint8, device="cuda")]
    import paper_2606_29565_amd as spp
    s = UNIT
    m = spp.Model(s.n_layers, s.d_model, s.n_q, s.n_kv, s.head_dim, s.ffn, s.vocab, s.rope_base,
                  s.bf16, b_w, rms_eps=s.eps, max_tokens=rows, mxfp4=True)
    return m, embed.float().cpu().numpy().astype(np.float64)


def _unit_run(m, rows, token):
    import torch
    import paper_2606_29565_amd as spp
    sess = spp.Session(m, rows)
    dist = torch.empty(UNIT.vocab, dtype=torch.float32, device="cuda")
    sess.preposition([token] * rows, dist)
    torch.cuda.synchronize()
    return sess, dist.cpu().numpy().astype(np.float64)


def _inv_rms(x):
    return 1.0 / np.sqrt(np.mean(x * x) + UNIT.eps)


# A projection input enters as it does with bf16 weights, as two bf16 halves, which leave at
# most 2^-18 of an element whatever its neighbours are.
HALVES = 2.0 ** -18
FP32 = 2.0 ** -21   # the few fp32 roundings on the way from an element to its logit


@pytest.mark.parametrize("rows", [1, 32, 33, 70, 130])
@pytest.mark.parametrize("ratio", [1.0, 128.0, 1024.0, 8192.0])
def test_mxfp4_projection_inputs_keep_their_small_elements(rows, ratio):
    """Gate/up and down inputs, the outliers in 1 of 32 channels of either."""
    d, F, token = UNIT.d_model, UNIT.ffn, 3
    rng = np.random.default_rng(5)
    gain = np.ones(d, np.float32)
    gain[7::32] = ratio
    plain = np.array([c for c in range(d) if c % 32 != 7])
    gate = rng.choice(plain, F)
    up = rng.choice(plain, F)
    up[5::32] = np.arange(7, d, 32)            # one SwiGLU output in 32 is an outlier
    m, E = _unit_model(rows, {"mlp_norm": gain}, {"w_gate": gate, "w_up": up, "w_down": np.arange(d)})
    sess, got = _unit_run(m, rows, token)
    x0 = E[token]
    y, inv = x0 * gain, _inv_rms(x0)
    a, u = inv * y[gate], inv * y[up]
    act = a / (1.0 + np.exp(-a)) * u
    x = x0 + act
    # relative error of one SwiGLU output: the gate's (d log silu / d log a <= 1 + |a|), the up's,
    # the output's own
    bound = (3.0 + np.abs(a)) * HALVES * np.abs(act) + FP32 * (np.abs(x0) + np.abs(act))
    # (the final 1/RMS is common to all logits and follows the outliers' own error: the median
    # of the ratios stands for it)
    err = np.abs(got / np.median(got / x) - x)
    log(f"unit model, {rows} rows, outliers {ratio:g}x: worst error {(err / bound).max():.3f} of its bound")
    assert (err / bound).max() <= 1.0
    sess.close()
    m.close()


@pytest.mark.parametrize("ratio", [1.0, 1024.0, 8192.0])
def test_mxfp4_attention_output_keeps_its_small_elements(ratio):
    """The O projection's input: with one key the attention output is the value cell itself."""
    import paper_2606_29565_amd as spp
    d, token = UNIT.d_model, 9
    gain = np.ones(d, np.float32)
    gain[7::32] = ratio
    kv_rows = UNIT.n_kv * UNIT.head_dim
    m, E = _unit_model(1, {"attn_norm": gain}, {"wv": np.arange(kv_rows), "wo": np.arange(d)})
    sess, got = _unit_run(m, 1, token)
    b = type("B", (), {"shape": UNIT, "model": m})
    _, V = read_kv(b, sess, 0, 1)
    head = np.arange(UNIT.n_q).repeat(UNIT.head_dim) // UNIT.group
    att = V[head, 0, np.tile(np.arange(UNIT.head_dim), UNIT.n_q)].astype(np.float64)
    x = E[token] + att
    bound = HALVES * np.abs(att) + FP32 * (np.abs(E[token]) + np.abs(att))
    err = np.abs(got / _inv_rms(x) - x)
    log(f"unit model, attention output, outliers {ratio:g}x: worst error {(err / bound).max():.3f} of its bound")
    assert (err / bound).max() <= 1.0
    sess.close()
    m.close()
