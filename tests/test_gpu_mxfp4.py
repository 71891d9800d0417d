"""4-bit weight-only variant (MXFP4 projections) on the GPU.

The headline model of Sec. 4 is a 70B-class model at 4-bit precision.  The library
streams its projections as MXFP4 (e2m1 codes, one power-of-two scale per 32 weights along
K) into scaled fp4 x fp6 matrix-core products, which are exact.  The oracle
dequantizes the same generated bytes itself (``oracle.dequant_mxfp4``) and runs its
plain forward pass; the GPU logits must match within the pre-position bar."""
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
    """Prefill rows of 100 / 70 / 33 (the split-K gate/up with the separate SwiGLU past 64
    rows; 64-row tiles; 48-row tiles) and entries of 3, 65 and 1 rows against the
    oracle, logits and every cache cell."""
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
    """A 4-bit MLP as wide as 2 x 16384 outputs at 24 rows takes the unfused gate/up with
    four column blocks per wave (then the separate SwiGLU); 12 rows keep the fused kernel.
    Both against the oracle, logits and every cache cell, with the library packing its
    own copies or handed tiled ones."""
    import torch
    import paper_2606_29565_amd as spp
    shape = synth.Shape("fp4wide", 1, 256, 4, 2, 64, 16384, 2048, 1e4, "bf16", wfmt="mxfp4")
    seed = 73
    b = build_model(shape, seed, max_tokens=64, packed=packed)
    for n_past, L in ((40, 24), (30, 12)):
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


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 64, 65, 127, 128, 129, 272])
def test_mxfp4_rows_at_the_edges_of_the_projection_tiles(rows):
    """Every edge of the row tiles (16, 32 and 64 rows of the streaming kernel, 128 of the tile
    kernel), with an odd number of K-steps (F = 384: 3 of 128), matrices narrower than a
    workgroup's columns, and heads of 64 dims: logits and cells against the oracle."""
    import torch
    import paper_2606_29565_amd as spp
    shape = synth.Shape("fp4edge", 2, 256, 4, 2, 64, 384, 2048, 1e4, "bf16", wfmt="mxfp4")
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
    log(f"mxfp4 edges, {rows} rows: max|dlogit| {err:.2e}")
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
    """An embedding with an infinity or a NaN: the six-bit parts hold neither, so their block
    scales carry it, and the distribution is flagged as it is with bf16 weights."""
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
