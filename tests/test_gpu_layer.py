"""GPU parity of the rest of the decoder layer (layer norm, KV append, attention, fused epilogues and the
whole layer) against oracle/layer.py, operator by operator on the same fp16 inputs and end to end.

Operators: fp16 outputs within rel-L2 <= 1e-3 and max-abs <= 1e-2 * max|ref| of the fp64 oracle; the
KV append is a copy and must be bit-exact.  The whole layer chains eight roundings to fp16, each of
which can flip on a 1-ulp difference upstream, so it is compared at rel-L2 <= 2e-3."""
import numpy as np
import pytest

import paper_2403_01136_amd as lpq
from paper_2403_01136_amd import workloads as wl
from gpu_util import check_output, to_dev, u16
from oracle import indicator as OI
from oracle import layer as OL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU (no fallback path)"
    lpq.load_library()


def f16(a):
    return np.asarray(a, dtype=np.float32).astype(np.float16)


def rng(*key):
    return np.random.default_rng(wl.stream_seed("layer", *key))


def layer_shapes(h):
    """(K, N) of a decoder layer's linears."""
    return {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, 4 * h), "fc2": (4 * h, h)}


@pytest.mark.parametrize("M,h", [(1, 64), (5, 768), (33, 5120), (3, 14336)])
def test_layernorm(M, h):
    r = rng("ln", M, h)
    x = f16(r.standard_normal((M, h)) * 2 + 0.5)
    x[:, :3] *= 30                                        # outlier channels
    g, b = f16(1 + 0.1 * r.standard_normal(h)), f16(0.1 * r.standard_normal(h))
    y = lpq.lpq_layernorm(to_dev(x), to_dev(g), to_dev(b), 1e-5)
    check_output(y, OL.layernorm(x, g, b, 1e-5), "layernorm %dx%d" % (M, h))


@pytest.mark.parametrize("M", [1, 512, 513, 701, 1100, 1101])
@pytest.mark.parametrize("h", [8, 520, 2048, 2056, 4096, 4104, 8192, 8200, 12288, 12296, 16384])
def test_layernorm_kernel_forms(M, h):
    """Every number of threads and of chunks a thread that a launch takes, at its edges: waves of few chunks, an odd number of waves, the longest rows."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + h)
    x = (torch.randn((M, h), generator=gen, device="cuda") * 2 + 0.5).half()
    x[:, :3] *= 30
    g, b = ((a + 0.1 * torch.randn(h, generator=gen, device="cuda")).half() for a in (1.0, 0.0))
    y = lpq.lpq_layernorm(x, g, b, 1e-5)
    d = x.double()
    ref = (d - d.mean(1, keepdim=True)) / (d.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt() * g.double() + b.double()
    check_output(y, ref.cpu().numpy(), "layernorm %dx%d" % (M, h))


@pytest.mark.parametrize("act", [lpq.LPQ_ACT_RELU, lpq.LPQ_ACT_GELU_TANH, lpq.LPQ_ACT_NONE], ids=["relu", "gelu", "none"])
@pytest.mark.parametrize("phase,M", [(lpq.LPQ_DECODE, 7), (lpq.LPQ_DECODE, 40), (lpq.LPQ_PREFILL, 70)], ids=["dec7", "dec40", "pre70"])
def test_fused_epilogue(orc, act, phase, M):
    """act(x . w^T + bias) + residual with one rounding, also when a unit is cut (long K) and in place."""
    import torch
    N, K = 192, 4096
    w = wl.weight_np(N, K, "fused")
    x = wl.act_np(M, K, False, "fused", M)
    r = rng("fused", M)
    bias, res = f16(0.1 * r.standard_normal(N)), f16(r.standard_normal((M, N)))
    qw = lpq.lpq_quantize_pack(to_dev(w), 4, 1, bias=to_dev(bias))
    ref = orc.qlinear(x, w, 4, 1, bias)
    kind = {lpq.LPQ_ACT_RELU: "relu", lpq.LPQ_ACT_GELU_TANH: "gelu_tanh"}.get(act)
    ref = (OL.activation(ref, kind) if kind else ref) + res.astype(np.float64)
    y = to_dev(res).clone()                               # in place: the residual is the output buffer
    lpq.lpq_qlinear_fused(qw, to_dev(x), phase, activation=act, residual=y, y=y)
    check_output(y, ref, "fused epilogue")


def make_state(B, H, d, S, seed, alibi=False, act=lpq.LPQ_ACT_RELU):
    import torch
    r = rng("state", seed)
    h = H * d
    ln = [(f16(1 + 0.1 * r.standard_normal(h)), f16(0.05 * r.standard_normal(h))) for _ in range(2)]
    slopes = (2.0 ** (-8.0 * (np.arange(H) + 1) / H)).astype(np.float32) if alibi else None
    st = lpq.LayerState(H, d, S, B, torch.device("cuda"), tuple(to_dev(a) for a in ln[0]), tuple(to_dev(a) for a in ln[1]),
                        activation=act, alibi_slopes=None if slopes is None else to_dev(slopes))
    return st, ln, slopes


@pytest.mark.parametrize("d", [64, 128])
def test_kv_append_bit_exact(d):
    import torch
    B, H, S, T, pos0 = 3, 5, 128, 7, 40
    st, _, _ = make_state(B, H, d, S, d)
    r = rng("kv", d)
    qkv = f16(r.standard_normal((B * T, 3 * H * d)))
    k0, v0 = f16(r.standard_normal((B, H, S, d))), f16(r.standard_normal((B, H, d, S)))
    st.k_cache.copy_(to_dev(k0)), st.vt_cache.copy_(to_dev(v0))
    lpq.lpq_kv_append(to_dev(qkv), st, B, T, pos0)
    OL.kv_append(k0, v0, qkv, B, T, pos0, H)
    assert np.array_equal(u16(st.k_cache), k0.view(np.uint16)) and np.array_equal(u16(st.vt_cache), v0.view(np.uint16))


@pytest.mark.parametrize("alibi", [False, True], ids=["plain", "alibi"])
@pytest.mark.parametrize("B,H,d,S,T,pos0", [
    (2, 3, 64, 128, 1, 0), (16, 5, 128, 640, 1, 599), (1, 2, 128, 4160, 1, 4100), (3, 4, 64, 256, 1, 77),      # decode
    (2, 3, 128, 256, 100, 0), (1, 2, 64, 320, 130, 150), (2, 2, 128, 128, 16, 5), (1, 1, 128, 64, 3, 0),        # prefill
], ids=["dec_first", "dec_B16_L600", "dec_split_L4101", "dec_d64", "pre_T100", "pre_chunk_d64", "pre_T16", "pre_T3"])
def test_attention(B, H, d, S, T, pos0, alibi):
    import torch
    st, _, slopes = make_state(B, H, d, S, T, alibi)
    r = rng("att", B, H, d, T, pos0)
    qkv = f16(r.standard_normal((B * T, 3 * H * d)))
    qkv[:, :H * d] *= 2.0                                  # sharper softmax
    k = f16(r.standard_normal((B, H, S, d)))
    vt = f16(r.standard_normal((B, H, d, S)))
    k[:, :, pos0 + T:], vt[:, :, :, pos0 + T:] = np.nan, np.nan          # unwritten positions must never matter
    st.k_cache.copy_(to_dev(k)), st.vt_cache.copy_(to_dev(vt))
    lpq.lpq_kv_append(to_dev(qkv), st, B, T, pos0)
    out = lpq.lpq_attention(to_dev(qkv), st, B, T, pos0)
    OL.kv_append(k, vt, qkv, B, T, pos0, H)
    ref = OL.attention(qkv, k[:, :, :pos0 + T], vt[:, :, :, :pos0 + T], B, T, pos0, H, slopes)
    check_output(out, ref, "attention B%d H%d d%d T%d pos0 %d" % (B, H, d, T, pos0))


@pytest.mark.parametrize("bits,scheme,act,alibi", [(4, 1, lpq.LPQ_ACT_RELU, False), (3, 1, lpq.LPQ_ACT_GELU_TANH, True),
                                                   (8, 2, lpq.LPQ_ACT_RELU, False), (16, 0, lpq.LPQ_ACT_RELU, False)],
                         ids=["w4_relu", "w3_gelu_alibi", "i8_relu", "fp16_relu"])
def test_decoder_layer_prefill_then_decode(orc, bits, scheme, act, alibi):
    """A prompt of s tokens in the prefill phase, then three decode steps, against the oracle layer."""
    import torch
    B, H, d, S, s_len, f = 2, 4, 64, 128, 37, 512
    h = H * d
    st, ln, slopes = make_state(B, H, d, S, bits, alibi, act)
    r = rng("layer", bits, scheme)
    shapes = {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}
    W = {n: f16(r.standard_normal((N, K)) * (1.0 / np.sqrt(K))) for n, (K, N) in shapes.items()}
    bias = {n: f16(0.05 * r.standard_normal(N)) for n, (K, N) in shapes.items()}
    layer = {n: lpq.lpq_quantize_pack(to_dev(W[n]), bits, scheme, bias=to_dev(bias[n])) for n in shapes}
    kind = "relu" if act == lpq.LPQ_ACT_RELU else "gelu_tanh"
    k_ref, vt_ref = np.zeros((B, H, S, d), np.float16), np.zeros((B, H, d, S), np.float16)

    def lin(name, a):
        return orc.qlinear(a.astype(np.float16), W[name], bits, scheme, bias[name])

    ws = None
    pos = 0
    for step, (phase, T) in enumerate([(lpq.LPQ_PREFILL, s_len)] + [(lpq.LPQ_DECODE, 1)] * 3):
        x = f16(r.standard_normal((B * T, h)))
        y, ws = lpq.lpq_decoder_layer(layer, st, phase, B, T, pos, to_dev(x), workspace=ws if step > 1 else None)
        ref = OL.decoder_layer(x, lin, ln[0], ln[1], k_ref, vt_ref, B, T, pos, H, 1e-5, kind, slopes)
        yd = y.cpu().numpy().astype(np.float64)
        rel = np.linalg.norm(yd - ref) / np.linalg.norm(ref)
        assert np.all(np.isfinite(yd)) and rel <= 2e-3, "step %d rel-L2 %.3e" % (step, rel)
        assert np.abs(yd - ref).max() <= 1e-2 * np.abs(ref).max()
        # the caches hold what the oracle's hold, up to the fp16 rounding of qkv (compared as values)
        kd = st.k_cache.cpu().numpy().astype(np.float64)[:, :, :pos + T]
        assert np.linalg.norm(kd - k_ref[:, :, :pos + T].astype(np.float64)) <= 2e-3 * np.linalg.norm(kd)
        pos += T


def test_decoder_layer_at_the_benchmark_shape(orc):
    """One 4-bit OPT-13B-shaped layer (h = 5120, 40 heads of 128, f = 20480) at the two points bench.py and the cost
    model time: a prefill of 4 prompts x 512 tokens, and a decode step of 16 sequences at position 562.  The oracle
    layer runs on what it can finish in seconds: the first 48 tokens of the second prompt (a causal layer's output
    for a token depends on no later token, so that prefix is a prefill of its own), and two of the sixteen sequences
    of the decode step over the 562 cached positions (the cache is filled with seeded values)."""
    import torch
    B, H, d, f, s_len, n_gen = 4, 40, 128, 20480, 512, 100
    h, S, bits, scheme = H * d, 640, 4, 1
    st, ln, _ = make_state(16, H, d, S, "bench_shape")
    r = rng("bench_shape")
    shapes = {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}
    W = {n: f16(r.standard_normal((N, K), dtype=np.float32) * np.float32(1.0 / np.sqrt(K))) for n, (K, N) in shapes.items()}
    bias = {n: f16(0.05 * r.standard_normal(N)) for n, (K, N) in shapes.items()}
    layer = {n: lpq.lpq_quantize_pack(to_dev(W[n]), bits, scheme, bias=to_dev(bias[n])) for n in shapes}

    def lin(name, a):
        return orc.qlinear(a.astype(np.float16), W[name], bits, scheme, bias[name])

    def compare(y_rows, ref, what):
        yd = y_rows.astype(np.float64)
        rel = np.linalg.norm(yd - ref) / np.linalg.norm(ref)
        assert np.all(np.isfinite(yd)) and rel <= 2e-3, "%s rel-L2 %.3e" % (what, rel)
        assert np.abs(yd - ref).max() <= 1e-2 * np.abs(ref).max(), what

    # prefill: 4 x 512 tokens
    x = f16(r.standard_normal((B * s_len, h), dtype=np.float32))
    y, ws = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_PREFILL, B, s_len, 0, to_dev(x))
    seq, T_chk = 1, 48
    rows = slice(seq * s_len, seq * s_len + T_chk)
    k_ref, vt_ref = np.zeros((1, H, S, d), np.float16), np.zeros((1, H, d, S), np.float16)
    ref = OL.decoder_layer(x[rows], lin, ln[0], ln[1], k_ref, vt_ref, 1, T_chk, 0, H, 1e-5, "relu")
    compare(y[rows].cpu().numpy(), ref, "prefill 4 x 512, prompt %d, first %d tokens" % (seq, T_chk))
    kd = st.k_cache[seq, :, :T_chk].cpu().numpy().astype(np.float64)
    assert np.linalg.norm(kd - k_ref[0, :, :T_chk].astype(np.float64)) <= 2e-3 * np.linalg.norm(kd)

    # decode: 16 sequences at position s + n / 2
    n_seq, pos = 16, s_len + n_gen // 2
    k0 = f16(r.standard_normal((n_seq, H, S, d), dtype=np.float32))
    v0 = f16(r.standard_normal((n_seq, H, d, S), dtype=np.float32))
    st.k_cache.copy_(to_dev(k0)), st.vt_cache.copy_(to_dev(v0))
    xd = f16(r.standard_normal((n_seq, h), dtype=np.float32))
    yd, _ = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, n_seq, 1, pos, to_dev(xd))
    yd = yd.cpu().numpy()
    for b in (0, 9):
        kb, vb = k0[b:b + 1].copy(), v0[b:b + 1].copy()
        ref = OL.decoder_layer(xd[b:b + 1], lin, ln[0], ln[1], kb, vb, 1, 1, pos, H, 1e-5, "relu")
        compare(yd[b:b + 1], ref, "decode step, sequence %d of 16 at position %d" % (b, pos))
        assert np.array_equal(u16(st.k_cache[b, :, pos]), kb[0, :, pos].view(np.uint16)) or \
            np.linalg.norm(st.k_cache[b, :, pos].cpu().numpy().astype(np.float64) - kb[0, :, pos].astype(np.float64)) <= 2e-3 * np.linalg.norm(kb[0, :, pos].astype(np.float64))


@pytest.mark.parametrize("stochastic", [False, True], ids=["deterministic", "stochastic"])
@pytest.mark.parametrize("N,K,M", [(1, 128, 1), (70, 640, 33), (5120, 5120, 16), (333, 14336, 5)])
def test_variance_indicator(N, K, M, stochastic):
    """All eight forms of D_W * S_W(b)^2 * G(X) against the fp64 oracle (reductions in fp32 / fp64: 1e-5)."""
    w = wl.weight_np(N, K, "ind", N, K)
    x = wl.act_np(M, K, True, "ind", M)
    if stochastic:
        x = (x.astype(np.float32) + 0.75).astype(np.float16)          # a mean that matters
    got = lpq.lpq_variance_indicator(to_dev(w), to_dev(x), stochastic).cpu().numpy()
    ref = OI.indicator(w, x, stochastic)
    for i, key in enumerate(OI.ORDER):
        assert abs(got[i] - ref[key]) <= 1e-5 * abs(ref[key]) + 1e-300, (key, got[i], ref[key])


def test_decoder_layer_decode_step_in_a_hip_graph(orc):
    """A decode step of the layer captured once (after an eager warm-up, so that nothing is allocated during
    capture) and replayed several times, with eager work and synchronisations between the replays: every
    replay must reproduce the eager result bit for bit, caches included."""
    import torch
    B, H, d, S, f, pos = 4, 4, 64, 128, 512, 40
    h = H * d
    st, ln, _ = make_state(B, H, d, S, "graph")
    r = rng("graph")
    shapes = {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}
    layer = {n: lpq.lpq_quantize_pack(to_dev(f16(r.standard_normal((N, K)) / np.sqrt(K))), 4, 1) for n, (K, N) in shapes.items()}
    st.k_cache.copy_(to_dev(f16(r.standard_normal((B, H, S, d)))))
    st.vt_cache.copy_(to_dev(f16(r.standard_normal((B, H, d, S)))))
    x = to_dev(f16(r.standard_normal((B, h))))
    y_eager, ws = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, B, 1, pos, x)          # warm-up: workspaces exist now
    torch.cuda.synchronize()
    k_eager, v_eager = st.k_cache.clone(), st.vt_cache.clone()
    y_graph = torch.empty_like(y_eager)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, B, 1, pos, x, y_graph, ws, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    for replay in range(4):
        y_graph.fill_(float("nan"))
        st.k_cache[:, :, pos].fill_(0), st.vt_cache[:, :, :, pos].fill_(0)                 # the step must rewrite its position
        other = lpq.lpq_qlinear_decode(layer["fc1"], x)                                     # eager work between replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(u16(y_graph), u16(y_eager)), "replay %d" % replay
        assert torch.equal(st.k_cache, k_eager) and torch.equal(st.vt_cache, v_eager), "replay %d caches" % replay
        assert torch.isfinite(other).all()


@pytest.mark.parametrize("B,H,d,T,pos0", [
    (1, 3, 128, 127, 0), (2, 9, 64, 128, 0), (1, 2, 128, 129, 63), (1, 1, 64, 257, 64), (3, 3, 128, 31, 97), (1, 2, 64, 33, 1),   # prefill: 32- and
    (1, 2, 128, 1, 62), (2, 1, 64, 1, 63), (1, 3, 128, 1, 64), (1, 1, 64, 1, 255), (2, 2, 128, 1, 256), (1, 1, 128, 1, 1999),     # 128-query, 64-key edges
])
def test_attention_tile_edges_and_growing_scores(B, H, d, T, pos0):
    """Lengths around the kernels' tiles, scores that grow along the positions (a running maximum that moves at every tile,
    by a little and by much) beside flat ones, NaN behind the written positions.
    Tolerance: the file's (weights and results in fp16)."""
    import torch
    S = (pos0 + T + 63) // 64 * 64
    st, _, slopes = make_state(B, H, d, S, T, B == 2)
    r = rng("edges", B, H, d, T, pos0)
    h = H * d
    qkv = f16(r.standard_normal((B * T, 3 * h)))
    qkv[:, :h:d] = 4.0                                     # feature 0 of every head's queries
    k = f16(r.standard_normal((B, H, S, d)))
    vt = f16(r.standard_normal((B, H, d, S)))
    grow = np.array([0.0, 0.02, 0.5])[np.arange(H) % 3]    # per head: score growth per position (natural units)
    k[:, :, :, 0] = (grow[None, :, None] * np.arange(S)[None, None, :] * np.sqrt(d) / 4.0).astype(np.float16)
    k[:, :, pos0 + T:], vt[:, :, :, pos0 + T:] = np.nan, np.nan
    st.k_cache.copy_(to_dev(k)), st.vt_cache.copy_(to_dev(vt))
    lpq.lpq_kv_append(to_dev(qkv), st, B, T, pos0)
    out = lpq.lpq_attention(to_dev(qkv), st, B, T, pos0)
    OL.kv_append(k, vt, qkv, B, T, pos0, H)
    ref = OL.attention(qkv, k[:, :, :pos0 + T], vt[:, :, :, :pos0 + T], B, T, pos0, H, slopes)
    check_output(out, ref, "attention edges B%d H%d d%d T%d pos0 %d" % (B, H, d, T, pos0))


@pytest.mark.parametrize("pos0", [0, 1, 63, 64, 200, 1300])
def test_decode_layer_appends_in_the_attention_kernel(pos0):
    """A decode step of the whole layer writes the same cache bits as lpq_kv_append of its own QKV output does, beside positions that
    hold NaN, and leaves every other position alone; one split over positions and several."""
    import torch
    B, H, d, f = 2, 2, 64, 256
    h, S = H * d, (pos0 + 1 + 63) // 64 * 64
    st, ln, _ = make_state(B, H, d, S, pos0)
    r = rng("fresh", pos0)
    W = {n: f16(r.standard_normal((N, K)) / np.sqrt(K)) for n, (K, N) in {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}.items()}
    layer = {n: lpq.lpq_quantize_pack(to_dev(w), 4, 1) for n, w in W.items()}
    k, vt = f16(r.standard_normal((B, H, S, d))), f16(r.standard_normal((B, H, d, S)))
    k[:, :, pos0:], vt[:, :, :, pos0:] = np.nan, np.nan
    x = f16(r.standard_normal((B, h)))
    st.k_cache.copy_(to_dev(k)), st.vt_cache.copy_(to_dev(vt))
    y, _ = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, B, 1, pos0, to_dev(x))
    got_k, got_v = u16(st.k_cache).copy(), u16(st.vt_cache).copy()
    # the same operators one by one
    st.k_cache.copy_(to_dev(k)), st.vt_cache.copy_(to_dev(vt))
    h1 = lpq.lpq_layernorm(to_dev(x), *st.ln1, 1e-5)
    qkv = lpq.lpq_qlinear_decode(layer["qkv"], h1)
    lpq.lpq_kv_append(qkv, st, B, 1, pos0)
    assert np.array_equal(got_k, u16(st.k_cache)) and np.array_equal(got_v, u16(st.vt_cache))
    att = lpq.lpq_attention(qkv, st, B, 1, pos0)
    x1 = lpq.lpq_qlinear_fused(layer["out"], att, lpq.LPQ_DECODE, residual=to_dev(x))
    ff = lpq.lpq_qlinear_fused(layer["fc1"], lpq.lpq_layernorm(x1, *st.ln2, 1e-5), lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU)
    ref = lpq.lpq_qlinear_fused(layer["fc2"], ff, lpq.LPQ_DECODE, residual=x1)
    # the two attention calls add the new token's part in another order: roundings of the layer's operators may flip
    a, b = y.double().cpu().numpy(), ref.double().cpu().numpy()
    assert np.all(np.isfinite(a)) and np.linalg.norm(a - b) <= 2e-3 * np.linalg.norm(b)


@pytest.mark.parametrize("N,K,M", [(7, 128, 4099), (9, 2176, 1), (8200, 256, 3), (8193, 384, 700), (17, 4096, 2048)])
def test_variance_indicator_block_edges(N, K, M):
    """Rows that do not fill a workgroup's eight waves, more rows than waves (a wave takes several), K behind and on multiples of the
    2048 columns whose loads go out together, X smaller and larger than W.  Tolerance as above."""
    r = rng("ind-edges", N, K, M)
    w, x = f16(0.02 * r.standard_normal((N, K))), f16(r.standard_normal((M, K)) + 0.25)
    for stochastic in (False, True):
        got = lpq.lpq_variance_indicator(to_dev(w), to_dev(x), stochastic).cpu().numpy()
        ref = OI.indicator(w, x, stochastic)
        for i, key in enumerate(OI.ORDER):
            assert abs(got[i] - ref[key]) <= 1e-5 * abs(ref[key]) + 1e-300, (key, got[i], ref[key])


@pytest.mark.parametrize("d,T,pos0,bad", [(128, 100, 1, 70), (64, 300, 0, 130), (128, 40, 30, 39), (64, 33, 64, 32), (128, 260, 5, 0)])
@pytest.mark.parametrize("alibi", [False, True])
def test_non_finite_values_of_a_later_token(d, T, pos0, bad, alibi):
    """Infinities and NaN in the value row of one prompt token reach the queries at and behind it, not the ones before: those are what they are
    without it, up to the order of 32-bit sums (tolerance: the file's); the other head is the same bits."""
    import torch
    B, H, S = 1, 2, (pos0 + T + 63) // 64 * 64
    st, _, slopes = make_state(B, H, d, S, T, alibi)
    r = rng("nonfinite", d, T, pos0)
    h = H * d
    qkv = f16(r.standard_normal((B * T, 3 * h)))
    k, vt = f16(r.standard_normal((B, H, S, d))), f16(r.standard_normal((B, H, d, S)))
    outs = []
    for value in (None, np.inf, np.nan):
        q = qkv.copy()
        if value is not None:
            q[bad, 2 * h:2 * h + d:3] = value                # every third feature of head 0
            q[bad, 2 * h + 1] = -value
        st.k_cache.copy_(to_dev(k)), st.vt_cache.copy_(to_dev(vt))
        lpq.lpq_kv_append(to_dev(q), st, B, T, pos0)
        outs.append(lpq.lpq_attention(to_dev(q), st, B, T, pos0).double().cpu().numpy())
    clean, inf, nan = outs
    for got in (inf, nan):
        assert np.all(np.isfinite(got[:bad, :d])), "queries before the token"
        if bad:
            assert np.linalg.norm(got[:bad] - clean[:bad]) <= 1e-3 * np.linalg.norm(clean[:bad])
        assert np.array_equal(got[:, d:], clean[:, d:])
    # the queries that see it: +-inf or NaN in its features (its weight may round to zero), the others unharmed
    hit = np.zeros(d, dtype=bool)
    hit[0::3], hit[1] = True, True
    assert not np.any(np.isfinite(inf[bad:, :d][:, hit])) and not np.any(np.isfinite(nan[bad:, :d][:, hit]))
    seen = inf[bad, :d]
    assert np.all(seen[0::3] == np.inf) and seen[1] == -np.inf
    rest = inf[bad:, :d][:, ~hit]
    assert np.linalg.norm(rest - clean[bad:, :d][:, ~hit]) <= 1e-3 * np.linalg.norm(clean[bad:, :d][:, ~hit])


def test_decode_layer_of_large_caches_appends_ahead():
    """A decode step over more than 1 GB of cache appends in a launch of its own: the same bits as the operators one by one, in the outputs too."""
    import torch
    B, H, d, f, pos0 = 34, 16, 64, 256, 8001
    h, S, dev = H * d, (pos0 + 64) // 64 * 64, torch.device("cuda")
    gen = torch.Generator(device="cuda").manual_seed(9)
    normal = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.float16)
    ln = [(1.0 + 0.1 * normal(h), 0.1 * normal(h)) for _ in range(2)]
    st = lpq.LayerState(H, d, S, B, dev, *ln)
    st.k_cache.normal_(generator=gen), st.vt_cache.normal_(generator=gen)
    layer = {n: lpq.lpq_quantize_pack(normal(N, K) * 0.03, 4, 1) for n, (K, N) in {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}.items()}
    x = normal(B, h)
    k0, v0 = st.k_cache.clone(), st.vt_cache.clone()
    y, _ = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, B, 1, pos0, x)
    k1, v1 = st.k_cache.clone(), st.vt_cache.clone()
    st.k_cache.copy_(k0), st.vt_cache.copy_(v0)
    qkv = lpq.lpq_qlinear_decode(layer["qkv"], lpq.lpq_layernorm(x, *st.ln1, 1e-5))
    lpq.lpq_kv_append(qkv, st, B, 1, pos0)
    assert torch.equal(k1, st.k_cache) and torch.equal(v1, st.vt_cache)
    x1 = lpq.lpq_qlinear_fused(layer["out"], lpq.lpq_attention(qkv, st, B, 1, pos0), lpq.LPQ_DECODE, residual=x)
    ff = lpq.lpq_qlinear_fused(layer["fc1"], lpq.lpq_layernorm(x1, *st.ln2, 1e-5), lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU)
    assert torch.equal(y, lpq.lpq_qlinear_fused(layer["fc2"], ff, lpq.LPQ_DECODE, residual=x1))


def test_attention_over_very_long_rows():
    """max_seq beyond 2^32 / 14: a lane's offset into eight rows of the transposed V cache no longer fits 32 bits."""
    import torch
    H, d, S = 1, 64, 306_783_424
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("two caches of 39 GB")
    dev = torch.device("cuda")
    one = torch.ones(d, dtype=torch.float16, device=dev)
    st = lpq.LayerState(H, d, 64, 1, dev, (one, one), (one, one))
    st.cfg.max_seq = S
    st.k_cache = torch.empty((1, H, S, d), dtype=torch.float16, device=dev)
    st.vt_cache = torch.empty((1, H, d, S), dtype=torch.float16, device=dev)
    try:
        gen = torch.Generator(device="cuda").manual_seed(2)
        pos0, T = 100, 5
        qkv = torch.randn((T, 3 * d), generator=gen, device=dev).half()
        st.k_cache[0, 0, :pos0].normal_(generator=gen)
        st.vt_cache[0, 0, :, :pos0] = torch.randn((d, pos0), generator=gen, device=dev).half()
        for rows in (1, T):                                       # the decode kernel, the prefill kernel
            x = qkv[:rows].contiguous()
            lpq.lpq_kv_append(x, st, 1, rows, pos0)
            out = lpq.lpq_attention(x, st, 1, rows, pos0).double()
            k, v = st.k_cache[0, 0, :pos0 + rows].double(), st.vt_cache[0, 0, :, :pos0 + rows].double()
            sc = x[:, :d].double() @ k.t() / d ** 0.5
            sc = sc.masked_fill(torch.arange(pos0 + rows, device=dev)[None, :] > torch.arange(pos0, pos0 + rows, device=dev)[:, None], float("-inf"))
            ref = torch.softmax(sc, 1) @ v.t()
            assert float((out - ref).norm() / ref.norm()) <= 1e-3, rows
    finally:
        st.k_cache = st.vt_cache = None
        torch.cuda.empty_cache()


@pytest.mark.parametrize("bits,scheme", [(3, 1), (4, 1), (8, 1), (8, 2), (16, 0)], ids=["w3", "w4", "w8", "i8", "f16"])
@pytest.mark.parametrize("heads,d,seqs", [(9, 128, 1), (9, 128, 5), (12, 64, 2), (12, 64, 3), (12, 64, 16), (32, 128, 4), (40, 128, 1), (40, 128, 2), (42, 64, 6),
                                          (16, 128, 7), (16, 128, 8), (12, 64, 9), (42, 64, 3), (40, 128, 4)])
def test_decode_layer_normalises_in_the_linears(bits, scheme, heads, d, seqs, norm_behind=False):
    """Decode layers of few rows, whose QKV and FC1 kernels normalise their rows themselves (one or two rows to a wave, rows that fill no
    whole number of 512 columns, up to the longest that do), and the first that do not, against the same layer of single calls.  Both round to fp16 at the same places;
    statistics added in another order move an element by one such rounding now and then: the layer's 2e-3 as in this file."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(heads * d + seqs)
    h, pos = heads * d, 70

    def rand(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).half()

    shapes = layer_shapes(h)
    norm1, norm2, _ = lpq.lpq_layer_route_of([(bits, scheme) + shapes[n] for n in lpq.LINEARS], seqs, pos)
    if norm_behind:
        assert norm2 == lpq.LPQ_NORM_BEHIND_SPLITS
    else:
        inside = seqs <= 4 or (seqs <= 8 and h <= 2048)
        assert (norm1 == lpq.LPQ_NORM_IN_LINEAR) == inside and (norm2 == norm1 or bits == 16)      # a fp16 FC1 of 200 MB is no small launch
    layer = {n: lpq.lpq_quantize_pack(rand(N, K, std=0.02), bits, scheme, bias=rand(N, std=0.05)) for n, (K, N) in shapes.items()}
    norms = [((1 + 0.1 * torch.randn(h, generator=gen, device="cuda")).half(), rand(h, std=0.1)) for _ in range(2)]
    st = lpq.LayerState(heads, d, 128, seqs, torch.device("cuda"), norms[0], norms[1])
    st.k_cache[:, :, :pos] = rand(seqs, heads, pos, d)
    st.vt_cache[:, :, :, :pos] = rand(seqs, heads, d, pos)
    k0, v0 = st.k_cache.clone(), st.vt_cache.clone()
    x = rand(seqs, h, std=2.0)
    x[:, 5] *= 30
    x += 0.5
    y, _ = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, seqs, 1, pos, x)
    k1, v1 = st.k_cache.clone(), st.vt_cache.clone()
    st.k_cache.copy_(k0)
    st.vt_cache.copy_(v0)
    qkv = lpq.lpq_qlinear_decode(layer["qkv"], lpq.lpq_layernorm(x, *norms[0], 1e-5))
    lpq.lpq_kv_append(qkv, st, seqs, 1, pos)
    att = lpq.lpq_attention(qkv, st, seqs, 1, pos)
    z = lpq.lpq_qlinear_fused(layer["out"], att, lpq.LPQ_DECODE, residual=x)
    ff = lpq.lpq_qlinear_fused(layer["fc1"], lpq.lpq_layernorm(z, *norms[1], 1e-5), lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU)
    z = lpq.lpq_qlinear_fused(layer["fc2"], ff, lpq.LPQ_DECODE, residual=z)
    for a, b in ((y, z), (k1, st.k_cache), (v1, st.vt_cache)):
        assert float((a.double() - b.double()).norm() / b.double().norm()) <= 2e-3


@pytest.mark.parametrize("heads,d,seqs", [(40, 128, 16), (20, 128, 33), (64, 128, 20), (128, 128, 33), (17, 128, 50)])
def test_decode_layer_norm_behind_split_sums(heads, d, seqs):
    """Decode layers whose out-projection is split over K: the kernel that adds the splits also forms the second norm (rows of up to 16384 columns,
    that fill its threads or not).  Against the same layer of single calls, as above."""
    test_decode_layer_normalises_in_the_linears(4, 1, heads, d, seqs, norm_behind=True)


@pytest.mark.parametrize("bits,scheme,heads,d,seqs", [(3, 1, 12, 64, 1), (4, 1, 9, 128, 5), (8, 2, 16, 128, 8), (16, 0, 42, 64, 3), (4, 1, 40, 128, 4),
                                                      (3, 1, 17, 128, 50), (4, 1, 40, 128, 16), (8, 1, 64, 128, 33), (4, 1, 112, 128, 64)])
def test_decode_layer_norms_against_64_bits(bits, scheme, heads, d, seqs):
    """Norms inside the linears and behind split sums against 64 bits, every operator's output rounded to fp16: K and V of the new token (the first norm and
    QKV alone) and y, with rows of small numbers beside outlier channels, so that y is what the layer adds to them.  K and V: the rounding of the norm
    (2.1e-4), of the output (2.1e-4) and of the weights (1.7e-4), 3.5e-4 together, 1e-3 as for single operators; y: 2e-3 as in this file."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(heads * d + seqs)
    h, pos, shapes = heads * d, 70, layer_shapes(heads * d)

    def rand(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).half()

    norm1, norm2, _ = lpq.lpq_layer_route_of([(bits, scheme) + shapes[n] for n in lpq.LINEARS], seqs, pos)
    assert norm1 == norm2 == lpq.LPQ_NORM_IN_LINEAR if seqs <= 8 else norm2 == lpq.LPQ_NORM_BEHIND_SPLITS
    layer = {n: lpq.lpq_quantize_pack(rand(N, K, std=0.02), bits, scheme, bias=rand(N, std=0.05)) for n, (K, N) in shapes.items()}
    norms = [((1 + 0.1 * torch.randn(h, generator=gen, device="cuda")).half(), rand(h, std=0.1)) for _ in range(2)]
    st = lpq.LayerState(heads, d, 128, seqs, torch.device("cuda"), norms[0], norms[1])
    st.k_cache[:, :, :pos] = rand(seqs, heads, pos, d)
    st.vt_cache[:, :, :, :pos] = rand(seqs, heads, d, pos)
    x = rand(seqs, h, std=0.05)
    x[:, 5] *= 30
    x += 0.02
    y, _ = lpq.lpq_decoder_layer(layer, st, lpq.LPQ_DECODE, seqs, 1, pos, x)

    def rounded(a):
        return a.half().double()

    def norm(a, p):
        m, v = a.mean(1, keepdim=True), a.var(1, unbiased=False, keepdim=True)
        return rounded((a - m) / (v + 1e-5).sqrt() * p[0].double() + p[1].double())

    def linear(name, a):
        return a @ lpq.lpq_unpack_dequant(layer[name]).double().t() + layer[name].bias.double()

    def off(a, ref):
        return float((a.double() - ref).norm() / ref.norm())

    qkv = rounded(linear("qkv", norm(x.double(), norms[0]))).view(seqs, 3, heads, d)
    k, v = st.k_cache[:, :, pos], st.vt_cache[:, :, :, pos]
    assert off(k, qkv[:, 1]) <= 1e-3 and off(v, qkv[:, 2]) <= 1e-3
    keys, values = st.k_cache[:, :, :pos + 1].double(), st.vt_cache[:, :, :, :pos + 1].double()
    p = torch.softmax((qkv[:, 0, :, None] * keys).sum(-1) / d ** 0.5, -1)
    att = rounded((p[:, :, None] * values).sum(-1).view(seqs, h))
    z = rounded(x.double() + linear("out", att))
    ff = rounded(torch.relu(linear("fc1", norm(z, norms[1]))))
    assert off(y, rounded(z + linear("fc2", ff))) <= 2e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S", [128, 256])
@pytest.mark.parametrize("pos0", [0, 1, 30, 31, 32, 63, 64, 127])
def test_kv_append_of_one_token(d, pos0, S):
    """One token per sequence, at every place of a 16-byte chunk's halves and at the edges of a line, into short rows and into long ones, whose line is read
    first: its K and V and nothing else change, beside positions that hold NaN and infinities."""
    B, H = 3, 5
    st, _, _ = make_state(B, H, d, S, d)
    r = rng("kv1", d, pos0)
    qkv = f16(r.standard_normal((B, 3 * H * d)))
    k0, v0 = f16(r.standard_normal((B, H, S, d))), f16(r.standard_normal((B, H, d, S)))
    v0[:, :, :, pos0:], v0[:, 0, :, ::3] = np.nan, np.inf
    st.k_cache.copy_(to_dev(k0)), st.vt_cache.copy_(to_dev(v0))
    lpq.lpq_kv_append(to_dev(qkv), st, B, 1, pos0)
    OL.kv_append(k0, v0, qkv, B, 1, pos0, H)
    assert np.array_equal(u16(st.k_cache), k0.view(np.uint16)) and np.array_equal(u16(st.vt_cache), v0.view(np.uint16))


@pytest.mark.parametrize("T", [1, 3])
def test_kv_append_beside_another_writer(T):
    """Other positions of the same V rows, in the same 32, are another stream's to write at the same time: both writers' values are there afterwards."""
    import torch
    B, H, d, S, pos0 = 8, 16, 128, 256, 69
    st, _, _ = make_state(B, H, d, S, 5)
    r = rng("kv2", T)
    qkv, other = to_dev(f16(r.standard_normal((B * T, 3 * H * d)))), to_dev(f16(r.standard_normal((2, B, H, d, S))))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for i in range(40):
        with torch.cuda.stream(side):
            st.vt_cache[:, :, :, 64:pos0].copy_(other[i % 2][:, :, :, 64:pos0])
            st.vt_cache[:, :, :, pos0 + T:96].copy_(other[i % 2][:, :, :, pos0 + T:96])
        for _ in range(3):
            lpq.lpq_kv_append(qkv, st, B, T, pos0)
        torch.cuda.synchronize()
        want = other[i % 2].clone()
        want[:, :, :, pos0:pos0 + T] = qkv.view(B, T, 3, H, d)[:, :, 2].permute(0, 2, 3, 1)
        assert torch.equal(st.vt_cache[:, :, :, 64:96], want[:, :, :, 64:96]), "turn %d" % i
