"""The work that a serving program has this library do, as measurable cases.

A pipeline stage of an LLM with per-layer weight precisions is loaded (weights are quantised and packed on the GPU, the
planner asks for their variance indicators), runs its prompts (prefill) and then generates (decode); a program either
calls whole decoder layers, or the linears of a stage in one call, or single linears and the attention with its cache
beside operators of its own.  The kinds below are those calls:

    layer      lpq_decoder_layer in either phase, with the cache it updates
    attention  lpq_kv_append + lpq_attention, one new token per sequence or a (chunk of a) prompt
    stage      lpq_stage_linears in either phase, layers of mixed precisions
    linear     lpq_qlinear_fused, one linear with its epilogue, in either phase
    quantize   lpq_quantize_pack of a layer's four weights
    indicator  lpq_variance_indicator of a layer's four weights

Sizes are the shapes that the benchmark and the tests of this repository use (hidden sizes 768, 5120, 7168, 9216, 14336;
feed-forward four times as wide) and others of the same range; storage formats are all five of the library ("w3", "w4",
"w8": grouped 3, 4, 8 bit; "i8": per-row symmetric 8 bit; "f16").  Inputs are seeded: weights N(0, 0.02^2) with a
thousandth of them twenty times larger, activations N(0, 1) with a few channels thirty times larger.
"""
import math
import zlib

import torch

import paper_2403_01136_amd as lpq

FORMATS = {"w3": (3, lpq.LPQ_ASYM_GROUP), "w4": (4, lpq.LPQ_ASYM_GROUP), "w8": (8, lpq.LPQ_ASYM_GROUP),
           "i8": (8, lpq.LPQ_SYM_CHANNEL), "f16": (16, lpq.LPQ_FP16)}
ACTS = {"none": lpq.LPQ_ACT_NONE, "relu": lpq.LPQ_ACT_RELU, "gelu": lpq.LPQ_ACT_GELU_TANH}
LN_EPS = 1e-5
DEVICE = "cuda"


def listed():
    return [
        # the smallest model's layer generating for one user: ten launches of almost no work
        dict(name="layer_decode_768_1seq_w4", kind="layer", h=768, head_dim=64, fmt="w4", seqs=1, T=1, pos=212, act="relu", alibi=False),
        # the benchmark's layer: OPT-13B shapes, 4 bit, 16 sequences half way through their answers
        dict(name="layer_decode_5120_16seq_w4", kind="layer", h=5120, head_dim=128, fmt="w4", seqs=16, T=1, pos=562, act="relu", alibi=False),
        # a busier server: more sequences than one pass of 32 rows takes, an odd context, BLOOM-like ALiBi and GELU, 3 bit
        dict(name="layer_decode_7168_43seq_w3", kind="layer", h=7168, head_dim=128, fmt="w3", seqs=43, T=1, pos=1337, act="gelu", alibi=True),
        # a prefill micro-batch of ragged length (the prompts are padded to the longest, not to a tile)
        dict(name="layer_prefill_5120_3x397_w4", kind="layer", h=5120, head_dim=128, fmt="w4", seqs=3, T=397, pos=0, act="relu", alibi=False),
        # long contexts of few users: the cache is split over positions
        dict(name="attention_decode_7168_3seq_6001", kind="attention", h=7168, head_dim=128, seqs=3, T=1, pos=6001, alibi=False),
        # long prompts: attention is the part of prefill that grows with the square
        dict(name="attention_prefill_5120_2x1500", kind="attention", h=5120, head_dim=128, seqs=2, T=1500, pos=0, alibi=False),
        # a twelve-layer stage of alternating 3- and 4-bit layers (OPT-30B shapes), a small decode micro-batch
        dict(name="stage_decode_7168_7row_w3w4", kind="stage", phase="decode", h=7168, M=7, layers="w3 w4 w3 w4 w3 w4 w3 w4 w3 w4 w3 w4"),
        # the widest shapes (BLOOM-176B), 3 bit, the largest decode micro-batch of the benchmark
        dict(name="stage_decode_14336_64row_w3", kind="stage", phase="decode", h=14336, M=64, layers="w3 w3 w3 w3"),
        # the mixed OPT-13B stage at the benchmark's prefill micro-batch of 4 x 512 tokens
        dict(name="stage_prefill_5120_2048row_mixed", kind="stage", phase="prefill", h=5120, M=2048, layers="f16 w8 w4 w4 w3 w3 w4 w8"),
        # a single short prompt through one wide linear with a fused epilogue
        dict(name="linear_prefill_9216_200row_i8", kind="linear", phase="prefill", K=9216, N=36864, M=200, fmt="i8", act="gelu", residual=False),
        # loading: a layer's weights to packed 3 bit
        dict(name="quantize_7168_w3", kind="quantize", h=7168, fmt="w3"),
        # planning: the indicators of a layer on a calibration batch
        dict(name="indicator_5120_2048row", kind="indicator", h=5120, M=2048),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _hidden(rng, lo, hi):
    """A hidden size: whole heads of 64 or 128, a multiple of 128."""
    return max(lo // 128, _logu(rng, lo, hi) // 128) * 128, rng.choice((64, 128, 128))


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "attention", "attention", "stage", "stage", "linear", "linear", "quantize", "indicator"))
    if kind in ("layer", "attention"):
        h, d = _hidden(rng, 768, 7168)
        case = dict(kind=kind, h=h, head_dim=d, alibi=rng.random() < 0.4)
        if rng.random() < 0.5:                                       # decode: at most 200k cached tokens x features of 5120
            seqs = _logu(rng, 1, 64)
            top = min(8000 if kind == "attention" else 2000, 300_000_000 // (seqs * h))
            case.update(seqs=seqs, T=1, pos=_logu(rng, 16, max(17, top)))
        else:                                                        # a prompt, or a later chunk of one
            T = _logu(rng, 9, 1500 if kind == "attention" else 900)
            case.update(seqs=rng.randint(1, max(1, min(4, 1800 // T))), T=T, pos=rng.choice((0, 0, 0, _logu(rng, 10, 1000))))
        if kind == "layer":
            case.update(fmt=rng.choice(tuple(FORMATS)), act=rng.choice(("relu", "gelu")))
        return case
    if kind == "stage":
        h, _ = _hidden(rng, 768, 7168)
        phase = rng.choice(("decode", "prefill"))
        n = rng.randint(1, 4)
        return dict(kind=kind, phase=phase, h=h, M=_logu(rng, 1, 64) if phase == "decode" else _logu(rng, 40, 2000),
                    layers=" ".join(rng.choice(tuple(FORMATS)) for _ in range(n)))
    if kind == "linear":
        phase = rng.choice(("decode", "prefill"))
        return dict(kind=kind, phase=phase, K=_logu(rng, 768, 28672) // 128 * 128, N=_logu(rng, 768, 36864) // 64 * 64,
                    M=_logu(rng, 1, 64) if phase == "decode" else _logu(rng, 20, 1500), fmt=rng.choice(tuple(FORMATS)),
                    act=rng.choice(tuple(ACTS)), residual=rng.random() < 0.5)
    h, _ = _hidden(rng, 768, 7168)
    if kind == "quantize":
        return dict(kind=kind, h=h, fmt=rng.choice(tuple(FORMATS)))
    return dict(kind=kind, h=h, M=_logu(rng, 64, 4096))


# ---- inputs -------------------------------------------------------------------------------------------------------

def _gen(seed, *key):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((zlib.crc32(repr(key).encode()) << 20) ^ int(seed))
    return g


def _normal(shape, std, seed, *key):
    return torch.empty(shape, dtype=torch.float16, device=DEVICE).normal_(0.0, std, generator=_gen(seed, *key))


def _weight(N, K, seed, *key):
    w = _normal((N, K), 0.02, seed, "w", *key)
    flat = w.view(-1)
    at = torch.randint(0, flat.numel(), (flat.numel() // 1000,), generator=_gen(seed, "at", *key), device=DEVICE)
    flat[at] = flat[at] * 20.0
    return w


def _acts(M, K, seed, *key):
    x = _normal((M, K), 1.0, seed, "x", *key)
    ch = torch.randperm(K, generator=_gen(seed, "ch", *key), device=DEVICE)[:6]
    x[:, ch] *= 30.0
    return x


def _shapes(h):
    """name -> (K, N) of a layer's four linears."""
    return {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, 4 * h), "fc2": (4 * h, h)}


def _layer_norms(h, seed):
    return [((1.0 + _normal((h,), 0.1, seed, "gamma", i)).half(), _normal((h,), 0.05, seed, "beta", i)) for i in (1, 2)]


def _max_seq(case):
    return (case["pos"] + case["T"] + 64) // 64 * 64


def _cache(case, seed):
    """K [seqs][heads][max_seq][d] and V transposed, filled up to the call's first position."""
    B, H, S, d, pos = case["seqs"], case["h"] // case["head_dim"], _max_seq(case), case["head_dim"], case["pos"]
    k = _normal((B, H, S, d), 1.0, seed, "k")
    v = _normal((B, H, d, S), 1.0, seed, "v")
    k[:, :, pos:] = 0.0
    v[:, :, :, pos:] = 0.0
    return k, v


def _slopes(case):
    H = case["h"] // case["head_dim"]
    return torch.tensor([2.0 ** (-8.0 * (i + 1) / H) for i in range(H)], dtype=torch.float32, device=DEVICE) if case["alibi"] else None


def _pack(w, fmt, bias=None):
    return lpq.lpq_quantize_pack(w, *FORMATS[fmt], bias=bias)


def _layer_state(case, seed, act):
    h, d = case["h"], case["head_dim"]
    ln1, ln2 = _layer_norms(h, seed)
    st = lpq.LayerState(h // d, d, _max_seq(case), case["seqs"], torch.device(DEVICE), ln1, ln2, activation=ACTS[act], ln_eps=LN_EPS,
                        alibi_slopes=_slopes(case))
    st.k_cache, st.vt_cache = _cache(case, seed)
    return st


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "layer":
        h, M = case["h"], case["seqs"] * case["T"]
        s["layer"] = {n: _pack(_weight(N, K, seed, n), case["fmt"], bias=_normal((N,), 0.05, seed, "bias", n)) for n, (K, N) in _shapes(h).items()}
        s["state"] = _layer_state(case, seed, case["act"])
        s["x"] = _acts(M, h, seed)
        s["phase"] = lpq.LPQ_DECODE if case["T"] == 1 else lpq.LPQ_PREFILL
        s["y"] = torch.empty_like(s["x"])
        s["ws"] = torch.empty(M * 9 * h * 2, dtype=torch.uint8, device=DEVICE)          # h1, qkv, attention output, feed-forward rows
    elif kind == "attention":
        s["state"] = _layer_state(case, seed, "relu")
        s["qkv"] = _normal((case["seqs"] * case["T"], 3 * case["h"]), 1.0, seed, "qkv")
        s["out"] = torch.empty((case["seqs"] * case["T"], case["h"]), dtype=torch.float16, device=DEVICE)
    elif kind == "stage":
        layers, xs, ys = [], [], []
        for i, fmt in enumerate(case["layers"].split()):
            shapes = _shapes(case["h"])
            layers.append({n: _pack(_weight(N, K, seed, i, n), fmt) for n, (K, N) in shapes.items()})
            xs.append({n: _acts(case["M"], K, seed, i, n) for n, (K, N) in shapes.items()})
            ys.append({n: torch.empty((case["M"], N), dtype=torch.float16, device=DEVICE) for n, (K, N) in shapes.items()})
        s["stage"], s["ys"] = lpq.Stage(layers, xs, ys), [y for lay in ys for y in lay.values()]
        s["phase"] = lpq.LPQ_DECODE if case["phase"] == "decode" else lpq.LPQ_PREFILL
    elif kind == "linear":
        s["w"] = _pack(_weight(case["N"], case["K"], seed), case["fmt"], bias=_normal((case["N"],), 0.05, seed, "bias"))
        s["x"] = _acts(case["M"], case["K"], seed)
        s["res"] = _normal((case["M"], case["N"]), 1.0, seed, "res") if case["residual"] else None
        s["y"] = torch.empty((case["M"], case["N"]), dtype=torch.float16, device=DEVICE)
        s["phase"] = lpq.LPQ_DECODE if case["phase"] == "decode" else lpq.LPQ_PREFILL
    else:
        s["w"] = [_weight(N, K, seed, n) for n, (K, N) in _shapes(case["h"]).items()]
        if kind == "indicator":
            s["x"] = [_acts(case["M"], K, seed, n) for n, (K, N) in _shapes(case["h"]).items()]
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "layer":
        st = s["state"]
        lpq.lpq_decoder_layer(s["layer"], st, s["phase"], case["seqs"], case["T"], case["pos"], s["x"], s["y"], s["ws"])
        return [s["y"], st.k_cache, st.vt_cache]
    if kind == "attention":
        st = s["state"]
        lpq.lpq_kv_append(s["qkv"], st, case["seqs"], case["T"], case["pos"])
        lpq.lpq_attention(s["qkv"], st, case["seqs"], case["T"], case["pos"], s["out"])
        return [s["out"], st.k_cache, st.vt_cache]
    if kind == "stage":
        lpq.lpq_stage_linears(s["stage"], s["phase"])
        return s["ys"]
    if kind == "linear":
        return lpq.lpq_qlinear_fused(s["w"], s["x"], s["phase"], activation=ACTS[case["act"]], residual=s["res"], y=s["y"])
    if kind == "quantize":
        out = []
        for w in s["w"]:
            q = _pack(w, case["fmt"])
            out += [t for t in (q.codes, q.scales, q.zeros) if t is not None]
        return out
    return [lpq.lpq_variance_indicator(w, x) for w, x in zip(s["w"], s["x"])]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def _packed_bytes(K, N, fmt):
    bits, scheme = FORMATS[fmt]
    return K * N * bits // 8 + (4 * (K // 128) * N if scheme == lpq.LPQ_ASYM_GROUP else 2 * N if scheme == lpq.LPQ_SYM_CHANNEL else 0)


def _attention_work(case):
    """(bytes, flops): cached positions read once, the new ones written once; q.k and p.v over the causal half."""
    B, h, T, pos = case["seqs"], case["h"], case["T"], case["pos"]
    return 4 * B * h * (pos + T), 4 * B * h * (T * pos + T * (T + 1) // 2)


def work(case):
    kind = case["kind"]
    if kind == "layer":
        h, M = case["h"], case["seqs"] * case["T"]
        b, f = _attention_work(case)
        for K, N in _shapes(h).values():
            b += _packed_bytes(K, N, case["fmt"]) + 2 * N
            f += 2 * M * K * N
        return {"bytes": b + 4 * M * h + 8 * h, "flops": f}
    if kind == "attention":
        b, f = _attention_work(case)
        return {"bytes": b + 8 * case["seqs"] * case["T"] * case["h"], "flops": f}
    if kind == "stage":
        M, b, f = case["M"], 0, 0
        for fmt in case["layers"].split():
            for K, N in _shapes(case["h"]).values():
                b += _packed_bytes(K, N, fmt) + 2 * M * (K + N)
                f += 2 * M * K * N
        return {"bytes": b, "flops": f}
    if kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": _packed_bytes(K, N, case["fmt"]) + 2 * N + 2 * M * (K + N * (2 if case["residual"] else 1)), "flops": 2 * M * K * N}
    if kind == "quantize":
        return {"bytes": sum(2 * K * N + _packed_bytes(K, N, case["fmt"]) for K, N in _shapes(case["h"]).values()), "flops": 0}
    return {"bytes": sum(2 * K * (N + case["M"]) for K, N in _shapes(case["h"]).values()), "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "indicator":
        return {"rel": 1e-5}                       # 32-bit group statistics, sums in 64 bits
    if kind == "attention":
        return {"rel": 1e-3, "max": 2e-2}          # probabilities and results in fp16: 2.5e-4 from 64 bits
    if kind == "layer":
        return {"rel": 4e-3, "max": 5e-2}          # eight operators that each round to fp16: up to 9e-4 from 64 bits
    return {"rel": 1.2e-3, "max": 1e-2}            # fp16 operands, 32-bit sums, one rounding to fp16: 3e-4 from 64 bits


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------

def _dequant64(w, fmt):
    """The weight values that the format stores, for rows of w (fp16 [n][K]), in 64 bits."""
    bits, scheme = FORMATS[fmt]
    if scheme == lpq.LPQ_FP16:
        return w.double()
    n, K = w.shape
    f = w.float()
    if scheme == lpq.LPQ_SYM_CHANNEL:
        top = torch.full((1,), 127.0, device=DEVICE)                 # a tensor: division by a number multiplies by its reciprocal
        s = (f.abs().amax(1, keepdim=True) / top).half().float()
        s = torch.where(s == 0, torch.ones_like(s), s)
        return torch.clamp(torch.round(f / s), -127, 127).double() * s.double()
    f = f.view(n, K // 128, 128)
    lo, hi, top = f.amin(2, keepdim=True), f.amax(2, keepdim=True), torch.full((1,), float(2 ** bits - 1), device=DEVICE)
    s = ((hi - lo) / top).half().float()
    s = torch.where(s == 0, torch.ones_like(s), s)
    return (torch.clamp(torch.round((f - lo) / s), 0, 2 ** bits - 1).double() * s.double() + lo.double()).view(n, K)


def _linear64(x64, w, fmt, bias=None):
    """x64 . dequant(w)^T in 64 bits, in bands of rows of w."""
    y = torch.empty((x64.shape[0], w.shape[0]), dtype=torch.float64, device=DEVICE)
    for r in range(0, w.shape[0], 4096):
        y[:, r:r + 4096] = x64 @ _dequant64(w[r:r + 4096], fmt).t()
    return y if bias is None else y + bias.double()


def _act64(y, act):
    if act == "relu":
        return torch.relu(y)
    if act == "gelu":
        return 0.5 * y * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (y + 0.044715 * y ** 3)))
    return y


def _attention64(case, qkv64, seed):
    """(attention output, K cache, transposed V cache) of a call in 64 bits."""
    B, T, pos, h, d = case["seqs"], case["T"], case["pos"], case["h"], case["head_dim"]
    H, L = h // d, pos + T
    k16, v16 = _cache(case, seed)
    k, vt = k16.double(), v16.double()
    new = qkv64.view(B, T, 3, H, d)
    k[:, :, pos:L] = new[:, :, 1].permute(0, 2, 1, 3)
    vt[:, :, :, pos:L] = new[:, :, 2].permute(0, 2, 3, 1)
    slopes = _slopes(case)
    j = torch.arange(L, device=DEVICE, dtype=torch.float64)
    i = torch.arange(pos, L, device=DEVICE, dtype=torch.float64)
    dist = j[None, :] - i[:, None]                                    # key position - query position
    out = torch.empty((B, T, H, d), dtype=torch.float64, device=DEVICE)
    for b in range(B):
        for hd in range(H):
            sc = new[b, :, 0, hd] @ k[b, hd, :L].t() / math.sqrt(d)
            if slopes is not None:
                sc = sc + float(slopes[hd]) * dist
            sc = sc.masked_fill(dist > 0, float("-inf"))
            out[b, :, hd] = torch.softmax(sc, 1) @ vt[b, hd, :, :L].t()
    return out.reshape(B * T, h), k, vt


def _norm64(x, gamma, beta):
    mean, var = x.mean(1, keepdim=True), x.var(1, unbiased=False, keepdim=True)
    return (x - mean) / torch.sqrt(var + LN_EPS) * gamma.double() + beta.double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        h = case["h"]
        ln1, ln2 = _layer_norms(h, seed)

        def lin(x, name):
            K, N = _shapes(h)[name]
            return _linear64(x, _weight(N, K, seed, name), case["fmt"], _normal((N,), 0.05, seed, "bias", name))

        x = _acts(case["seqs"] * case["T"], h, seed).double()
        att, k, vt = _attention64(case, lin(_norm64(x, *ln1), "qkv"), seed)
        x = x + lin(att, "out")
        return [x + lin(_act64(lin(_norm64(x, *ln2), "fc1"), case["act"]), "fc2"), k, vt]
    if kind == "attention":
        return list(_attention64(case, _normal((case["seqs"] * case["T"], 3 * case["h"]), 1.0, seed, "qkv").double(), seed))
    if kind == "stage":
        return [_linear64(_acts(case["M"], K, seed, i, n).double(), _weight(N, K, seed, i, n), fmt)
                for i, fmt in enumerate(case["layers"].split()) for n, (K, N) in _shapes(case["h"]).items()]
    if kind == "linear":
        y = _linear64(_acts(case["M"], case["K"], seed).double(), _weight(case["N"], case["K"], seed), case["fmt"],
                      _normal((case["N"],), 0.05, seed, "bias"))
        y = _act64(y, case["act"])
        return y + _normal((case["M"], case["N"]), 1.0, seed, "res").double() if case["residual"] else y
    if kind == "quantize":
        return None                                                   # bytes and stored fp16 values: compared bit for bit
    out = []
    for n, (K, N) in _shapes(case["h"]).items():
        w, x = _weight(N, K, seed, n), _acts(case["M"], K, seed, n).double()
        g = w.view(N, K // 128, 128)
        rng = (g.amax(2).double() - g.amin(2).double()).pow(2).sum()
        lo, hi, amax = w.min().double(), w.max().double(), w.abs().amax(1).double()
        var = x.var(unbiased=False) / 4.0
        vals = [128.0 * rng / q ** 2 for q in (7.0, 15.0, 255.0)] + [K * amax.pow(2).sum() / 127.0 ** 2]
        vals += [N * K * ((hi - lo) / q) ** 2 for q in (7.0, 15.0, 255.0)] + [N * K * (amax.max() / 127.0) ** 2]
        out.append(torch.stack(vals) * var)
    return out
