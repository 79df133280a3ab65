"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Bit-exact for codes, scales, zeros, packed words and the fp32 dequantised weights; fp16 outputs
within rel-L2 <= 1e-3 and max-abs <= 1e-2 * max|ref| of the oracle's fp64 result.
Shapes span several 64x128 blocks, ragged row blocks (N not a multiple of the workgroups' 256 rows), ragged token counts, split-K, and the first configuration at full size."""
import numpy as np
import pytest

import paper_2403_01136_amd as lpq
from paper_2403_01136_amd import workloads as wl
from gpu_util import VARIANTS, VARIANT_IDS, check_output, check_packed, to_dev, u16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU (no fallback path)"
    lpq.load_library()


# ---- a1 + a2: quantise and pack ---------------------------------------------------------

@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("N,K", [(64, 128), (192, 384), (320, 1280)])
def test_quantize_pack_bit_exact(orc, bits, scheme, N, K):
    w = wl.weight_np(N, K, "qp", bits, scheme, N, K)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme)
    check_packed(qw, orc, w)
    deq = lpq.lpq_unpack_dequant(qw).cpu().numpy()
    assert np.array_equal(deq.view(np.uint32), orc.dequant_weights(w, bits, scheme).view(np.uint32))


@pytest.mark.parametrize("bits,scheme", VARIANTS[:4], ids=VARIANT_IDS[:4])
def test_quantize_pack_edge_groups(orc, bits, scheme):
    """Flat groups, -0/+0, exact grids, ranges whose fp16 scale is subnormal or underflows,
    large magnitudes: bit-equality with the oracle is all that is asked here."""
    rng = np.random.default_rng(5)
    N, K = 64, 1024
    w = wl.weight_np(N, K, "edge", bits, scheme).astype(np.float32)
    w[:, 0:128] = 0.0
    w[:, 128:256] = 0.37
    w[:, 256:384] = -0.0
    w[3, 256] = 0.0
    w[:, 384:512] = (np.arange(128) % 16) * 0.125 - 0.9375
    tiny = rng.integers(0, 40, (N, 128)).astype(np.uint16).view(np.float16).astype(np.float32)
    w[:, 512:640] = tiny                                  # fp16 subnormals: scale subnormal or zero
    w[:, 640:768] = tiny * 64 - 3e-5
    w[:, 768:896] = rng.standard_normal((N, 128)) * 2000   # large magnitudes
    w[:, 896:1024] = np.abs(w[:, 896:1024])               # all positive
    w[5, :] = 0.0                                          # a whole flat row (per-row scheme)
    w = w.astype(np.float16)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme)
    check_packed(qw, orc, w)
    deq = lpq.lpq_unpack_dequant(qw).cpu().numpy()
    assert np.array_equal(deq.view(np.uint32), orc.dequant_weights(w, bits, scheme).view(np.uint32))


# ---- quantise a weight piecewise, and stream it from host memory (Sec. 5, on-the-fly quantizer) ----

@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
def test_quantize_pack_rows_any_order(orc, bits, scheme):
    """Row windows quantised out of order, from buffers that hold only those rows, give the same packed
    weight as one call over the whole matrix (and the oracle)."""
    import torch
    N, K = 448, 384
    w = wl.weight_np(N, K, "rows", bits, scheme)
    qw = lpq.QWeight(bits, scheme, K, N, torch.device("cuda"))
    for t in (qw.codes, qw.scales, qw.zeros):
        if t is not None:
            t.view(torch.uint8).fill_(0xA5)
    for row0, n_rows in ((256, 192), (0, 64), (64, 0), (128, 128), (64, 64)):
        lpq.lpq_quantize_pack_rows(to_dev(w[row0:row0 + n_rows]), qw, row0)
    check_packed(qw, orc, w)


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("pinned", [True, False], ids=["pinned", "pageable"])
def test_load_quantize_pack_from_host(orc, bits, scheme, pinned):
    """Streaming from host memory through a staging buffer (several bands of rows, a ragged last one) is
    bit-identical to quantising the resident weight; then the linear runs on the result."""
    import torch
    N, K, M = 704, 256, 8
    w = wl.weight_np(N, K, "load", bits, scheme)
    w_host = torch.from_numpy(w.copy())
    if pinned:
        w_host = w_host.pin_memory()
    staging = torch.empty(192 * K * 2 + 300, dtype=torch.uint8, device="cuda")          # 192-row bands: 3 full + 128 rows
    qw = lpq.lpq_load_quantize_pack(w_host, bits, scheme, staging)
    torch.cuda.synchronize()
    check_packed(qw, orc, w)
    x = wl.act_np(M, K, True, "load", M)
    check_output(lpq.lpq_qlinear_decode(qw, to_dev(x)), orc.qlinear(x, w, bits, scheme), "decode after load %d-bit" % bits)


# ---- a3: decode linear ---------------------------------------------------------------------

@pytest.fixture(params=["rows", "rows_3", "rows_5", "even_share"])
def decode_kernel_choice(request):
    """Up to 64 token rows, a launch that streams little goes to the kernels that give a workgroup a group of 16-row tiles (up to 16
    rows) or a few 64-row blocks, a larger one to the even-share kernel; lpq_set_decode_routing moves the limit, so small shapes
    can reach both.  rows_3 / rows_5 ask for groups of 3 / 5 tiles (up to 16 rows), which cut across the packed layout's 64-row blocks (the library
    falls back to 4 where the group size does not divide a linear's tiles: N = 320 has 20, N = 192 has 12)."""
    if request.param == "even_share":
        lpq.lpq_set_decode_routing(0, 0)
    elif request.param != "rows":
        lpq.lpq_set_decode_routing(-1, int(request.param[-1]))
    yield request.param
    lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M", [1, 2, 5, 16, 17, 32, 33, 64])
def test_decode_small(orc, bits, scheme, M, decode_kernel_choice):
    if M > 64 and decode_kernel_choice != "even_share":
        pytest.skip("more than 64 token rows always take the even-share kernel")
    N, K = 320, 640         # 5 (fp16: 10) row blocks: the last workgroup has idle waves; 5 steps: idle waves in a row block's workgroup
    w = wl.weight_np(N, K, "dec", bits, scheme)
    x = wl.act_np(M, K, True, "dec", M)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme)
    y = lpq.lpq_qlinear_decode(qw, to_dev(x))
    check_output(y, orc.qlinear(x, w, bits, scheme), "decode %d-bit M=%d" % (bits, M))


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M", [3, 21, 70, 130])
def test_decode_split_k_and_many_rows(orc, bits, scheme, M, decode_kernel_choice):
    """K long enough that the work is cut into several K ranges (fp32 partial sums + reduction, or waves that split
    K); M > 64 runs in several passes; a bias is added exactly once."""
    if M > 64 and decode_kernel_choice != "even_share":
        pytest.skip("more than 64 token rows always take the even-share kernel")
    N, K = 192, 16384
    w = wl.weight_np(N, K, "decsk", bits, scheme)
    x = wl.act_np(M, K, True, "decsk", M)
    bias = (np.arange(N) % 7 - 3).astype(np.float16)
    import torch
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    lpq.lpq_qlinear_decode(qw, to_dev(x), y)
    check_output(y, orc.qlinear(x, w, bits, scheme, bias), "decode split-K %d-bit M=%d" % (bits, M))


@pytest.mark.parametrize("bits,scheme", [(3, 1), (4, 1), (8, 1), (8, 2)], ids=["w3", "w4", "w8", "i8sym"])
def test_decode_zero_term_rows_of_unlike_magnitude(orc, bits, scheme):
    """Up to 32 token rows the stage-wide kernel adds the zero term once per unit, as a matrix product with the activations'
    group sums held as fp16 pairs scaled per token row.  Rows 2^-11 and 2^5 times the others in one micro-batch: every row
    keeps the tolerance on its own, whatever its neighbours' scale."""
    lpq.lpq_set_decode_routing(0, 0)
    try:
        N, K = 192, 2048
        w = wl.weight_np(N, K, "zrow", bits, scheme)
        for M in (7, 24):
            x = wl.act_np(M, K, False, "zrow", M).astype(np.float32)
            x *= np.array([2.0 ** -11, 1.0, 2.0 ** 5])[np.arange(M) % 3][:, None]
            x = x.astype(np.float16)
            y = lpq.lpq_qlinear_decode(lpq.lpq_quantize_pack(to_dev(w), bits, scheme), to_dev(x))
            ref = orc.qlinear(x, w, bits, scheme)
            for m in range(M):
                check_output(y[m:m + 1], ref[m:m + 1], "decode %d-bit M=%d row %d" % (bits, M, m))
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("bits,scheme", [(3, 1), (8, 2)], ids=["w3", "i8sym"])
def test_decode_zero_term_very_long_rows(orc, bits, scheme):
    """K = 66048 is 516 groups: more than a thread of the group-sum kernel keeps in registers, so it reads the row twice;
    the 516 groups are also not a multiple of the 16 a matrix instruction of the zero term covers."""
    lpq.lpq_set_decode_routing(0, 0)
    try:
        N, K = 128, 66048
        w = wl.weight_np(N, K, "zlong", bits, scheme)
        for M in (3, 18):
            x = wl.act_np(M, K, True, "zlong", M)
            y = lpq.lpq_qlinear_decode(lpq.lpq_quantize_pack(to_dev(w), bits, scheme), to_dev(x))
            check_output(y, orc.qlinear(x, w, bits, scheme), "decode %d-bit M=%d K=%d" % (bits, M, K))
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("bits,scheme", [(3, 1), (8, 2)], ids=["w3", "i8"])
def test_decode_longest_rows_and_the_limit_on_k(orc, bits, scheme):
    """The decode kernels' descriptors keep K / 128 in 16 bits.  At the largest K they hold (65535 steps of 128 columns)
    one-hot activation rows read single columns of the dequantised weight out of the product -- first, last and middle
    groups -- and each is compared with the oracle on that group's 128 columns alone (quantisation is per group);
    one step more is refused with LPQ_ERR_UNSUPPORTED and nothing is written."""
    import torch
    N, KT = 64, 65535
    K = KT * 128
    gen = torch.Generator(device="cuda").manual_seed(23)
    w = torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16)
    qw = lpq.lpq_quantize_pack(w, bits, scheme)
    cols = [0, 127, 128, 5 * 128 + 77, (KT // 2) * 128 + 3, (KT - 1) * 128, K - 1]
    x = torch.zeros((len(cols), K), dtype=torch.float16, device="cuda")
    for i, c in enumerate(cols):
        x[i, c] = 1.0 + i / 8.0
    y = lpq.lpq_qlinear_decode(qw, x)
    torch.cuda.synchronize()
    y_host = y.cpu().numpy().astype(np.float64)
    for i, c in enumerate(cols):
        g = c // 128
        if scheme == 2:      # one scale per row over the whole of K: the oracle needs the row's largest magnitude, kept in a 129th group
            wmax = w.abs().amax(dim=1, keepdim=True)
            wg = torch.cat([w[:, g * 128:(g + 1) * 128], wmax.expand(N, 128)], dim=1).cpu().numpy()
            xg = np.zeros((1, 256), dtype=np.float16)
        else:
            wg = w[:, g * 128:(g + 1) * 128].cpu().numpy()
            xg = np.zeros((1, 128), dtype=np.float16)
        xg[0, c % 128] = np.float16(1.0 + i / 8.0)
        ref = orc.qlinear(xg, wg, bits, scheme)
        check_output(torch.from_numpy(y_host[i:i + 1]), ref, "decode %d-bit K=%d, column %d" % (bits, K, c))
    del qw, w, x, y
    K2 = K + 128
    w2 = torch.zeros((N, K2), dtype=torch.float16, device="cuda")
    qw2 = lpq.lpq_quantize_pack(w2, bits, scheme)
    x2 = torch.zeros((2, K2), dtype=torch.float16, device="cuda")
    y2 = torch.full((2, N), float("nan"), dtype=torch.float16, device="cuda")
    with pytest.raises(lpq.LpqError) as err:
        lpq.lpq_qlinear_decode(qw2, x2, y2)
    assert err.value.status == 8
    torch.cuda.synchronize()
    assert torch.isnan(y2).all(), "a refused call wrote outputs"


# ---- a4: prefill linear --------------------------------------------------------------------

@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M", [1, 7, 128, 130, 300])
def test_prefill_small(orc, bits, scheme, M):
    N, K = 320, 640         # 5 row blocks: the second workgroup has one active wave
    w = wl.weight_np(N, K, "pre", bits, scheme)
    x = wl.act_np(M, K, True, "pre", M)
    bias = (np.arange(N) % 5 - 2).astype(np.float16) if M == 7 else None
    import torch
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=None if bias is None else to_dev(bias))
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    lpq.lpq_qlinear_prefill(qw, to_dev(x), y)
    check_output(y, orc.qlinear(x, w, bits, scheme, bias), "prefill %d-bit M=%d" % (bits, M))


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M,K", [(7, 8192), (260, 8192), (300, 4224)])
def test_prefill_split_k(orc, bits, scheme, M, K):
    """Few tiles and a long K: the library cuts K into ranges (fp32 partial sums, second kernel).  K = 4224 is
    33 steps, which no split count divides; the bias is added exactly once."""
    N = 320
    w = wl.weight_np(N, K, "presk", bits, scheme)
    x = wl.act_np(M, K, True, "presk", M)
    bias = (np.arange(N) % 5 - 2).astype(np.float16)
    import torch
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    lpq.lpq_qlinear_prefill(qw, to_dev(x), y)
    check_output(y, orc.qlinear(x, w, bits, scheme, bias), "prefill split-K %d-bit M=%d" % (bits, M))


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("mag", [2.0 ** -12, 2.0 ** -6, 2.0 ** 5], ids=["x_2e-12", "x_2e-6", "x_2e5"])
def test_activation_magnitude(orc, bits, scheme, mag, decode_kernel_choice):
    """The tolerance holds whatever the scale of the activations (tiny ones near the fp16 subnormal
    range, large ones short of overflow in the outputs): no step of the kernels may cost them bits."""
    if decode_kernel_choice in ("rows_3", "rows_5"):
        pytest.skip("N = 128 has 8 tiles: groups of 3 or 5 do not apply")
    N, K = 128, 512
    w = wl.weight_np(N, K, "mag", bits, scheme)
    for M, fn, tag in [(8, lpq.lpq_qlinear_decode, "decode"), (40, lpq.lpq_qlinear_decode, "decode"),
                       (64, lpq.lpq_qlinear_prefill, "prefill")]:
        x = (wl.act_np(M, K, False, "mag", M).astype(np.float32) * mag).astype(np.float16)
        y = fn(lpq.lpq_quantize_pack(to_dev(w), bits, scheme), to_dev(x))
        check_output(y, orc.qlinear(x, w, bits, scheme), "%s %d-bit M=%d x*%g" % (tag, bits, M, mag))


RANDOM_SHAPES = [(N, K, M, v) for i, (N, K, M) in enumerate([
    (192, 4096, 1), (320, 1024, 7), (960, 384, 16), (1280, 1024, 19), (1600, 128, 32), (2048, 2048, 45), (960, 4096, 64),
    (1280, 384, 5), (320, 4096, 27), (1600, 1024, 16), (2048, 128, 3), (192, 2048, 33)]) for v in [VARIANTS[i % len(VARIANTS)]]]


@pytest.mark.parametrize("N,K,M,variant", RANDOM_SHAPES, ids=["N%d_K%d_M%d_%s" % (N, K, M, VARIANT_IDS[VARIANTS.index(v)]) for N, K, M, v in RANDOM_SHAPES])
def test_decode_shapes_that_vary_the_workgroup_plan(orc, N, K, M, variant):
    """A single decode linear picks its workgroup shape from N, K and M (groups of 2-5 tiles, K splits, one or two
    token tiles, one or two passes): shapes whose tile counts divide by 3 or 5 or neither, long and one-step K,
    every range of M, with a bias and a residual, every element against the oracle."""
    import torch
    bits, scheme = variant
    w = wl.weight_np(N, K, "plan", N, K, bits, scheme)
    x = wl.act_np(M, K, True, "plan", N, K, M)
    bias = ((np.arange(N) % 5) - 2).astype(np.float16) * np.float16(0.5)
    res = wl.act_np(M, N, False, "plan-res", N, K, M)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    lpq.lpq_qlinear_fused(qw, to_dev(x), lpq.LPQ_DECODE, residual=to_dev(res), y=y)
    ref = orc.qlinear(x, w, bits, scheme, bias) + res.astype(np.float64)
    check_output(y, ref, "decode N=%d K=%d M=%d %d-bit" % (N, K, M, bits))


def test_decode_and_prefill_agree_and_are_deterministic(orc):
    N, K, M = 128, 2048, 24
    w = wl.weight_np(N, K, "agree")
    x = to_dev(wl.act_np(M, K, True, "agree"))
    qw = lpq.lpq_quantize_pack(to_dev(w), 4, 1)
    yd1, yd2 = lpq.lpq_qlinear_decode(qw, x), lpq.lpq_qlinear_decode(qw, x)
    yp1, yp2 = lpq.lpq_qlinear_prefill(qw, x), lpq.lpq_qlinear_prefill(qw, x)
    assert np.array_equal(u16(yd1), u16(yd2)) and np.array_equal(u16(yp1), u16(yp2))
    ref = orc.qlinear(x.cpu().numpy(), w, 4, 1)
    check_output(yd1, ref, "decode")
    check_output(yp1, ref, "prefill")


# ---- a5: stage of layers with per-layer bits -----------------------------------------------

def _build_stage(cfg_key, h, f, qkv_n, layer_specs, M, outliers):
    import torch
    shapes = {"qkv": (h, qkv_n), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}
    layers, xs, ys, host = [], [], [], []
    for li, (bits, scheme) in enumerate(layer_specs):
        lw, lx, ly, lh = {}, {}, {}, {}
        x_h = wl.act_np(M, h, outliers, cfg_key, li, "h")
        x_f = wl.act_np(M, f, outliers, cfg_key, li, "f")
        xd_h, xd_f = to_dev(x_h), to_dev(x_f)
        for name, (K, N) in shapes.items():
            w = wl.weight_np(N, K, cfg_key, li, name)
            lw[name] = lpq.lpq_quantize_pack(to_dev(w), bits, scheme)
            lx[name] = xd_f if name == "fc2" else xd_h
            ly[name] = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            lh[name] = (w, x_f if name == "fc2" else x_h)
        layers.append(lw), xs.append(lx), ys.append(ly), host.append(lh)
    return lpq.Stage(layers, xs, ys), ys, host


@pytest.mark.parametrize("phase,M", [(lpq.LPQ_DECODE, 1), (lpq.LPQ_DECODE, 16), (lpq.LPQ_DECODE, 24), (lpq.LPQ_DECODE, 40),
                                     (lpq.LPQ_PREFILL, 128)],
                         ids=["decode_M1", "decode_M16", "decode_M24", "decode_M40", "prefill_M128"])
def test_stage_mixed_bits_small(orc, phase, M, decode_kernel_choice):
    if decode_kernel_choice in ("rows_3", "rows_5"):
        pytest.skip("the stage's linears have 16, 48 and 64 tiles: no group of 3 or 5 fits them all")
    specs = [(16, 0), (8, 1), (4, 1), (3, 1), (8, 2), (3, 1)]
    stage, ys, host = _build_stage("stage_small", 256, 1024, 768, specs, M, True)
    lpq.lpq_stage_linears(stage, phase)
    for li, (bits, scheme) in enumerate(specs):
        for name in wl.LINEARS:
            w, x = host[li][name]
            check_output(ys[li][name], orc.qlinear(x, w, bits, scheme), "layer %d %s" % (li, name))


@pytest.mark.parametrize("phase,M", [(lpq.LPQ_DECODE, 3), (lpq.LPQ_DECODE, 20), (lpq.LPQ_DECODE, 70), (lpq.LPQ_PREFILL, 130), (lpq.LPQ_PREFILL, 300)],
                         ids=["decode_M3", "decode_M20", "decode_M70", "prefill_M130", "prefill_M300"])
def test_stage_with_more_linears_than_one_launch_holds(orc, phase, M, decode_kernel_choice):
    """A stage of 13 layers = 52 linears: a grouped decode launch holds at most 48, so the decode phase takes two
    launches that share the workspace, and a storage variant with more than 40 linears takes two prefill launches
    (here the 4-bit variant has 44).  Every element of every output is checked."""
    if decode_kernel_choice in ("rows_3", "rows_5"):
        pytest.skip("the stage's linears have 16, 32 and 48 tiles: no group of 3 or 5 fits them all")
    specs = [(4, 1)] * 11 + [(3, 1)] * 2
    stage, ys, host = _build_stage("stage_52", 256, 512, 768, specs, M, True)
    lpq.lpq_stage_linears(stage, phase)
    for li, (bits, scheme) in enumerate(specs):
        for name in wl.LINEARS:
            w, x = host[li][name]
            check_output(ys[li][name], orc.qlinear(x, w, bits, scheme), "layer %d %s" % (li, name))


@pytest.mark.parametrize("phase", [lpq.LPQ_DECODE, lpq.LPQ_PREFILL], ids=["decode", "prefill"])
def test_config0_full(orc, phase):
    """First configuration at full size: one OPT-125m-shaped layer, 4-bit grouped, decode M = 1 and
    prefill M = 128; packed data bit-exact, every output element compared."""
    cfg = wl.CONFIGS[0]
    M = cfg["decode_Ms"][0] if phase == lpq.LPQ_DECODE else cfg["prefill_M"]
    stage, ys, host = _build_stage(cfg["name"], cfg["h"], cfg["f"], cfg["qkv_n"], cfg["layers"], M, cfg["act_outliers"])
    for name in wl.LINEARS:
        check_packed(stage.keep[0][0][name], orc, host[0][name][0])
    lpq.lpq_stage_linears(stage, phase)
    bits, scheme = cfg["layers"][0]
    for name in wl.LINEARS:
        w, x = host[0][name]
        check_output(ys[0][name], orc.qlinear(x, w, bits, scheme), name)


@pytest.mark.parametrize("bits,scheme", [(3, 1), (4, 1), (8, 1), (8, 2), (16, 0)], ids=["w3", "w4", "w8", "i8", "f16"])
@pytest.mark.parametrize("K,N", [(128, 64), (384, 320), (4736, 192), (1152, 1088)])
def test_decode_17_to_64_rows_edges(orc, bits, scheme, K, N):
    """The kernel for 17-64 token rows at the edges of its token tiles, with row blocks that do not fill a workgroup, fewer steps of K than
    an iteration holds, steps that do not fill the last one, ranges of K over several workgroups (reduced by a second kernel) and one,
    with bias, activation and a residual in place.  Tolerances: the file's."""
    import torch
    w = wl.weight_np(N, K, "mid", bits, scheme)
    r = np.random.default_rng(wl.stream_seed("mid", K, N))
    bias = (0.1 * r.standard_normal(N)).astype(np.float16)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    x = wl.act_np(64, K, True, "mid", K)
    res = r.standard_normal((64, N)).astype(np.float16)
    ref = np.maximum(orc.qlinear(x, w, bits, scheme, bias), 0.0) + res.astype(np.float64)
    for M in (17, 31, 32, 33, 48, 49, 63, 64):
        y = to_dev(res[:M]).clone()
        lpq.lpq_qlinear_fused(qw, to_dev(x[:M]), lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU, residual=y, y=y)
        check_output(y, ref[:M], "decode %d rows, %d bits, %d -> %d" % (M, bits, K, N))


@pytest.mark.parametrize("M", [12, 13, 16])
@pytest.mark.parametrize("bits,scheme", [(3, 1), (8, 2), (16, 0)], ids=["w3", "i8", "f16"])
def test_decode_13_to_16_rows_without_a_split(orc, bits, scheme, M):
    """A single wide linear of a short K: from 13 rows on it changes kernels (no split of K needed)."""
    K, N = 384, 64 * 237
    w = wl.weight_np(N, K, "mid16", bits)
    x = wl.act_np(M, K, False, "mid16", M)
    y = lpq.lpq_qlinear_decode(lpq.lpq_quantize_pack(to_dev(w), bits, scheme), to_dev(x))
    check_output(y, orc.qlinear(x, w, bits, scheme), "decode %d rows" % M)


@pytest.mark.parametrize("M", [20, 40, 60])
def test_decode_17_to_64_rows_stage_of_unlike_linears(orc, M):
    """One launch of two layers in two formats whose linears have different K (different numbers of splits), against the even-share kernel's
    route on the same buffers and the oracle."""
    import torch
    h, f = 256, 1536
    shapes = {"qkv": (h, 3 * h), "out": (h, h), "fc1": (h, f), "fc2": (f, h)}
    host = [{n: wl.weight_np(N, K, "mid-stage", i, n) for n, (K, N) in shapes.items()} for i in range(2)]
    layers = [{n: lpq.lpq_quantize_pack(to_dev(w), b, s) for n, w in host[i].items()} for i, (b, s) in enumerate([(3, 1), (8, 2)])]
    xh = [{n: wl.act_np(M, K, False, "mid-stage", i, n, M) for n, (K, N) in shapes.items()} for i in range(2)]
    xs = [{n: to_dev(x) for n, x in d.items()} for d in xh]
    for route in (-1, 0):
        ys = [{n: torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for n, (K, N) in shapes.items()} for _ in range(2)]
        lpq.lpq_set_decode_routing(route, 0)
        try:
            lpq.lpq_stage_linears(lpq.Stage(layers, xs, ys), lpq.LPQ_DECODE)
        finally:
            lpq.lpq_set_decode_routing(-1, -1)
        for i, (b, s) in enumerate([(3, 1), (8, 2)]):
            for n in shapes:
                check_output(ys[i][n], orc.qlinear(xh[i][n], host[i][n], b, s), "stage layer %d %s route %d" % (i, n, route))


@pytest.mark.parametrize("bits,scheme", [(4, 1), (8, 2), (16, 0)], ids=["w4", "i8", "f16"])
@pytest.mark.parametrize("M,N,K", [(700, 23104, 2048), (1191, 14912, 2048), (100, 71744, 2048), (256, 320, 4224), (300, 1088, 3200), (300, 1088, 8192), (300, 4160, 8192), (700, 2880, 4096)])
def test_prefill_whole_and_split_tiles(orc, bits, scheme, M, N, K):
    """Linears with more tiles than the chip has compute units but fewer than twice as many (full rounds of whole tiles, the rest split over
    K: the border runs through a row block when the token blocks do not divide it), and with fewer (all split), N that is no multiple of
    256 and ragged token blocks: every output written exactly once; 256 tokens to a tile, and 128 (100 rows).  Activations below and above 4 MB, fewer and more than 32
    tiles, where the order of the work units changes, with up to two token blocks and more.  Every output against an fp32 product of the dequantised weights
    (both sides round fp32 sums once: the file's tolerance), the rows around the border and the last ones against the oracle."""
    import torch
    kernel, tile, splits, whole = lpq.lpq_route_of([(bits, scheme, K, N)], lpq.LPQ_PREFILL, M)
    assert kernel == lpq.LPQ_ROUTE_PREFILL and tile == (128 if M <= 128 else 256) and splits > 1 and (whole > 0) == (N > 10000)
    gen = torch.Generator(device="cuda").manual_seed(N + bits)
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.02).half()
    x = torch.randn((M, K), generator=gen, device="cuda").half()
    qw = lpq.lpq_quantize_pack(w, bits, scheme)
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    lpq.lpq_qlinear_prefill(qw, x, y)
    ref = x.float() @ lpq.lpq_unpack_dequant(qw).t()
    d = (y.float() - ref).double()
    assert torch.isfinite(y).all()
    assert float(d.norm() / ref.double().norm()) <= 1e-3 and float(d.abs().max()) <= 1e-2 * float(ref.abs().max())
    border = 256 * (256 // ((M + 255) // 256)) if M > 128 else 256 * 256
    rows = sorted({min(max(r, 0), N - 64) // 64 * 64 for r in (0, border - 64, border, border + 256, N - 64)})
    for r0 in rows:
        check_output(y[:, r0:r0 + 64], orc.qlinear(x.cpu().numpy(), w[r0:r0 + 64].cpu().numpy(), bits, scheme), "rows %d.. of %d" % (r0, N))


@pytest.mark.parametrize("phase", [lpq.LPQ_PREFILL, lpq.LPQ_DECODE], ids=["prefill", "decode"])
@pytest.mark.parametrize("K,N", [(20480, 5120), (57344, 14336)])
def test_symmetric_weights_with_activations_of_one_sign(phase, K, N):
    """The second feed-forward linear's input is a ReLU's output.  Per-row symmetric 8-bit codes are multiplied as signed integers by
    every prefill call and from 17 decode rows on, so no sums cancel and the error against 64 bits is that of the one rounding to
    fp16: uniform within half an ulp, an ulp between 2^-11 and 2^-10 of the value, so at most 2^-11 / sqrt(3) = 2.82e-4 in the 2-norm.
    The 32-bit sums' share is under 1e-5: 3e-4.  Decode launches of up to 16 rows multiply offset codes and are not part of this."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(K)
    w = (torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16) * 0.02)
    flat = w.view(-1)
    flat[torch.randint(0, flat.numel(), (flat.numel() // 1000,), generator=gen, device="cuda")] *= 20.0
    qw = lpq.lpq_quantize_pack(w, 8, lpq.LPQ_SYM_CHANNEL)
    rows = torch.arange(0, N, 37, device="cuda")
    scale = qw.scales[rows].double()[:, None]
    deq = torch.clamp(torch.round(w[rows].float() / qw.scales[rows].float()[:, None]), -127, 127).double() * scale
    for M in (9, 20, 40, 64):
        if phase == lpq.LPQ_DECODE and M <= 16:
            continue
        z = torch.randn((M, K), generator=gen, device="cuda")
        for name, x in (("relu", torch.relu(z).half()), ("shifted", (z + 3.0).half())):
            y = lpq.lpq_qlinear_fused(qw, x, phase)[:, rows].double()
            ref = x.double() @ deq.t()
            rel = float((y - ref).norm() / ref.norm())
            assert rel <= 3e-4, "%d rows, %s: %.2e" % (M, name, rel)


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("phase,M", [(lpq.LPQ_PREFILL, 5), (lpq.LPQ_PREFILL, 16), (lpq.LPQ_PREFILL, 30), (lpq.LPQ_PREFILL, 64),
                                     (lpq.LPQ_PREFILL, 100), (lpq.LPQ_DECODE, 40), (lpq.LPQ_DECODE, 64)])
def test_infinite_activations(phase, M, bits, scheme):
    """An infinite activation makes its token's outputs infinite with the dequantised weight's sign (NaN where infinities of both signs or
    a zero weight meet), whichever kernel a prefill call takes, and in decode calls of 33 to 64 rows; the other tokens' outputs
    are the same bits as without it.  Weights are kept away from zero, where rounding to fp16 would decide."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M + bits)
    N, K = 320, 2304
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    w = (w + 0.01 * torch.sign(w)).half()
    qw = lpq.lpq_quantize_pack(w, bits, scheme)
    x = torch.randn((M, K), generator=gen, device="cuda").half()
    plain = lpq.lpq_qlinear_fused(qw, x, phase)
    deq = lpq.lpq_unpack_dequant(qw)
    inf = float("inf")
    x[0, 1000] = inf
    x[M - 1, 2303], x[M - 1, 0] = -inf, -inf
    x[M // 2, 130] = float("nan")
    y = lpq.lpq_qlinear_fused(qw, x, phase)
    keep = torch.ones(M, dtype=torch.bool, device="cuda")
    keep[[0, M // 2, M - 1]] = False
    assert torch.equal(y[keep], plain[keep]), "a token without infinities changed"
    assert torch.isnan(y[M // 2]).all()
    sure = (deq[:, [0, 1000, 2303]].abs() > 1e-4).all(1)
    assert int(sure.sum()) > N // 2
    assert torch.equal(y[0, sure].float(), (torch.sign(deq[:, 1000]) * inf)[sure])
    a, b = deq[sure, 0], deq[sure, 2303]
    both = torch.where(torch.sign(a) == torch.sign(b), -torch.sign(a) * inf, torch.full_like(a, float("nan")))
    assert torch.equal(torch.nan_to_num(y[M - 1, sure].float(), nan=3.0), torch.nan_to_num(both, nan=3.0))


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("K,N", [(128, 64), (256, 960)])
def test_decode_17_to_32_rows_of_few_columns(orc, bits, scheme, K, N):
    """One or two groups of columns: the kernel for up to 16 rows, in two workgroups of 16 rows each, with bias, activation and a residual in place."""
    r = np.random.default_rng(wl.stream_seed("short", K, N))
    w, x, res = wl.weight_np(N, K, "short", bits), wl.act_np(32, K, True, "short", K), r.standard_normal((32, N)).astype(np.float16)
    bias = (0.1 * r.standard_normal(N)).astype(np.float16)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    ref = np.maximum(orc.qlinear(x, w, bits, scheme, bias), 0.0) + res.astype(np.float64)
    for phase in (lpq.LPQ_DECODE, lpq.LPQ_PREFILL):
        for M in (17, 31, 32):
            assert lpq.lpq_route_of([(bits, scheme, K, N)], phase, M)[0] == lpq.LPQ_ROUTE_ROWS
            y = to_dev(res[:M]).clone()
            lpq.lpq_qlinear_fused(qw, to_dev(x[:M]), phase, activation=lpq.LPQ_ACT_RELU, residual=y, y=y)
            check_output(y, ref[:M], "%d rows, %d bits, %d -> %d" % (M, bits, K, N))


def _prefill_reference(qw, x, bias):
    """The dequantised weights times x, in 64 bits on the GPU."""
    return (x.double() @ lpq.lpq_unpack_dequant(qw).double().t() + bias.double()).cpu().numpy()


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M", [65, 100, 127])
@pytest.mark.parametrize("N,K", [(320, 640), (320, 8192), (320, 4224)])
def test_prefill_128_token_tiles(orc, bits, scheme, M, N, K):
    """65 to 127 rows, the ragged 128-token tile: whole, split over K (two numbers of steps, one that no split count divides), a bias added once."""
    kernel, tile, splits, _ = lpq.lpq_route_of([(bits, scheme, K, N)], lpq.LPQ_PREFILL, M)
    assert (kernel, tile) == (lpq.LPQ_ROUTE_PREFILL, 128) and (splits > 1) == (K > 2048)
    w, x = wl.weight_np(N, K, "pre128", bits, scheme), wl.act_np(M, K, True, "pre128", M)
    bias = (np.arange(N) % 5 - 2).astype(np.float16)
    y = lpq.lpq_qlinear_prefill(lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias)), to_dev(x))
    check_output(y, orc.qlinear(x, w, bits, scheme, bias), "prefill %d rows" % M)


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M,N,K", [(1, 320, 640), (7, 320, 8192), (24, 320, 640), (40, 192, 4224), (64, 320, 640)])
def test_prefill_kernels_up_to_64_rows(orc, bits, scheme, M, N, K):
    """Calls of few rows that keep the prefill kernels (launches past the line of the decode kernels, longer lists of linears, no workspace):
    reached by turning those kernels off.  Activations from 2^-12 to 2^5."""
    w = wl.weight_np(N, K, "pre64", bits, scheme)
    bias = (np.arange(N) % 5 - 2).astype(np.float16)
    qw = lpq.lpq_quantize_pack(to_dev(w), bits, scheme, bias=to_dev(bias))
    lpq.lpq_set_decode_routing(0, 0)
    try:
        assert lpq.lpq_route_of([(bits, scheme, K, N)], lpq.LPQ_PREFILL, M)[0] == lpq.LPQ_ROUTE_PREFILL
        for mag in (2.0 ** -12, 1.0, 2.0 ** 5):
            x = (wl.act_np(M, K, False, "pre64", M).astype(np.float32) * mag).astype(np.float16)
            y = lpq.lpq_qlinear_prefill(qw, to_dev(x))
            check_output(y, orc.qlinear(x, w, bits, scheme, bias), "prefill %d rows x*%g" % (M, mag))
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("bits,scheme", VARIANTS, ids=VARIANT_IDS)
@pytest.mark.parametrize("M", [100, 300])
def test_prefill_layer_split_over_k(bits, scheme, M):
    """The four linears of a layer in one launch of few tiles: ranges of K of about one length for all, the long second feed-forward linear
    in several, the others in one or two."""
    import torch
    h, f = 1088, 4352                                     # no multiples of 256
    gen = torch.Generator(device="cuda").manual_seed(M + bits)
    shapes = {"qkv": (1152, 3 * h), "out": (1152, h), "fc1": (1152, f), "fc2": (f, h)}
    layer, xs, ys, ref = {}, {}, {}, {}
    for n, (K, N) in shapes.items():
        bias = torch.randn((N,), generator=gen, device="cuda").half()
        layer[n] = lpq.lpq_quantize_pack((torch.randn((N, K), generator=gen, device="cuda") * 0.02).half(), bits, scheme, bias=bias)
        xs[n] = torch.randn((M, K), generator=gen, device="cuda").half()
        ys[n] = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        ref[n] = _prefill_reference(layer[n], xs[n], bias)
    lpq.lpq_stage_linears(lpq.Stage([layer], [xs], [ys]), lpq.LPQ_PREFILL)
    for n in shapes:
        check_output(ys[n], ref[n], "%s, %d rows" % (n, M))


MID_FORMS = [(16, 1, False, 1408, 2496), (16, 1, True, 2432, 3200), (16, 2, False, 1152, 16448), (16, 2, True, 2432, 448), (16, 4, False, 1152, 32832),
             (16, 4, True, 2432, 64), (24, 1, False, 1152, 2496), (24, 1, True, 1152, 64), (24, 2, False, 1152, 16448), (24, 2, True, 14464, 6208),
             (24, 4, False, 1152, 32832), (24, 4, True, 9344, 16448), (40, 2, False, 1152, 8256), (40, 2, True, 1152, 64), (40, 4, False, 1152, 32832),
             (40, 4, True, 9344, 16448), (60, 2, False, 1152, 8256), (60, 2, True, 1152, 64), (60, 4, False, 1152, 32832), (60, 4, True, 9344, 16448)]


@pytest.mark.parametrize("M,blocks,split,K,N", MID_FORMS, ids=["M%d_rb%d_%s" % (c[0], c[1], "split" if c[2] else "whole") for c in MID_FORMS])
@pytest.mark.parametrize("bits,scheme", [(3, 1), (4, 1), (8, 2), (16, 0)], ids=["w3", "w4", "i8", "fp16"])
def test_decode_mid_kernel_forms(bits, scheme, M, blocks, split, K, N):
    """Every form of the kernel for 17-64 rows (13-16 too): 1, 2 and 4 row blocks per workgroup at 1 to 4 token tiles, with and without K splits,
    over several iterations of its loop with a ragged last one, and row blocks that do not fill the last workgroup; bias, activation
    and a residual in place.  Against the dequantised weights in 64 bits."""
    import torch
    kernel, got_blocks, splits, _ = lpq.lpq_route_of([(bits, scheme, K, N)], lpq.LPQ_DECODE, M)
    if M == 16 and kernel != lpq.LPQ_ROUTE_MID:
        pytest.skip("this format stays with the kernel for up to 16 rows here")
    assert kernel == lpq.LPQ_ROUTE_MID and (got_blocks, splits > 1) == (blocks, split)
    gen = torch.Generator(device="cuda").manual_seed(K + N + bits)
    w = (torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16) * 0.02)
    bias = torch.randn((N,), generator=gen, device="cuda").half()
    x, res = torch.randn((M, K), generator=gen, device="cuda").half(), torch.randn((M, N), generator=gen, device="cuda").half()
    qw = lpq.lpq_quantize_pack(w, bits, scheme, bias=bias)
    ref = np.maximum(_prefill_reference(qw, x, bias), 0.0) + res.double().cpu().numpy()
    y = res.clone()
    lpq.lpq_qlinear_fused(qw, x, lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU, residual=y, y=y)
    check_output(y, ref, "%d rows, %d -> %d" % (M, K, N))


@pytest.fixture
def even_share():
    """Launches that stream little go to the even-share kernel too."""
    lpq.lpq_set_decode_routing(0, 0)
    yield
    lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("bits", [3, 4], ids=["w3", "w4"])
@pytest.mark.parametrize("size", [300.0, 1000.0, 10000.0, 60000.0])
def test_decode_beside_large_activations(bits, size, even_share):
    """Activations are read as they are, whatever stands next to them: one element of each row is up to 60000 times the others, in a column whose
    weights are zero in W and in W~, so that the outputs are made of the others alone.  Against 64 bits, row by row: the rounding of the output (2.1e-4 of
    it) and, in calls of 33 rows and more, that of the weights to fp16 (1.7e-4), 2.7e-4 together; 4e-4 leaves room for sums of 1152 terms in 32 bits."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(bits)
    K, N = 1152, 1088
    col = torch.arange(64, device="cuda") * 17 % K                                        # every place of a lane's 32 columns
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.02).abs().half()           # a group's least weight is the 0 there
    w[:, col] = 0.0
    qw = lpq.lpq_quantize_pack(w, bits, lpq.LPQ_ASYM_GROUP)
    deq = lpq.lpq_unpack_dequant(qw).double()
    assert float(deq[:, col].abs().max()) == 0.0
    x = torch.randn((64, K), generator=gen, device="cuda").half()
    x[torch.arange(64, device="cuda"), col] = size
    ref = x.double() @ deq.t()
    for M in (8, 24, 33, 48, 64):
        assert lpq.lpq_route_of([(bits, lpq.LPQ_ASYM_GROUP, K, N)], lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
        y = lpq.lpq_qlinear_decode(qw, x[:M]).double()
        err = (y - ref[:M]).norm(dim=1) / ref[:M].norm(dim=1)
        assert float(err.max()) <= 4e-4, "%d rows: row %d off by %.2e" % (M, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("bits", [3, 4, 8], ids=["w3", "w4", "w8"])
@pytest.mark.parametrize("size", [1000.0, 60000.0])
@pytest.mark.parametrize("K", [128, 1152])
def test_decode_33_to_64_rows_beside_large_activations_on_codes_that_are_not_zero(bits, size, K, even_share):
    """As above, 33 rows and more, where the large element's weights are zero in W~ only as scale * code + zero: groups are symmetric about zero.  The weights lie on
    the grid, so that W~ = W exactly and the output's rounding (2.1e-4) is all there is, but for sums of 1152 terms in 32 bits: 3e-4."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(bits + K)
    N, top, mid, scale = 1088, 2 ** bits - 1, 2 ** (bits - 1) - 1, 2.0 ** (-4 - bits)
    col = torch.arange(64, device="cuda") * 17 % K                                        # every place of a lane's 32 columns
    codes = (torch.randn((N, K), generator=gen, device="cuda") * (top / 6.0) + mid).round().clamp(0, top)
    codes[:, col] = mid
    others = [[k for k in range(128 * g, 128 * g + 128) if k not in set(col.tolist())] for g in range(K // 128)]
    codes[:, [o[0] for o in others]], codes[:, [o[1] for o in others]] = 0.0, float(top)   # a group's range: its scale and zero
    w = ((codes - mid) * scale).half()
    qw = lpq.lpq_quantize_pack(w, bits, lpq.LPQ_ASYM_GROUP)
    deq = lpq.lpq_unpack_dequant(qw).double()
    assert torch.equal(deq, w.double()) and float(deq[:, col].abs().max()) == 0.0
    x = torch.randn((64, K), generator=gen, device="cuda").half()
    x[torch.arange(64, device="cuda"), col] = size
    ref = x.double() @ deq.t()
    for M in (33, 48, 64):
        assert lpq.lpq_route_of([(bits, lpq.LPQ_ASYM_GROUP, K, N)], lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
        y = lpq.lpq_qlinear_decode(qw, x[:M]).double()
        err = (y - ref[:M]).norm(dim=1) / ref[:M].norm(dim=1)
        assert float(err.max()) <= 3e-4, "%d rows: row %d off by %.2e" % (M, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("bits", [3, 4], ids=["w3", "w4"])
@pytest.mark.parametrize("K,N", [(128, 64), (384, 320), (4736, 192), (1152, 1088), (2048 * 128 + 1152, 64)])
def test_decode_33_to_64_rows_even_share(bits, K, N, even_share):
    """The even-share kernel of 33 to 64 rows, 3- and 4-bit weights, at the edges of its token
    tiles, with waves without a row block, chunks of one step to a whole one and rows of up to 263296 columns;
    rows of unlike magnitude, rows of zeros and of the smallest fp16 numbers, elements thirty and a thousand times their neighbours,
    bias, activation and a residual in place.  Against 64 bits, row by row: the roundings of the output and of the weights to fp16
    (2.1e-4 and 1.7e-4 of it, 2.7e-4 together); 4e-4 leaves room for sums in 32 bits."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(K + N + bits)
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.02).half()
    bias = (0.1 * torch.randn(N, generator=gen, device="cuda")).half()
    qw = lpq.lpq_quantize_pack(w, bits, lpq.LPQ_ASYM_GROUP, bias=bias)
    deq = lpq.lpq_unpack_dequant(qw).double()
    x = torch.randn((64, K), generator=gen, device="cuda")
    x[:, torch.randperm(K, generator=gen, device="cuda")[:3]] *= 30.0
    x[1, 5] *= 1000.0
    scale = torch.tensor([1.0, 2.0 ** -11, 2.0 ** 5], device="cuda")[torch.arange(64, device="cuda") % 3]
    x = (x * scale[:, None]).half()
    x[2] = 0.0
    x[3] = 2.0 ** -24
    acc = x.double() @ deq.t()
    for M in (33, 47, 48, 49, 63, 64):
        assert lpq.lpq_route_of([(bits, lpq.LPQ_ASYM_GROUP, K, N)], lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
        y = lpq.lpq_qlinear_fused(qw, x[:M], lpq.LPQ_DECODE).double()
        ref = acc[:M] + bias.double()
        err = (y - ref).norm(dim=1) / ref.norm(dim=1)
        assert float(err.max()) <= 4e-4, "%d rows: row %d off by %.2e" % (M, int(err.argmax()), float(err.max()))
        res = torch.randn((M, N), generator=gen, device="cuda").half()
        z = res.clone()
        lpq.lpq_qlinear_fused(qw, x[:M], lpq.LPQ_DECODE, activation=lpq.LPQ_ACT_RELU, residual=z, y=z)
        check_output(z, (torch.relu(ref) + res.double()).cpu().numpy(), "even share, %d rows" % M)


@pytest.mark.parametrize("small", [False, True], ids=["even_share", "small"])
@pytest.mark.parametrize("bits", [3, 4, 8], ids=["w3", "w4", "w8"])
@pytest.mark.parametrize("K,N", [(4736, 1088), (1920, 576)])
def test_decode_zero_term_of_one_signed_activations(bits, K, N, small):
    """Codes multiplied without their zero points, zero times the sum of a group's activations behind: the even-share kernel up to 32 rows, the kernels of small
    launches.  Where that term is largest, activations of one sign against weights about zero: it is 100 to 170 times the result, in rows of magnitudes up to 2^12 apart.  Against
    64 bits, row by row: the output's rounding is 2.1e-4; 32-bit sums of terms 170 times the result leave some 170 * 2^-24 * sqrt(K / 32) = 1.2e-4, 2.5e-4 together, 3e-4 with
    room for the worst row (sums kept as one fp16 number instead of two would leave 8e-3).  From 33 rows on the even-share kernel multiplies weights rounded to fp16, the same few
    values many times over: the library's tolerance."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(K + N + bits)
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.02).half()
    qw = lpq.lpq_quantize_pack(w, bits, lpq.LPQ_ASYM_GROUP)
    deq = lpq.lpq_unpack_dequant(qw).double()
    x = torch.rand((64, K), generator=gen, device="cuda") + 0.5
    scale = torch.tensor([1.0, 2.0 ** -8, -(2.0 ** 4)], device="cuda")[torch.arange(64, device="cuda") % 3]
    x = (x * scale[:, None]).half()
    ref = x.double() @ deq.t()
    zeros = qw.zeros.view(K // 128, N).double()                                          # the term itself, of the first row
    term = x[0].double().view(K // 128, 128).sum(1) @ zeros
    assert 90.0 <= float(term.norm() / ref[0].norm()) <= 200.0
    lpq.lpq_set_decode_routing(-1 if small else 0, 0)
    try:
        for M in (1, 8, 16, 17, 32, 33, 64):
            assert (lpq.lpq_route_of([(bits, lpq.LPQ_ASYM_GROUP, K, N)], lpq.LPQ_DECODE, M)[0] != lpq.LPQ_ROUTE_EVEN_SHARE) == small
            y = lpq.lpq_qlinear_decode(qw, x[:M]).double()
            err = (y - ref[:M]).norm(dim=1) / ref[:M].norm(dim=1)
            assert float(err.max()) <= (3e-4 if small or M <= 32 else 1e-3), "%d rows: row %d off by %.2e" % (M, int(err.argmax()), float(err.max()))
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("M", [40, 64])
@pytest.mark.parametrize("bits", [3, 4], ids=["w3", "w4"])
def test_infinite_activations_even_share(bits, M, even_share):
    assert lpq.lpq_route_of([(bits, lpq.LPQ_ASYM_GROUP, 2304, 320)], lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
    test_infinite_activations(lpq.LPQ_DECODE, M, bits, lpq.LPQ_ASYM_GROUP)


@pytest.mark.parametrize("M", [40, 64])
def test_decode_of_long_rows_without_allocation(M, even_share):
    """A launch of 40 linears of 65536 columns, on the workspace and on the static scratch array (128 MiB): the same bits, right ones."""
    import torch
    layer = {n: lpq.lpq_quantize_pack((torch.randn((N, K), device="cuda") * 0.02).half(), 3, lpq.LPQ_ASYM_GROUP)
             for n, (K, N) in {"qkv": (65536, 64), "out": (65536, 64), "fc1": (65536, 64), "fc2": (65536, 64)}.items()}
    n = 10
    xs = [{k: torch.randn((M, 65536), device="cuda").half() for k in layer}] * n
    out = []
    for static in (False, True):
        ys = [{k: torch.empty((M, 64), dtype=torch.float16, device="cuda") for k in layer} for _ in range(n)]
        (lpq.lpq_stage_linears_noalloc if static else lpq.lpq_stage_linears)(lpq.Stage([layer] * n, xs, ys), lpq.LPQ_DECODE)
        out.append(ys)
    for name in layer:
        assert all(torch.equal(a[name], b[name]) for a, b in zip(*out)), "%s, %d rows: other bits" % (name, M)
        ref = xs[0][name].double() @ lpq.lpq_unpack_dequant(layer[name]).double().t()
        for ys in out:
            check_output(ys[n - 1][name], ref.cpu().numpy(), "%s, %d rows" % (name, M))


@pytest.mark.parametrize("bits,scheme,M", [(8, 1, 20), (8, 2, 20), (8, 2, 43), (16, 0, 30), (16, 0, 64)], ids=["w8_20", "i8_20", "i8_43", "fp16_30", "fp16_64"])
def test_decode_mid_kernel_between_the_lines(bits, scheme, M):
    """Launches of four linears of 1.2 GB of codes, with which a single linear would take the even-share kernel."""
    import torch
    K, N = 8192, 18432 * 16 // bits
    assert lpq.lpq_route_of([(bits, scheme, K, N)] * 4, lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_MID
    assert lpq.lpq_route_of([(bits, scheme, K, 4 * N)], lpq.LPQ_DECODE, M)[0] == lpq.LPQ_ROUTE_EVEN_SHARE
    gen = torch.Generator(device="cuda").manual_seed(bits + M)
    bias = torch.randn((N,), generator=gen, device="cuda").half()
    qw = lpq.lpq_quantize_pack(torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float16) * 0.02, bits, scheme, bias=bias)
    names = ("qkv", "out", "fc1", "fc2")
    xs = {n: torch.randn((M, K), generator=gen, device="cuda").half() for n in names}
    ys = {n: torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for n in names}
    lpq.lpq_stage_linears(lpq.Stage([{n: qw for n in names}], [xs], [ys]), lpq.LPQ_DECODE)
    for n in names:
        check_output(ys[n], _prefill_reference(qw, xs[n], bias), "%s, %d rows" % (n, M))
