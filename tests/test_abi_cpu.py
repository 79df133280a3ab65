"""C-ABI checks that need no GPU: the library loads, exports every symbol the header declares,
reports sizes, and rejects bad arguments on the host before any HIP call."""
import ctypes
import os
import re

import pytest

import paper_2403_01136_amd as lpq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    text = open(os.path.join(ROOT, "include", "lpq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(lpq_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = lpq.load_library()
    names = header_functions()
    assert set(names) == set(lpq.EXPORTS), names
    for name in names:
        assert getattr(lib, name) is not None


def test_packed_sizes_are_dense():
    # Sec. 4.1: bytes = weights * bit / 8; scale and zero are fp16 per (row, 128 columns)
    for bits, scheme in ((3, 1), (4, 1), (8, 1), (8, 2), (16, 0)):
        for K, N in ((128, 64), (5120, 15360), (57344, 14336)):
            c, s, z = lpq.lpq_packed_sizes(bits, scheme, K, N)
            assert c * 8 == K * N * bits
            assert s == (N * (K // 128) * 2 if scheme == 1 else (N * 2 if scheme == 2 else 0))
            assert z == (s if scheme == 1 else 0)


@pytest.mark.parametrize("bits,scheme,K,N,status", [
    (5, 1, 128, 64, 2), (2, 1, 128, 64, 2), (4, 7, 128, 64, 3), (16, 1, 128, 64, 3), (3, 2, 128, 64, 3), (4, 0, 128, 64, 3),
    (4, 1, 100, 64, 4), (4, 1, 128, 16, 4), (4, 1, 128, 96, 4), (4, 1, 0, 64, 4), (4, 1, 128, -64, 4),
])
def test_bad_descriptors(bits, scheme, K, N, status):
    with pytest.raises(lpq.LpqError) as e:
        lpq.lpq_packed_sizes(bits, scheme, K, N)
    assert e.value.status == status


def test_group_size_must_be_128_for_grouped_scheme():
    lib = lpq.load_library()
    c = ctypes.c_size_t()
    d = lpq.lpq_qdesc(4, 1, 64, 128, 64)
    assert lib.lpq_packed_sizes(ctypes.byref(d), ctypes.byref(c), ctypes.byref(c), ctypes.byref(c)) == 3
    assert lib.lpq_packed_sizes(None, ctypes.byref(c), ctypes.byref(c), ctypes.byref(c)) == 1
    d = lpq.lpq_qdesc(4, 1, 128, 128, 64)
    assert lib.lpq_packed_sizes(ctypes.byref(d), None, ctypes.byref(c), ctypes.byref(c)) == 1


def test_entry_points_validate_before_touching_the_device():
    lib = lpq.load_library()
    d = lpq.make_desc(4, 1, 128, 64)
    fake = 0x10000          # never dereferenced: every call below must fail validation first
    good = lpq.lpq_qweight(d, fake, fake, fake, None)
    # NULL pointers
    assert lib.lpq_quantize_pack(None, ctypes.byref(d), ctypes.byref(good), None) == 1
    assert lib.lpq_qlinear_decode(ctypes.byref(good), None, 1, fake, None) == 1
    assert lib.lpq_qlinear_prefill(ctypes.byref(good), fake, 1, None, None) == 1
    nz = lpq.lpq_qweight(d, fake, fake, None, None)
    assert lib.lpq_qlinear_decode(ctypes.byref(nz), fake, 1, fake, None) == 1
    assert lib.lpq_unpack_dequant(ctypes.byref(good), None, None) == 1
    assert lib.lpq_stage_linears(None, 1, 1, 1, None, None) == 1
    # M < 1
    assert lib.lpq_qlinear_decode(ctypes.byref(good), fake, 0, fake, None) == 4
    assert lib.lpq_qlinear_prefill(ctypes.byref(good), fake, -3, fake, None) == 4
    # alignment
    assert lib.lpq_qlinear_decode(ctypes.byref(good), fake + 2, 1, fake, None) == 5
    odd = lpq.lpq_qweight(d, fake + 8, fake, fake, None)
    assert lib.lpq_qlinear_prefill(ctypes.byref(odd), fake, 1, fake, None) == 5
    assert lib.lpq_quantize_pack(fake + 4, ctypes.byref(d), ctypes.byref(good), None) == 5
    # descriptor mismatch between desc and out
    d2 = lpq.make_desc(3, 1, 128, 64)
    assert lib.lpq_quantize_pack(fake, ctypes.byref(d2), ctypes.byref(good), None) == 4
    # row windows: on 64-row boundaries and inside W
    d3 = lpq.make_desc(4, 1, 128, 192)
    w3 = lpq.lpq_qweight(d3, fake, fake, fake, None)
    for row0, n_rows in ((32, 64), (0, 100), (128, 128), (-64, 64), (0, -64)):
        assert lib.lpq_quantize_pack_rows(fake, ctypes.byref(d3), row0, n_rows, ctypes.byref(w3), None) == 4
    assert lib.lpq_quantize_pack_rows(None, ctypes.byref(d3), 0, 64, ctypes.byref(w3), None) == 1
    assert lib.lpq_quantize_pack_rows(fake + 2, ctypes.byref(d3), 0, 64, ctypes.byref(w3), None) == 5
    # loader: NULL host or staging pointer, misaligned pointers, staging too small for 64 rows
    assert lib.lpq_load_quantize_pack(None, ctypes.byref(d3), ctypes.byref(w3), fake, 1 << 20, None) == 1
    assert lib.lpq_load_quantize_pack(fake, ctypes.byref(d3), ctypes.byref(w3), None, 1 << 20, None) == 1
    assert lib.lpq_load_quantize_pack(fake + 8, ctypes.byref(d3), ctypes.byref(w3), fake, 1 << 20, None) == 5
    assert lib.lpq_load_quantize_pack(fake, ctypes.byref(d3), ctypes.byref(w3), fake + 4, 1 << 20, None) == 5
    assert lib.lpq_load_quantize_pack(fake, ctypes.byref(d3), ctypes.byref(w3), fake, 64 * 128 * 2 - 1, None) == 6
    assert lib.lpq_load_quantize_pack(fake, ctypes.byref(d2), ctypes.byref(w3), fake, 1 << 20, None) == 4
    # fused epilogue: unknown activation, misaligned residual, unknown phase
    ep = lpq.lpq_epilogue(7, None)
    assert lib.lpq_qlinear_fused(ctypes.byref(good), fake, 1, fake, ctypes.byref(ep), 1, None) == 8
    ep = lpq.lpq_epilogue(1, fake + 2)
    assert lib.lpq_qlinear_fused(ctypes.byref(good), fake, 1, fake, ctypes.byref(ep), 1, None) == 5
    assert lib.lpq_qlinear_fused(ctypes.byref(good), fake, 1, fake, None, 3, None) == 8
    assert lib.lpq_qlinear_fused(ctypes.byref(good), None, 1, fake, None, 1, None) == 1
    # layer norm
    assert lib.lpq_layernorm(None, fake, fake, 1e-5, 1, 64, fake, None) == 1
    for M, h in ((0, 64), (1, 60), (1, 0), (1, 16392)):
        assert lib.lpq_layernorm(fake, fake, fake, 1e-5, M, h, fake, None) == 4
    assert lib.lpq_layernorm(fake, fake + 2, fake, 1e-5, 1, 64, fake, None) == 5
    # attention and KV cache: head size, cache length, positions
    st = lpq.lpq_layer_state(fake, fake, fake, fake, fake, fake, None)
    for cfg, n_seqs, T, pos0 in ((lpq.lpq_layer_cfg(4, 96, 128, 1, 1e-5), 1, 1, 0), (lpq.lpq_layer_cfg(4, 64, 100, 1, 1e-5), 1, 1, 0),
                                 (lpq.lpq_layer_cfg(4, 64, 128, 1, 1e-5), 1, 2, 127), (lpq.lpq_layer_cfg(4, 64, 128, 1, 1e-5), 0, 1, 0),
                                 (lpq.lpq_layer_cfg(0, 64, 128, 1, 1e-5), 1, 1, 0), (lpq.lpq_layer_cfg(4, 64, 128, 1, 1e-5), 1, 1, -1)):
        assert lib.lpq_kv_append(fake, ctypes.byref(cfg), ctypes.byref(st), n_seqs, T, pos0, None) == 4
        assert lib.lpq_attention(fake, ctypes.byref(cfg), ctypes.byref(st), n_seqs, T, pos0, fake, None) == 4
    cfg = lpq.lpq_layer_cfg(4, 64, 128, 1, 1e-5)
    no_cache = lpq.lpq_layer_state(fake, fake, fake, fake, None, fake, None)
    assert lib.lpq_attention(fake, ctypes.byref(cfg), ctypes.byref(no_cache), 1, 1, 0, fake, None) == 1
    assert lib.lpq_attention(fake + 2, ctypes.byref(cfg), ctypes.byref(st), 1, 1, 0, fake, None) == 5
    # decoder layer: weights must fit hidden = heads * head_dim; workspace size is checked
    h, f = 256, 512
    mk = lambda K, N: lpq.lpq_qweight(lpq.make_desc(4, 1, K, N), fake, fake, fake, None)
    layer = lpq.lpq_layer(mk(h, 3 * h), mk(h, h), mk(h, f), mk(f, h))
    need = lib.lpq_decoder_layer_workspace(ctypes.byref(layer), ctypes.byref(cfg), 8)
    assert need == 8 * (5 * h + f) * 2 and lib.lpq_decoder_layer_workspace(None, ctypes.byref(cfg), 8) == 0
    args = (ctypes.byref(layer), ctypes.byref(cfg), ctypes.byref(st), 1, 8, 1, 0, fake, fake, fake)
    assert lib.lpq_decoder_layer(*args, need - 1, None) == 6
    wrong = lpq.lpq_layer(mk(h, 3 * h), mk(h, h), mk(h, f), mk(f, 2 * h))
    assert lib.lpq_decoder_layer(ctypes.byref(wrong), *args[1:], need, None) == 4
    bad_act = lpq.lpq_layer_cfg(4, 64, 128, 9, 1e-5)
    assert lib.lpq_decoder_layer(args[0], ctypes.byref(bad_act), *args[2:], need, None) == 8
    assert lib.lpq_decoder_layer(args[0], args[1], args[2], 1, 8, 1, 0, None, fake, fake, need, None) == 1
    # variance indicator
    assert lib.lpq_variance_indicator(None, 128, 64, fake, 1, 0, fake, None) == 1
    assert lib.lpq_variance_indicator(fake, 128, 64, fake, 1, 0, None, None) == 1
    for K, N, M in ((100, 64, 1), (0, 64, 1), (128, 0, 1), (128, 64, 0)):
        assert lib.lpq_variance_indicator(fake, K, N, fake, M, 0, fake, None) == 4
    assert lib.lpq_variance_indicator(fake + 2, 128, 64, fake, 1, 0, fake, None) == 5
    assert lib.lpq_variance_indicator(fake, 128, 64, fake, 1, 0, fake + 4, None) == 5
    # bad bits inside a weight
    bad = lpq.lpq_qweight(lpq.lpq_qdesc(5, 1, 128, 128, 64), fake, fake, fake, None)
    assert lib.lpq_qlinear_decode(ctypes.byref(bad), fake, 1, fake, None) == 2
    # stage: bad layer count, bad phase, one bad layer rejects the whole call
    layers = (lpq.lpq_layer * 1)()
    io = (lpq.lpq_layer_io * 1)()
    assert lib.lpq_stage_linears(layers, 0, 1, 1, io, None) == 4
    assert lib.lpq_stage_linears(layers, 1, 5, 1, io, None) == 8
    assert lib.lpq_stage_linears(layers, 1, 1, 1, io, None) != 0      # zeroed layer: bits = 0
    for i in range(9):
        assert isinstance(lpq.status_str(i), str) and lpq.status_str(i)
    assert lpq.status_str(99) == "unknown status"


def test_workspace_growth_policy():
    """The per-device workspace never frees a block it has handed out: a larger need allocates a new block
    (need + 25 %, at least 8 MiB), a need that fits reuses the block, and once a reservation is in force a
    larger need is an error instead of an allocation.  (Pure host function: what the library does on a device
    is this policy followed by one hipMalloc.)"""
    MiB = 1 << 20
    assert lpq.lpq_workspace_policy(0, False, 1) == 8 * MiB                    # first use: the floor
    assert lpq.lpq_workspace_policy(8 * MiB, False, 8 * MiB) == 0              # fits: reuse
    assert lpq.lpq_workspace_policy(8 * MiB, False, 8 * MiB + 1) == 8 * MiB + 1 + (8 * MiB + 1) // 4
    assert lpq.lpq_workspace_policy(8 * MiB, False, 64 * MiB) == 80 * MiB      # growth leaves headroom
    assert lpq.lpq_workspace_policy(80 * MiB, True, 80 * MiB) == 0             # reserved and large enough
    with pytest.raises(lpq.LpqError) as err:
        lpq.lpq_workspace_policy(80 * MiB, True, 80 * MiB + 1)                 # reserved: no growth
    assert err.value.status == 6
    assert lpq.load_library().lpq_workspace_policy(0, 0, 1, None) == 1
    # a sequence of needs never shrinks the block and allocates only when a need exceeds it
    have, allocs = 0, 0
    for need in (1, 4 * MiB, 9 * MiB, 3 * MiB, 11 * MiB, 12 * MiB, 200 * MiB, 10 * MiB):
        a = lpq.lpq_workspace_policy(have, False, need)
        if a:
            assert a >= need and a > have
            have, allocs = a, allocs + 1
        assert have >= need
    assert allocs == 4


def test_decode_routing_arguments():
    lib = lpq.load_library()
    assert lib.lpq_set_decode_routing(0, 0) == 0 and lib.lpq_set_decode_routing(-1, 5) == 0
    for mib, tiles in ((5000, 0), (192, 1), (192, 6)):
        assert lib.lpq_set_decode_routing(mib, tiles) == 4
    assert lib.lpq_set_decode_routing(-1, -1) == 0


ROUTE_SHAPES = [(K, N) for K in (128, 384, 640, 768, 2048, 5120, 20480, 57344) for N in (64, 320, 768, 2304, 5120, 15360, 36864)]


def test_a_forced_group_size_holds_up_to_16_rows():
    """lpq_set_decode_routing(-1, T): every small launch of up to 16 rows takes the kernel for those rows with T tiles per workgroup (4 where T
    does not divide the linear's tiles, fp16 weights at most 2), also at 13 to 16 rows, where the library may choose otherwise."""
    try:
        for T in (2, 3, 4, 5):
            lpq.lpq_set_decode_routing(-1, T)
            for bits, scheme in ((3, 1), (4, 1), (8, 1), (8, 2), (16, 0)):
                for K, N in ROUTE_SHAPES:
                    if K * N * bits // 8 > 192 << 20:
                        continue
                    rt = 2 if bits == 16 and T > 2 else T
                    want = T if N // 16 % rt == 0 else 4
                    for M in (1, 12, 13, 16):
                        kernel, tiles, _, _ = lpq.lpq_route_of([(bits, scheme, K, N)], lpq.LPQ_DECODE, M)
                        assert (kernel, tiles) == (lpq.LPQ_ROUTE_ROWS, want), (T, bits, scheme, K, N, M)
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


def test_routes():
    """The families a call can take, by phase, rows and size, and what lpq_set_decode_routing(0, 0) does to them."""
    small, large = [(4, 1, 5120, 15360)], [(4, 1, 14336, 57344)] * 4
    kernel = lambda d, phase, M: lpq.lpq_route_of(d, phase, M)[0]
    for M in (1, 8, 12):
        assert kernel(small, lpq.LPQ_DECODE, M) == kernel(small, lpq.LPQ_PREFILL, M) == lpq.LPQ_ROUTE_ROWS
    for M in (17, 32, 33, 64):
        assert kernel(small, lpq.LPQ_DECODE, M) == kernel(small, lpq.LPQ_PREFILL, M) == lpq.LPQ_ROUTE_MID
    assert kernel(small, lpq.LPQ_DECODE, 65) == lpq.LPQ_ROUTE_EVEN_SHARE and kernel(small, lpq.LPQ_PREFILL, 65) == lpq.LPQ_ROUTE_PREFILL
    for M in (1, 16, 17, 64):
        assert kernel(large, lpq.LPQ_DECODE, M) == lpq.LPQ_ROUTE_EVEN_SHARE and kernel(large, lpq.LPQ_PREFILL, M) == lpq.LPQ_ROUTE_PREFILL
    assert kernel(large[:1], lpq.LPQ_PREFILL, 12) == lpq.LPQ_ROUTE_ROWS              # a single linear, however large
    try:
        lpq.lpq_set_decode_routing(0, 0)
        for M in (1, 16, 17, 64):
            assert kernel(small, lpq.LPQ_DECODE, M) == lpq.LPQ_ROUTE_EVEN_SHARE and kernel(small, lpq.LPQ_PREFILL, M) == lpq.LPQ_ROUTE_PREFILL
    finally:
        lpq.lpq_set_decode_routing(-1, -1)
    lib, r, d = lpq.load_library(), lpq.lpq_route(), lpq.make_desc(4, 1, 128, 64)
    assert lib.lpq_route_of(None, 1, 1, 1, 256, ctypes.byref(r)) == 1 and lib.lpq_route_of(ctypes.byref(d), 1, 1, 1, 256, None) == 1
    for n, phase, M, cus in ((0, 1, 1, 256), (49, 1, 1, 256), (1, 1, 0, 256), (1, 1, 1, 0), (1, 2, 1, 256)):
        assert lib.lpq_route_of(ctypes.byref(d), n, phase, M, cus, ctypes.byref(r)) == 4
    d = lpq.make_desc(4, 1, 65536 * 128, 64)
    assert lib.lpq_route_of(ctypes.byref(d), 1, 1, 1, 256, ctypes.byref(r)) == 8


@pytest.mark.parametrize("bits,scheme,several,one", [
    (3, 1, (1.0e9, 1.0e9, 0.55e9), (1.0e9, 1.0e9, 0.55e9)), (4, 1, (1.0e9, 1.0e9, 0.55e9), (1.0e9, 1.0e9, 0.55e9)),
    (8, 1, (1.9e9, 1.0e9, 1.0e9), (1.0e9,) * 3), (8, 2, (1.9e9, 1.9e9, 1.0e9), (1.0e9,) * 3), (16, 0, (0.7e9,) * 3, (0.5e9,) * 3)])
def test_routes_of_17_to_64_rows_by_weights(bits, scheme, several, one):
    """The number of weights up to which a launch of 17-32, 33-48 and 49-64 rows goes to the kernel of few row blocks, of several linears and of
    one; it moves with the first routing setting."""
    kernel = lambda weights, n, M: lpq.lpq_route_of([(bits, scheme, 8192, round(weights / n / 8192 / 64) * 64)] * n, lpq.LPQ_DECODE, M)[0]
    for n, lines in ((1, one), (3, several)):
        for line, rows in zip(lines, ((17, 32), (33, 48), (49, 64))):
            for M in rows:
                assert kernel(0.99 * line, n, M) == lpq.LPQ_ROUTE_MID and kernel(1.01 * line, n, M) == lpq.LPQ_ROUTE_EVEN_SHARE, (n, M, line)
    try:
        lpq.lpq_set_decode_routing(2 * 192, -1)
        assert kernel(1.99 * several[0], 3, 17) == lpq.LPQ_ROUTE_MID
    finally:
        lpq.lpq_set_decode_routing(-1, -1)


@pytest.mark.parametrize("grouped", [(3, 1), (4, 1), (8, 1)], ids=["w3", "w4", "w8"])
@pytest.mark.parametrize("other", [(8, 2), (16, 0)], ids=["i8", "f16"])
def test_grouped_weights_of_33_rows_and_more_keep_the_near_line(grouped, other):
    """Up to 64 rows symmetric 8-bit and fp16 weights go farther with the kernel of few row blocks, but not beside a grouped linear, whose weights the
    even-share kernel dequantises from 33 rows on and that one does not."""
    far, small = other + (8192, 73728 if other[0] == 8 else 36864), grouped + (128, 64)       # two of them: 1.2 GB
    kernel = lambda descs, M: lpq.lpq_route_of(descs, lpq.LPQ_DECODE, M)[0]
    for M in (17, 32):
        assert kernel([far, far], M) == kernel([far, small, far], M) == lpq.LPQ_ROUTE_MID
    for M in (33, 48):
        assert kernel([far, far], M) == lpq.LPQ_ROUTE_MID and kernel([far, small, far], M) == lpq.LPQ_ROUTE_EVEN_SHARE


def layer_route(fmt, h, n_seqs, pos0=70):
    return lpq.lpq_layer_route_of([fmt + kn for kn in ((h, 3 * h), (h, h), (h, 4 * h), (4 * h, h))], n_seqs, pos0)


def test_layer_routes():
    """Where a decode layer forms its norms: inside the linears of few rows, behind the sums of a split out-projection, else in launches of their own."""
    for fmt in ((3, 1), (4, 1), (8, 1), (8, 2), (16, 0)):
        for h, B in ((768, 1), (768, 8), (2048, 8), (2560, 4), (4096, 4)):
            assert layer_route(fmt, h, B)[:2] == (lpq.LPQ_NORM_IN_LINEAR, lpq.LPQ_NORM_IN_LINEAR), (fmt, h, B)
        for h, B in ((768, 9), (768, 12), (2048, 9), (2176, 5), (5248, 1), (7168, 1), (4096, 5)):
            assert layer_route(fmt, h, B)[:2] == (lpq.LPQ_NORM_LAUNCH, lpq.LPQ_NORM_LAUNCH), (fmt, h, B)
        assert layer_route(fmt, 5120, 4)[0] == lpq.LPQ_NORM_IN_LINEAR
        assert layer_route(fmt, 768, 16)[0] == lpq.LPQ_NORM_LAUNCH
        for h, B in ((2560, 16), (5120, 16), (7168, 43), (16384, 64)):
            assert layer_route(fmt, h, B)[:2] == (lpq.LPQ_NORM_LAUNCH, lpq.LPQ_NORM_BEHIND_SPLITS), (fmt, h, B)
    # the new token: in the attention kernel for little cache, for few feature rows and at the first position of a tile, but not of a long context
    for h, B, pos0, append in ((768, 64, 300, 1), (2048, 16, 1000, 1), (5120, 8, 1000, 1), (5120, 16, 562, 0), (14336, 32, 100, 0), (4096, 8, 4000, 1),
                               (1152, 32, 4000, 1), (4096, 8, 8100, 0), (7168, 64, 640, 1), (7168, 64, 704, 0), (7168, 64, 4096, 0), (5120, 16, 1024, 1), (5120, 16, 0, 1)):
        assert layer_route((4, 1), h, B, pos0)[2] == append, (h, B, pos0)
    lib, r, d = lpq.load_library(), lpq.lpq_layer_route(), (lpq.lpq_qdesc * 4)(*[lpq.make_desc(4, 1, 128, 64)] * 4)
    assert lib.lpq_layer_route_of(None, 1, 0, 256, ctypes.byref(r)) == 1 and lib.lpq_layer_route_of(d, 1, 0, 256, None) == 1
    for n_seqs, pos0, cus in ((0, 0, 256), (1, -1, 256), (1, 0, 0)):
        assert lib.lpq_layer_route_of(d, n_seqs, pos0, cus, ctypes.byref(r)) == 4


def test_routes_of_13_to_32_rows():
    """Where the kernel for 17 and more rows would be the slower one: 8-bit and fp16 linears of 13 to 16 rows with neither few workgroups of long
    ranges nor more than a round of them, and one or two groups of columns up to 32 rows.  Below 512 columns, too, the blocks
    per workgroup follow from the estimate: as many workgroups as fit the chip, not four blocks in each."""
    route = lambda fmt, K, N, M: lpq.lpq_route_of([fmt + (K, N)], lpq.LPQ_DECODE, M)
    for fmt in ((8, 1), (8, 2), (16, 0)):
        for K, N in ((768, 2304), (768, 3072), (2048, 6144), (1920, 6272), (384, 15168)):
            for M in (13, 16):
                assert route(fmt, K, N, M)[0] == lpq.LPQ_ROUTE_ROWS, (fmt, K, N, M)
    for fmt in ((3, 1), (4, 1), (8, 1), (8, 2), (16, 0)):
        for M in (13, 16, 17, 32):
            assert route(fmt, 128, 4096, M)[0] == lpq.LPQ_ROUTE_ROWS and route(fmt, 256, 4096, M)[0] == lpq.LPQ_ROUTE_ROWS
        assert route(fmt, 128, 4096, 33)[0] == route(fmt, 384, 4096, 17)[0] == lpq.LPQ_ROUTE_MID
        for M in (17, 32, 33, 64):
            kernel, blocks, splits, _ = route(fmt, 384, 15168, M)
            assert kernel == lpq.LPQ_ROUTE_MID and splits == 1 and 15168 // 64 / blocks >= 118, (fmt, M, blocks)
