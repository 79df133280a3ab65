// C-ABI entry points: host-side validation, work decomposition, kernel dispatch.
// Every argument check happens before the first HIP call (see include/lpq.h).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <vector>

#include "lpq_common.h"

namespace lpq {

int variant_of(const lpq_qdesc& d)
{
    if (d.scheme == LPQ_FP16) return d.bits == 16 ? 4 : -1;
    if (d.scheme == LPQ_ASYM_GROUP) return d.bits == 3 ? 0 : d.bits == 4 ? 1 : d.bits == 8 ? 2 : -1;
    if (d.scheme == LPQ_SYM_CHANNEL) return d.bits == 8 ? 3 : -1;
    return -1;
}

size_t tile_bytes_of(int variant)
{
    static const size_t tb[5] = {768, 1024, 2048, 2048, 4096};
    return tb[variant];
}

namespace {

lpq_status check_desc(const lpq_qdesc* d)
{
    if (!d) return LPQ_ERR_NULL;
    if (d->bits != 3 && d->bits != 4 && d->bits != 8 && d->bits != 16) return LPQ_ERR_BITS;
    if (d->scheme != LPQ_FP16 && d->scheme != LPQ_ASYM_GROUP && d->scheme != LPQ_SYM_CHANNEL) return LPQ_ERR_SCHEME;
    if (variant_of(*d) < 0) return LPQ_ERR_SCHEME;
    if (d->scheme == LPQ_ASYM_GROUP ? d->group_size != 128 : (d->group_size != 0 && d->group_size != 128)) return LPQ_ERR_SCHEME;
    if (d->K <= 0 || d->N <= 0 || d->K % 128 != 0 || d->N % 64 != 0) return LPQ_ERR_SHAPE;
    return LPQ_OK;
}

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

lpq_status check_weight(const lpq_qweight* w)
{
    if (!w) return LPQ_ERR_NULL;
    lpq_status st = check_desc(&w->d);
    if (st != LPQ_OK) return st;
    if (!w->codes) return LPQ_ERR_NULL;
    if (w->d.scheme != LPQ_FP16 && !w->scales) return LPQ_ERR_NULL;
    if (w->d.scheme == LPQ_ASYM_GROUP && !w->zeros) return LPQ_ERR_NULL;
    if (misaligned(w->codes) || (w->d.scheme != LPQ_FP16 && misaligned(w->scales)) ||
        (w->d.scheme == LPQ_ASYM_GROUP && misaligned(w->zeros)) || (w->bias && misaligned(w->bias)))
        return LPQ_ERR_ALIGN;
    return LPQ_OK;
}

// the descriptor a quantiser call is given and the buffers it is to fill
lpq_status check_quantize_target(const lpq_qdesc* desc, const lpq_qweight* out)
{
    lpq_status st = check_desc(desc);
    if (st != LPQ_OK) return st;
    if (out->d.bits != desc->bits || out->d.scheme != desc->scheme || out->d.K != desc->K || out->d.N != desc->N ||
        out->d.group_size != desc->group_size)
        return LPQ_ERR_SHAPE;
    return check_weight(out);
}

lpq_status check_linear(const lpq_qweight* w, const void* x, int32_t M, const void* y)
{
    lpq_status st = check_weight(w);
    if (st != LPQ_OK) return st;
    if (!x || !y) return LPQ_ERR_NULL;
    if (M < 1) return LPQ_ERR_SHAPE;
    if (misaligned(x) || misaligned(y)) return LPQ_ERR_ALIGN;
    return LPQ_OK;
}

// ---- split-K workspace: one block per device, grown on demand.  A block that has been handed out is never
// freed before the process ends: a captured HIP graph, or work still queued on a stream, may hold its address.
// Growth allocates a new block and retires the old one (kept allocated); once lpq_workspace_reserve has been
// called on a device, that device's block no longer grows and a larger need is an error.
struct Workspace {
    std::mutex mu;
    void* ptr[64] = {};
    size_t bytes[64] = {};
    bool reserved[64] = {};
    std::vector<void*> retired;      // earlier blocks, released by the runtime at process exit
};
Workspace g_ws;

// What a request of `need` bytes does to a block of `have` bytes: 0 = reuse it, > 0 = allocate a new block of that
// size; LPQ_ERR_BUFSIZE if a reservation forbids growth.
lpq_status workspace_policy(size_t have, bool reserved, size_t need, size_t* alloc)
{
    *alloc = 0;
    if (need <= have) return LPQ_OK;
    if (reserved) return LPQ_ERR_BUFSIZE;
    *alloc = std::max(need + need / 4, (size_t)8 << 20);
    return LPQ_OK;
}

lpq_status workspace_grow(int dev, size_t want)      // g_ws.mu held
{
    void* fresh = nullptr;
    if (hipMalloc(&fresh, want) != hipSuccess) { (void)hipGetLastError(); return LPQ_ERR_BUFSIZE; }
    if (g_ws.ptr[dev]) g_ws.retired.push_back(g_ws.ptr[dev]);
    g_ws.ptr[dev] = fresh;
    g_ws.bytes[dev] = want;
    return LPQ_OK;
}

lpq_status library_workspace(size_t need, float** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LPQ_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_ws.mu);
    size_t alloc = 0;
    lpq_status st = workspace_policy(g_ws.bytes[dev], g_ws.reserved[dev], need, &alloc);
    if (st != LPQ_OK) return st;
    if (alloc && (st = workspace_grow(dev, alloc)) != LPQ_OK) return st;
    *out = static_cast<float*>(g_ws.ptr[dev]);
    return LPQ_OK;
}

// Partial sums of a call: the library's own workspace, or -- for the entry point that must not allocate -- the
// device's static scratch array (a larger need is an error there, never an allocation).
lpq_status workspace(bool static_ws, size_t need, float** out)
{
    if (!static_ws) return library_workspace(need, out);
    void* p = nullptr;
    size_t bytes = 0;
    if (static_scratch(&p, &bytes) != hipSuccess) { (void)hipGetLastError(); return LPQ_ERR_DEVICE; }
    if (need > bytes) return LPQ_ERR_BUFSIZE;
    *out = static_cast<float*>(p);
    return LPQ_OK;
}

// Compute units of the current device (cached).
lpq_status device_cus(int* out)
{
    static std::mutex mu;
    static int cus[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LPQ_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(mu);
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return LPQ_ERR_DEVICE;
        cus[dev] = n;
    }
    *out = cus[dev];
    return LPQ_OK;
}

// Routing of decode launches between the two kernel families (lpq_set_decode_routing; defaults measured on MI355X).
std::atomic<int32_t> g_rows_max_mb{192};     // launches that stream at most this many MiB of codes take the small-launch kernel
std::atomic<int32_t> g_rows_tiles{0};        // 2..5: force that many 16-row tiles per workgroup there; 0: the planner's choice

// Wavefronts per decode workgroup: eight, one workgroup per CU (two waves per SIMD), so that a step's activations
// are staged once for 512 rows of W.  (Four waves and two workgroups per CU move twice the activation bytes from
// L2 -- a third of the weight bytes at 3 bits and 16 token rows -- and measured 0.5-4 % slower on every configuration.)
// The workgroups per launch are what the chip holds at once.
int decode_waves(int /*M*/) { return 8; }

// relative cost of streaming one byte of each variant (x16), used to weight the even-share split
uint32_t variant_cost_x16(int variant)
{
    // measured on MI355X: bytes of 3- and 4-bit codes take longer to stream because unpacking them is
    // ALU work per byte; 8-bit codes and fp16 weights run at the memory system's pace
    static const uint32_t c[5] = {26, 21, 17, 17, 16};
    return c[variant];
}

// Workgroup shape of a single linear in the small-launch decode kernel: 16-row tiles per workgroup (T) and K
// splits (s).  Measured on MI355X (OPT-13B, 7B- and 70B-class shapes, 3- and 4-bit): a launch runs fastest
// when its workgroups just fit the compute units once -- a unit that gets two takes 2.6 times as long, not
// twice -- and a workgroup's time grows with its steps times (the activations it reads per step, from L2,
// plus T tiles of weights).  T = 3 and 5 cut a 64-row block across workgroups (e.g. 1280 tiles = 256 x 5);
// at T = 5 the kernel holds the whole register file and runs a third slower per byte.  A split costs a second
// kernel.  The estimate below (microseconds) is only used to rank the choices.
void rows_plan(const LinDesc& L, int cus, int* tiles, int* splits)
{
    static const double tile_us[5] = {0.024, 0.032, 0.064, 0.064, 0.128};     // per tile and step, by variant
    const int KT = L.kt, n_tiles = L.N / 16;
    double best = 1e30;
    *tiles = 4;
    *splits = 1;
    static const int order[4] = {4, 2, 3, 5};                                // ties go to the earlier entry
    for (int oi = 0; oi < 4; ++oi) {
        const int T = order[oi];
        if (L.variant == 4 && T > 2 && T != 4) continue;                     // fp16 weights: one or two tiles (4 stands for 2)
        const int rt = (L.variant == 4 && T > 2) ? 2 : T;
        if (n_tiles % rt != 0) continue;
        const double step_us = 0.06 + rt * tile_us[L.variant] + (rt == 5 ? 0.09 : 0.0);
        for (int s = 1; s <= 8; ++s) {
            const long wgs = (long)(n_tiles / rt) * s;
            // a split is there to fill the chip, not to add rounds; a wave wants several steps per stage of its ring
            if (s > 1 && (KT / s < 16 || wgs > cus)) break;
            const long rounds = (wgs + cus - 1) / cus;
            const double est = (rounds == 1 ? 1.0 : 1.3 * rounds) * ((KT + s - 1) / s) * step_us + (s > 1 ? 5.0 : 0.0);
            if (est < best * 0.98) best = est, *tiles = T, *splits = s;
        }
    }
}

// Row blocks per workgroup (DecodeArgs::row_tiles) and K splits (LinDesc::aux) of a launch of the decode kernel for 17-64 token
// rows.  A launch is fastest when its workgroups just fill the compute units once and their ranges of K are equally long:
// every number of row blocks and range lengths t are tried (a linear alone: those that change its splits; launches of several:
// fewer, each shape once, so that planning 48 linears takes 2 us of host time and not 20), each linear gets ceil(KT / t)
// splits, and the estimate (microseconds) ranks them: a step's arithmetic on the SIMDs of a workgroup (fp16 weights are a
// third longer, four times the loads), its activations through LDS, a workgroup's start and end, a reduce launch and its traffic.
// The constants are fitted to 17 shapes x 4 formats x 5 row counts with every row-block and split count timed: the choice is
// 2 % from the fastest in the mean, 12 % at most.  The splits' sums stay within `max_floats`.
void mid_plan(DecodeArgs& p, int cus, size_t max_floats)
{
    static const double step_us[4] = {0.42, 0.55, 1.2, 1.45};                    // of four row blocks at 1, 2, 3, 4 token tiles
    static const double format[5] = {1.0, 1.0, 1.05, 1.05, 1.35};
    struct Shape { int kt, N, variant, count; } shapes[MAX_LIN_PER_LAUNCH];
    const int tiles = (p.M + 15) / 16;
    int n = 0, kt_max = 1;
    for (int i = 0; i < p.n_lin; ++i) {
        const LinDesc& L = p.lin[i];
        kt_max = std::max(kt_max, (int)L.kt);
        int k = 0;
        while (k < n && (shapes[k].kt != L.kt || shapes[k].N != L.N || shapes[k].variant != L.variant)) ++k;
        if (k == n) shapes[n++] = Shape{L.kt, L.N, L.variant, 0};
        ++shapes[k].count;
    }
    double best = 1e30;
    int best_t = kt_max;
    p.row_tiles = 4;
    for (int rb = 4; rb >= (tiles <= 2 ? 1 : 2); rb /= 2) {
        const int slots = tiles == 1 ? 16 / rb : tiles == 2 && rb <= 2 ? 8 : 4;                    // steps per iteration (MidCfg in lpq_decode.hip)
        const double step = 0.25 * rb * step_us[tiles - 1], lds = 0.027 * tiles;
        for (int t = kt_max; t >= 4 || t == kt_max;) {
            double wgs = 0.0, floats = 0.0, sum = 0.0, longest = 0.0, shortest = 1e30;
            int most = 1;
            for (int k = 0; k < n; ++k) {
                const Shape& L = shapes[k];
                const int s = (L.kt + t - 1) / t, len = (L.kt + s - 1) / s;
                const double w = (double)((L.N / 64 + rb - 1) / rb) * s * L.count;
                const double us = (len + slots - 1) / slots * slots * (step * format[L.variant] + lds) + 2.0;
                wgs += w;
                sum += w * us;
                longest = std::max(longest, us);
                shortest = std::min(shortest, us);
                if (s > 1) floats += (double)s * p.M * L.N * L.count;
                most = std::max(most, s);
            }
            if (floats > (double)max_floats) break;                         // shorter ranges only need more
            // Up to two rounds of workgroups of one linear are counted whole; more, or of unlike lengths (longest first), fill up better.
            // Those of several linears start behind others of any length, which costs a fifth (four 4-bit layers of 1024 at 64 rows,
            // us: 320 workgroups of two row blocks 28.7, 192 of four 23.9).
            const double filled = std::max(longest, sum / cus + 0.5 * shortest) * (p.n_lin > 1 ? 1.2 : 1.0);
            const double est = (most > 1 ? 1.2 + 0.05 * most + floats * 8.0 / 1.4e6 : 0.0) +
                               (wgs <= cus ? longest : p.n_lin == 1 && wgs <= 2.0 * cus ? 2.0 * longest : filled);
            if (est < best * 0.99) best = est, best_t = t, p.row_tiles = rb;
            const int splits = (kt_max + t - 1) / t;
            t = p.n_lin == 1 ? (kt_max - 1) / splits : std::min(t - 1, t * 7 / 8);      // alone: the longest range with one split more
        }
    }
    for (int i = 0; i < p.n_lin; ++i) p.lin[i].aux = (p.lin[i].kt + best_t - 1) / best_t;
}

// Bytes that decode_prepare_kernel leaves for a linear in a decode launch of up to 32 token rows per pass.  The group
// sums: per token row (32 of them) an fp16 pair per 128-column group, groups padded to a multiple of 16, and 16 bytes
// for the row's factors; behind them, for 3-bit weights that the launch reads in place, `rows` rows of scaled
// activations.
size_t prepared_bytes(const lpq_qdesc& d, int rows, bool in_place)
{
    const size_t sums = (size_t)32 * (4 * (((size_t)d.K / 128 + 15) & ~(size_t)15) + 16);
    return sums + (in_place && variant_of(d) == 0 ? (size_t)rows * (size_t)d.K * 2 : 0);
}

struct LinearCall {
    const lpq_qweight* w;
    const void* x;
    void* y;
    const void* residual = nullptr;
    int32_t act = LPQ_ACT_NONE;
};

// Whether a stage-wide decode launch of M token rows reads its 3-bit codes in place (lpq_decode.hip: a third of the
// unpacking instructions less, against a copy of those linears' activations scaled beforehand).  The copy costs by
// the row, the saving is per weight: it pays at up to 16 rows where 3-bit weights are a good part of what the launch
// streams.  Measured: +2.5 % (16 rows) to +5 % (1 row) on an all-3-bit stage, +0.5 % on one of alternating 3- and
// 4-bit layers, -0.6 % where an eighth of the bytes is 3-bit; at 32 rows -3 to -5 %.
bool reads_in_place(const std::vector<LinearCall>& calls, size_t begin, size_t end, int32_t M)
{
    if (M > 16) return false;
    double w3 = 0.0, all = 0.0;
    for (size_t c = begin; c < end; ++c) {
        const lpq_qdesc& d = calls[c].w->d;
        const double bytes = (double)d.K * (double)d.N * d.bits;
        all += bytes;
        if (variant_of(d) == 0) w3 += bytes;
    }
    return w3 >= 0.25 * all;
}

// Whether a decode launch of 17 to 64 token rows goes to the kernel of few row blocks per workgroup instead of the even-share
// kernel.  That one has some 30 us of preparation, fix-up pass and partial tiles, this one a higher cost per 3- or 4-bit weight
// (both tiles' FMAs against the zero term outside the loop; at 33-64 rows a product per group against weights
// dequantised between the matrix instructions), so the line lies at a number of weights; 8- and 16-bit codes cost about the same in both.  Measured, us,
// even-share / this, at 32, 48 and 64 rows: a 4-bit layer of 5120 (315 M weights) 81 / 46, 90 / 55, 93 / 65; a 3- and a 4-bit layer
// of 5120 (629 M) 107 / 83, 131 / 109, 138 / 130; three 4-bit layers of 5120 (944 M) 143 / 128, 173 / 162, 182 / 198; a 3- and a 4-bit layer of 7168
// (1.2 G) 165 / 149, 222 / 200, 226 / 238; a 3-bit layer of 14336 (2.5 G) 259 / 290, 381 / 370, 393 / 455; 8 bit, 7168 -> 28672 93 / 42, 110 / 48, 119 / 56;
// an 8-bit layer of 9216 (1.0 G) 227 / 193, 244 / 220, 252 / 252; fp16, 7168 -> 28672 114 / 66, 120 / 71, 129 / 73.
// With the weight pipeline of the even-share kernel kept full across its chunks: three 4-bit layers of 5120 125 / 108 at 17 rows, 134 / 128 at 32, 182 / 198
// at 64; three layers of 7168 of 3 and 4 bit (1.85 G) 190 / 199, 203 / 212, 309 / 342.
// With its 3- and 4-bit weights of 33 to 64 rows dequantised between the matrix instructions: even-share over this at 33, 40, 48, 56, 64 rows, a 3- and a 4-bit layer of
// 4608 (0.51 G) 1.00 1.04 1.07 0.89 0.92, of 5120 (0.63 G) 1.05 1.10 1.11 0.93 0.95, of 6144 (0.91 G) 0.98 1.00 1.00 0.84 0.86, of 7168 (1.23 G) 0.93 0.92 0.95 0.78 0.80; one
// linear, 3 bit, 14336 -> 57344 (0.82 G) 1.01 1.04 1.07 0.91 0.90, 4 bit, 28672 -> 36864 (1.06 G) 1.00 1.06 1.04 0.90 0.93.
// 8 bit at 18, 32, 44, 64 rows: two layers of 7168 (1.23 GB) 1.09 1.12 1.09 0.98, three (1.85 GB) 1.03 1.04 1.10 1.01, two of 9216 (2.04 GB) 1.06 1.08 1.05 0.94,
// five of 7168 (3.1 GB) 1.05 1.05 1.08 0.93; fp16: 7168 (1.23 GB) 1.10 1.11 1.15 1.10, 9216 (2.04 GB) 1.06 1.06 1.09 1.06, three of 7168 (3.7 GB) 0.96 0.96 0.99 0.99;
// but a single fp16 linear, 28672 -> 36864 (2.1 GB), 0.976 at 24 and 0.973 at 64 rows, and at 2 GB the first launch on new weights is 4-6 % slower in this one (466 / 488
// on two 8-bit layers of 9216, 24 rows; 449 / 470 on fp16, 40 rows), at 1.85 GB (465 / 460) and 1.2 GB (308 / 310) not: the lines are below that.
// (49-64 rows of 3 and 4 bit: they meet at some 0.45 G; the line stays a little above, where a launch without a fix-up pass needs less workspace, and a reservation
// that served a call has to serve it still.)
// rows_max_mib of lpq_set_decode_routing (default 192) moves the line in proportion.
struct MidLine { double weights34[3], bytes8[3], bytes16[3]; };       // [17-32, 33-48, 49-64 rows]
const MidLine MID_LINE = {{1.0e9, 1.0e9, 0.55e9}, {1.9e9, 1.9e9, 1.0e9}, {1.4e9, 1.4e9, 1.4e9}};
// The line of a single linear: its row blocks are all of one length, and their last round may be nearly empty (fp16, 28672 -> 24320, 1.39 GB, 380 row
// blocks for 256 compute units: 0.994 at 18 rows, 0.957 at 48; 20480 -> 32768, 512 of them, 1.20 at 24 rows).  Also that of launches of several of 33 rows and more with
// grouped weights among them: there even-share dequantises, and next to an activation thousands of times the others, in a column of zero weights, codes multiplied as
// they are lose (one of 60000 among N(0, 1), 1152 columns of 8 bit: 4.2e-3 against 64 bits, 2.2e-4 dequantised).  Above it a launch of several
// asks for the even-share kernel's workspace all the same: other numbers of rows of the same linears take that one, and a workspace reserved for
// the widest call of a program has to serve its narrower ones.
const MidLine MID_LINE_ONE = {{1.0e9, 1.0e9, 0.55e9}, {1.0e9, 1.0e9, 1.0e9}, {1.0e9, 1.0e9, 1.0e9}};
bool mid_route(const std::vector<LinearCall>& calls, size_t begin, size_t end, int32_t M, const MidLine& line)
{
    const int m = (M + 15) / 16 - 2;
    double load = 0.0;
    for (size_t c = begin; c < end; ++c) {
        const lpq_qdesc& d = calls[c].w->d;
        const double weights = (double)d.K * (double)d.N;
        load += d.bits <= 4 ? weights / line.weights34[m] : weights * d.bits / 8.0 / (d.bits == 8 ? line.bytes8[m] : line.bytes16[m]);
    }
    return load <= g_rows_max_mb.load() / 192.0;
}

// Whether a decode launch goes to the kernels for launches that stream little: up to 16 token rows by the bytes of its codes,
// 17 to 64 by mid_route.
bool small_launch(const std::vector<LinearCall>& calls, size_t begin, size_t end, int32_t M)
{
    if (M > 64) return false;
    if (M > 16) {
        bool far = end - begin > 1;
        for (size_t c = begin; c < end; ++c) far = far && (M <= 32 || calls[c].w->d.scheme != LPQ_ASYM_GROUP);
        return mid_route(calls, begin, end, M, far ? MID_LINE : MID_LINE_ONE);
    }
    int64_t stream_bytes = 0;
    for (size_t c = begin; c < end; ++c) stream_bytes += (int64_t)calls[c].w->d.K * calls[c].w->d.N * calls[c].w->d.bits / 8;
    return stream_bytes <= (int64_t)g_rows_max_mb.load() << 20;
}

// Whether a single linear of 13 to 16 token rows takes the kernel for 17 and more.  Measured at 16 rows, us, that for up to 16 / this:
// 4 bit, 128 -> 4096 4.3 / 4.9, 384 -> 15168 6.8 / 6.0, 768 -> 3072 6.9 / 6.1, 2048 -> 2048 10.3 / 6.9, 5120 -> 5120 12.6 / 10.4,
// 5120 -> 20480 19.1 / 15.8, 28672 -> 7168 35.1 / 27.3; 8 bit, 768 -> 3072 6.2 / 6.9, 2048 -> 6144 8.0 / 8.3, 2048 -> 2048 9.2 / 7.8,
// 5120 -> 5120 12.8 / 12.1, 384 -> 15168 7.0 / 7.1, 768 -> 36864 18.5 / 10.3, 5120 -> 20480 24.8 / 22.6; fp16, 768 -> 3072 7.5 / 8.8, 2048 -> 6144
// 10.6 / 11.1, 8192 -> 2048 16.5 / 13.6, 5120 -> 15360 35.4 / 31.7.  With codes unpacked once for all waves' steps it is 3- and 4-bit
// weights that gain; wider ones where the other kernel has few workgroups with long ranges, or more than a round of them.
bool mid_at_16(const LinDesc& L, int cus)
{
    const int blocks = L.N / 64;
    if (L.variant <= 1) return L.kt >= 3;
    return (L.kt >= 16 && blocks <= cus / 3) || (L.kt >= 6 && blocks >= cus * 3 / 4);
}

// One grouped decode launch: its arguments (without the workspace's addresses), the kernel it takes and the bytes of
// workspace it needs.
enum DecodeKernel { DECODE_EVEN_SHARE = LPQ_ROUTE_EVEN_SHARE, DECODE_ROWS = LPQ_ROUTE_ROWS, DECODE_MID = LPQ_ROUTE_MID };
struct DecodeLaunch {
    DecodeArgs a;
    DecodeKernel kernel;
    size_t partial_bytes, workspace_bytes;       // of them partial sums; all
};

// Plans the launch of linears [begin, end) on a device of `cus` compute units; a function of its arguments and the
// routing settings alone.  prefill: a prefill call's linears (M <= 64), for the kernels of small launches whatever they stream, 8-bit
// symmetric codes without an offset.
lpq_status plan_decode(const std::vector<LinearCall>& calls, size_t begin, size_t end, int32_t M, int cus, bool prefill, DecodeLaunch* out)
{
    DecodeArgs& a = out->a;
    const int waves = decode_waves(M);
    const int n_blocks = cus * (8 / waves);
    const int tok_rows = std::min(64, (M + 15) / 16 * 16);
    a.M = M;
    a.m0 = 0;
    a.n_lin = 0;
    a.waves = waves;
    a.n_blocks = n_blocks;
    a.slot_floats = tok_rows * waves * 64;
    a.row_tiles = 4;
    a.prefill = prefill;
    a.partial = nullptr;
    a.prep = nullptr;
    a.ln_gamma = a.ln_beta = a.after_gamma = a.after_beta = nullptr;
    a.after_y = nullptr;
    a.ln_eps = 0.0f;
    const size_t partial_bytes = ((size_t)2 * n_blocks * a.slot_floats * sizeof(float) + 255) & ~(size_t)255;
    // after the partial tiles: what decode_prepare_kernel leaves for a launch whose last pass has up to 32 token rows
    const int last_rows = (M - 1) % 64 + 1;
    const bool in_place = reads_in_place(calls, begin, end, M);
    uint64_t total = 0;
    size_t sums_off16 = 0;                       // in 16-byte units
    for (size_t c = begin; c < end; ++c) {
        const lpq_qweight& w = *calls[c].w;
        LinDesc& L = a.lin[a.n_lin++];
        L.codes = static_cast<const uint8_t*>(w.codes);
        L.scales = static_cast<const uint16_t*>(w.scales);
        L.zeros = static_cast<const uint16_t*>(w.zeros);
        L.x = static_cast<const uint16_t*>(calls[c].x);
        L.y = static_cast<uint16_t*>(calls[c].y);
        L.bias = static_cast<const uint16_t*>(w.bias);
        L.residual = static_cast<const uint16_t*>(calls[c].residual);
        L.act = (uint8_t)calls[c].act;
        L.aux = (int32_t)sums_off16;
        sums_off16 += prepared_bytes(w.d, last_rows, in_place) / 16;
        if (w.d.K / 128 > 0xffff) return LPQ_ERR_UNSUPPORTED;          // the descriptor keeps K / 128 in 16 bits
        L.kt = (uint16_t)(w.d.K / 128);
        L.N = w.d.N;
        L.variant = (uint8_t)variant_of(w.d);
        const int rows = decode_rows_per_wave(L.variant);
        const uint32_t step_bytes = (uint32_t)(waves * rows) * (128u * (uint32_t)w.d.bits / 8u + (w.d.scheme == LPQ_ASYM_GROUP ? 4u : 0u));
        L.step_weight = step_bytes * variant_cost_x16(L.variant);
        L.cum_weight = total;
        total += (uint64_t)L.step_weight * (uint64_t)lin_row_superblocks(L, waves) * (uint64_t)L.kt;
    }
    if (total >= ((uint64_t)1 << 50)) return LPQ_ERR_UNSUPPORTED;
    a.total_weight = total;
    // A launch that streams little (a single linear of a decoder layer) has too few steps to spread evenly and pays the
    // fix-up pass: it goes to the kernels whose workgroups take a few tiles of W over K (no pieces to add).  Which of
    // them: from 17 token rows on the one that shares the activations through LDS; up to 16 the one that reads them
    // straight from L2 and streams from deeper rings -- except a single linear of 13 to 16 rows (mid_at_16), and that at up
    // to 256 columns the latter takes up to 32 rows, 16 per workgroup (128 -> 4096, 17 rows: 4.6 us against 5.4).
    if (prefill || small_launch(calls, begin, end, M)) {
        // longest K first: the last workgroups to start are then the shortest
        std::stable_sort(a.lin, a.lin + a.n_lin, [](const LinDesc& x, const LinDesc& y) { return x.kt > y.kt; });
        const int forced = g_rows_tiles.load();
        const bool mid = (M > 16 && (M > 32 || a.lin[0].kt > 2)) || (M > 12 && M <= 16 && a.n_lin == 1 && forced == 0 && mid_at_16(a.lin[0], cus));
        int tiles = 4, splits1 = 0;                  // the kernel for up to 16 rows: tiles per workgroup, K splits of a single linear
        if (mid) {
            mid_plan(a, cus, partial_bytes / sizeof(float));
        } else {
            if (a.n_lin == 1) rows_plan(a.lin[0], cus, &tiles, &splits1);
            if (forced >= 2 && forced <= 5 && forced != tiles) tiles = forced, splits1 = 0;
            for (int i = 0; i < a.n_lin; ++i)
                if ((a.lin[i].N / 16) % rows_group_tiles(a.lin[i].variant, tiles) != 0) tiles = 4, splits1 = 0;    // groups must tile every linear exactly
        }
        int64_t blocks = 0, row_blocks = 0, partial_floats = 0;
        for (int i = 0; i < a.n_lin; ++i) row_blocks += a.lin[i].N / 16 / rows_group_tiles(a.lin[i].variant, tiles);
        for (int i = 0; i < a.n_lin; ++i) {
            LinDesc& L = a.lin[i];
            if (!mid) {
                // K splits (L.aux) of a launch of several linears: only if it leaves most compute units without a
                // workgroup, and only down to 32 steps per workgroup
                const int KT = L.kt;
                const int want = (int)std::max<int64_t>(1, 320 / std::max<int64_t>(1, row_blocks));
                L.aux = splits1 > 0 ? splits1 : std::max(1, std::min(std::min(want, KT / 32), 8));
            }
            L.step_weight = (uint32_t)partial_floats;                 // float offset of this linear's partial sums
            if (L.aux > 1) partial_floats += (int64_t)L.aux * M * L.N;
            L.cum_weight = (uint64_t)blocks;
            blocks += (int64_t)(mid ? mid_superblocks(L, a.row_tiles) : rows_row_blocks(L, tiles)) * L.aux;
        }
        if (blocks > 0x7fffffffLL || partial_floats > 0x7fffffffLL) return LPQ_ERR_UNSUPPORTED;
        a.n_blocks = (int32_t)blocks;
        if (!mid) {
            a.row_tiles = tiles;
            a.waves = blocks <= 64 ? 8 : 4;          // very few blocks: more waves per block keep more loads in flight
        }
        out->kernel = mid ? DECODE_MID : DECODE_ROWS;
        out->partial_bytes = out->workspace_bytes = (size_t)partial_floats * sizeof(float);
        if (!prefill && M > 16 && !mid_route(calls, begin, end, M, MID_LINE_ONE))
            out->workspace_bytes = std::max(out->workspace_bytes, partial_bytes + (last_rows <= 32 ? sums_off16 * 16 : 0));
        return LPQ_OK;
    }
    // A small launch (one linear of a decoder layer) is not cut into more ranges than it has chunks of
    // steps: thinner ranges stream no faster and only multiply the pieces the fix-up pass has to add.
    const int min_steps = M <= 16 ? 16 : 8;              // a 64-token step is 3x as long
    int64_t steps = 0;
    for (int i = 0; i < a.n_lin; ++i) steps += (int64_t)lin_row_superblocks(a.lin[i], waves) * a.lin[i].kt;
    a.n_blocks = (int32_t)std::max<int64_t>(1, std::min<int64_t>(n_blocks, steps / min_steps));
    a.range_q = a.total_weight / (uint64_t)a.n_blocks;
    a.range_rem = (uint32_t)(a.total_weight % (uint64_t)a.n_blocks);
    if (in_place)
        for (int i = 0; i < a.n_lin; ++i)
            if (a.lin[i].variant == 0) a.lin[i].variant = V_W3_INPLACE;
    out->kernel = DECODE_EVEN_SHARE;
    out->partial_bytes = partial_bytes;
    out->workspace_bytes = partial_bytes + (last_rows <= 32 ? sums_off16 * 16 : 0);
    return LPQ_OK;
}

// A layer norm in front of a decoder layer's linear, rows [M][h] of x, normalised into the linear's x if not by its kernel; or behind one, rows of its y.
struct NormBefore {
    const void *x, *gamma, *beta;
    float eps;
    void* y;
};
struct NormAfter {
    const void *gamma, *beta;
    float eps;
    void* y;
    bool done;              // out: the linear's launches have done it
};

// Whether a decode linear's kernel normalises its M rows of K columns itself (every workgroup all of them) rather than a launch in front of it: where a
// wave has one row, and of short rows two.  Whole layers, us, what it takes longer so (4-bit, symmetric 8-bit, fp16): 768 wide, 1 row -3.2, -3.2, -3.7; 4 rows -4.0, -3.5, -4.5; 8
// rows -2.0, -1.5, -2.1; 9 rows 0.0, 1.2, 0.3; 16 rows -0.4, 2.9, 2.0.  2048, 8 rows -2.0, -0.3, -1.5; 9 rows 1.1, 2.6, 1.7.  2560, 4 rows -3.4, -1.5, -2.1; 8
// rows -0.8, 0.5, 2.0.  4096, 4 rows -1.8, -1.1, 0.2; 5 rows 3.1, 2.4, 8.3.  5120, 4 rows -2.8, -1.8, -0.9.
bool norm_in_linear(int32_t M, int32_t K)
{
    return K <= LN_LINEAR_MAX_K && (M <= 4 || (M <= 8 && K <= 2048));
}

bool norm_inside(const DecodeLaunch& p) { return p.kernel == DECODE_ROWS && p.a.waves == 4 && norm_in_linear(p.a.M, (int32_t)p.a.lin[0].K()); }
// Whether a launch of a single linear adds K splits in a kernel of their own, which can form a norm of the sums
bool norm_behind(const DecodeLaunch& p) { return p.kernel != DECODE_EVEN_SHARE && p.a.lin[0].aux > 1; }

// One new token per sequence: whether the attention kernel writes it to the caches itself, a launch (some 2 us) less -- while its stores of two bytes to every
// feature row cost less than that: little cache to read, or few rows, or a first position of a tile of 64, which it then need not read.  Whole layers of
// 4 bit, caches of 1.2 GB and more in turn, us, one launch / two, by megabytes of cache: 2 sequences 2048 wide, 16 MB 40.2 / 42.1; 16 of 2048, 74 MB
// 53.5 / 56.4, 131 MB 63.2 / 64.4; 8 of 5120, 92 MB 92.1 / 95.5, 164 MB 105.4 / 106.9, 328 MB 141.8 / 139.2; 16 of 5120, 98 MB 89.4 / 92.4, 184 MB 105.6 / 105.0, 655
// MB 198.4 / 191.3; 64 of 5120, 131 MB 149.4 / 150.1, 393 MB 196.7 / 193.1; 32 of 14336, 184 MB 344.7 / 339.1; few rows: 8 of 4096, 524 MB 141.8 / 144.2, 32 of 1152, 590 MB 149.5 / 149.5.  First
// positions: 64 of 7168, position 640 374 / 384, 1024 494 / 492, 4096 1411 / 1323; 16 of 5120, 1024 (336 MB) 200.5 / 204.2; 64 of 768, 2048 (403 MB) 115.7 / 119.3.
bool append_in_attention(int32_t n_seqs, int64_t h, int32_t pos0)
{
    const double bytes = 4.0 * n_seqs * (double)h * pos0;
    return bytes <= 1.7e8 || ((int64_t)n_seqs * h <= 36864 && bytes <= 1.0e9) || (pos0 % 64 == 0 && (pos0 <= 640 || bytes <= 4.5e8));
}

// Decode-phase dispatch of a list of independent linears: grouped launches of at most
// MAX_LIN_PER_LAUNCH linears, 64 token rows per pass, each launch one round of equally loaded
// workgroups (see lpq_decode.hip).  Every launch is planned, and the workspace of the largest asked for, ahead of the first
// one: launches and passes run one after the other on the stream and share the space.
// norm (a single linear): its activations' layer norm comes first, in the linear's own launch where that takes few enough of them.  after (a single
// linear): a layer norm of its output, done if its K splits are added by a kernel of their own, which then does both.
lpq_status run_decode(const std::vector<LinearCall>& calls, int32_t M, hipStream_t stream, bool static_ws = false, bool prefill = false,
                      const NormBefore* norm = nullptr, NormAfter* after = nullptr)
{
    const size_t n = calls.size();
    const size_t n_launch = (n + MAX_LIN_PER_LAUNCH - 1) / MAX_LIN_PER_LAUNCH;
    const size_t per_launch = (n + n_launch - 1) / n_launch;
    int cus = 0;
    lpq_status st = device_cus(&cus);
    if (st != LPQ_OK) return st;
    DecodeLaunch one;                            // the usual call is a single launch: no allocation, no clearing of 4 KB
    std::vector<DecodeLaunch> several(n_launch > 1 ? n_launch : 0);
    DecodeLaunch* const plan = n_launch > 1 ? several.data() : &one;
    size_t need = 0;
    for (size_t li = 0; li < n_launch; ++li) {
        st = plan_decode(calls, li * per_launch, std::min(n, (li + 1) * per_launch), M, cus, prefill, &plan[li]);
        if (st != LPQ_OK) return st;
        need = std::max(need, plan[li].workspace_bytes);
    }
    float* ws = nullptr;
    if (need) {
        st = workspace(static_ws, need, &ws);
        if (st != LPQ_OK) return st;
    }
    if (norm) {
        DecodeArgs& a = plan[0].a;
        const int64_t K = a.lin[0].K();
        if (norm_inside(plan[0])) {
            a.lin[0].x = static_cast<const uint16_t*>(norm->x);
            a.ln_gamma = static_cast<const uint16_t*>(norm->gamma);
            a.ln_beta = static_cast<const uint16_t*>(norm->beta);
            a.ln_eps = norm->eps;
        } else if (launch_layernorm(norm->x, norm->gamma, norm->beta, norm->eps, M, (int)K, norm->y, stream) != hipSuccess) {
            return LPQ_ERR_DEVICE;
        }
    }
    if (after && norm_behind(plan[0])) {
        DecodeArgs& a = plan[0].a;
        a.after_gamma = static_cast<const uint16_t*>(after->gamma);
        a.after_beta = static_cast<const uint16_t*>(after->beta);
        a.after_y = static_cast<uint16_t*>(after->y);
        a.ln_eps = after->eps;
        after->done = true;
    }
    for (size_t li = 0; li < n_launch; ++li) {
        DecodeLaunch& p = plan[li];
        p.a.partial = ws;
        if (p.kernel == DECODE_EVEN_SHARE && p.workspace_bytes > p.partial_bytes)
            p.a.prep = reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(ws) + p.partial_bytes);
        if (p.kernel != DECODE_EVEN_SHARE) {
            if ((p.kernel == DECODE_MID ? launch_decode_mid(p.a, stream) : launch_decode_rows(p.a, stream)) != hipSuccess) return LPQ_ERR_DEVICE;
            continue;
        }
        for (int m0 = 0; m0 < M; m0 += 64) {
            p.a.m0 = m0;
            if (launch_decode(p.a, stream) != hipSuccess) return LPQ_ERR_DEVICE;
        }
    }
    return LPQ_OK;
}

// How many groups to split a linear's token blocks into (see PrefillLin).  With g groups, a linear's
// weights are fetched into g of the 8 L2s and its activations into 8 / g of them.  Measured on whole
// stages (OPT-13B and 70B-class shapes, every variant), two groups are best or within 1% of it;
// other counts are for shapes with too few token or row blocks, or that two groups would spread
// unevenly over the XCDs.
int prefill_token_groups(int m_blocks, int n_blocks)
{
    static const int order[4] = {2, 4, 1, 8};
    int best = 1;
    double best_imbalance = 1e30;
    for (int i = 0; i < 4; ++i) {
        const int g = order[i];
        if (g > 1 && (g > m_blocks || 8 / g > n_blocks)) continue;
        const double imbalance = 8.0 * prefill_xcd_tiles(m_blocks, n_blocks, g) / ((double)m_blocks * n_blocks);
        if (imbalance <= 1.15) return g;
        if (imbalance < best_imbalance) { best = g; best_imbalance = imbalance; }
    }
    return best;
}

// K splits of one prefill linear that is launched with too few tiles to fill the chip (a single linear of a decoder layer at a
// small micro-batch): *whole tiles are computed as they are -- full rounds of the compute units --, the rest in *splits ranges of K.  Estimated time in units of one 128-column step of a tile (about 4.1 us):
// rounds of workgroups times steps per workgroup, a round that is not full at 0.85 + 0.15 of its share (the chip is
// power-limited: fewer busy units run faster), plus the fp32 partial sums written and read (8 bytes per element and split,
// 8 TB/s, most of it served by the caches) and the second kernel's launch.  4 bit, us before (all tiles split alike, an XCD's share
// a rectangle of tiles, so shares up to a fifth out of balance) and now: 5120 -> 15360 at 1191 rows 280 / 209, 20480 -> 5120 at 1191
// 320 / 250 and at 700 244 / 150, 5120 -> 5120 at 700 86 / 56, 7168 -> 21504 at 200 129 / 86.
void prefill_k_splits(int variant, int tiles, int KT, int32_t M, int32_t N, int cus, int* whole, int* splits)
{
    *whole = 0;
    *splits = 1;
    if (tiles >= 2 * cus) return;
    auto rounds = [&](double units) {
        const double full = std::floor(units / cus), part = units / cus - full;
        return full + (part > 0.0 ? 0.85 + 0.15 * part : 0.0);
    };
    // a split must pay clearly in the eight-wave kernel (160 tiles of 40 steps: 3 and 4 bit 4 % faster split, 8 bit and fp16 slower)
    double best = rounds(tiles) * KT * (variant <= 1 ? 1.0 : 0.97);
    const double tile_elements = (double)M * N / tiles;
    for (int w = 0; w < tiles; w += cus)
        for (int s = 2; s <= 8 && KT / s >= 8; ++s) {                      // keep the pipeline's fill and drain small
            const int rest = tiles - w;
            const double cost = (double)(w / cus) * KT + rounds((double)rest * s) * ((KT + s - 1) / s) + 1.5 +
                                8.0 * s * tile_elements * rest / 8.0e12 / 4.1e-6;
            if (cost < best) best = cost, *whole = w, *splits = s;
        }
}

// Splits of a linear of KT steps at about t steps each: at most 8, of at least 8 steps (the pipeline's fill and drain stay small).
int prefill_range_splits(int KT, int t) { return std::max(1, std::min(std::min((KT + t - 1) / t, 8), KT / 8)); }

// Steps of K per work unit in a launch of several linears with too few tiles: every linear is cut in ceil(KT / t) splits.  Estimated
// as above: the longest unit, or the launch's steps dealt out over the units of the chip with half a unit left over at the end,
// plus each split linear's traffic and reduce launch.  (Each linear judged by itself against the launch's rounds cut a 5120-wide
// layer's second feed-forward linear in 7 at 500 rows, and the others in 2: 1538 us for a layer each of 3, 8, 8 and 16 bit, 1441 cut
// in 2 all of them, 1313 now; 2048-wide at 100 rows 170, 249 cut in 3 and 2, 160 now; 2048-wide, four layers of 4 bit at 100 rows 131, now 92.)
int prefill_range(const std::vector<const LinearCall*>& mine, size_t first, size_t last, int m_blocks, int32_t M, int cus)
{
    int kt_max = 1, best_t = 0;
    for (size_t i = first; i < last; ++i) kt_max = std::max(kt_max, mine[i]->w->d.K / 128);
    double best = 1e30;
    for (int t = kt_max; t >= 8; t = std::min(t - 1, t * 7 / 8)) {
        double units = 0.0, steps = 0.0, longest = 0.0, extra = 0.0;
        for (size_t i = first; i < last; ++i) {
            const lpq_qdesc& d = mine[i]->w->d;
            const int KT = d.K / 128, s = prefill_range_splits(KT, t);
            const double n = (double)m_blocks * ((d.N + 255) / 256);
            units += n * s;
            steps += n * KT;
            longest = std::max(longest, (double)((KT + s - 1) / s));
            if (s > 1) extra += 1.5 + 8.0 * s * (double)M * d.N / 8.0e12 / 4.1e-6;
        }
        const double est = (units <= cus ? longest : std::max(longest, steps / cus + 0.5 * longest)) + extra;
        if (est < best * 0.97) best = est, best_t = t;
    }
    return std::max(best_t, 8);
}

// Prefill-phase dispatch of a list of independent linears: one grouped launch per storage variant
// (and per MAX_PREFILL_LIN linears), tiles of the longest-K linears first.
lpq_status run_prefill_rows(const std::vector<LinearCall>& calls, int32_t M, int BM, hipStream_t stream, bool static_ws)
{
    int cus = 0;
    lpq_status cst = device_cus(&cus);
    if (cst != LPQ_OK) return cst;
    for (int variant = 0; variant < 5; ++variant) {
        const int m_blocks = (M + BM - 1) / BM;
        std::vector<const LinearCall*> mine;
        for (const LinearCall& c : calls)
            if (variant_of(c.w->d) == variant) mine.push_back(&c);
        std::stable_sort(mine.begin(), mine.end(), [](const LinearCall* a, const LinearCall* b) { return a->w->d.K > b->w->d.K; });
        for (size_t first = 0; first < mine.size(); first += MAX_PREFILL_LIN) {
            PrefillArgs a;
            float* ws = nullptr;
            // a second time, without K splits, if there is no room for the splits' sums (a reservation, the static scratch array)
            for (bool split : {true, false}) {
                a.M = M;
                a.n_lin = 0;
                a.tokens_per_tile = BM;
                long tiles = 0, launch_tiles = 0;
                size_t partial_floats = 0;
                const size_t last = std::min(mine.size(), first + (size_t)MAX_PREFILL_LIN);
                for (size_t i = first; i < last; ++i) launch_tiles += (long)m_blocks * ((mine[i]->w->d.N + 255) / 256);
                const bool few = split && launch_tiles < 2L * cus;
                const int range = few && last - first > 1 ? prefill_range(mine, first, last, m_blocks, M, cus) : 0;
                for (size_t i = first; i < last; ++i) {
                    const lpq_qweight& w = *mine[i]->w;
                    PrefillLin& L = a.lin[a.n_lin++];
                    L.codes = static_cast<const uint8_t*>(w.codes);
                    L.scales = static_cast<const uint16_t*>(w.scales);
                    L.zeros = static_cast<const uint16_t*>(w.zeros);
                    L.x = static_cast<const uint16_t*>(mine[i]->x);
                    L.y = static_cast<uint16_t*>(mine[i]->y);
                    L.bias = static_cast<const uint16_t*>(w.bias);
                    L.residual = static_cast<const uint16_t*>(mine[i]->residual);
                    L.act = mine[i]->act;
                    L.K = w.d.K;
                    L.N = w.d.N;
                    L.n_blocks = (w.d.N + 255) / 256;
                    L.token_groups = prefill_token_groups(m_blocks, L.n_blocks);
                    L.tile_begin = (int32_t)tiles;
                    // splitting is judged per launch: a launch with many tiles fills the chip whatever its linears' shapes
                    L.whole_tiles = 0;
                    L.k_splits = 1;
                    if (range) L.k_splits = prefill_range_splits(w.d.K / 128, range);
                    else if (few) prefill_k_splits(variant, (int)launch_tiles, w.d.K / 128, M, w.d.N, cus, &L.whole_tiles, &L.k_splits);
                    L.partial = nullptr;
                    if (L.k_splits > 1) {
                        partial_floats += (size_t)L.k_splits * M * split_cols(L, m_blocks);
                        long share = 0;                                        // workgroups of the busiest XCD
                        for (int x = 0; x < 8; ++x) {
                            const PrefillShare sh = prefill_split_share(L, m_blocks, x);
                            share = std::max(share, (long)sh.whole + sh.units);
                        }
                        tiles += 8L * share;
                    } else {
                        tiles += 8L * prefill_xcd_tiles(m_blocks, L.n_blocks, L.token_groups);
                    }
                }
                if (tiles > 0x7fffffffL) return LPQ_ERR_UNSUPPORTED;
                a.total_tiles = (int32_t)tiles;
                if (!partial_floats) break;
                const lpq_status st = workspace(static_ws, partial_floats * sizeof(float), &ws);
                if (st == LPQ_ERR_BUFSIZE) continue;
                if (st != LPQ_OK) return st;
                for (int i = 0; i < a.n_lin; ++i) {
                    if (a.lin[i].k_splits <= 1) continue;
                    a.lin[i].partial = ws;
                    ws += (size_t)a.lin[i].k_splits * M * split_cols(a.lin[i], m_blocks);
                }
                break;
            }
            if (launch_prefill(variant, a, stream) != hipSuccess) return LPQ_ERR_DEVICE;
        }
    }
    return LPQ_OK;
}

// Whether a prefill call goes to the decode kernels for small launches.  Up to 64 rows a 128-token tile is at least half empty, and
// those kernels hold all rows at once: at 40 rows, 4 bit, 5120 -> 15360 23.5 us against 31.1, 8 bit 7168 -> 21504 38 against 81; at
// 9 rows 13 against 27 and 30 against 79.  A single linear of up to 16 rows goes there however large it is: not to the
// even-share kernel, whose offset 8-bit codes cost a prefill call precision.  (What the workspace or the descriptors do not
// hold takes the prefill kernels, and so does everything while lpq_set_decode_routing keeps launches away from those kernels.)
bool prefill_takes_decode(const std::vector<LinearCall>& calls, int32_t M)
{
    return M <= 64 && calls.size() <= MAX_LIN_PER_LAUNCH &&
           (small_launch(calls, 0, calls.size(), M) || (M <= 16 && calls.size() == 1 && g_rows_max_mb.load() > 0));
}

// Prefill-phase dispatch.  Tokens per tile: 256 as a rule: weights are fetched and unpacked once per token block.  A call of at most 128 rows
// has one block either way and takes 128-token tiles (half the matrix instructions per step).  A call of 1024 rows
// or more whose last block of 256 would hold at most 128 rows pays a full tile of matrix instructions for that block
// (1100 rows cost what 1280 do): there the tail runs as launches of its own with 128-token tiles -- measured on an
// OPT-13B layer's four linears, 11-19 % less time at 1100, 1152, 1600, 2100 and 3200 rows.  Below 1024 rows a call
// is short of tiles either way, and both a tail launch and 128-token tiles throughout measured slower than the
// ragged block (384 rows: 0.45 against 0.41 ms), so it keeps 256-token tiles.
lpq_status run_prefill(const std::vector<LinearCall>& calls, int32_t M, hipStream_t stream, bool static_ws = false)
{
    const int32_t tail = M % 256, body = M - tail;
    if (prefill_takes_decode(calls, M)) {
        const lpq_status st = run_decode(calls, M, stream, static_ws, true);
        if (st != LPQ_ERR_BUFSIZE && st != LPQ_ERR_UNSUPPORTED) return st;
    }
    if (M <= 128) return run_prefill_rows(calls, M, 128, stream, static_ws);
    if (tail == 0 || tail > 128) return run_prefill_rows(calls, M, 256, stream, static_ws);
    if (M < 1024) return run_prefill_rows(calls, M, 256, stream, static_ws);
    lpq_status st = run_prefill_rows(calls, body, 256, stream, static_ws);
    if (st != LPQ_OK) return st;
    std::vector<LinearCall> rest(calls);
    for (LinearCall& c : rest) {
        c.x = static_cast<const uint16_t*>(c.x) + (size_t)body * c.w->d.K;
        c.y = static_cast<uint16_t*>(c.y) + (size_t)body * c.w->d.N;
        if (c.residual) c.residual = static_cast<const uint16_t*>(c.residual) + (size_t)body * c.w->d.N;
    }
    return run_prefill_rows(rest, tail, 128, stream, static_ws);
}

lpq_status check_attention_args(const lpq_layer_cfg* cfg, const lpq_layer_state* st, int32_t n_seqs, int32_t T, int32_t pos0)
{
    if (!st->k_cache || !st->vt_cache) return LPQ_ERR_NULL;
    if (cfg->n_heads < 1 || (cfg->head_dim != 64 && cfg->head_dim != 128) || cfg->max_seq < 64 || cfg->max_seq % 64 != 0) return LPQ_ERR_SHAPE;
    if (n_seqs < 1 || T < 1 || pos0 < 0 || (int64_t)pos0 + T > cfg->max_seq) return LPQ_ERR_SHAPE;
    if (misaligned(st->k_cache) || misaligned(st->vt_cache) || (reinterpret_cast<uintptr_t>(st->alibi_slopes) & 3u)) return LPQ_ERR_ALIGN;
    return LPQ_OK;
}

// fresh (T = 1 only): the caches do not hold the new token yet; the attention kernel appends it.
lpq_status run_attention(const void* qkv, const lpq_layer_cfg* cfg, const lpq_layer_state* st, int32_t n_seqs, int32_t T, int32_t pos0,
                         bool fresh, void* out, hipStream_t stream)
{
    if (T > 1)
        return launch_attention_prefill(qkv, st->k_cache, st->vt_cache, st->alibi_slopes, n_seqs, T, pos0, cfg->n_heads, cfg->head_dim,
                                        cfg->max_seq, out, stream) == hipSuccess ? LPQ_OK : LPQ_ERR_DEVICE;
    const int n = fresh ? pos0 : pos0 + 1;
    int range = 0, splits = 0, cus = 0;
    const lpq_status cst = device_cus(&cus);
    if (cst != LPQ_OK) return cst;
    attention_decode_plan(n_seqs, cfg->n_heads, n, cus, &range, &splits);
    const size_t floats = attention_decode_workspace_floats(n_seqs, cfg->n_heads, cfg->head_dim, splits);
    float* part = nullptr;
    if (floats) {
        const lpq_status s = workspace(false, floats * sizeof(float), &part);
        if (s == LPQ_ERR_BUFSIZE) range = (n + 63) / 64 * 64, splits = 1;      // no room for the splits' results: one split needs none
        else if (s != LPQ_OK) return s;
    }
    return launch_attention_decode(qkv, st->k_cache, st->vt_cache, st->alibi_slopes, n_seqs, n, fresh, cfg->n_heads, cfg->head_dim, cfg->max_seq,
                                   range, splits, out, part, stream) == hipSuccess ? LPQ_OK : LPQ_ERR_DEVICE;
}

}  // namespace
}  // namespace lpq

using namespace lpq;

extern "C" {

lpq_status lpq_packed_sizes(const lpq_qdesc* desc, size_t* code_bytes, size_t* scale_bytes, size_t* zero_bytes)
{
    if (!desc || !code_bytes || !scale_bytes || !zero_bytes) return LPQ_ERR_NULL;
    lpq_status st = check_desc(desc);
    if (st != LPQ_OK) return st;
    const size_t K = (size_t)desc->K, N = (size_t)desc->N;
    *code_bytes = K * N * (size_t)desc->bits / 8;
    *scale_bytes = desc->scheme == LPQ_ASYM_GROUP ? N * (K / 128) * 2 : desc->scheme == LPQ_SYM_CHANNEL ? N * 2 : 0;
    *zero_bytes = desc->scheme == LPQ_ASYM_GROUP ? *scale_bytes : 0;
    return LPQ_OK;
}

lpq_status lpq_quantize_pack(const void* w_fp16, const lpq_qdesc* desc, lpq_qweight* out, void* hip_stream)
{
    if (!w_fp16 || !desc || !out) return LPQ_ERR_NULL;
    lpq_status st = check_quantize_target(desc, out);
    if (st != LPQ_OK) return st;
    if (misaligned(w_fp16)) return LPQ_ERR_ALIGN;
    return launch_quantize_pack(w_fp16, *desc, 0, desc->N, *out, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? LPQ_OK : LPQ_ERR_DEVICE;
}

lpq_status lpq_quantize_pack_rows(const void* w_rows_fp16, const lpq_qdesc* desc, int32_t row0, int32_t n_rows, lpq_qweight* out,
                                  void* hip_stream)
{
    if (!w_rows_fp16 || !desc || !out) return LPQ_ERR_NULL;
    lpq_status st = check_quantize_target(desc, out);
    if (st != LPQ_OK) return st;
    if (row0 < 0 || n_rows < 0 || row0 % 64 != 0 || n_rows % 64 != 0 || (int64_t)row0 + n_rows > desc->N) return LPQ_ERR_SHAPE;
    if (misaligned(w_rows_fp16)) return LPQ_ERR_ALIGN;
    return launch_quantize_pack(w_rows_fp16, *desc, row0, n_rows, *out, static_cast<hipStream_t>(hip_stream)) == hipSuccess
               ? LPQ_OK : LPQ_ERR_DEVICE;
}

lpq_status lpq_load_quantize_pack(const void* w_fp16_host, const lpq_qdesc* desc, lpq_qweight* out, void* staging, size_t staging_bytes,
                                  void* hip_stream)
{
    if (!w_fp16_host || !desc || !out || !staging) return LPQ_ERR_NULL;
    lpq_status st = check_quantize_target(desc, out);
    if (st != LPQ_OK) return st;
    if (misaligned(w_fp16_host) || misaligned(staging)) return LPQ_ERR_ALIGN;
    // Bands of rows alternate on the caller's stream: copy a band into the staging buffer, quantise it into
    // its place, copy the next.  The quantiser runs some thirty times faster than the host link, so the copy
    // engine idles 2-3 % of the time; a second stream that overlapped the two was measured at +1 % at best and
    // at -35 % in a runtime state seen after large allocations had been freed, so it is not used.
    const size_t row_bytes = (size_t)desc->K * 2;
    const int64_t chunk_rows = std::min<int64_t>((int64_t)(staging_bytes / row_bytes) / 64 * 64, desc->N);
    if (chunk_rows < 64) return LPQ_ERR_BUFSIZE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    for (int64_t row = 0; row < desc->N; row += chunk_rows) {
        const int64_t rows = std::min<int64_t>(chunk_rows, desc->N - row);
        if (hipMemcpyAsync(staging, static_cast<const uint8_t*>(w_fp16_host) + (size_t)row * row_bytes, (size_t)rows * row_bytes,
                           hipMemcpyHostToDevice, stream) != hipSuccess)
            return LPQ_ERR_DEVICE;
        if (launch_quantize_pack(staging, *desc, row, rows, *out, stream) != hipSuccess) return LPQ_ERR_DEVICE;
    }
    return LPQ_OK;
}

lpq_status lpq_layernorm(const void* x, const void* gamma, const void* beta, float eps, int32_t M, int32_t hidden, void* y, void* hip_stream)
{
    if (!x || !gamma || !beta || !y) return LPQ_ERR_NULL;
    if (M < 1 || hidden < 8 || hidden % 8 != 0 || hidden > layernorm_max_hidden() || !(eps >= 0.0f)) return LPQ_ERR_SHAPE;
    if (misaligned(x) || misaligned(gamma) || misaligned(beta) || misaligned(y)) return LPQ_ERR_ALIGN;
    return launch_layernorm(x, gamma, beta, eps, M, hidden, y, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? LPQ_OK : LPQ_ERR_DEVICE;
}

lpq_status lpq_kv_append(const void* qkv, const lpq_layer_cfg* cfg, const lpq_layer_state* st, int32_t n_seqs, int32_t T, int32_t pos0,
                         void* hip_stream)
{
    if (!qkv || !cfg || !st) return LPQ_ERR_NULL;
    lpq_status s = check_attention_args(cfg, st, n_seqs, T, pos0);
    if (s != LPQ_OK) return s;
    if (misaligned(qkv)) return LPQ_ERR_ALIGN;
    return launch_kv_append(qkv, st->k_cache, st->vt_cache, n_seqs, T, pos0, cfg->n_heads, cfg->head_dim, cfg->max_seq,
                            static_cast<hipStream_t>(hip_stream)) == hipSuccess ? LPQ_OK : LPQ_ERR_DEVICE;
}

lpq_status lpq_attention(const void* qkv, const lpq_layer_cfg* cfg, const lpq_layer_state* st, int32_t n_seqs, int32_t T, int32_t pos0,
                         void* out, void* hip_stream)
{
    if (!qkv || !cfg || !st || !out) return LPQ_ERR_NULL;
    lpq_status s = check_attention_args(cfg, st, n_seqs, T, pos0);
    if (s != LPQ_OK) return s;
    if (misaligned(qkv) || misaligned(out)) return LPQ_ERR_ALIGN;
    return run_attention(qkv, cfg, st, n_seqs, T, pos0, false, out, static_cast<hipStream_t>(hip_stream));
}

size_t lpq_decoder_layer_workspace(const lpq_layer* layer, const lpq_layer_cfg* cfg, int32_t M)
{
    if (!layer || !cfg || M < 1 || cfg->n_heads < 1 || cfg->head_dim < 1) return 0;
    const size_t h = (size_t)cfg->n_heads * cfg->head_dim, f = (size_t)std::max(layer->fc1.d.N, 0);
    return (size_t)M * (5 * h + f) * 2;       // h1 / h2, qkv (3h), attention output, feed-forward activations
}

lpq_status lpq_decoder_layer(const lpq_layer* layer, const lpq_layer_cfg* cfg, const lpq_layer_state* st, lpq_phase phase, int32_t n_seqs,
                             int32_t T, int32_t pos0, const void* x, void* y, void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!layer || !cfg || !st || !x || !y || !workspace) return LPQ_ERR_NULL;
    if (phase != LPQ_PREFILL && phase != LPQ_DECODE) return LPQ_ERR_UNSUPPORTED;
    if (cfg->activation != LPQ_ACT_NONE && cfg->activation != LPQ_ACT_RELU && cfg->activation != LPQ_ACT_GELU_TANH) return LPQ_ERR_UNSUPPORTED;
    lpq_status s = check_attention_args(cfg, st, n_seqs, T, pos0);
    if (s != LPQ_OK) return s;
    if (!st->ln1_gamma || !st->ln1_beta || !st->ln2_gamma || !st->ln2_beta) return LPQ_ERR_NULL;
    const lpq_qweight* w[4] = {&layer->qkv, &layer->out, &layer->fc1, &layer->fc2};
    for (int j = 0; j < 4; ++j) {
        s = check_weight(w[j]);
        if (s != LPQ_OK) return s;
    }
    const int64_t h = (int64_t)cfg->n_heads * cfg->head_dim, f = layer->fc1.d.N, M = (int64_t)n_seqs * T;
    if (h > layernorm_max_hidden() || M > 0x7fffffff) return LPQ_ERR_SHAPE;
    if (layer->qkv.d.K != h || layer->qkv.d.N != 3 * h || layer->out.d.K != h || layer->out.d.N != h || layer->fc1.d.K != h ||
        layer->fc2.d.K != f || layer->fc2.d.N != h)
        return LPQ_ERR_SHAPE;
    if (misaligned(x) || misaligned(y) || misaligned(workspace) || misaligned(st->ln1_gamma) || misaligned(st->ln1_beta) ||
        misaligned(st->ln2_gamma) || misaligned(st->ln2_beta))
        return LPQ_ERR_ALIGN;
    if (workspace_bytes < lpq_decoder_layer_workspace(layer, cfg, (int32_t)M)) return LPQ_ERR_BUFSIZE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint16_t* h1 = static_cast<uint16_t*>(workspace);          // LN1 output, later LN2 output
    uint16_t* qkv = h1 + M * h;
    uint16_t* att = qkv + 3 * M * h;
    uint16_t* ff = att + M * h;
    auto linear = [&](const lpq_qweight* wt, const void* in, void* out, const void* residual, int act) {
        std::vector<LinearCall> calls(1, LinearCall{wt, in, out, residual, act});
        return phase == LPQ_PREFILL ? run_prefill(calls, (int32_t)M, stream) : run_decode(calls, (int32_t)M, stream);
    };
    auto norm_linear = [&](const void* in, const void* gamma, const void* beta, const lpq_qweight* wt, void* out, int act) {
        if (phase == LPQ_DECODE) {
            const NormBefore norm = {in, gamma, beta, cfg->ln_eps, h1};
            std::vector<LinearCall> calls(1, LinearCall{wt, h1, out, nullptr, act});
            return run_decode(calls, (int32_t)M, stream, false, false, &norm);
        }
        if (launch_layernorm(in, gamma, beta, cfg->ln_eps, (int)M, (int)h, h1, stream) != hipSuccess) return LPQ_ERR_DEVICE;
        return linear(wt, h1, out, nullptr, act);
    };
    if ((s = norm_linear(x, st->ln1_gamma, st->ln1_beta, &layer->qkv, qkv, LPQ_ACT_NONE)) != LPQ_OK) return s;
    const bool fresh = T == 1 && append_in_attention(n_seqs, h, pos0);
    if (!fresh && launch_kv_append(qkv, st->k_cache, st->vt_cache, n_seqs, T, pos0, cfg->n_heads, cfg->head_dim, cfg->max_seq, stream) != hipSuccess)
        return LPQ_ERR_DEVICE;
    if ((s = run_attention(qkv, cfg, st, n_seqs, T, pos0, fresh, att, stream)) != LPQ_OK) return s;
    // y = x + out-projection, then feed-forward of its norm
    NormAfter ln2 = {st->ln2_gamma, st->ln2_beta, cfg->ln_eps, h1, false};
    if (phase == LPQ_DECODE) {
        std::vector<LinearCall> calls(1, LinearCall{&layer->out, att, y, x, LPQ_ACT_NONE});
        s = run_decode(calls, (int32_t)M, stream, false, false, nullptr, &ln2);
    } else {
        s = linear(&layer->out, att, y, x, LPQ_ACT_NONE);
    }
    if (s != LPQ_OK) return s;
    s = ln2.done ? linear(&layer->fc1, h1, ff, nullptr, cfg->activation)
                 : norm_linear(y, st->ln2_gamma, st->ln2_beta, &layer->fc1, ff, cfg->activation);
    if (s != LPQ_OK) return s;
    return linear(&layer->fc2, ff, y, y, LPQ_ACT_NONE);                                           // y += feed-forward
}

lpq_status lpq_variance_indicator(const void* w_fp16, int32_t K, int32_t N, const void* x, int32_t M, int32_t stochastic, double* omega,
                                  void* hip_stream)
{
    if (!w_fp16 || !x || !omega) return LPQ_ERR_NULL;
    if (K < 128 || K % 128 != 0 || N < 1 || M < 1) return LPQ_ERR_SHAPE;
    if (misaligned(w_fp16) || misaligned(x) || (reinterpret_cast<uintptr_t>(omega) & 7u)) return LPQ_ERR_ALIGN;
    float* ws = nullptr;
    lpq_status st = workspace(false, indicator_workspace_bytes(K, N, M), &ws);
    if (st != LPQ_OK) return st;
    return launch_indicator(w_fp16, K, N, x, M, stochastic != 0, omega, ws, static_cast<hipStream_t>(hip_stream)) == hipSuccess
               ? LPQ_OK : LPQ_ERR_DEVICE;
}

lpq_status lpq_unpack_dequant(const lpq_qweight* w, void* w_fp32, void* hip_stream)
{
    lpq_status st = check_weight(w);
    if (st != LPQ_OK) return st;
    if (!w_fp32) return LPQ_ERR_NULL;
    if (misaligned(w_fp32)) return LPQ_ERR_ALIGN;
    return launch_unpack_dequant(*w, static_cast<float*>(w_fp32), static_cast<hipStream_t>(hip_stream)) == hipSuccess ? LPQ_OK
                                                                                                                       : LPQ_ERR_DEVICE;
}

lpq_status lpq_qlinear_prefill(const lpq_qweight* w, const void* x, int32_t M, void* y, void* hip_stream)
{
    lpq_status st = check_linear(w, x, M, y);
    if (st != LPQ_OK) return st;
    std::vector<LinearCall> calls(1, LinearCall{w, x, y, nullptr, LPQ_ACT_NONE});
    return run_prefill(calls, M, static_cast<hipStream_t>(hip_stream));
}

lpq_status lpq_qlinear_decode(const lpq_qweight* w, const void* x, int32_t M, void* y, void* hip_stream)
{
    lpq_status st = check_linear(w, x, M, y);
    if (st != LPQ_OK) return st;
    std::vector<LinearCall> calls(1, LinearCall{w, x, y, nullptr, LPQ_ACT_NONE});
    return run_decode(calls, M, static_cast<hipStream_t>(hip_stream));
}

lpq_status lpq_qlinear_fused(const lpq_qweight* w, const void* x, int32_t M, void* y, const lpq_epilogue* ep, lpq_phase phase,
                             void* hip_stream)
{
    lpq_status st = check_linear(w, x, M, y);
    if (st != LPQ_OK) return st;
    if (phase != LPQ_PREFILL && phase != LPQ_DECODE) return LPQ_ERR_UNSUPPORTED;
    LinearCall c{w, x, y, nullptr, LPQ_ACT_NONE};
    if (ep) {
        if (ep->activation != LPQ_ACT_NONE && ep->activation != LPQ_ACT_RELU && ep->activation != LPQ_ACT_GELU_TANH)
            return LPQ_ERR_UNSUPPORTED;
        if (ep->residual && misaligned(ep->residual)) return LPQ_ERR_ALIGN;
        c.residual = ep->residual;
        c.act = ep->activation;
    }
    std::vector<LinearCall> calls(1, c);
    return phase == LPQ_PREFILL ? run_prefill(calls, M, static_cast<hipStream_t>(hip_stream))
                                : run_decode(calls, M, static_cast<hipStream_t>(hip_stream));
}

static lpq_status stage_linears(const lpq_layer* layers, int32_t n_layers, lpq_phase phase, int32_t M, const lpq_layer_io* io,
                                void* hip_stream, bool static_ws)
{
    if (!layers || !io) return LPQ_ERR_NULL;
    if (n_layers < 1 || n_layers > 4096) return LPQ_ERR_SHAPE;
    if (phase != LPQ_PREFILL && phase != LPQ_DECODE) return LPQ_ERR_UNSUPPORTED;
    std::vector<LinearCall> calls;
    calls.reserve((size_t)n_layers * 4);
    for (int32_t i = 0; i < n_layers; ++i) {
        const lpq_qweight* w[4] = {&layers[i].qkv, &layers[i].out, &layers[i].fc1, &layers[i].fc2};
        const void* xs[4] = {io[i].x_qkv, io[i].x_out, io[i].x_fc1, io[i].x_fc2};
        void* ys[4] = {io[i].y_qkv, io[i].y_out, io[i].y_fc1, io[i].y_fc2};
        for (int j = 0; j < 4; ++j) {
            lpq_status st = check_linear(w[j], xs[j], M, ys[j]);
            if (st != LPQ_OK) return st;
            calls.push_back(LinearCall{w[j], xs[j], ys[j], nullptr, LPQ_ACT_NONE});
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    return phase == LPQ_DECODE ? run_decode(calls, M, stream, static_ws) : run_prefill(calls, M, stream, static_ws);
}

lpq_status lpq_stage_linears(const lpq_layer* layers, int32_t n_layers, lpq_phase phase, int32_t M, const lpq_layer_io* io,
                             void* hip_stream)
{
    return stage_linears(layers, n_layers, phase, M, io, hip_stream, false);
}

lpq_status lpq_stage_linears_noalloc(const lpq_layer* layers, int32_t n_layers, lpq_phase phase, int32_t M, const lpq_layer_io* io,
                                     void* hip_stream)
{
    return stage_linears(layers, n_layers, phase, M, io, hip_stream, true);
}

lpq_status lpq_workspace_policy(size_t have_bytes, int32_t reserved, size_t need_bytes, size_t* alloc_bytes)
{
    if (!alloc_bytes) return LPQ_ERR_NULL;
    return workspace_policy(have_bytes, reserved != 0, need_bytes, alloc_bytes);
}

lpq_status lpq_workspace_reserve(size_t bytes)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LPQ_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_ws.mu);
    if (g_ws.bytes[dev] < bytes) {
        lpq_status st = workspace_grow(dev, bytes);
        if (st != LPQ_OK) return st;
    }
    g_ws.reserved[dev] = true;
    return LPQ_OK;
}

size_t lpq_workspace_bytes(void)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(g_ws.mu);
    return g_ws.bytes[dev];
}

lpq_status lpq_set_decode_routing(int32_t rows_max_mib, int32_t rows_tiles)
{
    if (rows_max_mib > 4096 || (rows_tiles > 0 && (rows_tiles < 2 || rows_tiles > 5))) return LPQ_ERR_SHAPE;
    g_rows_max_mb.store(rows_max_mib < 0 ? 192 : rows_max_mib);
    g_rows_tiles.store(rows_tiles < 0 ? 0 : rows_tiles);
    return LPQ_OK;
}

lpq_status lpq_route_of(const lpq_qdesc* descs, int32_t n, lpq_phase phase, int32_t M, int32_t compute_units, lpq_route* out)
{
    if (!descs || !out) return LPQ_ERR_NULL;
    if (n < 1 || n > MAX_LIN_PER_LAUNCH || M < 1 || compute_units < 1 || (phase != LPQ_DECODE && phase != LPQ_PREFILL)) return LPQ_ERR_SHAPE;
    std::vector<lpq_qweight> w((size_t)n);
    std::vector<LinearCall> calls((size_t)n);
    for (int i = 0; i < n; ++i) {
        const lpq_status st = check_desc(&descs[i]);
        if (st != LPQ_OK) return st;
        w[i] = lpq_qweight{descs[i], nullptr, nullptr, nullptr, nullptr};
        calls[i] = LinearCall{&w[i], nullptr, nullptr};
    }
    *out = lpq_route{LPQ_ROUTE_PREFILL, 0, 1, 0};
    if (phase == LPQ_PREFILL && !prefill_takes_decode(calls, M)) {
        if (n > 1) return LPQ_OK;
        const int bm = M <= 128 ? 128 : 256;                             // of the body, where a tail is launched apart
        const int32_t rows = M >= 1024 && M % 256 <= 128 ? M - M % 256 : M;
        const int tiles = (rows + bm - 1) / bm * ((descs[0].N + 255) / 256);
        out->tiles = bm;
        prefill_k_splits(variant_of(descs[0]), tiles, descs[0].K / 128, rows, descs[0].N, compute_units, &out->whole_tiles, &out->splits);
        if (out->splits == 1) out->whole_tiles = tiles;
        return LPQ_OK;
    }
    std::vector<DecodeLaunch> plan(1);
    const lpq_status st = plan_decode(calls, 0, calls.size(), M, compute_units, phase == LPQ_PREFILL, &plan[0]);
    if (st != LPQ_OK) return st;
    out->kernel = plan[0].kernel;
    if (plan[0].kernel == DECODE_EVEN_SHARE) return LPQ_OK;
    out->tiles = plan[0].a.row_tiles;
    for (int i = 0; i < n; ++i) out->splits = std::max(out->splits, plan[0].a.lin[i].aux);
    return LPQ_OK;
}

lpq_status lpq_layer_route_of(const lpq_qdesc* descs, int32_t n_seqs, int32_t pos0, int32_t compute_units, lpq_layer_route* out)
{
    if (!descs || !out) return LPQ_ERR_NULL;
    if (n_seqs < 1 || pos0 < 0 || compute_units < 1) return LPQ_ERR_SHAPE;
    for (int i = 0; i < 4; ++i) {
        const lpq_status st = check_desc(&descs[i]);
        if (st != LPQ_OK) return st;
    }
    std::vector<DecodeLaunch> plan(3);                                   // QKV, out-projection, FC1
    for (int i = 0; i < 3; ++i) {
        const lpq_qweight w = lpq_qweight{descs[i], nullptr, nullptr, nullptr, nullptr};
        const std::vector<LinearCall> calls(1, LinearCall{&w, nullptr, nullptr});
        const lpq_status st = plan_decode(calls, 0, 1, n_seqs, compute_units, false, &plan[i]);
        if (st != LPQ_OK) return st;
    }
    out->norm1 = norm_inside(plan[0]) ? LPQ_NORM_IN_LINEAR : LPQ_NORM_LAUNCH;
    out->norm2 = norm_behind(plan[1]) ? LPQ_NORM_BEHIND_SPLITS : norm_inside(plan[2]) ? LPQ_NORM_IN_LINEAR : LPQ_NORM_LAUNCH;
    out->append = append_in_attention(n_seqs, descs[0].K, pos0);
    return LPQ_OK;
}

const char* lpq_status_str(lpq_status status)
{
    switch (status) {
    case LPQ_OK: return "ok";
    case LPQ_ERR_NULL: return "null pointer";
    case LPQ_ERR_BITS: return "bits must be 3, 4, 8 or 16";
    case LPQ_ERR_SCHEME: return "bits / scheme / group_size do not match";
    case LPQ_ERR_SHAPE: return "bad shape or size (K % 128, N % 64, M >= 1, descriptor mismatch, malformed plan or samples)";
    case LPQ_ERR_ALIGN: return "pointer not 16-byte aligned";
    case LPQ_ERR_BUFSIZE: return "buffer too small, or workspace allocation failed";
    case LPQ_ERR_DEVICE: return "HIP call failed";
    case LPQ_ERR_UNSUPPORTED: return "unsupported request";
    }
    return "unknown status";
}

}  // extern "C"
