// The rest of the decoder layer around the four linears: layer normalisation, KV-cache append and
// causal attention over the pre-allocated cache (LLM-PQ, arXiv 2403.01136: Sec. 4.1 "KV Storage
// Modeling" reserves the cache for s + n positions; Sec. 5 serves models with a pre-allocated cache).
// The operators are the published pre-LayerNorm decoder block of the paper's models.
//
// Cache layout per layer: K [B][H][S][d] (a position's d values contiguous) and V transposed,
// VT [B][H][d][S] (a feature's positions contiguous).  With that, both contractions of attention read
// their operands along the contracted index: q.K over d, p.V over positions -- as 16-byte loads, which the
// prefill kernel stages through LDS as MFMA A operands (no transposes).
#include <algorithm>
#include <type_traits>

#include "lpq_common.h"
#include "lpq_device.h"

namespace lpq {

namespace {

// ---- layer normalisation: one workgroup per row, the row held in registers -------------------
// HBM-bound at many rows (2 bytes read + 2 bytes written per element), a chain of latencies at few.  Two forms.  AHEAD asks for a thread's part of gamma and
// beta together with the row and keeps all of it as fp16; the other keeps the row as fp32, converted once, and reads gamma and beta behind the sums.
// launch_layernorm has the lines between them and the figures.
constexpr int LN_MAX_HIDDEN = 16384;

// THREADS: of a workgroup; of a single chunk a thread, the most there may be.  512: no more than 64 registers, for four workgroups on a compute unit.
template <int THREADS, int CHUNKS, bool AHEAD>
__global__ __launch_bounds__(THREADS, THREADS == 512 ? 8 : 4) void layernorm_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gamma, const uint16_t* __restrict__ beta,
                                                            float eps, int h, uint16_t* __restrict__ y)
{
    constexpr int MAX_WAVES = THREADS / 64;
    __shared__ __attribute__((aligned(16))) float red[2][MAX_WAVES];
    const size_t row = blockIdx.x;
    const int nch = h / 8, threads = CHUNKS == 1 ? (int)blockDim.x : THREADS, waves = threads / 64;       // 16-byte chunks in a row
    typedef float f8 __attribute__((ext_vector_type(8)));
    typename std::conditional<AHEAD, h8, f8>::type t[CHUNKS];
    h8 g[CHUNKS], b[CHUNKS];
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int ch = threadIdx.x + threads * c;
        if (ch < nch) {
            const h8 v = *reinterpret_cast<const h8*>(x + row * h + 8 * ch);
            if constexpr (AHEAD) {
                t[c] = v;
                g[c] = *reinterpret_cast<const h8*>(gamma + 8 * ch);
                b[c] = *reinterpret_cast<const h8*>(beta + 8 * ch);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) { t[c][e] = (float)v[e]; s += t[c][e]; }
            }
        }
    }
    if constexpr (AHEAD)
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
            if ((int)threadIdx.x + threads * c < nch)
#pragma unroll
                for (int e = 0; e < 8; ++e) s += (float)t[c][e];
    const float mean = row_sum<MAX_WAVES>(s, waves, red[0]) / (float)h;
    float q = 0.0f;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c)
        if ((int)threadIdx.x + threads * c < nch) q = norm_squares(t[c], mean, q, c == 0);
    const float rstd = 1.0f / sqrtf(row_sum<MAX_WAVES>(q, waves, red[1]) / (float)h + eps);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int ch = threadIdx.x + threads * c;
        if (ch < nch) {
            if constexpr (!AHEAD) {
                g[c] = *reinterpret_cast<const h8*>(gamma + 8 * ch);
                b[c] = *reinterpret_cast<const h8*>(beta + 8 * ch);
            }
            h8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = norm_element((float)t[c][e], mean, rstd, g[c][e], b[c][e]);
            *reinterpret_cast<h8*>(y + row * h + 8 * ch) = o;
        }
    }
}

// ---- KV append: the K and V parts of qkv [tokens][3h] into the caches at positions pos0.. -----
// Grid (sequences * heads, ceil(T / 64)): a workgroup moves 64 tokens of one head.  K rows are copied as
// they are; V is transposed through LDS so that a wave writes 64 consecutive positions of one feature row.
template <int D>
__global__ __launch_bounds__(256) void kv_append_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ kc, uint16_t* __restrict__ vtc,
                                                        int T, int pos0, int H, int S)
{
    __shared__ uint16_t vs[64][D + 2];                 // +2: feature-major reads of a column hit different banks
    typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
    const int bh = blockIdx.x, b = bh / H, head = bh % H, t0 = 64 * blockIdx.y;
    const int h = H * D, nt = min(64, T - t0);
    constexpr int CH = D / 8;                          // 16-byte chunks per token and head
    for (int i = threadIdx.x; i < nt * CH; i += 256) {
        const int t = i / CH, c = i % CH;
        const uint16_t* src = qkv + ((size_t)b * T + t0 + t) * 3 * h + head * D + 8 * c;
        const u16x8 k = *reinterpret_cast<const u16x8*>(src + h), v = *reinterpret_cast<const u16x8*>(src + 2 * h);
        *reinterpret_cast<u16x8*>(kc + (((size_t)b * H + head) * S + pos0 + t0 + t) * D + 8 * c) = k;
#pragma unroll
        for (int e = 0; e < 8; ++e) vs[t][8 * c + e] = v[e];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < nt)
        for (int dd = wave; dd < D; dd += 4) vtc[(((size_t)b * H + head) * D + dd) * S + pos0 + t0 + lane] = vs[lane][dd];
}

// ---- lane exchanges without LDS: DPP inside 16 lanes, the row / half swaps above them -----------
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// {v of lane % 32, v of lane % 32 + 32}, and the same for lanes 16 apart within 32.  The results go through scalars: a
// bit cast of a vector's element reads element 0 whichever is named.
__device__ __forceinline__ f2 both_halves(float v)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto t = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t a = t[0], b = t[1];
    return f2{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ f2 both_rows(float v)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto t = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a = t[0], b = t[1];
    return f2{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
// v <- op(v, v of a partner lane), doubling the group that shares the result: 2, 4, 8, 16 lanes by DPP
// (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror), 32 and 64 by the swaps
template <int LANES, typename Op>
__device__ __forceinline__ float group_reduce(float v, Op op)
{
    if constexpr (LANES >= 2) v = op(v, dpp_move<0xB1>(v));
    if constexpr (LANES >= 4) v = op(v, dpp_move<0x4E>(v));
    if constexpr (LANES >= 8) v = op(v, dpp_move<0x141>(v));
    if constexpr (LANES >= 16) v = op(v, dpp_move<0x140>(v));
    if constexpr (LANES >= 32) { const f2 t = both_rows(v); v = op(t[0], t[1]); }
    if constexpr (LANES >= 64) { const f2 t = both_halves(v); v = op(t[0], t[1]); }
    return v;
}
struct OpAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

constexpr float LOG2E = 1.4426950408889634f;

// KV append of one token per sequence: a workgroup per (sequence, head).  In the transposed V cache the token is one value in each feature row, two
// bytes of a line.  Stored by themselves they miss the L2, and the memory reads, changes and writes the line behind the kernel, which holds the
// attention's reads up.  So the line is read first and the store hits it; only the two bytes are stored (the other positions may be another
// stream's to write: what is read of them is not used).  kv_append and attention, us, with the store alone / behind the read: 43 sequences of 56 heads at
// 1338 positions 292.3 / 262.2 (attention alone 241), 64 of 56 at 1339 428.5 / 395.8, 64 of 40 at 601 161.8 / 142.3, 16 of 40 at 563 40.8 / 36.6; with 64 of
// the 128 bytes read 266.3, 403.7, 142.5, 36.5.  READ false: caches whose feature rows are no more than a few
// lines, most of which the attention reads (43 sequences of 40 heads, the store alone / behind the read: max_seq 64, position 10 20.4 / 23.3; 192, position 10 22.8 /
// 26.2, position 100 32.4 / 31.6; 256, position 10 23.2 / 24.5, position 250 52.5 / 49.6; 64 of 56, 2048, position 10 56.3 / 50.2).
template <int D, bool READ>
__global__ __launch_bounds__(256) void kv_append_token_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ kc, uint16_t* vtc, int pos, int H, int S)
{
    constexpr int ROUNDS = D / 64;                     // 64 feature rows at a time, four lanes a row
    const int bh = blockIdx.x, b = bh / H, head = bh % H, h = H * D, tid = threadIdx.x;
    const uint16_t* src = qkv + (size_t)b * 3 * h + head * D;
    uint16_t* row = vtc + ((size_t)bh * D + tid / 4) * S;
    const uint16_t* line = row + (pos & ~63) + 16 * (tid % 4);         // S is a multiple of 64
    u32x4 seen[ROUNDS];
    uint16_t v[ROUNDS];
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        if constexpr (READ) seen[i] = *reinterpret_cast<const u32x4*>(line + (size_t)64 * i * S);
        v[i] = src[2 * h + 64 * i + tid / 4];
    }
    if (tid < D / 8) *reinterpret_cast<h8*>(kc + ((size_t)bh * S + pos) * D + 8 * tid) = *reinterpret_cast<const h8*>(src + h + 8 * tid);
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        if constexpr (READ) {
            const u32x4 rest = *reinterpret_cast<const u32x4*>(line + (size_t)64 * i * S + 8);
            asm volatile("" ::"v"(seen[i]), "v"(rest) : "memory");              // the reads are waited for ahead of the store
        }
        if (tid % 4 == 0) row[(size_t)64 * i * S + pos] = v[i];
    }
}

// A lane's byte offset into eight feature rows of the transposed V cache: 32 bits where 14 * max_seq + 126 fits them, so that a load takes a
// scalar base and a 32-bit offset as they are; LONG: 64 bits.
template <bool LONG> using VOffset = typename std::conditional<LONG, uint64_t, uint32_t>::type;
bool long_rows(int S) { return S > (1 << 28); }

// ---- decode attention: one new token per sequence over the cached positions --------------------
// HBM-bound on the cache: 2 * n * d * 2 bytes per (sequence, head).  Grid (sequences * heads, splits); a
// workgroup takes a contiguous range of positions, its four waves take the range's tiles of 64 positions in
// turn, each with a running maximum and sum of its own, so no wave waits for another before the end.  A wave's
// loads go through two half-tile buffers in registers (8 KB each at d = 128): K's first half, K's second, V's two, each
// asked for as soon as the buffer's contents are used up, so 8 to 16 KB per wave are under way all the time at four waves
// per SIMD.  (One pass over K for the scores of a whole range, then one over V, with four loads in flight per lane, moved
// 4.9-5.3 TB/s; this moves 6.4 on 3 sequences of 6002 positions.)  Scores: lanes along d, D/8 lanes per key; p.V: eight lanes along positions, the sum
// over them formed once per wave, at its end.  Exponents are taken to base 2.
// FRESH: the new token's K and V are still in qkv only; split 0 adds that token and writes it to the
// caches (kv_append in the same launch).  `n`: cached positions that are read (without the new token if FRESH).
// With several splits the unnormalised partial outputs and their (max, sum) go to a workspace and a second
// kernel combines them.
template <int D, bool FRESH, bool LONG>
__global__ __launch_bounds__(256, 4) void attention_decode_kernel(const uint16_t* __restrict__ qkv, uint16_t* kc, uint16_t* vtc,
                                                                  const float* __restrict__ slopes, int H, int S, int n, int range, int splits,
                                                                  uint16_t* __restrict__ out, float* __restrict__ part)
{
    constexpr int LPK = D / 8, LOADS = D / 8;          // lanes per key; loads per lane and tile, for K and for V
    __shared__ __attribute__((aligned(16))) float pw[4][64];
    __shared__ __attribute__((aligned(16))) float red[4][D + 2];
    const int bh = blockIdx.x, b = bh / H, head = bh % H, split = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j1 = min(n, (split + 1) * range);        // this workgroup's positions [split * range, j1); range is a multiple of 64
    const int t_end = (j1 + 63) / 64;
    const int h = H * D;
    const float slope = slopes ? slopes[head] * LOG2E : 0.0f;
    const float c = LOG2E / sqrtf((float)D);
    const int q_pos = FRESH ? n : n - 1;               // the query's position
    const uint16_t* qrow = qkv + (size_t)b * 3 * h + head * D;
    float q[8];                                        // the lane's 8 query features
    {
        const h8 t = *reinterpret_cast<const h8*>(qrow + 8 * (lane % LPK));
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = (float)t[e];
    }
    auto dot8 = [&](const h8& k) {
        float d = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d += q[e] * (float)k[e];
        return group_reduce<LPK>(d, OpAdd());
    };
    uint16_t* kbase = kc + (size_t)bh * S * D;         // b * H + head == bh
    uint16_t* vbase = vtc + (size_t)bh * D * S;
    float m = -INFINITY, l = 0.0f;                     // running maximum (wave), this lane's part of the sum
    float acc[LOADS];                                  // features 8 u + lane / 8: this lane's part of the sum over positions
#pragma unroll
    for (int u = 0; u < LOADS; ++u) acc[u] = 0.0f;
    constexpr int HL = LOADS / 2;                      // loads per half of a tile
    h8 buf[2][HL];
    // a load's address is a scalar base and a 32-bit lane offset in bytes: key LOADS * (lane / LPK) + u of the tile;
    // feature 8 u + lane / 8, positions 8 (lane % 8) ..
    uint32_t koff = (uint32_t)((lane / LPK) * LOADS * D + 8 * (lane % LPK)) * 2u;
    VOffset<LONG> voff = ((VOffset<LONG>)(lane / 8) * (uint32_t)S + 8u * (uint32_t)(lane % 8)) * 2u;
    auto load_k = [&](int t, int x) {
        const uint8_t* base = reinterpret_cast<const uint8_t*>(kbase + (size_t)64 * t * D);
        asm volatile("" : "+v"(koff));                 // keeps the widening to 64 bits next to the loads
#pragma unroll
        for (int u = 0; u < HL; ++u) buf[x][u] = __builtin_nontemporal_load(reinterpret_cast<const h8*>(base + koff + (x * HL + u) * D * 2));
    };
    auto load_v = [&](int t, int x) {
        const uint8_t* base = reinterpret_cast<const uint8_t*>(vbase + (size_t)64 * t);
#pragma unroll
        for (int u = 0; u < HL; ++u) {
            asm volatile("" : "+v"(voff));
            buf[x][u] = __builtin_nontemporal_load(reinterpret_cast<const h8*>(base + (size_t)(x * HL + u) * 16 * S + voff));
        }
    };
    // tile t (the caches hold whole tiles: S is a multiple of 64); NEXT: tile t + 4 is this wave's too and is asked for
    auto tile = [&](int t, auto next) {
        constexpr bool NEXT = decltype(next)::value;
        float sc = 0.0f;                               // score of position 64 t + lane
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int u = 0; u < HL; ++u) {
                const float d = dot8(buf[x][u]);
                sc = lane % LPK == x * HL + u ? d : sc;
                if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four keys in work at a time: registers
            }
            load_v(t, x);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int j = 64 * t + lane;
        sc = sc * c + slope * (float)(j - q_pos);
        sc = j < j1 ? sc : -INFINITY;
        const float mn = fmaxf(m, group_reduce<64>(sc, OpMax()));
        const float ms = mn == -INFINITY ? 0.0f : mn;
        const float alpha = __builtin_amdgcn_exp2f(m - ms), p = __builtin_amdgcn_exp2f(sc - ms);
        m = mn;
        l = l * alpha + p;
        pw[wave][lane] = p;                            // a wave's LDS operations stay in order
        __builtin_amdgcn_wave_barrier();
        const f4 p0 = *reinterpret_cast<const f4*>(&pw[wave][8 * (lane % 8)]), p1 = *reinterpret_cast<const f4*>(&pw[wave][8 * (lane % 8) + 4]);
        __builtin_amdgcn_wave_barrier();
        const float pr[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
        const bool any_zero = __any(p == 0.0f);        // positions past the end hold anything, also NaN: a zero weight takes them out
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            if (any_zero) {
#pragma unroll
                for (int u = 0; u < HL; ++u) {
                    float a = acc[x * HL + u] * alpha;
#pragma unroll
                    for (int e = 0; e < 8; ++e) a += pr[e] != 0.0f ? pr[e] * (float)buf[x][u][e] : 0.0f;
                    acc[x * HL + u] = a;
                    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int u = 0; u < HL; ++u) {
                    float a = acc[x * HL + u] * alpha;
#pragma unroll
                    for (int e = 0; e < 8; ++e) a += pr[e] * (float)buf[x][u][e];
                    acc[x * HL + u] = a;
                    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (NEXT) load_k(t + 4, x);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int t = split * (range / 64) + wave;
    if (t < t_end) {
        load_k(t, 0);
        load_k(t, 1);
        for (; t + 4 < t_end; t += 4) tile(t, std::true_type());
        tile(t, std::false_type());
    }
    if constexpr (FRESH) {
        // Behind the tiles, by the wave with the fewest of them: ahead of them its loads and scattered stores hold the
        // stream back (43 sequences of 56 heads at 1338 positions: 314 us; so: 305; kv_append and this kernel without it: 264; the host takes two
        // launches where the caches are not small.  64 aligned bytes read, changed and stored per feature row, as kv_append does it, are slower here.)
        if (split == 0 && wave == 3) {
            const h8 k = *reinterpret_cast<const h8*>(qrow + h + 8 * (lane % LPK));
            uint16_t v[LOADS];
#pragma unroll
            for (int u = 0; u < LOADS; ++u) v[u] = qrow[2 * h + 8 * u + lane / 8];
            const float sc = dot8(k) * c;
            const float mn = fmaxf(m, sc), ms = mn == -INFINITY ? 0.0f : mn;
            const float alpha = __builtin_amdgcn_exp2f(m - ms), p = __builtin_amdgcn_exp2f(sc - ms);
            m = mn;
            l = l * alpha + (lane == 0 ? p : 0.0f);
            if (lane < LPK) *reinterpret_cast<h8*>(kbase + (size_t)n * D + 8 * lane) = k;
#pragma unroll
            for (int u = 0; u < LOADS; ++u) {
                acc[u] *= alpha;
                if (lane % 8 == 0) {
                    if (p != 0.0f) acc[u] += p * (float)__builtin_bit_cast(_Float16, v[u]);
                    vbase[(size_t)(8 * u + lane / 8) * S + n] = v[u];
                }
            }
        }
    }
    l = group_reduce<64>(l, OpAdd());
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const float a = group_reduce<8>(acc[u], OpAdd());
        if (lane % 8 == 0) red[wave][8 * u + lane / 8] = a;
    }
    if (lane == 0) { red[wave][D] = m; red[wave][D + 1] = l; }
    __syncthreads();
    if (tid >= D) return;
    const float mt = fmaxf(fmaxf(red[0][D], red[1][D]), fmaxf(red[2][D], red[3][D])), ms = mt == -INFINITY ? 0.0f : mt;
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float e = __builtin_amdgcn_exp2f(red[w][D] - ms);
        num += e * red[w][tid];
        den += e * red[w][D + 1];
    }
    if (splits == 1) {
        out[(size_t)bh * D + tid] = __builtin_bit_cast(uint16_t, (_Float16)(num / den));   // row b, column head * D + tid
        return;
    }
    float* ps = part + ((size_t)bh * splits + split) * (D + 2);
    ps[tid] = num;
    if (tid == 0) { ps[D] = mt; ps[D + 1] = den; }
}

template <int D>
__global__ void attention_combine_kernel(const float* __restrict__ part, int splits, uint16_t* __restrict__ out)
{
    const int bh = blockIdx.x, dd = threadIdx.x;       // out is [B][H * D]: row b, column head * D + dd = bh * D + dd
    const float* ps = part + (size_t)bh * splits * (D + 2);
    float m = -INFINITY;
    for (int s = 0; s < splits; ++s) m = fmaxf(m, ps[s * (D + 2) + D]);
    const float ms = m == -INFINITY ? 0.0f : m;
    float num = 0.0f, den = 0.0f;
#pragma unroll 4
    for (int s = 0; s < splits; ++s) {
        const float w = __builtin_amdgcn_exp2f(ps[s * (D + 2) + D] - ms);
        num += w * ps[s * (D + 2) + dd];
        den += w * ps[s * (D + 2) + D + 1];
    }
    out[(size_t)bh * D + dd] = __builtin_bit_cast(uint16_t, (_Float16)(num / den));
}

// ---- prefill attention: T new tokens per sequence, causal, over positions 0 .. pos0 + t ----------
// Matrix-core and vector bound (the exponentials take about as long as the products).  A workgroup takes 128
// queries of one head, each of its four waves 32 of them, and walks the visible keys 64 at a time with a running
// maximum and sum; K and V tiles are shared through LDS (two buffers each, filled by global-to-LDS loads while the
// tile before is multiplied; 64 KB at d = 128, so two workgroups per compute unit).
// Both products are formed transposed, on 32x32x16 MFMAs: S^T = K . Q^T and O^T = V^T . P^T.  A lane then holds scores of
// ONE query (column lane % 32) against half of the tile's keys, so the softmax needs a single exchange between the
// two halves of the wave, the rescaling of O is a multiplication by the lane's own factor, and P^T goes from
// accumulator to operand registers as it is: with the rows of the K operand taken in the order pi (bits 2 and 3 of
// the row swapped), registers 8 c .. 8 c + 7 of a lane are keys 16 c + 8 (lane / 32) + 0 .. 7, which is the B operand of
// a 16-key step. 
// 16-byte chunks are XOR-swizzled by row, so that the operand reads of eight consecutive lanes fall on
// different banks.  Workgroup ids go round-robin over the 8 XCDs: a head stays on one of them (its K and V are fetched into
// one L2), longest walks first.
// 2 x 1500 tokens, 40 heads of 128 (46 GFLOP over the visible half): 71 us = 0.65 PFLOP/s; 397 us with 16 queries per wave,
// operands straight from global memory and P through LDS.  Tiles: 32 matrix instructions (1024 cycles) and some 230 vector
// ones, 32 of them exponentials at a quarter rate, per wave and 64 keys; on this chip the two add up.
__device__ __forceinline__ int swap_bits23(int x) { return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1); }

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// One query at position p by one wave, on the vector units, over the keys it sees and no others: lanes along the keys for the scores, along
// the features for p . V.  For queries whose sums came out not finite: a later token's infinite or NaN value row, at weight
// zero, does that in the matrix product of a tile that both share.  (Same scaling, exponents and rounding of the weights.)
template <int D>
__device__ __forceinline__ void attention_one_query(const uint16_t* __restrict__ qp, const uint16_t* __restrict__ kbase, const uint16_t* __restrict__ vbase,
                                                    int S, int p, float c, float slope, uint16_t* __restrict__ op)
{
    const int lane = threadIdx.x & 63;
    float m = -INFINITY, l = 0.0f, acc[D / 64] = {};
#pragma unroll 1
    for (int j0 = 0; j0 <= p; j0 += 64) {
        const int j = j0 + lane;                       // within the cache: it holds whole tiles of 64
        float sc = 0.0f;
#pragma unroll 1
        for (int f = 0; f < D; f += 8) {
            const h8 q = *reinterpret_cast<const h8*>(qp + f), k = *reinterpret_cast<const h8*>(kbase + (size_t)j * D + f);
#pragma unroll
            for (int e = 0; e < 8; ++e) sc += (float)q[e] * (float)k[e];
        }
        sc = j <= p ? __builtin_fmaf(sc, c, slope * (float)(j - p)) : -INFINITY;
        const float mn = fmaxf(m, group_reduce<64>(sc, OpMax())), alpha = __builtin_amdgcn_exp2f(m - mn);
        const float w = j <= p ? __builtin_amdgcn_exp2f(sc - mn) : 0.0f;
        m = mn;
        l = l * alpha + w;
#pragma unroll
        for (int i = 0; i < D / 64; ++i) acc[i] *= alpha;
        const int n = min(64, p + 1 - j0);
#pragma unroll 1
        for (int u = 0; u < n; ++u) {
            const float wu = (float)(_Float16)__shfl(w, u);
#pragma unroll
            for (int i = 0; i < D / 64; ++i)
                acc[i] = __builtin_fmaf(wu, (float)__builtin_bit_cast(_Float16, vbase[(size_t)(64 * i + lane) * S + j0 + u]), acc[i]);
        }
    }
    l = group_reduce<64>(l, OpAdd());
#pragma unroll
    for (int i = 0; i < D / 64; ++i) op[64 * i + lane] = __builtin_bit_cast(uint16_t, (_Float16)(acc[i] / l));
}

template <int D, bool ALIBI, bool LONG>
__global__ __launch_bounds__(256, 2) void attention_prefill_kernel(const uint16_t* __restrict__ qkv, const uint16_t* __restrict__ kc,
                                                                   const uint16_t* __restrict__ vtc, const float* __restrict__ slopes,
                                                                   int BH, int H, int S, int T, int pos0, int q_blocks, uint16_t* __restrict__ out)
{
    // kbuf: [key][feature chunk ^ f(key)]; vbuf: [feature][key chunk ^ (feature & 7)].  Dynamic, because ahead of a read of a
    // named LDS array the compiler waits for every global-to-LDS load under way into it, also into the other buffer.
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
    struct Smem { uint16_t kbuf[2][64 * D], vbuf[2][64 * D]; };
    Smem& sm = *reinterpret_cast<Smem*>(smem_raw);
    constexpr int CH = D / 8;                          // 16-byte chunks of a key's features
    constexpr int KS = D / 16, DT = D / 32;            // 16-feature steps of S^T; 32-feature tiles of O^T
    constexpr int FILLS = D / 32;                      // 1 KB loads per wave and operand tile
    const int per_xcd = (BH + 7) / 8, slot = (int)(blockIdx.x >> 3);
    const int bh = (int)(blockIdx.x & 7) + 8 * (slot % per_xcd), qb = q_blocks - 1 - slot / per_xcd;
    if (bh >= BH) return;                              // the whole workgroup
    const int b = bh / H, head = bh % H;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int h = H * D;
    const int t0 = 128 * qb + 32 * wave;               // this wave's first query (token index within the sequence)
    const int p = pos0 + min(t0 + col, T - 1);         // the lane's query position (columns past the end repeat the last query)
    const float c = LOG2E / sqrtf((float)D);
    const float slope = ALIBI ? slopes[head] * LOG2E : 0.0f;
    const uint16_t* kbase = kc + (size_t)bh * S * D;
    const uint16_t* vbase = vtc + (size_t)bh * D * S;
    const int tiles = (pos0 + min(128 * qb + 127, T - 1)) / 64 + 1;                        // of the workgroup
    const int my_tiles = t0 < T ? (pos0 + min(t0 + 31, T - 1)) / 64 + 1 : 0;               // of this wave

    // A fill's address is a scalar base and a 32-bit lane offset in bytes.  K: the rows of a load are the lane's (lane / CH) and,
    // wave-uniform, r0; the swizzle's share of r0 is XOR-ed into the chunk.  V: r0 is a multiple of 8 and has no share.
    constexpr int ROWS = 512 / D;                      // keys per load
    const uint32_t kl = (uint32_t)((lane / CH) * D + 8 * ((lane % CH) ^ (swap_bits23(lane / CH) & (CH - 1)))) * 2u;
    VOffset<LONG> vl = ((VOffset<LONG>)(lane / 8) * (uint32_t)S + 8u * (uint32_t)((lane % 8) ^ (lane / 8))) * 2u;
    auto fill = [&](int j, int buf) {
        const uint8_t* kb = reinterpret_cast<const uint8_t*>(kbase + (size_t)64 * j * D);
        const uint8_t* vb = reinterpret_cast<const uint8_t*>(vbase + 64 * j);
#pragma unroll
        for (int i = 0; i < FILLS; ++i) {
            const int r0 = (FILLS * wave + i) * ROWS;
            uint32_t off = kl ^ (uint32_t)((swap_bits23(r0) & (CH - 1)) * 16);
            asm volatile("" : "+v"(off));              // keeps the widening to 64 bits next to the load
            __builtin_amdgcn_global_load_lds((gptr_t)(kb + (size_t)r0 * D * 2 + off), (lptr_t)&sm.kbuf[buf][r0 * D], 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < FILLS; ++i) {
            const int r0 = (FILLS * wave + i) * 8;
            asm volatile("" : "+v"(vl));
            __builtin_amdgcn_global_load_lds((gptr_t)(vb + (size_t)r0 * S * 2 + vl), (lptr_t)&sm.vbuf[buf][r0 * 64], 16, 0, 0);
        }
    };

    h8 qb_[KS];                                        // B operands of Q^T: lane (query col, features 16 k + 8 half ..)
    {
        const uint16_t* qp = qkv + ((size_t)b * T + min(t0 + col, T - 1)) * 3 * h + head * D + 8 * half;
#pragma unroll
        for (int k = 0; k < KS; ++k) qb_[k] = *reinterpret_cast<const h8*>(qp + 16 * k);
    }
    f16x o[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[d][v] = 0.0f;
    float m = -INFINITY, l = 0.0f;                     // running maximum of the lane's query; this lane's part of its sum
    const int krow = swap_bits23(col);

    fill(0, 0);
    for (int j = 0; j < tiles; ++j) {
        const int buf = j & 1;
        __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wave's part of tile j has landed
        __syncthreads();                               // everybody's has, and tile j - 1 is no longer read
        if (j + 1 < tiles) fill(j + 1, buf ^ 1);
        const int j0 = 64 * j, valid = pos0 + T;       // positions from `valid` on are unwritten and hold anything, also NaN
        if (j0 + 64 > valid) {                         // the last tile: their V is set to zero (their weight is)
#pragma unroll
            for (int i = 0; i < FILLS; ++i) {          // the 16-byte chunks that this thread's loads brought
                const int r0 = (FILLS * wave + i) * 8, row = r0 + lane / 8, key = 8 * ((lane % 8) ^ (row & 7));
                uint16_t* v = &sm.vbuf[buf][r0 * 64 + 8 * lane];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (j0 + key + e >= valid) v[e] = 0;
            }
            __syncthreads();
        }
        if (j >= my_tiles) continue;
        // Operands are read a batch ahead of the matrix instructions that take them, and the wait for a batch stands ahead of
        // the next batch's issue: with global-to-LDS loads under way the compiler waits for every LDS read at each use.
        auto wait_reads = [] { __builtin_amdgcn_s_waitcnt(0xC07F); __builtin_amdgcn_sched_barrier(0); };
        h8 ra[8], rb[8];
        auto read_k = [&](h8 (&r)[8], int kt) {
#pragma unroll
            for (int k = 0; k < KS; ++k)
                r[k] = *reinterpret_cast<const h8*>(&sm.kbuf[buf][(32 * kt + krow) * D + 8 * ((2 * k + half) ^ (col & (CH - 1)))]);
        };
        auto read_v = [&](h8 (&r)[8], int d0) {        // features 32 d0 .. 32 d0 + 63, the tile's four 16-key steps
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = 32 * (d0 + i / 4) + col;
                r[i] = *reinterpret_cast<const h8*>(&sm.vbuf[buf][row * 64 + 8 * ((2 * (i % 4) + half) ^ (row & 7))]);
            }
        };
        f16x s[2];                                     // scores: register 8 c + e of s[kt] is key 32 kt + 16 c + 8 half + e
        constexpr f16x zero = {};
        read_k(ra, 0);
        wait_reads();
        read_k(rb, 1);
#pragma unroll
        for (int k = 0; k < KS; ++k) s[0] = mfma32(ra[k], qb_[k], k == 0 ? zero : s[0]);
        wait_reads();
        read_v(ra, 0);
#pragma unroll
        for (int k = 0; k < KS; ++k) s[1] = mfma32(rb[k], qb_[k], k == 0 ? zero : s[1]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ALIBI) {                         // to base 2, with the linear bias
            const float base = slope * (float)(j0 + 8 * half - p);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    s[kt][v] = __builtin_fmaf(s[kt][v], c, __builtin_fmaf(slope, (float)(32 * kt + 16 * (v / 8) + v % 8), base));
        }
        if (j0 + 63 > pos0 + t0) {                     // some key of the tile lies behind some query of the wave
            const int rel = p - j0 - 8 * half;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v) s[kt][v] = 32 * kt + 16 * (v / 8) + v % 8 <= rel ? s[kt][v] : -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[kt][v]);
        const f2 m2 = both_halves(mx);
        mx = fmaxf(m2[0], m2[1]);
        // Rescaling only once a maximum has outgrown the one in use by 2^8 (among 32 queries there is a new one nearly always)
        // was 4 % faster and not kept: the largest weight is then not exactly 1, error against 64 bits 2.6e-4 for 2.5e-4.
        const float mn = fmaxf(m, ALIBI ? mx : mx * c);                      // finite from the first tile on: key 0 is visible to every query
        if (__any(mn > m)) {
            const float alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[d][v] *= alpha;
        }
        h8 pb[4];                                      // P^T operands of the four 16-key steps
        float ls = 0.0f;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float e = __builtin_amdgcn_exp2f(ALIBI ? s[kt][v] - m : __builtin_fmaf(s[kt][v], c, -m));
                ls += e;
                pb[2 * kt + v / 8][v % 8] = (_Float16)e;
            }
        l += ls;
#pragma unroll
        for (int d0 = 0; d0 < DT; d0 += 2) {
            h8 (&cur)[8] = (d0 & 2) ? rb : ra;
            wait_reads();
            if (d0 + 2 < DT) read_v((d0 & 2) ? ra : rb, d0 + 2);
#pragma unroll
            for (int i = 0; i < 8; ++i) o[d0 + i / 4] = mfma32(cur[i], pb[i % 4], o[d0 + i / 4]);
        }
    }
    const f2 l2 = both_halves(l);
    l = l2[0] + l2[1];
    // the lane holds features 32 d + 8 a + 4 half + 0 .. 3 of its query; the halves trade so that each stores 16 bytes
    const float inv = 1.0f / l;
    float total[4] = {0.0f, 0.0f, 0.0f, 0.0f};         // finite if all the lane's sums are
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) total[v % 4] += o[d][v];
    uint64_t again = __ballot(!__builtin_isfinite((total[0] + total[1]) + (total[2] + total[3])) && t0 + col < T);
    again = (again | again >> 32) & 0xffffffffu;       // queries to be done again: a bit per column, of either half
    const bool store = t0 + col < T && !(again >> col & 1);
    uint16_t* op = out + ((size_t)b * T + t0 + col) * h + head * D + 8 * half;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int a = 0; a < 4; a += 2) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const h2 x = {(_Float16)(o[d][4 * a + 2 * i] * inv), (_Float16)(o[d][4 * a + 2 * i + 1] * inv)};
                const h2 y = {(_Float16)(o[d][4 * a + 4 + 2 * i] * inv), (_Float16)(o[d][4 * a + 5 + 2 * i] * inv)};
                const u32x2 t = __builtin_amdgcn_permlane32_swap(as_u32(x), as_u32(y), false, false);
                w[i] = t[0];
                w[2 + i] = t[1];
            }
            if (store) *reinterpret_cast<u32x4*>(op + 32 * d + 8 * a) = w;
        }
    while (__builtin_expect(again != 0, 0)) {
        const int t = t0 + __builtin_ctzll(again);
        again &= again - 1;
        const size_t row = (size_t)b * T + t;
        attention_one_query<D>(qkv + row * 3 * h + head * D, kbase, vbase, S, pos0 + t, c, slope, out + row * h + head * D);
    }
}

}  // namespace

hipError_t launch_layernorm(const void* x, const void* gamma, const void* beta, float eps, int M, int h, void* y, hipStream_t s)
{
    // Threads of a row's workgroup and 16-byte chunks of a thread.  Rows not in any cache, us:
    //   up to 512 rows: 512 threads, or as many as there are chunks (7168 columns: 1024 threads / so, 16 rows 3.7 / 3.1, 512 rows 6.3 / 5.4).
    //   more, up to 8192 columns: 256 threads, up to four chunks, AHEAD (5120 columns: 512 threads / so, 1191 rows 8.3 / 7.2; 7168 columns: not AHEAD / so,
    //   4000 rows 23.2 / 21.0).
    //   more, beyond: four chunks at 512 threads (9216 columns: 1024 threads / so, 4000 rows 31.3 / 27.0; 16384 columns, 600 rows 10.6 / 9.9).  About 1000 rows
    //   are four to a compute unit: six chunks at 256 threads up to 12288 columns (9216, 1000 rows: 512 threads / so 9.5 / 9.2).  Beyond 12288 columns and 1100
    //   rows two chunks at 1024 threads, AHEAD (16384, 2000 rows: 512 threads / so 26.0 / 23.1).
    const int chunks = h / 8, all = (chunks + 63) / 64 * 64;
    const uint16_t *xs = static_cast<const uint16_t*>(x), *g = static_cast<const uint16_t*>(gamma), *b = static_cast<const uint16_t*>(beta);
    uint16_t* out = static_cast<uint16_t*>(y);
    auto run = [&](auto kernel, int threads) { kernel<<<(unsigned)M, threads, 0, s>>>(xs, g, b, eps, h, out); };
    if (M > 512 && chunks <= 1024) {
        if (chunks <= 256)      run(layernorm_kernel<256, 1, true>, all);
        else if (chunks <= 512) run(layernorm_kernel<256, 2, true>, 256);
        else                    run(layernorm_kernel<256, 4, true>, 256);
    } else if (M > 1100 && chunks > 1536) {
        run(layernorm_kernel<1024, 2, true>, 1024);
    } else if (M > 700 && M <= 1100 && chunks > 1024 && chunks <= 1536) {
        run(layernorm_kernel<256, 6, false>, 256);
    } else {
        if (chunks <= 512)       run(layernorm_kernel<512, 1, false>, all);
        else if (chunks <= 1024) run(layernorm_kernel<512, 2, false>, 512);
        else                     run(layernorm_kernel<512, 4, false>, 512);
    }
    return hipGetLastError();
}

constexpr int KV_SHORT_ROWS = 192;                     // positions of a feature row up to which an append reads nothing of it

int layernorm_max_hidden() { return LN_MAX_HIDDEN; }

hipError_t launch_kv_append(const void* qkv, void* kc, void* vtc, int n_seqs, int T, int pos0, int H, int d, int S, hipStream_t s)
{
    const dim3 grid((unsigned)(n_seqs * H), (unsigned)((T + 63) / 64));
    const uint16_t* q = static_cast<const uint16_t*>(qkv);
    if (T == 1) {
        uint16_t *k = static_cast<uint16_t*>(kc), *v = static_cast<uint16_t*>(vtc);
        auto run = [&](auto kernel) { kernel<<<(unsigned)(n_seqs * H), 256, 0, s>>>(q, k, v, pos0, H, S); };
        if (S <= KV_SHORT_ROWS) d == 128 ? run(kv_append_token_kernel<128, false>) : run(kv_append_token_kernel<64, false>);
        else                    d == 128 ? run(kv_append_token_kernel<128, true>) : run(kv_append_token_kernel<64, true>);
        return hipGetLastError();
    }
    if (d == 128) kv_append_kernel<128><<<grid, 256, 0, s>>>(q, static_cast<uint16_t*>(kc), static_cast<uint16_t*>(vtc), T, pos0, H, S);
    else          kv_append_kernel<64><<<grid, 256, 0, s>>>(q, static_cast<uint16_t*>(kc), static_cast<uint16_t*>(vtc), T, pos0, H, S);
    return hipGetLastError();
}

// Positions per workgroup and number of splits of a decode-attention launch over n cached positions.  The estimate (in tiles of 64
// positions that a compute unit streams one after the other, about 1.3 us each at d = 128) only ranks the choices: a
// workgroup takes its tiles four at a time and about three tiles' time to start and to end; up to four workgroups share a
// compute unit, more are dealt out as others end; a split costs the combining kernel, about four tiles' time.
// (3 sequences of 56 heads at 6002 positions: three splits, 80 us; 43 at 1338: one, 253 us on its own.)
void attention_decode_plan(int n_seqs, int H, int n, int cus, int* range, int* splits)
{
    const long bh = (long)n_seqs * H, tiles = std::max(1, (n + 63) / 64);
    double best = 1e30;
    *range = (int)tiles * 64;
    *splits = 1;
    for (long sp = 1; sp <= std::min<long>(64, (tiles + 3) / 4); ++sp) {
        const long per = (tiles + sp - 1) / sp, used = (tiles + per - 1) / per, wgs = bh * used;     // splits that have any
        const double rounds = wgs <= 4L * cus ? (double)((wgs + cus - 1) / cus) : (double)wgs / cus + 1.0;
        const double est = rounds * (double)((per + 3) / 4 * 4 + 3) + (used > 1 ? 4.0 : 0.0);
        if (est < best * 0.99) best = est, *range = (int)per * 64, *splits = (int)used;
    }
}

size_t attention_decode_workspace_floats(int n_seqs, int H, int d, int splits) { return splits > 1 ? (size_t)n_seqs * H * splits * (d + 2) : 0; }

hipError_t launch_attention_decode(const void* qkv, void* kc, void* vtc, const float* slopes, int n_seqs, int n, bool fresh, int H, int d, int S,
                                   int range, int splits, void* out, float* part, hipStream_t s)
{
    const uint16_t* q = static_cast<const uint16_t*>(qkv);
    uint16_t *k = static_cast<uint16_t*>(kc), *v = static_cast<uint16_t*>(vtc), *o = static_cast<uint16_t*>(out);
    const dim3 grid((unsigned)(n_seqs * H), (unsigned)splits);
#define LPQ_ATT(D, F)                                                                                                        \
    do {                                                                                                                     \
        if (long_rows(S)) attention_decode_kernel<D, F, true><<<grid, 256, 0, s>>>(q, k, v, slopes, H, S, n, range, splits, o, part); \
        else              attention_decode_kernel<D, F, false><<<grid, 256, 0, s>>>(q, k, v, slopes, H, S, n, range, splits, o, part); \
    } while (0)
    if (d == 128) { if (fresh) LPQ_ATT(128, true); else LPQ_ATT(128, false); }
    else          { if (fresh) LPQ_ATT(64, true); else LPQ_ATT(64, false); }
#undef LPQ_ATT
    if (splits > 1) {
        if (d == 128) attention_combine_kernel<128><<<(unsigned)(n_seqs * H), 128, 0, s>>>(part, splits, o);
        else          attention_combine_kernel<64><<<(unsigned)(n_seqs * H), 64, 0, s>>>(part, splits, o);
    }
    return hipGetLastError();
}

hipError_t launch_attention_prefill(const void* qkv, const void* kc, const void* vtc, const float* slopes, int n_seqs, int T, int pos0, int H, int d,
                                    int S, void* out, hipStream_t s)
{
    const uint16_t *q = static_cast<const uint16_t*>(qkv), *k = static_cast<const uint16_t*>(kc), *v = static_cast<const uint16_t*>(vtc);
    uint16_t* o = static_cast<uint16_t*>(out);
    const int bh = n_seqs * H, q_blocks = (T + 127) / 128;
    const unsigned grid = 8u * (unsigned)((bh + 7) / 8) * (unsigned)q_blocks;
#define LPQ_ATT(D, A)                                                                                                        \
    do {                                                                                                                     \
        constexpr size_t smem = 2 * 2 * 64 * D * 2;                                                                          \
        if (long_rows(S)) attention_prefill_kernel<D, A, true><<<grid, 256, smem, s>>>(q, k, v, slopes, bh, H, S, T, pos0, q_blocks, o); \
        else              attention_prefill_kernel<D, A, false><<<grid, 256, smem, s>>>(q, k, v, slopes, bh, H, S, T, pos0, q_blocks, o); \
    } while (0)
    if (d == 128) { if (slopes) LPQ_ATT(128, true); else LPQ_ATT(128, false); }
    else          { if (slopes) LPQ_ATT(64, true); else LPQ_ATT(64, false); }
#undef LPQ_ATT
    return hipGetLastError();
}

}  // namespace lpq
