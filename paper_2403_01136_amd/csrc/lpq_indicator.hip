// Variance indicator (LLM-PQ, arXiv 2403.01136, Sec. 4.2, Theorem 1 and Eq. 3): the extra output variance of a
// linear operator under b-bit weight quantisation is estimated as D_W * S_W(b)^2 * G(X), G(X) = Var[X] / 4
// (deterministic rounding) or (E[X]^2 + Var[X]) / 6 (stochastic rounding).
//
// Everything it needs is a few reductions, bound by reading W and X once from HBM:
//   over W:  sum over its 128-column groups of (max - min)^2, sum over its rows of max |w|^2, min, max
//   over X:  sum x, sum x^2                                                       (fp64 per lane)
// One launch reads both (some workgroups take rows of W, the others a share of X) and leaves one partial result per workgroup; a
// second, of one workgroup, adds those in fp64 and evaluates the eight forms: the printed one-scale-per-matrix form
// and the form with the quantiser's own granularity (a scale per (row, 128 columns) group, or per row for the symmetric scheme),
// for bits 3, 4, 8 and symmetric 8.
// The four weights of a 5120-wide layer against 2048 rows of X (776 MB): 155 us (137 in the reading launch, 5.7 TB/s); with a statistic per row of W, summed
// by the second kernel's one workgroup (9-25 us of it), X in a launch of its own, minima and maxima exchanged through LDS: 222.
#include <algorithm>
#include "lpq_common.h"
#include "lpq_device.h"

namespace lpq {

namespace {

constexpr int IND_THREADS = 512, IND_WAVES = IND_THREADS / 64;
constexpr int IND_MAX_BLOCKS = 1024;                   // of either kind: four workgroups of eight waves per compute unit

// W: a = sum of group ranges squared, b = sum of the rows' max |w|^2; X: a = sum x, b = sum x^2
struct IndPart { double a, b; float lo, hi; };

__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// minimum and maximum over the 16 lanes of a 128-column group, two values to a register: exact in fp16
template <int CTRL> __device__ __forceinline__ h2 dpp_pair(h2 v)
{
    return as_h2((uint32_t)__builtin_amdgcn_update_dpp(0, (int)as_u32(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ void group_min_max(h2& lo, h2& hi)
{
    lo = __builtin_elementwise_min(lo, dpp_pair<0xB1>(lo));  hi = __builtin_elementwise_max(hi, dpp_pair<0xB1>(hi));
    lo = __builtin_elementwise_min(lo, dpp_pair<0x4E>(lo));  hi = __builtin_elementwise_max(hi, dpp_pair<0x4E>(hi));
    lo = __builtin_elementwise_min(lo, dpp_pair<0x141>(lo)); hi = __builtin_elementwise_max(hi, dpp_pair<0x141>(hi));
    lo = __builtin_elementwise_min(lo, dpp_pair<0x140>(lo)); hi = __builtin_elementwise_max(hi, dpp_pair<0x140>(hi));
}

__global__ __launch_bounds__(IND_THREADS) void indicator_stats_kernel(const uint16_t* __restrict__ w, int K, int N, int w_blocks,
                                                                      const uint16_t* __restrict__ x, long n8, IndPart* __restrict__ part)
{
    __shared__ IndPart red[IND_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int U = 4;                               // loads issued together
    double a = 0.0, b = 0.0;
    float lo_all = INFINITY, hi_all = -INFINITY;
    if ((int)blockIdx.x < w_blocks) {
        for (long n = (long)blockIdx.x * IND_WAVES + wave; n < N; n += (long)w_blocks * IND_WAVES) {
            const uint16_t* row = w + n * K;
            float range_sq = 0.0f, lo_row = INFINITY, hi_row = -INFINITY;
            for (int k0 = 8 * lane; k0 < K; k0 += 512 * U) {           // 16 lanes cover one 128-column group
                h8 t[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    t[u] = __builtin_nontemporal_load(reinterpret_cast<const h8*>(row + (k0 + 512 * u < K ? k0 + 512 * u : k0)));
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (k0 + 512 * u >= K) continue;   // whole groups: K is a multiple of 128
                    const h2 p0 = {t[u][0], t[u][1]}, p1 = {t[u][2], t[u][3]}, p2 = {t[u][4], t[u][5]}, p3 = {t[u][6], t[u][7]};
                    h2 lo = __builtin_elementwise_min(__builtin_elementwise_min(p0, p1), __builtin_elementwise_min(p2, p3));
                    h2 hi = __builtin_elementwise_max(__builtin_elementwise_max(p0, p1), __builtin_elementwise_max(p2, p3));
                    group_min_max(lo, hi);
                    const float l = fminf((float)lo[0], (float)lo[1]), h = fmaxf((float)hi[0], (float)hi[1]);
                    range_sq += (h - l) * (h - l);
                    lo_row = fminf(lo_row, l);
                    hi_row = fmaxf(hi_row, h);
                }
            }
            if ((lane & 15) == 0) a += (double)range_sq;               // the group's 16 lanes hold the same value
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) { lo_row = fminf(lo_row, __shfl_xor(lo_row, off)); hi_row = fmaxf(hi_row, __shfl_xor(hi_row, off)); }
            const double amax = fmax(fabs((double)lo_row), fabs((double)hi_row));
            if (lane == 0) b += amax * amax;
            lo_all = fminf(lo_all, lo_row);
            hi_all = fmaxf(hi_all, hi_row);
        }
    } else {
        const long stride = (long)(gridDim.x - w_blocks) * IND_THREADS;
        for (long i = (long)(blockIdx.x - w_blocks) * IND_THREADS + threadIdx.x; i < n8; i += U * stride) {
            h8 t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) t[u] = __builtin_nontemporal_load(reinterpret_cast<const h8*>(x + 8 * (i + u * stride < n8 ? i + u * stride : i)));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i + u * stride >= n8) continue;
#pragma unroll
                for (int e = 0; e < 8; ++e) { const double v = (double)(float)t[u][e]; a += v; b += v * v; }
            }
        }
    }
    a = wave_sum_f64(a);
    b = wave_sum_f64(b);
    if (lane == 0) red[wave] = IndPart{a, b, lo_all, hi_all};           // a wave's lanes agree on lo and hi
    __syncthreads();
    if (threadIdx.x == 0) {
        IndPart r = red[0];
        for (int i = 1; i < IND_WAVES; ++i) { r.a += red[i].a; r.b += red[i].b; r.lo = fminf(r.lo, red[i].lo); r.hi = fmaxf(r.hi, red[i].hi); }
        part[blockIdx.x] = r;
    }
}

// one workgroup: add the partial results in fp64, evaluate the eight forms
__global__ __launch_bounds__(IND_THREADS) void indicator_finish_kernel(const IndPart* __restrict__ part, int w_blocks, int blocks, int K, int N,
                                                                       double x_count, int stochastic, double* __restrict__ omega)
{
    __shared__ double red[4][IND_WAVES];
    __shared__ float redf[2][IND_WAVES];
    double s[4] = {0.0, 0.0, 0.0, 0.0};                // range^2, max|w|^2, x, x^2
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2 * IND_MAX_BLOCKS / IND_THREADS; ++u) {
        const int i = threadIdx.x + IND_THREADS * u;
        if (i >= blocks) continue;
        const IndPart p = part[i];
        const bool is_w = i < w_blocks;
        s[0] += is_w ? p.a : 0.0;
        s[1] += is_w ? p.b : 0.0;
        s[2] += is_w ? 0.0 : p.a;
        s[3] += is_w ? 0.0 : p.b;
        lo = fminf(lo, p.lo);                          // an X part holds the neutral values
        hi = fmaxf(hi, p.hi);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = wave_sum_f64(s[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { lo = fminf(lo, __shfl_xor(lo, off)); hi = fmaxf(hi, __shfl_xor(hi, off)); }
    if ((threadIdx.x & 63) == 0) {
        const int wave = threadIdx.x >> 6;
        for (int i = 0; i < 4; ++i) red[i][wave] = s[i];
        redf[0][wave] = lo;
        redf[1][wave] = hi;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int i = 0; i < 4; ++i) {
        s[i] = red[i][0];
        for (int v = 1; v < IND_WAVES; ++v) s[i] += red[i][v];
    }
    for (int v = 0; v < IND_WAVES; ++v) { lo = fminf(lo, redf[0][v]); hi = fmaxf(hi, redf[1][v]); }
    const double mean = s[2] / x_count, var = fmax(s[3] / x_count - mean * mean, 0.0);
    const double g = stochastic ? (mean * mean + var) / 6.0 : var / 4.0;
    const double d = (double)N * (double)K, range = (double)hi - (double)lo, amax = fmax(fabs((double)lo), fabs((double)hi));
    const double q[3] = {7.0, 15.0, 255.0};
    for (int b = 0; b < 3; ++b) {
        omega[b] = 128.0 * s[0] / (q[b] * q[b]) * g;
        omega[4 + b] = d * (range / q[b]) * (range / q[b]) * g;
    }
    omega[3] = (double)K * s[1] / (127.0 * 127.0) * g;
    omega[7] = d * (amax / 127.0) * (amax / 127.0) * g;
}

}  // namespace

// Workgroups of W: a row per wave up to what the chip holds at once; of X: so that one reads about what a workgroup of W does.
static void indicator_blocks(int K, int N, int M, int* wb, int* xb)
{
    const long n8 = (long)M * K / 8, w8 = (long)N * K / 8;
    *wb = (int)std::min<long>(IND_MAX_BLOCKS, (N + IND_WAVES - 1) / IND_WAVES);
    const long per = std::max<long>(IND_THREADS, (w8 + *wb - 1) / *wb);
    *xb = (int)std::min<long>(IND_MAX_BLOCKS, std::max<long>(1, (n8 + per - 1) / per));
}

size_t indicator_workspace_bytes(int K, int N, int M)
{
    int wb, xb;
    indicator_blocks(K, N, M, &wb, &xb);
    return (size_t)(wb + xb) * sizeof(IndPart);
}

hipError_t launch_indicator(const void* w, int K, int N, const void* x, int M, int stochastic, double* omega, void* ws, hipStream_t s)
{
    int wb, xb;
    indicator_blocks(K, N, M, &wb, &xb);
    const long n8 = (long)M * K / 8;
    IndPart* part = static_cast<IndPart*>(ws);
    indicator_stats_kernel<<<(unsigned)(wb + xb), IND_THREADS, 0, s>>>(static_cast<const uint16_t*>(w), K, N, wb, static_cast<const uint16_t*>(x), n8, part);
    indicator_finish_kernel<<<1, IND_THREADS, 0, s>>>(part, wb, wb + xb, K, N, (double)M * (double)K, stochastic, omega);
    return hipGetLastError();
}

}  // namespace lpq
