// Codebook learning (Alg. 3, App. D) for gfx950: block-normalised gradient histogram,
// exact interval DP over the non-empty bins, and installation of a codebook into the
// tables the step kernels read (fp32 entries, midpoints, guide table).
//
// Floating-point choices: the histogram bin and the whole DP are evaluated in float64
// with contraction disabled, in the operation order of the definitions, so that the
// bins, DP costs, split points and codebook entries are reproducible bit for bit.
#include "gefen_internal.h"

#include <math.h>

namespace gefen {
namespace {

constexpr int kMaxBins = 16 * kMaxK;   // 4096

// ---------------------------------------------------------------------------------
// Histogram: x = g / max|g_block| (blocks with max 0 are skipped),
// bin = min(NB - 1, floor((x + 1) * NB / 2)). Each workgroup accumulates its tiles into
// an LDS histogram with integer atomics, then adds the non-zero bins to the global
// uint64 histogram. Integer atomics make the result independent of scheduling.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ float grad_at(const Seg& sg, int64_t i)
{
    if (sg.gdtype == DT_F32) return static_cast<const float*>(sg.grad)[i];
    return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(sg.grad)[i]) << 16);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Four gradient elements at vector index v (16-byte fp32 or 8-byte bf16 load).
__device__ __forceinline__ void grad4_at(const Seg& sg, int64_t v, float g[4])
{
    if (sg.gdtype == DT_F32) {
        const f32x4 x = reinterpret_cast<const f32x4*>(sg.grad)[v];
        g[0] = x.x; g[1] = x.y; g[2] = x.z; g[3] = x.w;
    } else {
        const u32x2 x = reinterpret_cast<const u32x2*>(sg.grad)[v];
        g[0] = __uint_as_float(x.x << 16); g[1] = __uint_as_float(x.x & 0xffff0000u);
        g[2] = __uint_as_float(x.y << 16); g[3] = __uint_as_float(x.y & 0xffff0000u);
    }
}

// Range [start, start + len) split into an aligned vector body [vb, ve) (vector units)
// and element-wise head/tail, when the gradient pointer is aligned for vector loads.
struct GSpan {
    int64_t vb, ve, start, nh, tail0, nt;
};

__device__ __forceinline__ GSpan grad_span(const Seg& sg, int64_t start, int64_t len)
{
    const int64_t end = start + len;
    const uintptr_t al = sg.gdtype == DT_F32 ? 15 : 7;
    int64_t b = end, e = end;
    if ((reinterpret_cast<uintptr_t>(sg.grad) & al) == 0) {
        b = (start + 3) & ~int64_t(3);
        e = end & ~int64_t(3);
        if (b > end) b = end;
        if (e < b) e = b;
    }
    GSpan s;
    s.vb = b >> 2;
    s.ve = e >> 2;
    s.start = start;
    s.nh = b - start;
    s.tail0 = e;
    s.nt = end - e;
    return s;
}

// Absmax over a span by `stride` threads, this one being `tid` (per-thread partial; the
// caller reduces).
__device__ __forceinline__ float span_absmax(const Seg& sg, const GSpan& sp, int tid, int stride)
{
    float a = 0.0f;
#pragma unroll 2
    for (int64_t v = sp.vb + tid; v < sp.ve; v += stride) {
        float g[4];
        grad4_at(sg, v, g);
        a = fmaxf(a, fmaxf(fmaxf(fabsf(g[0]), fabsf(g[1])), fmaxf(fabsf(g[2]), fabsf(g[3]))));
    }
    for (int64_t i = tid; i < sp.nh + sp.nt; i += stride) {
        const int64_t e = i < sp.nh ? sp.start + i : sp.tail0 + (i - sp.nh);
        a = fmaxf(a, fabsf(grad_at(sg, e)));
    }
    return a;
}

__device__ __forceinline__ void span_bins(const Seg& sg, const GSpan& sp, float absmax,
                                          double half_nb, int nbins, uint32_t* h, int tid, int stride)
{
    const HistBlock a = hist_block(absmax);
#pragma unroll 2
    for (int64_t v = sp.vb + tid; v < sp.ve; v += stride) {
        float g[4];
        grad4_at(sg, v, g);
#pragma unroll
        for (int c = 0; c < 4; ++c) atomicAdd(&h[hist_bin(g[c], a, half_nb, nbins)], 1u);
    }
    for (int64_t i = tid; i < sp.nh + sp.nt; i += stride) {
        const int64_t e = i < sp.nh ? sp.start + i : sp.tail0 + (i - sp.nh);
        atomicAdd(&h[hist_bin(grad_at(sg, e), a, half_nb, nbins)], 1u);
    }
}

__device__ __forceinline__ void tile_block(const Seg& sg, const Tile& tl, int bi, int64_t& start,
                                           int64_t& len)
{
    if (sg.period > 0) {
        start = tl.elem0 + static_cast<int64_t>(bi) * sg.period;
        len = sg.period;
    } else {
        const int64_t local = tl.blk0 + bi - sg.blk_begin;
        start = sg.csr[local];
        len = sg.csr[local + 1] - start;
    }
}

// Uniform blocks of whole 4-element vectors (nv = p / 4 <= 64 kHistVecs), taken by one wave
// with kHistVecs vectors a lane in registers, all loaded before the first is used, so the
// gradients are read once and each trip to memory brings kHistVecs vectors. J > 0: a block
// takes J vectors of every lane, kHistVecs / J blocks at a time; J = 0: a block takes one
// vector of each lane of a group of 2^lpb_log2 >= nv lanes, so a vector slot holds
// 64 >> lpb_log2 blocks. Blocks [0, nblk) from element e0 of the tensor.
//
// The kernel is bound by the latency of its chain (loads, block maximum, bins): one block a
// wave with two loads in flight and a second read for the bins took 405 us on the GPT-2
// small shapes (124M float32 gradients in rows of 768) and 2.30 ms on the Llama-3 1.5B ones
// (bfloat16, rows of 2048 and 8192); this takes 148 us and 1.22 ms. Not the flush: storing
// each workgroup's bins and adding them up in a second kernel instead of the atomics left
// both kernels' times as they were.
constexpr int kHistVecs = static_cast<int>(kHistVecBlock / 256);
constexpr int64_t kHistVecGroups = 1024;   // four workgroups a CU

// Elements e .. e + 3 (one vector when `aligned`).
template <int GDT>
__device__ __forceinline__ void hist_load(const void* grad, int64_t e, bool aligned, float g[4])
{
    if (!aligned) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (GDT == DT_F32)
                g[c] = static_cast<const float*>(grad)[e + c];
            else
                g[c] = __uint_as_float(
                    static_cast<uint32_t>(static_cast<const uint16_t*>(grad)[e + c]) << 16);
        }
    } else if (GDT == DT_F32) {
        const f32x4 x = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4*>(static_cast<const float*>(grad) + e));
        g[0] = x.x; g[1] = x.y; g[2] = x.z; g[3] = x.w;
    } else {
        const u32x2 x = __builtin_nontemporal_load(
            reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(grad) + e));
        g[0] = __uint_as_float(x.x << 16); g[1] = __uint_as_float(x.x & 0xffff0000u);
        g[2] = __uint_as_float(x.y << 16); g[3] = __uint_as_float(x.y & 0xffff0000u);
    }
}

__device__ __forceinline__ float max4(const float g[4])
{
    return fmaxf(fmaxf(fabsf(g[0]), fabsf(g[1])), fmaxf(fabsf(g[2]), fabsf(g[3])));
}

template <int GDT, int J>
__device__ __forceinline__ void hist_blocks(const void* grad, bool aligned, int64_t e0, int nblk,
                                            int nv, int lpb_log2, double half_nb, int nbins,
                                            uint32_t* h, int lane)
{
    constexpr int V = kHistVecs;
    constexpr int B = J ? V / J : 0;            // blocks at a time (J > 0)
    const int per = J ? B : V * (64 >> lpb_log2);
    const int sub = J ? 0 : lane >> lpb_log2;
    const int li = J ? lane : lane & ((1 << lpb_log2) - 1);
    for (int b0 = 0; b0 < nblk; b0 += per) {
        float g[V][4];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int blk = J ? b0 + u / (J ? J : 1) : b0 + u * (64 >> lpb_log2) + sub;
            const int v = J ? u % (J ? J : 1) * 64 + li : li;
            g[u][0] = g[u][1] = g[u][2] = g[u][3] = 0.0f;
            if (blk < nblk && v < nv && (!J || u < B * J)) {
                hist_load<GDT>(grad, e0 + (static_cast<int64_t>(blk) * nv + v) * 4, aligned, g[u]);
            }
        }
        constexpr int N = J ? B : V;   // maxima a lane takes part in
        float a[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            a[k] = 0.0f;
#pragma unroll
            for (int i = 0; i < (J ? J : 1); ++i) a[k] = fmaxf(a[k], max4(g[k * (J ? J : 1) + i]));
        }
        const int wl = J ? 64 : 1 << lpb_log2;
        for (int off = 1; off < wl; off <<= 1)
#pragma unroll
            for (int k = 0; k < N; ++k) a[k] = fmaxf(a[k], __shfl_xor(a[k], off));
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const HistBlock hb = hist_block(a[k]);
            const int blk = J ? b0 + k : b0 + k * (64 >> lpb_log2) + sub;
            if (!(a[k] > 0.0f) || blk >= nblk) continue;
#pragma unroll
            for (int i = 0; i < (J ? J : 1); ++i)
                if ((J ? i * 64 + li : li) < nv)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        atomicAdd(&h[hist_bin(g[k * (J ? J : 1) + i][c], hb, half_nb, nbins)], 1u);
        }
    }
}

// Longer blocks: kHistVecs vectors a lane in flight, once for the maximum and once for the
// bins (the last ones from registers).
template <int GDT>
__device__ __forceinline__ void hist_long(const void* grad, bool aligned, int64_t e0, int nblk,
                                          int64_t nv, double half_nb, int nbins, uint32_t* h,
                                          int lane)
{
    constexpr int V = kHistVecs;
    for (int blk = 0; blk < nblk; ++blk) {
        const int64_t b0 = e0 + 4 * nv * blk;
        const int64_t last = (nv - 1) / (64 * V) * (64 * V);
        float g[V][4];
        float a = 0.0f;
        for (int64_t v0 = 0; v0 <= last; v0 += 64 * V) {
#pragma unroll
            for (int u = 0; u < V; ++u) {
                const int64_t v = v0 + u * 64 + lane;
                g[u][0] = g[u][1] = g[u][2] = g[u][3] = 0.0f;
                if (v < nv) hist_load<GDT>(grad, b0 + 4 * v, aligned, g[u]);
            }
#pragma unroll
            for (int u = 0; u < V; ++u) a = fmaxf(a, max4(g[u]));
        }
        for (int off = 1; off < 64; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
        if (!(a > 0.0f)) continue;
        const HistBlock hb = hist_block(a);
        for (int64_t v0 = last; v0 >= 0; v0 -= 64 * V) {
            if (v0 < last) {
#pragma unroll
                for (int u = 0; u < V; ++u)
                    hist_load<GDT>(grad, b0 + 4 * (v0 + u * 64 + lane), aligned, g[u]);
            }
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (v0 + u * 64 + lane < nv)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        atomicAdd(&h[hist_bin(g[u][c], hb, half_nb, nbins)], 1u);
        }
    }
}

template <int GDT>
__device__ __forceinline__ void hist_uniform(const Seg& sg, const Tile& tl, double half_nb,
                                             int nbins, uint32_t* h, int lane)
{
    const uintptr_t al = GDT == DT_F32 ? 15 : 7;
    const bool aligned = (reinterpret_cast<uintptr_t>(sg.grad) & al) == 0;
    const int64_t nvec = sg.period >> 2;
    const int n = tl.nblk;
    if (nvec > 64 * kHistVecs) {
        hist_long<GDT>(sg.grad, aligned, tl.elem0, n, nvec, half_nb, nbins, h, lane);
        return;
    }
    const int nv = static_cast<int>(nvec);
#define GEFEN_HIST(J, LL) \
    hist_blocks<GDT, J>(sg.grad, aligned, tl.elem0, n, nv, LL, half_nb, nbins, h, lane)
    if (nv <= 32) {
        int ll = 0;
        while ((1 << ll) < nv) ++ll;
        GEFEN_HIST(0, ll);
    } else if (nv <= 64) {
        GEFEN_HIST(1, 6);
    } else if (nv <= 128) {
        GEFEN_HIST(2, 6);
    } else if (nv <= 256) {
        GEFEN_HIST(4, 6);
    } else {
        GEFEN_HIST(8, 6);
    }
#undef GEFEN_HIST
}

// Absolute maximum of |g| over one chunk of a huge block.
__global__ __launch_bounds__(kThreads) void k_hist_h_absmax(const Tile* __restrict__ tiles,
                                                            const HTile* __restrict__ htiles,
                                                            const Seg* __restrict__ segs,
                                                            float* __restrict__ am_partials)
{
    __shared__ float red[kThreads / 64];
    const Tile tl = tiles[blockIdx.x];
    const HTile ht = htiles[blockIdx.x];
    const Seg sg = segs[tl.seg];
    float a = span_absmax(sg, grad_span(sg, tl.elem0, tl.nelem), threadIdx.x, kThreads);
    for (int off = 1; off < 64; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) a = fmaxf(a, red[w]);
        am_partials[ht.first + ht.chunk] = fmaxf(a, red[0]);
    }
}

// VEC: the tiles of hist_by_vectors, else the others: a launch each, since the registers of
// the first would halve the waves that hide the second's chains.
template <bool VEC>
__global__ __launch_bounds__(kThreads) void k_histogram(const Tile* __restrict__ tiles,
                                                        int64_t n_tiles,
                                                        const int32_t* __restrict__ tile_kind,
                                                        const HTile* __restrict__ htiles,
                                                        const float* __restrict__ am_partials,
                                                        const Seg* __restrict__ segs,
                                                        int32_t nbins, int64_t longest,
                                                        uint64_t* __restrict__ hist)
{
    __shared__ uint32_t h[kMaxBins];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    for (int i = tid; i < nbins; i += kThreads) h[i] = 0;
    __syncthreads();
    const double half_nb = 0.5 * static_cast<double>(nbins);

    // Every wave takes its own tiles (wave-strided persistent loop) and reduces within
    // itself, so no barrier is needed until the flush.
    constexpr int kWaves = kThreads / 64;
    for (int64_t ti = static_cast<int64_t>(blockIdx.x) * kWaves + wave; ti < n_tiles;
         ti += static_cast<int64_t>(gridDim.x) * kWaves) {
        const Tile tl = tiles[ti];
        const Seg sg = segs[tl.seg];
        const int kind = tile_kind[ti];
        if (hist_by_vectors(kind, sg.period, longest) != VEC) continue;
        if constexpr (VEC) {
            if (sg.gdtype == DT_F32)
                hist_uniform<DT_F32>(sg, tl, half_nb, nbins, h, lane);
            else
                hist_uniform<DT_BF16>(sg, tl, half_nb, nbins, h, lane);
        } else if (kind == KIND_L) {
            // one lane per small block
            for (int bi = lane; bi < tl.nblk; bi += 64) {
                int64_t start, len;
                tile_block(sg, tl, bi, start, len);
                float a = 0.0f;
                for (int64_t i = 0; i < len; ++i) a = fmaxf(a, fabsf(grad_at(sg, start + i)));
                if (a > 0.0f) {
                    const HistBlock hb = hist_block(a);
                    for (int64_t i = 0; i < len; ++i)
                        atomicAdd(&h[hist_bin(grad_at(sg, start + i), hb, half_nb, nbins)], 1u);
                }
            }
        } else if (kind == KIND_H) {
            // one chunk of a huge block: block absmax from the chunk maxima
            const HTile ht = htiles[ti];
            float a = 0.0f;
            for (int c = lane; c < ht.nchunk; c += 64) a = fmaxf(a, am_partials[ht.first + c]);
            for (int off = 1; off < 64; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
            if (a > 0.0f)
                span_bins(sg, grad_span(sg, tl.elem0, tl.nelem), a, half_nb, nbins, h, lane, 64);
        } else {
            // the tile's blocks one after another, each by the whole wave
            for (int bi = 0; bi < tl.nblk; ++bi) {
                int64_t start, len;
                tile_block(sg, tl, bi, start, len);
                const GSpan sp = grad_span(sg, start, len);
                float a = span_absmax(sg, sp, lane, 64);
                for (int off = 1; off < 64; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
                if (a > 0.0f) span_bins(sg, sp, a, half_nb, nbins, h, lane, 64);
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < nbins; i += kThreads) {
        const uint32_t c = h[i];
        if (c) atomicAdd(reinterpret_cast<unsigned long long*>(&hist[i]),
                         static_cast<unsigned long long>(c));
    }
}

// ---------------------------------------------------------------------------------
// The DP (Alg. 3, App. D): D[j][r] = min over l of D[j-1][l-1] + C(l, r), argmin to the
// smallest l, over the b non-empty bins. Workspace (all 256-byte aligned):
//   hdr    int32[16]: [0] b (non-empty bins), [1] keff (entries the DP solves for),
//          [2] status, [3] 1 when rows may be pruned (dp_may_prune), [4] row tiles handed
//          out by k_dp_run, [5] 1 when one of its waits ran out
//   Z0,Z1,Z2,cnt,ctr   double[NB + 1] each (1-based, index 0 = 0)
//   D      double[k][NB + 1]   D[j][r]; from level kDpEntry on kDpUnset until written
//   from   uint16[2][NB + 1]   smallest l that a row of level j + 1 needs to look at, by
//          the parity of j (levels before kDpEntry)
//   split  uint16[k + 1][NB + 1]   the argmin l
//   jump   uint16[k / kDpCheck + 1][NB + 1]   k_dp_jump
// ---------------------------------------------------------------------------------
struct DpLayout {
    size_t hdr, z0, z1, z2, cnt, ctr, d, from, split, jump, total;
};

constexpr int kDpThreads = 256;
constexpr int kDpRows = kDpThreads / 64;   // rows r per workgroup, one wave each
constexpr int kDpCheck = 16;               // levels between checkpoints of the backtrack
constexpr int kDpEntry = 8;                // levels before it take a launch each
constexpr int kDpFill = 64;                // workgroups that mark D unset
constexpr unsigned long long kDpUnset = ~0ULL;   // a NaN; D holds none

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

__host__ __device__ inline DpLayout dp_layout(int32_t nbins, int32_t k)
{
    DpLayout L;
    const size_t row = static_cast<size_t>(nbins) + 1;
    size_t o = 0;
    L.hdr = o; o += align256(16 * sizeof(int32_t));
    L.z0 = o; o += align256(row * sizeof(double));
    L.z1 = o; o += align256(row * sizeof(double));
    L.z2 = o; o += align256(row * sizeof(double));
    L.cnt = o; o += align256(row * sizeof(double));
    L.ctr = o; o += align256(row * sizeof(double));
    L.d = o; o += align256(static_cast<size_t>(k) * row * sizeof(double));
    L.from = o; o += align256(2 * row * sizeof(uint16_t));
    L.split = o; o += align256(static_cast<size_t>(k + 1) * row * sizeof(uint16_t));
    L.jump = o; o += align256(static_cast<size_t>(k / kDpCheck + 1) * row * sizeof(uint16_t));
    L.total = o;
    return L;
}

template <typename T>
__device__ __forceinline__ T* at(void* ws, size_t off)
{
    return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// The interval cost of bins l .. r from the prefix sums before l (z*) and at r (zr*), in
// the definition's operations: SSE about the mean, or about the forced entry a = -1, +1.
__device__ __forceinline__ double dp_cost_free(double zr0, double zr1, double zr2, double z0,
                                               double z1, double z2)
{
    const double S0 = zr0 - z0;
    const double S1 = zr1 - z1;
    const double S2 = zr2 - z2;
    return S2 - S1 * S1 / S0;
}

// At most dp_cost_free's value (or not a number), without its division: the quotient from a
// float32 reciprocal, raised by 2^-20 (its error is below 2^-22), so that the rounded
// difference is no larger; an S0 of 0 gives minus infinity or NaN. A candidate whose value
// from this one is above the minimum so far is none, and a whole window mostly is.
__device__ __forceinline__ double dp_cost_below(double zr0, double zr1, double zr2, double z0,
                                                double z1, double z2)
{
    const double S0 = zr0 - z0;
    const double S1 = zr1 - z1;
    const double S2 = zr2 - z2;
    const double inv = static_cast<double>(__builtin_amdgcn_rcpf(static_cast<float>(S0)));
    return S2 - S1 * S1 * inv * (1.0 + 0x1p-20);
}

__device__ __forceinline__ double dp_cost_forced(double a, double zr0, double zr1, double zr2,
                                                 double z0, double z1, double z2)
{
    const double S0 = zr0 - z0;
    const double S1 = zr1 - z1;
    const double S2 = zr2 - z2;
    return S2 - 2.0 * a * S1 + a * a * S0;
}

// Whether rows may be pruned (k_dp_level). The proof takes the stored prefix sums as exact
// numbers: bin i then has weight c_i and the point mu_i = (Z1[i] - Z1[i-1]) / c_i. It needs
// the counts' sums exact and the points in bin order; each stored Z1 is off by at most one
// rounding of itself (2^-53 N) and of c m, so with c_i >= 1 neighbouring points, 2 / nbins
// apart, keep their order while 8 N 2^-53 < 2 / nbins. N nbins < 2^50 is half of that.
__device__ __forceinline__ bool dp_may_prune(double total, int32_t nbins)
{
    return total * static_cast<double>(nbins) < 1125899906842624.0;
}

// Compaction of non-empty bins and prefix sums, in increasing bin order. The workgroup
// compacts the non-empty bins (a prefix count over 16-bin runs) and forms each one's
// centre, count and the two products c m and (c m) m in LDS; three waves then take a running
// sum each in increasing bin order, so the summation order is the definition's. A wave holds
// 64 terms in its lanes and adds them one after another from scalar registers. The chain of
// 4096 dependent float64 additions bounds the kernel: 65 us; 82 us with one lane that reads
// and writes its terms in LDS sixteen at a time, 155 us with one thread for all three sums.
// Level 1 (one interval, entry -1) is written on the way out.
constexpr int kPrepRun = kMaxBins / kThreads;   // bins per thread in the compaction
constexpr int kPrepBatch = 64;

__global__ __launch_bounds__(kThreads) void k_dp_prep(const uint64_t* __restrict__ hist,
                                                      int32_t nbins, int32_t k, void* ws)
{
    // t[q][0 .. b]: c, c m, c m m, then their running sums; slots past b are read ahead
    __shared__ double t[3][kMaxBins + 2 * kPrepBatch];
    __shared__ int runs[kThreads];
    __shared__ int nr;
    const int tid = threadIdx.x;
    const DpLayout L = dp_layout(nbins, k);
    if (blockIdx.x > 0) {   // beside the chain of workgroup 0: the levels of k_dp_run unset
        const int64_t row = nbins + 1;
        unsigned long long* d = at<unsigned long long>(ws, L.d);
        for (int64_t i = kDpEntry * row + (blockIdx.x - 1) * kThreads + tid; i < k * row;
             i += static_cast<int64_t>(gridDim.x - 1) * kThreads)
            d[i] = kDpUnset;
        return;
    }
    double* cnt = at<double>(ws, L.cnt);
    double* ctr = at<double>(ws, L.ctr);
    const double w = 2.0 / static_cast<double>(nbins);
    // thread tid owns bins [tid * kPrepRun, + kPrepRun): count, then scan the counts
    const int i0 = tid * kPrepRun;
    uint64_t hv[kPrepRun];
    int mine = 0;
#pragma unroll
    for (int q = 0; q < kPrepRun; ++q) hv[q] = i0 + q < nbins ? hist[i0 + q] : 0;
#pragma unroll
    for (int q = 0; q < kPrepRun; ++q) mine += hv[q] != 0;
    runs[tid] = mine;
    __syncthreads();
    if (tid < 64) {   // one wave: four counts a lane, then a shuffle scan
        int c[kThreads / 64], sum = 0;
        for (int q = 0; q < kThreads / 64; ++q) {
            c[q] = runs[tid * (kThreads / 64) + q];
            sum += c[q];
        }
        int acc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(acc, off);
            if (tid >= off) acc += up;
        }
        if (tid == 63) nr = acc;
        acc -= sum;
        for (int q = 0; q < kThreads / 64; ++q) {
            runs[tid * (kThreads / 64) + q] = acc;
            acc += c[q];
        }
    }
    __syncthreads();
    const int b = nr;
    int r = runs[tid];   // compacted slots before this thread's bins (0-based)
#pragma unroll
    for (int q = 0; q < kPrepRun; ++q) {
        if (hv[q] == 0) continue;
        const double c = static_cast<double>(hv[q]);
        const double m = -1.0 + (static_cast<double>(i0 + q) + 0.5) * w;
        ++r;
        const double cm = c * m;
        t[0][r] = c;
        t[1][r] = cm;
        t[2][r] = cm * m;
        ctr[r] = m;
        cnt[r] = c;
    }
    if (tid < 3) t[tid][0] = 0.0;
    if (tid < 3 * kPrepBatch) t[tid / kPrepBatch][b + 1 + tid % kPrepBatch] = 0.0;
    __syncthreads();
    if (tid < 192) {   // wave q: 64 terms in its lanes, added one after another
        double* __restrict__ x = t[tid >> 6];
        const int lane = tid & 63;
        double z = 0.0, next = x[1 + lane];
        for (int q = 0; q < b; q += kPrepBatch) {
            const double term = next;
            next = x[q + kPrepBatch + 1 + lane];   // x has 2 kPrepBatch slots past kMaxBins
            double keep = 0.0;
#pragma unroll
            for (int u = 0; u < kPrepBatch; ++u) {
                const uint64_t w = __builtin_bit_cast(uint64_t, term);
                const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(w), u);
                const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(w >> 32), u);
                z = z + __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
                keep = lane == u ? z : keep;
            }
            x[q + 1 + lane] = keep;
        }
    }
    __syncthreads();
    if (tid == 0) {
        int32_t* hdr = at<int32_t>(ws, L.hdr);
        hdr[0] = b;
        hdr[1] = b >= k ? k : (b >= 2 ? b : 0);
        hdr[2] = b >= k ? 0 : 1;
        hdr[3] = dp_may_prune(t[0][b], nbins) ? 1 : 0;
        hdr[4] = hdr[5] = 0;
    }
    double* Z0 = at<double>(ws, L.z0);
    double* Z1 = at<double>(ws, L.z1);
    double* Z2 = at<double>(ws, L.z2);
    const size_t row = static_cast<size_t>(nbins) + 1;
    double* D1 = at<double>(ws, L.d) + row;
    uint16_t* from1 = at<uint16_t>(ws, L.from) + row;
    uint16_t* split1 = at<uint16_t>(ws, L.split) + row;
    for (int q = tid; q <= b; q += kThreads) {
        const double z0 = t[0][q], z1 = t[1][q], z2 = t[2][q];
        Z0[q] = z0;
        Z1[q] = z1;
        Z2[q] = z2;
        D1[q] = q == 0 ? INFINITY : 0.0 + dp_cost_forced(-1.0, z0, z1, z2, 0.0, 0.0, 0.0);
        from1[q] = 1;
        split1[q] = 1;
    }
}

// Smallest of a wave's doubles (no NaN), in every lane.
template <int CTRL>
__device__ __forceinline__ double dpp_min(double v)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const int lo = static_cast<int>(x), hi = static_cast<int>(x >> 32);
    const uint32_t l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const uint32_t h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return fmin(v, __builtin_bit_cast(double, (static_cast<uint64_t>(h2) << 32) | l2));
}

__device__ __forceinline__ double wave_min(double v)
{
    v = dpp_min<0xB1>(v);    // quad_perm 1,0,3,2
    v = dpp_min<0x4E>(v);    // quad_perm 2,3,0,1
    v = dpp_min<0x141>(v);   // row_half_mirror
    v = dpp_min<0x140>(v);   // row_mirror
    v = dpp_min<0x142>(v);   // row_bcast15
    v = dpp_min<0x143>(v);   // row_bcast31: lane 63 has the minimum
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(x), 63);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(x >> 32), 63);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// ---------------------------------------------------------------------------------
// DP level j, 2 <= j < keff and j < kDpEntry: a wave takes one row r and its candidates l, 64 at a time
// from l = r down to the row's lower bound. Only the rows r <= b - (keff - j) are taken: a
// longer prefix leaves too few bins for the entries still to come, so no path to
// D[keff][b] passes through it.
//
// Lower bound. Write cand_j(l, r) for the exact value of D[j-1][l-1] + C(l, r) over the
// stored prefix sums. Where dp_may_prune holds, C is the SSE of points in sorted order and
// satisfies the quadrangle inequality (the forced first interval too, whose entry -1 lies
// below every mean), so
//   (a) for l' < l, cand_j(l', r) - cand_j(l, r) does not fall when r grows, and
//   (b) it does not fall when j grows: D[j] - D[j-1] does not rise along a row. (Take an
//       optimal path of j - 1 edges to y and one of j edges to x < y: an edge of the second
//       lies inside one of the first, and exchanging the two paths' tails there gives j
//       edges to y and j - 1 to x at no higher cost.)
// So a candidate l' that is worse than the minimum, at l, by more than the rounding of both
// stays worse than l's at all higher levels and rows, and is never the computed minimum
// there. Rounding: the computed C is off by at most 7.2 u (S2 + S1^2 / S0), u = 2^-53, and
// at most 12.1 u S0 in the forced interval; along a path the intervals are disjoint, so these
// add up to less than 28 u Z0[r], and each level adds at most 1.1 u of the value itself. At
// a higher level l's value is no larger than at this one (its D is not), so a difference of
// computed candidates of row r is within u (112 Z0[r] + 10 k D) of the exact one over two
// levels; `slack` is about twice that. from[r] = the smallest l whose computed candidate
// lies within slack of the minimum.
//
// A row that the level before did not have takes the from of the row below it, so that
// bound is handed from row to row and has to hold with the rounding of all the rows still
// to come. There Z0 is at most Z0[b]; l's value exceeds the one here by at most Z2[b], once
// (its D is still this row's), and the D before l' is no larger than the one before l. So
// the level's last row, which hands its bound on, takes the slack with Z0[b] for Z0[r]. (With
// Z0[r] a bin of 2e10 counts above rows of a few counts each moved entries by 1e-3.)
//
// Values and argmins are those of the full scan, bit for bit.
//
// Where rows may not be pruned (counts times bins of 2^50 or more: histograms accumulated
// over many steps) every row takes its whole window, 2.1e9 candidates at 4096 bins and 256
// entries, here and in k_dp_run; dp_cost_below spares most of them the division, and the
// windows are read once. The whole DP then takes 3.3 ms (17.1 ms with the windows taken chunk
// by chunk twice as below, 4.7 ms for the full scan of a launch a level).
//
// The candidates fall from 1.9e9 to 5e7 at b = 4096, k = 256, and a level is bound by its
// launch and two dependent trips to memory, at the first levels by long windows too: the
// first 64 candidates are loaded before the header and the lower bound are known (loading
// four or eight chunks ahead as well changed nothing). 30, 23, 13, 10, 9 and 9 us for the
// levels 2 to 7; 18.1 us a level for the full scan with the candidates staged in LDS.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kDpThreads) void k_dp_level(int32_t nbins, int32_t k, int32_t j,
                                                         void* ws)
{
    const DpLayout L = dp_layout(nbins, k);
    const size_t row = static_cast<size_t>(nbins) + 1;
    const size_t cur = (j & 1) * row, prev = row - cur;   // of `from`
    const double* __restrict__ Z0 = at<double>(ws, L.z0);
    const double* __restrict__ Z1 = at<double>(ws, L.z1);
    const double* __restrict__ Z2 = at<double>(ws, L.z2);
    const double* __restrict__ Dp = at<double>(ws, L.d) + (j - 1) * row;
    const uint16_t* __restrict__ fp = at<uint16_t>(ws, L.from) + prev;
    const int32_t* __restrict__ hdr = at<int32_t>(ws, L.hdr);
    const int lane = threadIdx.x & 63;
    const int r = j + static_cast<int>(blockIdx.x) * kDpRows +
                  __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (r > nbins) return;
    // l - 1 of this lane's first candidate, kept inside the arrays
    const int x0 = r - 1 - lane > 0 ? r - 1 - lane : 0;
    double z0 = Z0[x0], z1 = Z1[x0], z2 = Z2[x0], dv = Dp[x0];
    const double zr0 = Z0[r], zr1 = Z1[r], zr2 = Z2[r];
    const int f0 = fp[r], f1 = fp[r - 1];
    const int b = hdr[0], keff = hdr[1], prune = hdr[3];
    const int rmax = b - keff + j;
    if (j >= keff || r > rmax) return;
    int lo = j;
    if (prune) {
        const int f = r < rmax ? f0 : f1;
        lo = f > j ? f : j;
    }
    double best = INFINITY;
    int arg = 0;
    double first = INFINITY;   // the first chunk's candidate
    if (r - lane >= lo) {
        const double c = dv + dp_cost_free(zr0, zr1, zr2, z0, z1, z2);
        if (c < INFINITY) {   // counts past 2^53 can make an empty interval: NaN
            first = best = c;
            arg = r - lane;
        }
    }
    if (!prune) {   // whole windows, the loads of four chunks in flight
        constexpr int kAhead = 4;
        for (int l0 = r - 64 - lane; l0 >= lo; l0 -= 64 * kAhead) {
            double y0[kAhead], y1[kAhead], y2[kAhead], y[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int x = l0 - 64 * u >= lo ? l0 - 64 * u - 1 : lo - 1;
                y0[u] = Z0[x];
                y1[u] = Z1[x];
                y2[u] = Z2[x];
                y[u] = Dp[x];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int l = l0 - 64 * u;
                if (l < lo || y[u] + dp_cost_below(zr0, zr1, zr2, y0[u], y1[u], y2[u]) > best)
                    continue;
                const double c = y[u] + dp_cost_free(zr0, zr1, zr2, y0[u], y1[u], y2[u]);
                if (c <= best && c < INFINITY) {
                    best = c;
                    arg = l;
                }
            }
        }
    }
    for (int l = r - 64 - lane; prune && l >= lo; l -= 64) {   // falling l: the last minimum kept
        const double c = Dp[l - 1] + dp_cost_free(zr0, zr1, zr2, Z0[l - 1], Z1[l - 1], Z2[l - 1]);
        if (c <= best && c < INFINITY) {
            best = c;
            arg = l;
        }
    }
    const double m = wave_min(best);
    const double zs0 = r < rmax ? zr0 : Z0[b];   // the last row's bound is handed on
    const double slack = 1.1102230246251565e-16 *
                         (256.0 * zs0 + 32.0 * static_cast<double>(k) * m);
    const double near = m + slack;
    int bestl, from;
    if (!(m < INFINITY)) {   // no candidate has a value (see above)
        bestl = from = lo;
    } else if (r - lo < 64) {   // one chunk (wave-uniform): l falls with the lane
        bestl = r - (63 - __builtin_clzll(__ballot(first == m)));
        from = r - (63 - __builtin_clzll(__ballot(first <= near)));
    } else {
        int a = best == m ? arg : 0x7fffffff;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_xor(a, off);
            a = o < a ? o : a;
        }
        bestl = a;
        // the smallest l within slack, from the lower bound up (bestl ends the search)
        from = lo;
        for (int base = lo; prune; base += 64) {
            const int l = base + lane;
            bool ok = false;
            if (l <= r) {
                const double c = Dp[l - 1] + dp_cost_free(zr0, zr1, zr2, Z0[l - 1], Z1[l - 1],
                                                          Z2[l - 1]);
                ok = c <= near;
            }
            const unsigned long long hit = __ballot(ok);
            if (hit) {
                from = base + __builtin_ctzll(hit);
                break;
            }
            if (base + 63 >= bestl) break;
        }
    }
    if (lane == 0) {
        at<double>(ws, L.d)[j * row + r] = m;
        at<uint16_t>(ws, L.from)[cur + r] = static_cast<uint16_t>(from);
        at<uint16_t>(ws, L.split)[j * row + r] = static_cast<uint16_t>(bestl);
    }
}

// ---------------------------------------------------------------------------------
// DP levels kDpEntry <= j < keff in one launch. A workgroup owns kDpTile consecutive rows at
// every level, in LDS: the prefix sums, D of the level before for its rows and, below them,
// for the rows its candidates reach. Its own rows stay there; the others' come from global
// memory, where every D is written once and is kDpUnset before, so that a value is its own
// flag: a reader loads it ahead (while it computes the level before) and polls it only where
// it was not there yet. D goes through agent-scope atomics, since the tiles run on all XCDs.
//
// Progress. A tile reads only lower tiles' rows, and tiles are handed out in the order in
// which the workgroups start, so whoever a workgroup waits for has started and itself waits
// for nothing higher: no assumption on residency or dispatch order is needed. Waits are
// bounded all the same (kDpSpin polls, seconds); one that runs out ends its workgroup, and
// k_dp_last then computes these levels itself (dp_levels_alone).
//
// Lower bounds, candidates, slack and tie rules are k_dp_level's. A lane takes a row and one
// of its candidates, kDpChunk of them from the row's lower bound up, into `cand`; after a
// barrier sixteen lanes a row form its minimum and argmins. (A wave a row, as in k_dp_level,
// needs about six times the instructions where windows hold few candidates, which one CU
// cannot hide.)
//
// Upper bound. Windows [from, r] are as long as the intervals: hundreds of bins at the first
// levels and in thinly filled stretches. No row below R needs a candidate above the largest l
// that lies within slack of R's minimum: by (a), read downwards, l stays worse than R's
// argmin by as much at r < R, and the rounding at r is no larger than at R (Z0[r] <= Z0[R],
// and R's argmin costs less at r). So where a tile has a window of more than kDpChunk, half
// of the waves scan the window of its highest row while the other half take the rows' first
// kDpChunk / 2 candidates; mostly the scan then shows these to be all that is needed (the
// tile's rows plus the shift of the argmin between two levels), else the bound is found and
// the windows taken chunk by chunk, once for the minimum and once for `from`. (Without it
// level 8 alone took 52 us.)
//
// A launch and two trips to memory made every level 4.1-6.5 us, 1.1 ms from level 8 to 255
// at 4096 bins; this takes 0.55 ms, 1.9-2.4 us a level in every tile: the latency of the two
// barriers, the interval cost's float64 division and the sixteen lanes' minimum. Waves
// without candidates that skip their part leave it at that, tiles of 32 rows (two candidates
// a lane) take 0.75-0.95 ms. The whole DP: 1.37 -> 0.77 ms (4096 bins, 256 entries). Before
// kDpEntry the windows are so long that all CUs on one level are faster (8-30 us).
// ---------------------------------------------------------------------------------
constexpr int kDpTile = 16;
constexpr int kDpRunThreads = 1024;
constexpr int kDpHalf = kDpRunThreads / 2;
constexpr int kDpWaves = kDpRunThreads / 64;
constexpr int kDpChunk = kDpRunThreads / kDpTile;   // candidates of a row at once
constexpr int kDpEach = kDpChunk / 16;              // of one lane in the minimum
constexpr int kDpPitch = kDpTile + 1;   // doubles; a row's candidates hit distinct banks

// Workgroup barrier for LDS only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ unsigned long long dp_load(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Smallest of a row of sixteen lanes' doubles (no NaN), in each of them; the same for ints.
__device__ __forceinline__ double row_min(double v)
{
    v = dpp_min<0xB1>(v);
    v = dpp_min<0x4E>(v);
    v = dpp_min<0x141>(v);
    return dpp_min<0x140>(v);
}

template <int CTRL>
__device__ __forceinline__ int dpp_imin(int v)
{
    const int o = __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
    return o < v ? o : v;
}

__device__ __forceinline__ int row_imin(int v)
{
    v = dpp_imin<0xB1>(v);
    v = dpp_imin<0x4E>(v);
    v = dpp_imin<0x141>(v);
    return dpp_imin<0x140>(v);
}

// `polls`: of one wait, at most (negative: every tile ends at its first level).
__global__ __launch_bounds__(kDpRunThreads) void k_dp_run(int32_t nbins, int32_t k, int32_t polls,
                                                          void* ws)
{
    __shared__ double zs[3][kMaxBins + 1];
    __shared__ double ds[kMaxBins + 1];
    __shared__ double cand[kDpChunk * kDpPitch];
    __shared__ uint16_t carg[kDpChunk * kDpPitch];   // whole windows: the candidates' l
    __shared__ double wmin[8], whigh[8];   // the scan's minima, by wave: all, and above the chunk
    __shared__ int lo[kDpTile];
    // by level parity: largest window and smallest lower bound of the level's rows, smallest
    // lower bound of all rows still to come
    __shared__ int wide[2], low[2], reach[2];
    __shared__ int first_in, last_in;   // largest and smallest l within slack, as rt - l
    __shared__ int tile_s, dead;
    const DpLayout L = dp_layout(nbins, k);
    const int64_t row = nbins + 1;
    int32_t* hdr = at<int32_t>(ws, L.hdr);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {   // the tile in order of the workgroups' starts
        tile_s = atomicAdd(&hdr[4], 1);
        dead = polls < 0;
        wide[0] = wide[1] = 0;
        low[0] = low[1] = reach[0] = reach[1] = first_in = 0x7fffffff;
        last_in = -1;
    }
    __syncthreads();
    const int b = hdr[0], keff = hdr[1];
    const bool prune = hdr[3] != 0;
    const double total = at<double>(ws, L.z0)[b];
    const int R0 = 1 + tile_s * kDpTile;
    // rows [j, b - keff + j] at level j: the first level with a row of this tile
    const int lift = b - keff;
    const int j0 = R0 - lift > kDpEntry ? R0 - lift : kDpEntry;
    if (j0 >= keff || R0 + kDpTile - 1 < j0) return;
    unsigned long long* D = at<unsigned long long>(ws, L.d);
    uint16_t* split = at<uint16_t>(ws, L.split);
    {
        // lower bounds from the last level of its own launch; rows it did not have take
        // those of its last row (they hold for all higher rows and levels)
        const int rm = lift + kDpEntry - 1;
        const uint16_t* from = at<uint16_t>(ws, L.from) + ((kDpEntry - 1) & 1) * row;
        if (tid < kDpTile) {
            const int r = R0 + tid;
            const int f = prune && r >= kDpEntry ? from[r < rm ? r : rm] : 0;
            const int v = f > j0 ? f : j0;
            lo[tid] = v;
            if (r >= j0) {
                atomicMin(&reach[j0 & 1], v);
                if (r <= lift + j0) {
                    atomicMin(&low[j0 & 1], v);
                    atomicMax(&wide[j0 & 1], r - v + 1);
                }
            }
        }
        __syncthreads();
    }
    int lmin = reach[j0 & 1];
    const int top = R0 + kDpTile - 1 < b ? R0 + kDpTile - 1 : b;
    for (int x = lmin - 1 + tid; x <= top; x += kDpRunThreads) {
        zs[0][x] = at<double>(ws, L.z0)[x];
        zs[1][x] = at<double>(ws, L.z1)[x];
        zs[2][x] = at<double>(ws, L.z2)[x];
        if (j0 == kDpEntry && x >= R0)
            ds[x] = at<double>(ws, L.d)[(kDpEntry - 1) * row + x];
    }
    const int q = tid % kDpTile, slot = tid / kDpTile;   // candidates: this lane's row
    const int cq = tid >> 4, sub = tid & 15;             // minima: this lane's row
    const bool minima = tid < 16 * kDpTile;
    const double slack_all = 1.1102230246251565e-16 * 256.0 * total;
    const double slack_own =
        minima && R0 + cq <= top
            ? 1.1102230246251565e-16 * 256.0 * at<double>(ws, L.z0)[R0 + cq] : 0.0;
    unsigned long long ahead = kDpUnset;
    for (int j = j0; j < keff; ++j) {
        const int rmax = lift + j;
        if (top < j) break;
        {   // D[j-1] of the rows below the tile
            const int x0 = (lmin > j ? lmin : j) - 1;
            const unsigned long long* Dp = D + (j - 1) * row;
            unsigned long long v = ahead;
            for (int x = R0 - 1 - tid; x >= x0; x -= kDpRunThreads) {
                for (int spin = 0; v == kDpUnset; ++spin) {
                    v = dp_load(Dp + x);
                    if (v != kDpUnset) break;
                    if (spin >= polls) {
                        dead = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                ds[x] = __builtin_bit_cast(double, v);
                v = kDpUnset;
            }
            const int x = R0 - 1 - tid;
            ahead = kDpUnset;
            if (x >= x0 && x >= j) ahead = dp_load(Dp + row + x);
        }
        lds_barrier();
        if (dead) {
            if (tid == 0) atomicExch(&hdr[5], 1);
            return;
        }
        int W = wide[j & 1];
        const int llow = low[j & 1];
        lmin = reach[j & 1];
        if (tid == 0) {
            wide[(j + 1) & 1] = 0;
            low[(j + 1) & 1] = reach[(j + 1) & 1] = 0x7fffffff;
        }
        const int r = R0 + q, cr = R0 + cq;
        int lq = r >= j && r <= rmax ? lo[q] : 0x7fffffff;
        int lc = minima ? lo[cq] : 0;
        int hi = 0x7fffffff;   // no row needs a candidate above
        const double zr0 = zs[0][r], zr1 = zs[1][r], zr2 = zs[2][r];
        const double slack1 = 1.1102230246251565e-16 * 32.0 * static_cast<double>(k);
        const double slack0 = cr < rmax ? slack_own : slack_all;   // as in k_dp_level
        auto candidates = [&](int c0) {
            const int l = lq + c0 + slot;
            double c = INFINITY;
            if (lq < 0x7fffffff && l <= r && l <= hi) {
                const double f = ds[l - 1] + dp_cost_free(zr0, zr1, zr2, zs[0][l - 1], zs[1][l - 1],
                                                          zs[2][l - 1]);
                if (f < INFINITY) c = f;
            }
            cand[slot * kDpPitch + q] = c;
        };
        double m = INFINITY, near = INFINITY;
        int ib = 0x7fffffff, in = 0x7fffffff;   // l = lc + index
        // the first `each` x 16 candidates of `cand`, starting at c0: minimum, argmins
        auto reduce = [&](int c0, int each, bool value, bool argnear) {
            double v[kDpEach];
#pragma unroll
            for (int u = 0; u < kDpEach; ++u)
                v[u] = u < each ? cand[(u * 16 + sub) * kDpPitch + cq] : INFINITY;
            if (value) {
                double n = v[0];
#pragma unroll
                for (int u = 1; u < kDpEach; ++u) n = fmin(n, v[u]);
                n = row_min(n);
                int f = 0x7fffffff;
#pragma unroll
                for (int u = kDpEach - 1; u >= 0; --u)
                    if (v[u] == n) f = c0 + u * 16 + sub;
                f = row_imin(f);
                if (n < m) {   // rising l: the first minimum kept
                    m = n;
                    ib = f;
                }
                near = m + (slack0 + slack1 * m);
            }
            if (argnear) {
                int f = 0x7fffffff;
#pragma unroll
                for (int u = kDpEach - 1; u >= 0; --u)
                    if (v[u] <= near) f = c0 + u * 16 + sub;
                f = row_imin(f);
                in = f < in ? f : in;
            }
        };
        bool done = !prune;
        if (!prune) {   // whole windows: a lane's minimum over every kDpChunk-th candidate
            double best = INFINITY;
            int arg = j;
            if (lq < 0x7fffffff) {
                for (int l = r - slot; l >= j; l -= kDpChunk) {   // falling l: the last one kept
                    const double y = ds[l - 1], y0 = zs[0][l - 1], y1 = zs[1][l - 1],
                                 y2 = zs[2][l - 1];
                    if (y + dp_cost_below(zr0, zr1, zr2, y0, y1, y2) > best) continue;
                    const double c = y + dp_cost_free(zr0, zr1, zr2, y0, y1, y2);
                    if (c <= best && c < INFINITY) {
                        best = c;
                        arg = l;
                    }
                }
            }
            cand[slot * kDpPitch + q] = best;
            carg[slot * kDpPitch + q] = static_cast<uint16_t>(arg);
            lds_barrier();
            if (minima) {
                for (int u = 0; u < kDpEach; ++u) m = fmin(m, cand[(u * 16 + sub) * kDpPitch + cq]);
                m = row_min(m);
                for (int u = 0; u < kDpEach; ++u) {
                    const int x = (u * 16 + sub) * kDpPitch + cq;
                    const int f = carg[x] - lc;
                    if (cand[x] == m && f < ib) ib = f;
                }
                ib = row_imin(ib);
                in = 0;
            }
        }
        if (prune && W > kDpChunk) {
            const int rt = top < rmax ? top : rmax, lt = lo[rt - R0];
            const int g = llow + kDpChunk / 2 - 1;
            const double t0 = zs[0][rt], t1 = zs[1][rt], t2 = zs[2][rt];
            auto cost = [&](int l) {
                const double c = ds[l - 1] + dp_cost_free(t0, t1, t2, zs[0][l - 1], zs[1][l - 1],
                                                          zs[2][l - 1]);
                return c < INFINITY ? c : INFINITY;
            };
            if (tid < kDpHalf) {
                candidates(0);
            } else {
                double a = INFINITY, h = INFINITY;
                for (int l = rt - (tid - kDpHalf); l >= lt; l -= kDpHalf) {
                    const double c = cost(l);
                    a = fmin(a, c);
                    if (l > g) h = fmin(h, c);
                }
                a = wave_min(a);
                h = wave_min(h);
                if (lane == 0) {
                    wmin[wave - 8] = a;
                    whigh[wave - 8] = h;
                }
            }
            lds_barrier();
            const double mt = row_min(wmin[lane & 7]);
            const double mh = row_min(whigh[lane & 7]);
            const double neart =
                mt + ((rt < rmax ? 1.1102230246251565e-16 * 256.0 * t0 : slack_all) + slack1 * mt);
            if (mh > neart) {
                if (minima) reduce(0, kDpEach / 2, true, true);
                done = true;
            } else if (mt < INFINITY) {
                int fi = 0x7fffffff, la = -1;
                for (int x = wave * 64; rt - x >= lt; x += kDpRunThreads) {
                    const int l = rt - x - lane;
                    const unsigned long long hit = __ballot(l >= lt && cost(l >= lt ? l : lt) <= neart);
                    if (hit) {
                        const int f = x + __builtin_ctzll(hit);
                        fi = f < fi ? f : fi;
                        la = x + 63 - __builtin_clzll(hit);
                    }
                }
                if (lane == 0 && la >= 0) {
                    atomicMin(&first_in, fi);
                    atomicMax(&last_in, la);
                }
                lds_barrier();
                hi = rt - first_in;
                int from = llow;
                if (rt == R0 || rt == j) {   // the level's only row here
                    from = rt - last_in;
                    if (r == rt) lq = from;
                    if (cr == rt) lc = from;
                }
                W = W < hi - from + 1 ? W : hi - from + 1;
                lds_barrier();   // `cand` is rewritten, the two bounds are reset
                if (tid == 0) {
                    first_in = 0x7fffffff;
                    last_in = -1;
                }
            }
        }
        for (int pass = 0; pass < 2 && !done; ++pass) {
            done = W <= kDpChunk;
            for (int c0 = 0; c0 < W; c0 += kDpChunk) {
                if (pass > 0 || c0 > 0) lds_barrier();   // the chunk before is read
                candidates(c0);
                lds_barrier();
                if (minima) reduce(c0, kDpEach, pass == 0, pass > 0 || done);
            }
        }
        if (minima && sub == 0 && cr >= j && cr <= rmax) {
            const int bestl = m < INFINITY ? lc + ib : lc;
            const int from = m < INFINITY ? lc + in : lc;
            ds[cr] = m;
            __hip_atomic_store(D + j * row + cr, __builtin_bit_cast(unsigned long long, m),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            split[j * row + cr] = static_cast<uint16_t>(bestl);
            const int p = (j + 1) & 1;
            int v = prune && from > j + 1 ? from : j + 1;
            lo[cq] = v;
            if (cr > j) {
                atomicMax(&wide[p], cr - v + 1);
                atomicMin(&low[p], v);
                atomicMin(&reach[p], v);
            }
            if (cr == rmax && cq + 1 < kDpTile) {   // the row that level j + 1 adds
                const int o = lo[cq + 1];
                v = v > o ? v : o;
                lo[cq + 1] = v;
                atomicMax(&wide[p], cr + 1 - v + 1);
                atomicMin(&low[p], v);
                atomicMin(&reach[p], o);   // those after it still have their first bound
            }
        }
    }
}

// jump[s][x], s >= 1: the path's row at level s kDpCheck from row x at the upper end of that
// stretch, level (s + 1) kDpCheck or keff - 1. A thread each, at most kDpCheck dependent
// reads.
__global__ __launch_bounds__(256) void k_dp_jump(int32_t nbins, int32_t k, void* ws)
{
    const DpLayout L = dp_layout(nbins, k);
    const int64_t row = nbins + 1;
    const int32_t* hdr = at<int32_t>(ws, L.hdr);
    const int b = hdr[0], keff = hdr[1];
    const int base = (blockIdx.y + 1) * kDpCheck;
    if (base > keff - 2 || hdr[5]) return;
    const int top = base + kDpCheck < keff - 1 ? base + kDpCheck : keff - 1;
    int x = blockIdx.x * 256 + threadIdx.x;
    if (x < top || x > b - keff + top) return;   // rows of level `top`
    const int x0 = x;
    const uint16_t* split = at<uint16_t>(ws, L.split);
    for (int j = top; j > base; --j) x = split[j * row + x] - 1;
    at<uint16_t>(ws, L.jump)[(blockIdx.y + 1) * row + x0] = static_cast<uint16_t>(x);
}

// Levels kDpEntry .. keff - 1 by one workgroup of 1024, every candidate of every row, where a
// wait of k_dp_run ran out (by reading it never does): the same values and argmins, about
// half a second at 4096 bins and 256 entries.
__device__ __forceinline__ void dp_levels_alone(int32_t nbins, int32_t k, int32_t b, int32_t keff,
                                             void* ws)
{
    const DpLayout L = dp_layout(nbins, k);
    const size_t row = static_cast<size_t>(nbins) + 1;
    const double* Z0 = at<double>(ws, L.z0);
    const double* Z1 = at<double>(ws, L.z1);
    const double* Z2 = at<double>(ws, L.z2);
    double* D = at<double>(ws, L.d);
    uint16_t* split = at<uint16_t>(ws, L.split);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int j = kDpEntry; j < keff; ++j) {
        const double* Dp = D + (j - 1) * row;
        for (int r = j + wave; r <= b - keff + j; r += 1024 / 64) {
            const double zr0 = Z0[r], zr1 = Z1[r], zr2 = Z2[r];
            double best = INFINITY;
            int arg = 0x7fffffff;
            for (int l = j + lane; l <= r; l += 64) {   // rising l: the first minimum kept
                const double c = Dp[l - 1] + dp_cost_free(zr0, zr1, zr2, Z0[l - 1], Z1[l - 1],
                                                          Z2[l - 1]);
                if (c < best) {
                    best = c;
                    arg = l;
                }
            }
            const double m = wave_min(best);
            if (best != m) arg = 0x7fffffff;
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_xor(arg, off);
                arg = o < arg ? o : arg;
            }
            if (lane == 0) {
                D[j * row + r] = m;
                split[j * row + r] = static_cast<uint16_t>(m < INFINITY ? arg : j);
            }
        }
        __syncthreads();
    }
}

// The last level (row b only, entry +1) and the backtrack, one workgroup. The path's rows
// at the checkpoint levels come from jump, one dependent read per kDpCheck levels;
// then one lane per stretch between checkpoints walks its split entries, and the entries
// (-1, +1 or the weighted mean of the interval) are formed in parallel: 32 dependent reads
// at k = 256 where a walk along the levels took 255 (77-110 us). Degenerate histograms
// (b < k) are padded with +1.
__global__ __launch_bounds__(1024) void k_dp_last(int32_t nbins, int32_t k, void* ws,
                                                  double* codebook, double* cost, int32_t* status)
{
    __shared__ double sv[16];
    __shared__ int sa[16];
    __shared__ int node[kMaxK + 1];   // row of the path at each level
    const DpLayout L = dp_layout(nbins, k);
    const int32_t* hdr = at<int32_t>(ws, L.hdr);
    const int b = hdr[0];
    const int keff = hdr[1];
    const double* Z0 = at<double>(ws, L.z0);
    const double* Z1 = at<double>(ws, L.z1);
    const double* Z2 = at<double>(ws, L.z2);
    const size_t row = static_cast<size_t>(nbins) + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (keff < 2) {
        if (tid != 0) return;
        const double* cnt = at<double>(ws, L.cnt);
        const double* ctr = at<double>(ws, L.ctr);
        codebook[0] = -1.0;
        for (int j = 1; j < k; ++j) codebook[j] = 1.0;
        double e = 0.0;
        for (int i = 1; i <= b; ++i) {
            const double dl = ctr[i] + 1.0, dr = 1.0 - ctr[i];
            const double d2 = (dl * dl < dr * dr) ? dl * dl : dr * dr;
            e += cnt[i] * d2;
        }
        *cost = e;
        *status = hdr[2];
        return;
    }
    const bool alone = hdr[5] != 0;   // a wait of k_dp_run ran out
    if (alone) dp_levels_alone(nbins, k, b, keff, ws);
    const double* Dp = at<double>(ws, L.d) + (keff - 1) * row;
    const double zr0 = Z0[b], zr1 = Z1[b], zr2 = Z2[b];
    double best = INFINITY;
    int arg = 0x7fffffff;
    for (int l = keff + tid; l <= b; l += 1024) {   // rising l: the first minimum kept
        const double c = Dp[l - 1] + dp_cost_forced(1.0, zr0, zr1, zr2, Z0[l - 1], Z1[l - 1],
                                                    Z2[l - 1]);
        if (c < best) {
            best = c;
            arg = l;
        }
    }
    const double m = wave_min(best);
    if (best != m) arg = 0x7fffffff;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_xor(arg, off);
        arg = o < arg ? o : arg;
    }
    if (lane == 0) {
        sv[wave] = m;
        sa[wave] = arg;
    }
    __syncthreads();
    if (tid == 0) {
        double v = sv[0];
        int a = sa[0];
        for (int q = 1; q < 16; ++q)
            if (sv[q] < v || (sv[q] == v && sa[q] < a)) {
                v = sv[q];
                a = sa[q];
            }
        if (!(v < INFINITY)) a = keff;   // no candidate has a value
        *cost = v;
        *status = hdr[2];
        node[keff] = b;
        node[keff - 1] = a - 1;
        // checkpoint levels below keff - 1, multiples of kDpCheck
        int x = a - 1;
        if (alone) {   // without jump
            for (int j = keff - 1; j > 1; --j) {
                x = at<uint16_t>(ws, L.split)[static_cast<size_t>(j) * row + x] - 1;
                node[j - 1] = x;
            }
        } else {
            for (int st = (keff - 2) / kDpCheck; st >= 1; --st) {
                x = at<uint16_t>(ws, L.jump)[static_cast<size_t>(st) * row + x];
                node[st * kDpCheck] = x;
            }
        }
        node[0] = 0;
    }
    __syncthreads();
    // stretch s: the levels strictly between checkpoint s and the next one (or keff - 1)
    const int stretches = (keff - 2) / kDpCheck + 1;
    if (tid < stretches) {
        const int base = tid * kDpCheck;
        int top = base + kDpCheck;
        if (top > keff - 1) top = keff - 1;
        int x = node[top];
        for (int j = top; j > base + 1; --j) {
            x = at<uint16_t>(ws, L.split)[static_cast<size_t>(j) * row + x] - 1;
            node[j - 1] = x;
        }
    }
    __syncthreads();
    for (int j = 1 + tid; j <= k; j += 1024) {
        double e = 1.0;
        if (j == 1) {
            e = -1.0;
        } else if (j < keff) {
            const int r = node[j], x = node[j - 1];
            const double S0 = Z0[r] - Z0[x];
            const double S1 = Z1[r] - Z1[x];
            e = S1 / S0;
        }
        codebook[j - 1] = e;
    }
}

// ---------------------------------------------------------------------------------
// Codebook installation: fp32 entries, fp64 copy, midpoints and the guide table.
// guide[bk] = number of midpoints whose bucket is < bk, bucket(x) =
// min(ng - 1, (int)((x + 1) * ng / 2)) in fp32 -- the same function the step applies
// to the (clamped) value being encoded, so the lookup is exact for fp32 midpoints. The
// midpoints' buckets are counted in LDS and scanned by the workgroup, 16 buckets a thread
// (85 us with one thread taking the 4096 buckets in turn).
// ---------------------------------------------------------------------------------
constexpr int kGuideRun = kMaxBins / kThreads;   // buckets per thread

__global__ __launch_bounds__(kThreads) void k_install(const double* __restrict__ in64,
                                                      const float* __restrict__ in32, int32_t k,
                                                      int32_t ng, float* cb32, double* cb64,
                                                      float* mid, uint8_t* guide)
{
    __shared__ float c[kMaxK];
    __shared__ uint32_t cnt[kMaxBins];
    __shared__ uint32_t wsum[kThreads / 64];
    const int t = threadIdx.x;
    for (int i = t; i < k; i += kThreads) {
        const float f = in64 ? static_cast<float>(in64[i]) : in32[i];
        c[i] = f;
        cb32[i] = f;
        cb64[i] = in64 ? in64[i] : static_cast<double>(in32[i]);
    }
    for (int i = t; i < kMaxBins; i += kThreads) cnt[i] = 0;
    __syncthreads();
    const float half_ng = 0.5f * static_cast<float>(ng);
    for (int i = t; i < k; i += kThreads) {
        const float mdp = i + 1 < k ? 0.5f * (c[i] + c[i + 1]) : 2.0f;
        mid[i] = mdp;
        if (i + 1 < k) {
            const float x = fminf(fmaxf(mdp, -1.0f), 1.0f);
            int bk = static_cast<int>((x + 1.0f) * half_ng);
            bk = bk < ng - 1 ? bk : ng - 1;
            atomicAdd(&cnt[bk], 1u);
        }
    }
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kGuideRun; ++q) sum += cnt[t * kGuideRun + q];
    uint32_t acc = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_up(acc, off);
        if ((t & 63) >= off) acc += up;
    }
    if ((t & 63) == 63) wsum[t >> 6] = acc;
    __syncthreads();
    acc -= sum;
    for (int w = 0; w < (t >> 6); ++w) acc += wsum[w];
    // the global guide is padded to 16 bytes past its ng + 1 entries
    for (int q = 0; q < kGuideRun; ++q) {
        const int bk = t * kGuideRun + q;
        if (bk < ng) guide[bk] = static_cast<uint8_t>(acc);
        acc += cnt[bk];
    }
    if (t == 0) {
        uint32_t all = 0;
        for (int w = 0; w < kThreads / 64; ++w) all += wsum[w];
        guide[ng] = static_cast<uint8_t>(all);
        for (int bk = ng + 1; bk < ((ng + 1 + 15) & ~15); ++bk) guide[bk] = 0;
    }
}

}  // namespace

size_t dp_workspace_bytes(int32_t nbins, int32_t k) { return dp_layout(nbins, k).total; }

hipError_t launch_hist_h_absmax(const Tile* tiles, const HTile* htiles, int64_t n_tiles,
                                const Seg* segs, float* am_partials, hipStream_t stream)
{
    if (n_tiles <= 0) return hipSuccess;
    if (n_tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_hist_h_absmax, dim3(static_cast<unsigned>(n_tiles)), dim3(kThreads), 0,
                       stream, tiles, htiles, segs, am_partials);
    return hipGetLastError();
}

hipError_t launch_histogram(const Tile* tiles, int64_t n_tiles, const int32_t* tile_kind,
                            const HTile* htiles, const float* am_partials, const Seg* segs,
                            int32_t nbins, uint64_t* hist, int32_t ways, hipStream_t stream)
{
    if (n_tiles <= 0) return hipSuccess;
    const int64_t w = (n_tiles + kThreads / 64 - 1) / (kThreads / 64);
    const auto grid = [&](int64_t most) {
        return dim3(static_cast<unsigned>(w < most ? w : most));
    };
    const int64_t longest = ways & kHistLong ? INT64_MAX : kHistVecBlock;
    if (ways & kHistVec)   // as many workgroups as are resident
        hipLaunchKernelGGL(k_histogram<true>, grid(kHistVecGroups), dim3(kThreads), 0, stream,
                           tiles, n_tiles, tile_kind, htiles, am_partials, segs, nbins, longest,
                           hist);
    if (ways & kHistStream)
        hipLaunchKernelGGL(k_histogram<false>, grid(4096), dim3(kThreads), 0, stream, tiles,
                           n_tiles, tile_kind, htiles, am_partials, segs, nbins, longest,
                           hist);
    return hipGetLastError();
}

hipError_t launch_dp(const uint64_t* hist, int32_t nbins, int32_t k, void* ws,
                     double* codebook_out, double* cost_out, int32_t* status_out,
                     hipStream_t stream, int32_t polls)
{
    hipLaunchKernelGGL(k_dp_prep, dim3(1 + (k > kDpEntry ? kDpFill : 0)), dim3(kThreads), 0, stream,
                       hist, nbins, k, ws);
    for (int j = 2; j < k && j < kDpEntry; ++j) {
        // rows j .. nbins - k + j at most (b <= nbins, keff <= k; with b < k: rows j .. j)
        const int rows = nbins > k ? nbins - k + 1 : 1;
        hipLaunchKernelGGL(k_dp_level, dim3((rows + kDpRows - 1) / kDpRows), dim3(kDpThreads), 0,
                           stream, nbins, k, j, ws);
    }
    if (k > kDpEntry)
        hipLaunchKernelGGL(k_dp_run, dim3((nbins + kDpTile - 1) / kDpTile), dim3(kDpRunThreads), 0,
                           stream, nbins, k, polls, ws);
    if (k - 2 >= kDpCheck)
        hipLaunchKernelGGL(k_dp_jump, dim3(nbins / 256 + 1, (k - 2) / kDpCheck), dim3(256), 0,
                           stream, nbins, k, ws);
    hipLaunchKernelGGL(k_dp_last, dim3(1), dim3(1024), 0, stream, nbins, k, ws, codebook_out,
                       cost_out, status_out);
    return hipGetLastError();
}

hipError_t launch_install_codebook(const double* cb64_in, int32_t k, int32_t ng, float* cb32,
                                   double* cb64, float* mid, uint8_t* guide, hipStream_t stream)
{
    hipLaunchKernelGGL(k_install, dim3(1), dim3(kThreads), 0, stream, cb64_in,
                       static_cast<const float*>(nullptr), k, ng, cb32, cb64, mid, guide);
    return hipGetLastError();
}

hipError_t launch_install_codebook_f32(const float* cb32_in, int32_t k, int32_t ng, float* cb32,
                                       double* cb64, float* mid, uint8_t* guide,
                                       hipStream_t stream)
{
    hipLaunchKernelGGL(k_install, dim3(1), dim3(kThreads), 0, stream,
                       static_cast<const double*>(nullptr), cb32_in, k, ng, cb32, cb64, mid,
                       guide);
    return hipGetLastError();
}

}  // namespace gefen
