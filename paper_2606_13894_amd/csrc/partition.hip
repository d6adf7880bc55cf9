// Automatic Block Partitioning (Sec. 5.1, Alg. 2) for gfx950.
//
// For every tensor of n elements and every divisor p of n:
//   z_j  = log(g_j^2 + eps)                     (float64)
//   mu_i = (sum of z over block i of p elements) / p
//   S(p) = sum_{i < n/p - 1} |mu_{i+1} - mu_i| / (n/p - 1),   S(n) = 0
// then the strict local maxima of S over the sorted divisors (1 < p < n), and the one
// with the largest S (ties: smallest p), else 1.
//
// The sums are built from each other (part_plan.h): one pass over the gradient with one
// float64 logarithm per element forms those of every divisor of L in LDS, and the other
// divisors' sums come from stored ones. Evaluating z once per divisor, as the definition
// reads, took 32.5 ms on the GPT-2 small shapes and 235 ms on the Llama-3 1.5B shapes; this
// form takes 1.9 and 17 ms. All sums run in a fixed order (the same tree for every
// block of one divisor), so the scores are deterministic.
#include "gefen_internal.h"

#include <math.h>

namespace gefen {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double z_at(const void* g, int gdt, int64_t i, double eps)
{
    double x;
    if (gdt == DT_F32)
        x = static_cast<double>(static_cast<const float*>(g)[i]);
    else
        x = static_cast<double>(
            __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(g)[i]) << 16));
    return log(x * x + eps);
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// Fixed-order workgroup sum (wave butterflies, then waves 0..3 in order).
__device__ __forceinline__ double block_sum(double v, double* red)
{
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    double t = red[0];
    for (int w = 1; w < kThreads / 64; ++w) t += red[w];
    __syncthreads();
    return t;
}

// The last of `n` records (by their first item) whose first item is at most `item`.
template <typename T, typename F>
__device__ __forceinline__ int find_item(const T* recs, int32_t n, int64_t item, F first)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first(recs[mid]) <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// A wave's sum by lane permutes inside the vector unit, in every lane of the result's row
// and complete in lane 63 (quads, rows of 16, then the rows in order).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), CTRL, ROWS, 0xf,
                                                    false);
    return v + __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ __forceinline__ double wave_sum63(double v)
{
    v = dpp_add<0xB1, 0xf>(v);    // quad_perm 1,0,3,2
    v = dpp_add<0x4E, 0xf>(v);    // quad_perm 2,3,0,1
    v = dpp_add<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);   // row_mirror
    v = dpp_add<0x142, 0xa>(v);   // row_bcast15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);   // row_bcast31 into rows 2 and 3
}

// The base pass. About 40 float64 operations for each logarithm against 2 to 4 bytes; the
// sums of all divisors of L add about two LDS reads and an addition per element. What bounds
// it is the chain of phases, so a chunk is small (about three 512-thread workgroups
// a CU hide each other's barriers; the vector units are busy 56 % of the time), the waves of a phase work on different divisors, the units'
// descriptors lie in LDS with the next one loaded ahead, and a workgroup takes a run of
// chunks: the search for its tensor is paid once, the next chunk's gradients are loaded
// under the work on this one, and contrasts add up over the run. On the GPT-2 small shapes:
// 2.09 ms with one 2048-element chunk per workgroup and all its threads on one divisor at a
// time; this: 1.57 ms.
__global__ __launch_bounds__(kPartThreads) void k_part_base(const PartTensor* __restrict__ tensors,
                                                            int32_t n_tensors,
                                                            const PartUnit* __restrict__ units,
                                                            const int32_t* __restrict__ phase_end,
                                                            const int64_t* __restrict__ keep,
                                                            double eps, double* __restrict__ sums,
                                                            double* __restrict__ part)
{
    extern __shared__ double S[];
    __shared__ u32x4 un[kPartMaxUnit];
    __shared__ int pe[kPartMaxPhase];
    __shared__ double gap[kPartMaxUnit];      // contrasts of the run, by GAP unit
    __shared__ double edge[kPartMaxEntry];    // last sum of the chunk before, by entry
    const int64_t item = blockIdx.x;
    const PartTensor t = tensors[find_item(tensors, n_tensors, item,
                                           [](const PartTensor& x) { return x.group0; })];
    const int64_t grp = item - t.group0;
    const int64_t c0 = grp * t.run;
    const int64_t c1 = c0 + t.run < t.nchunk ? c0 + t.run : t.nchunk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kPer = kPartChunkMax / kPartThreads;
    float g[kPer];
    auto load = [&](int64_t c) {   // elements past the tensor read its last one
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            int64_t i = c * t.chunk + tid + u * kPartThreads;
            i = i < t.n ? i : t.n - 1;
            if (t.gdtype == DT_F32)
                g[u] = static_cast<const float*>(t.grad)[i];
            else
                g[u] = __uint_as_float(
                    static_cast<uint32_t>(static_cast<const uint16_t*>(t.grad)[i]) << 16);
        }
    };
    load(c0);
    for (int u = tid; u < t.nunit; u += kPartThreads) {
        un[u] = reinterpret_cast<const u32x4*>(units + t.unit0)[u];
        gap[u] = 0.0;
    }
    if (tid < t.nphase) pe[tid] = phase_end[t.phase0 + tid];
    for (int64_t c = c0; c < c1; ++c) {
        const int64_t start = c * t.chunk;
        const int len = static_cast<int>(t.n - start < t.chunk ? t.n - start : t.chunk);
        const bool whole = len == t.chunk;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + u * kPartThreads;
            const double x = static_cast<double>(g[u]);
            if (i < len) S[i] = log(x * x + eps);   // p = 1 lies at 0
        }
        if (c + 1 < c1) load(c + 1);
        int u = wave;
        __syncthreads();
        for (int f = 1; f < t.nphase; ++f) {
            const int end = pe[f];
            u32x4 next = un[u < end ? u : 0];
            while (u < end) {
                const u32x4 w = next;
                const int u1 = u + kPartThreads / 64;
                next = un[u1 < end ? u1 : u];
                const uint32_t w0 = __builtin_amdgcn_readfirstlane(static_cast<int>(w.x));
                const uint32_t w1 = __builtin_amdgcn_readfirstlane(static_cast<int>(w.y));
                const uint32_t w2 = __builtin_amdgcn_readfirstlane(static_cast<int>(w.z));
                const uint32_t w3 = __builtin_amdgcn_readfirstlane(static_cast<int>(w.w));
                const int kind = w0 & 0xffff, p = w0 >> 16, q = w1 & 0xffff;
                const int i0 = w2 >> 16, slot = w3 >> 16;
                const int cnt = whole ? static_cast<int>(w3 & 0xffff) : len / p;
                const double* __restrict__ s = S + (w1 >> 16);
                const int stop = i0 + kPartUnit < cnt ? i0 + kPartUnit : cnt;
                if (kind == PART_ADD) {
                    double* __restrict__ d = S + (w2 & 0xffff);
                    if (q == 2) {
#pragma unroll 4
                        for (int i = i0 + lane; i < stop; i += 64) d[i] = s[2 * i] + s[2 * i + 1];
                    } else if (q == 3) {
#pragma unroll 4
                        for (int i = i0 + lane; i < stop; i += 64)
                            d[i] = s[3 * i] + s[3 * i + 1] + s[3 * i + 2];
                    } else {
                        for (int i = i0 + lane; i < stop; i += 64) {
                            double a = s[i * q];
#pragma unroll 4
                            for (int j = 1; j < q; ++j) a += s[i * q + j];
                            d[i] = a;
                        }
                    }
                } else if (kind == PART_GAP) {
                    const int top = stop < cnt ? stop : cnt - 1;
                    double acc = 0.0;
#pragma unroll 4
                    for (int i = i0 + lane; i < top; i += 64) acc += fabs(s[i + 1] - s[i]);
                    acc = wave_sum63(acc);
                    if (lane == 63) {   // the unit is this wave's in every chunk
                        const int e = w2 & 0xffff;
                        if (i0 == 0) {
                            double* __restrict__ o = part + t.out0 + (t.ngap + e) * t.ngroup + grp;
                            if (c == c0)
                                o[0] = s[0];
                            else
                                acc += fabs(s[0] - edge[e]);
                            edge[e] = s[cnt - 1];
                            if (c + 1 == c1) o[t.nentry * t.ngroup] = s[cnt - 1];
                        }
                        const double sum = gap[slot] + acc;
                        gap[slot] = sum;
                        if (c + 1 == c1) part[t.out0 + slot * t.ngroup + grp] = sum;
                    }
                } else {
                    double* __restrict__ o = sums + keep[t.keep0 + slot] + start / p;
                    for (int i = i0 + lane; i < stop; i += 64) o[i] = s[i];
                }
                u = u1;
            }
            u = end + wave;
            __syncthreads();
        }
    }
}

// The direct divisors: z of a span and two blocks beyond it in LDS, one logarithm an element
// for all of them, then a wave a divisor at a time: g lanes a block, 64 / g blocks, each
// contrasted with the next one's lanes. Bound by the logarithms: 262M bfloat16 gradients and
// one divisor 0.94 ms.
__global__ __launch_bounds__(kPartDirectThreads) void k_part_direct(
    const PartSpan* __restrict__ spans, int32_t n_spans, const int32_t* __restrict__ direct,
    const int64_t* __restrict__ store, const PartTensor* __restrict__ tensors, double eps,
    double* __restrict__ sums, double* __restrict__ part)
{
    extern __shared__ double S[];
    const int64_t item = blockIdx.x;
    const PartSpan sp =
        spans[find_item(spans, n_spans, item, [](const PartSpan& x) { return x.item0; })];
    const PartTensor t = tensors[sp.tensor];
    const int64_t it = item - sp.item0;
    const int64_t e0 = it * kPartSpan;
    const int64_t e1 = e0 + kPartSpan < t.n ? e0 + kPartSpan : t.n;
    const int64_t stop = e1 + 2 * direct[sp.first + sp.count - 1];
    const int len = static_cast<int>((stop < t.n ? stop : t.n) - e0);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll 4
    for (int i = tid; i < len; i += kPartDirectThreads) S[i] = z_at(t.grad, t.gdtype, e0 + i, eps);
    __syncthreads();
    for (int d = wave; d < sp.count; d += kPartDirectThreads / 64) {
        const int p = direct[sp.first + d];
        const int64_t first = (e0 + p - 1) / p, nb = t.n / p;
        const int64_t next_first = (e1 + p - 1) / p;
        // contrasts of first .. last - 1; block `last` is read
        const int64_t last = next_first < nb - 1 ? next_first : nb - 1;
        const int cnt = static_cast<int>(last - first);
        const int64_t at = store[sp.store0 + d];
        double* __restrict__ o = at < 0 ? nullptr : sums + at + first;
        const int own = static_cast<int>(next_first - first);   // sums of this item
        const double* __restrict__ s = S + (first * p - e0);
        const int gl = p <= 32 ? 0 : p <= 256 ? 2 : 4;
        const int g = 1 << gl, per = 64 >> gl, sub = lane & (g - 1), blk = lane >> gl;
        double acc = 0.0;
        for (int b = 0; b < cnt || b < own; b += per - 1) {
            const int i = b + blk;
            double v = 0.0;
            if (i <= cnt) {
#pragma unroll 4
                for (int k = sub; k < p; k += g) v += s[i * p + k];
            }
            for (int off = 1; off < g; off <<= 1) v += __shfl_xor(v, off);
            const double next = __shfl(v, (lane + g) & 63);
            if (sub == 0 && blk + 1 < per) {
                if (i < cnt) acc += fabs(next - v);
                if (o && i < own) o[i] = v;
            }
        }
        acc = wave_sum63(acc);
        if (lane == 63) part[sp.out + d * sp.n_items + it] = acc;
    }
}

// Terms [a, b) of a job's source, summed by `stride` threads of which this is `tid`.
__device__ __forceinline__ double term_sum(const PartJob& j, const PartTensor& t,
                                           const double* __restrict__ sums, double eps, int64_t a,
                                           int64_t b, int tid, int stride)
{
    double acc = 0.0;
    if (j.src >= 0) {
        const double* __restrict__ s = sums + j.src;
        for (int64_t i = a + tid; i < b; i += stride) acc += s[i];
    } else {
        for (int64_t i = a + tid; i < b; i += stride) acc += z_at(t.grad, t.gdtype, i, eps);
    }
    return acc;
}

__global__ __launch_bounds__(kThreads) void k_part_jobs(const PartJob* __restrict__ jobs,
                                                        int32_t n_jobs,
                                                        const PartTensor* __restrict__ tensors,
                                                        double eps, double* __restrict__ sums,
                                                        double* __restrict__ part)
{
    __shared__ double red[kThreads / 64];
    const int64_t item = blockIdx.x;
    const PartJob j = jobs[find_item(jobs, n_jobs, item, [](const PartJob& x) { return x.item0; })];
    const PartTensor t = tensors[j.tensor];
    const int64_t it = item - j.item0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (j.kind == PART_DIFF) {
        const double* __restrict__ s = sums + j.src;
        const int64_t a = it * j.per;
        const int64_t b = a + j.per < j.count - 1 ? a + j.per : j.count - 1;
        double acc = 0.0;
        for (int64_t i = a + tid; i < b; i += kThreads) acc += fabs(s[i + 1] - s[i]);
        acc = block_sum(acc, red);
        if (tid == 0) part[j.dst + it] = acc;
        return;
    }
    if (j.kind == PART_SUB) {
        const int64_t blk = it / j.sub, a = blk * j.q + (it % j.sub) * kPartSub;
        const int64_t end = (blk + 1) * j.q;
        const double s = block_sum(term_sum(j, t, sums, eps, a, a + kPartSub < end ? a + kPartSub
                                                                                  : end,
                                            tid, kThreads), red);
        if (tid == 0) sums[j.dst + it] = s;
        return;
    }
    const int64_t b0 = it * j.per;
    const int64_t b1 = b0 + j.per < j.count ? b0 + j.per : j.count;
    if (j.per == 1) {          // long blocks: the workgroup
        const double s = block_sum(term_sum(j, t, sums, eps, b0 * j.q, (b0 + 1) * j.q, tid, kThreads),
                                   red);
        if (tid == 0) sums[j.dst + b0] = s;
    } else if (j.q <= 16) {    // short ones: a thread each
        for (int64_t b = b0 + tid; b < b1; b += kThreads)
            sums[j.dst + b] = term_sum(j, t, sums, eps, b * j.q, (b + 1) * j.q, 0, 1);
    } else {                   // a wave each
        for (int64_t b = b0 + wave; b < b1; b += kThreads / 64) {
            const double s = wave_sum(term_sum(j, t, sums, eps, b * j.q, (b + 1) * j.q, lane, 64));
            if (lane == 0) sums[j.dst + b] = s;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_part_finalize(const PartScore* __restrict__ scores,
                                                            const double* __restrict__ part,
                                                            double* __restrict__ out)
{
    __shared__ double red[kThreads / 64];
    const PartScore s = scores[blockIdx.x];
    const int tid = threadIdx.x;
    if (s.nb < 2) {
        if (tid == 0) out[blockIdx.x] = 0.0;
        return;
    }
    const double* __restrict__ x = part + s.out;
    double acc = 0.0;
#pragma unroll 4
    for (int64_t i = tid; i < s.terms; i += kThreads) acc += x[i];
    const double* __restrict__ f = part + s.firsts;
    const double* __restrict__ l = part + s.lasts;
#pragma unroll 4
    for (int64_t i = tid; i + 1 < s.runs; i += kThreads) acc += fabs(f[i + 1] - l[i]);
    const double t = block_sum(acc, red);
    if (tid == 0) out[blockIdx.x] = t / static_cast<double>(s.p) / static_cast<double>(s.nb - 1);
}

// Strict local maxima over the sorted divisor list (1 and n included as neighbours), then
// the largest score (first on ties), else period 1. One wave per tensor.
__global__ __launch_bounds__(64) void k_part_select(const PartScore* __restrict__ divs,
                                                    const double* __restrict__ scores,
                                                    const int32_t* __restrict__ first,
                                                    const int32_t* __restrict__ count,
                                                    int64_t* __restrict__ periods)
{
    const int t = blockIdx.x, lane = threadIdx.x;
    const int f = first[t];
    const int c = count[t];
    int best = 0x7fffffff;   // index of the lane's best maximum
    double best_s = 0.0;
    for (int i = 1 + lane; i + 1 < c; i += 64) {
        const double s = scores[f + i];
        if (s > scores[f + i - 1] && s > scores[f + i + 1] && (best == 0x7fffffff || s > best_s)) {
            best = i;
            best_s = s;
        }
    }
    for (int off = 1; off < 64; off <<= 1) {
        const int ob = __shfl_xor(best, off);
        const double os = __shfl_xor(best_s, off);
        if (ob != 0x7fffffff && (best == 0x7fffffff || os > best_s || (os == best_s && ob < best))) {
            best = ob;
            best_s = os;
        }
    }
    if (lane == 0) periods[t] = best == 0x7fffffff ? 1 : divs[f + best].p;
}

}  // namespace

hipError_t launch_partition(const PartPlan& plan, const PartDevice& d, double eps,
                            hipStream_t stream)
{
    const int32_t nt = static_cast<int32_t>(plan.tensors.size());
    const int32_t ns = static_cast<int32_t>(plan.scores.size());
    if (plan.groups > 0x7fffffffLL || plan.span_items > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_part_base, dim3(static_cast<unsigned>(plan.groups)), dim3(kPartThreads),
                       sizeof(double) * plan.lds_doubles, stream, d.tensors, nt, d.units,
                       d.phase_end, d.keep, eps, d.sums, d.part);
    if (plan.span_items)
        hipLaunchKernelGGL(k_part_direct, dim3(static_cast<unsigned>(plan.span_items)),
                           dim3(kPartDirectThreads),
                           sizeof(double) * (kPartSpan + 2 * plan.direct_max), stream, d.spans,
                           static_cast<int32_t>(plan.spans.size()), d.direct, d.store, d.tensors,
                           eps, d.sums, d.part);
    const PartJob* jobs = d.jobs;
    for (const std::vector<PartJob>& l : plan.launches) {
        if (l.empty()) continue;
        const int64_t items = l.back().item0 + l.back().n_items;
        if (items > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_part_jobs, dim3(static_cast<unsigned>(items)), dim3(kThreads), 0,
                           stream, jobs, static_cast<int32_t>(l.size()), d.tensors, eps, d.sums,
                           d.part);
        jobs += l.size();
    }
    hipLaunchKernelGGL(k_part_finalize, dim3(static_cast<unsigned>(ns)), dim3(kThreads), 0, stream,
                       d.scores, d.part, d.values);
    hipLaunchKernelGGL(k_part_select, dim3(static_cast<unsigned>(nt)), dim3(64), 0, stream, d.scores,
                       d.values, d.first, d.count, d.periods);
    return hipGetLastError();
}

}  // namespace gefen
