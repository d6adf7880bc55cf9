// Internal declarations shared by the HIP sources of libgefen (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "part_plan.h"
#include "tile_plan.h"

namespace gefen {

// Kernel classes, tiles and the planner: tile_plan.h (host-only, shared with the
// host tests).


// Per-tensor descriptor on device (64 bytes). Pointers are refreshed when the caller
// passes different parameter or gradient buffers.
struct Seg {
    float* theta;             // parameters (fp32)
    const void* grad;         // gradients (fp32 or bf16)
    int64_t code_off;         // code index of the tensor's first code (a multiple of 32)
    int64_t period;           // > 0: uniform blocks of this size; 0: explicit blocks
    int64_t blk_begin;        // global index of the tensor's first block
    const int64_t* csr;       // explicit blocks: tensor-relative starts (n_blocks + 1)
    int64_t numel;
    int32_t gdtype;
    int32_t pad;
};
static_assert(sizeof(Seg) == 64, "Seg layout");

// Scalars of one step, computed on the host in float64 and rounded once.
struct StepScalars {
    float beta1, one_minus_beta1;
    float beta2, one_minus_beta2;
    float step_size;          // lr / (1 - beta1^t)
    float inv_bc2;            // 1 / (1 - beta2^t)
    float eps;
    float decay;              // 1 - lr * weight_decay
};

// Codebook tables used by the step: decode entries (fp32[k]) and, for encoding, the
// midpoints between consecutive entries (fp32[k], last unused) plus a guide table
// (uint8[ng + 1]) giving, per bucket of [-1, 1], the number of midpoints in lower
// buckets.
struct CodebookDev {
    const float* dec;
    const float* enc_mid;
    const uint8_t* enc_guide;
    int32_t k;
    int32_t ng;
};

// Tiles whose blocks the histogram kernel takes by 4-element vectors from the block's first
// element on: uniform blocks of whole vectors that one workgroup's tile holds whole, of at
// most `longest` elements: kHistVecBlock, what its registers hold, or any (hist_ways).
constexpr int64_t kHistVecBlock = 2048;
__host__ __device__ __forceinline__ bool hist_by_vectors(int32_t kind, int64_t period,
                                                         int64_t longest)
{
    return kind != KIND_H && period > 0 && period % 4 == 0 && period <= longest;
}

// The histogram kernels of a launch and whether the vector kernel takes its longer blocks too,
// for `regs` elements in tiles of hist_by_vectors, `longer` in those of longer blocks and
// whether there are other tiles. The other kernel, with more waves, is the faster one for the
// longer blocks (4M elements in rows of 3072, float32: 28 us against 45; 64M: 98 against
// 122), but beside shorter ones it is one launch more, about 20 us: worth it for the longer
// blocks' larger part and from 2^26 elements on (GPT-2 small, 96M elements in rows of 768 and
// 28M of 3072: 150 us in one launch, 170 in two; 1.5B elements, 268M of them in rows of 8192:
// 1.17 ms either way).
enum : int32_t { kHistVec = 1, kHistStream = 2, kHistLong = 4 };
inline int32_t hist_ways(int64_t regs, int64_t longer, bool other)
{
    int32_t ways = (regs ? kHistVec : 0) | (other ? kHistStream : 0);
    if (longer) ways |= longer <= regs && longer < (int64_t(1) << 26) ? kHistLong : kHistStream;
    return ways;
}

// Histogram bin (Alg. 3) of gradient g in a block whose largest |g| is a > 0: the bin of
// x = g / a among nbins equal bins of [-1, 1], the last one closed; half_nb = nbins / 2.
// Evaluated in float64 (these sources are built with contraction off), so that the
// histogram kernel and the step kernels that take the histogram on the way bin every
// element identically. (A float32 estimate with a float64 evaluation near bin edges
// measured slower in both kernels: a wave almost always holds some lane near an edge.)
//
// The quotient is the correctly rounded g / a without a division per element: with inv =
// RN(1 / a) once per block, q = RN(g inv) is within 2 ulp, r = g - q a is exact (a multiple
// of ulp(q) times the last place of a, at most 2^25 of them: a has 24 bits), and q + r inv
// is off by less than 2^-51 ulp before its one rounding. The quotient of two 24-bit numbers
// lies on no rounding boundary of float64 and no nearer to one than 2^-25 ulp, so that
// rounding is g / a's. float32 values leave the exponents far from float64's limits. An
// infinite a takes zeros instead: finite g gives x = 0, infinite g a NaN, as g / a does.
// (Three multiply-adds against about a dozen dependent operations of the division.)
struct HistBlock {
    double a, inv;
};

__host__ __device__ __forceinline__ HistBlock hist_block(float a)
{
    if (a > 3.4028234663852886e38f) return {0.0, 0.0};
    const double d = static_cast<double>(a);
    return {d, 1.0 / d};
}

__host__ __device__ __forceinline__ double hist_quotient(float g, const HistBlock& b)
{
    const double d = static_cast<double>(g);
    const double q = d * b.inv;
    return fma(fma(-q, b.a, d), b.inv, q);
}

__device__ __forceinline__ int hist_bin(float g, const HistBlock& blk, double half_nb, int nbins)
{
    const int b = static_cast<int>((hist_quotient(g, blk) + 1.0) * half_nb);
    return b < nbins - 1 ? b : nbins - 1;
}

// Launchers (all enqueue on `stream` and return the launch status).
// `bs` is the KIND_U workgroup size (256, 512 or 1024); other kinds use kThreads.
// `code_bits` is 8 (one code per byte) or 4 (two codes per byte, low nibble first);
// codes are addressed by code index Seg::code_off + element index.
hipError_t launch_step(int kind, int gdtype, int code_bits, int vpl, int bs, const Tile* tiles,
                       int64_t n_tiles, const Seg* segs, uint8_t* codes, float* scale,
                       float* vmom, CodebookDev cb, StepScalars sc, hipStream_t stream);

// KIND_H needs `htiles` (parallel to `tiles`), `partials` (float2 per tile) and
// `ws_old` (float2 per huge block).
hipError_t launch_step_h(int gdtype, int code_bits, const Tile* tiles, const HTile* htiles,
                         int64_t n_tiles, const Seg* segs, uint8_t* codes, float* scale,
                         float* vmom, CodebookDev cb, StepScalars sc, float2* partials,
                         float2* ws_old, hipStream_t stream);

// The KIND_G step of launch_step that also adds every element of its blocks to `hist`
// (uint64[nbins], accumulated into; Alg. 3 on this step's gradients). Persistent
// workgroups, each flushing one LDS histogram at its end.
hipError_t launch_step_g_hist(int gdtype, int code_bits, const Tile* tiles, int64_t n_tiles,
                              const Seg* segs, uint8_t* codes, float* scale, float* vmom,
                              CodebookDev cb, StepScalars sc, uint64_t* hist, int32_t nbins,
                              hipStream_t stream);

// Histogram over all tiles. KIND_H tiles need their block absmax first:
// launch_hist_h_absmax over each KIND_H class range writes am_partials[first + chunk].
hipError_t launch_hist_h_absmax(const Tile* tiles, const HTile* htiles, int64_t n_tiles,
                                const Seg* segs, float* am_partials, hipStream_t stream);
// `ways`: hist_ways of the range.
hipError_t launch_histogram(const Tile* tiles, int64_t n_tiles, const int32_t* tile_kind,
                            const HTile* htiles, const float* am_partials, const Seg* segs,
                            int32_t nbins, uint64_t* hist, int32_t ways, hipStream_t stream);

// DP over a device histogram. ws must hold dp_workspace_bytes(nbins, k) bytes. `polls`: of
// one wait between its row tiles, at most (a test passes -1: every tile gives up).
constexpr int32_t kDpPolls = 1 << 20;
size_t dp_workspace_bytes(int32_t nbins, int32_t k);
hipError_t launch_dp(const uint64_t* hist, int32_t nbins, int32_t k, void* ws,
                     double* codebook_out, double* cost_out, int32_t* status_out,
                     hipStream_t stream, int32_t polls = kDpPolls);

// Install a float64 codebook into a slot: fp32 entries, fp64 copy, midpoints, guide.
hipError_t launch_install_codebook(const double* cb64_in, int32_t k, int32_t ng,
                                   float* cb32, double* cb64, float* mid, uint8_t* guide,
                                   hipStream_t stream);
// Same from an fp32 codebook (imports).
hipError_t launch_install_codebook_f32(const float* cb32_in, int32_t k, int32_t ng,
                                       float* cb32, double* cb64, float* mid,
                                       uint8_t* guide, hipStream_t stream);

// Block partitioning (Alg. 2) of several tensors: the plan's tables, sums, partial contrasts,
// scores (one double each) and periods on the device.
struct PartDevice {
    const PartTensor* tensors;
    const PartUnit* units;
    const int32_t* phase_end;
    const int64_t* keep;
    const PartSpan* spans;
    const int32_t* direct;
    const int64_t* store;
    const PartJob* jobs;          // the launches' jobs one after another
    const PartScore* scores;
    const int32_t *first, *count;
    double *sums, *part, *values;
    int64_t* periods;
};
hipError_t launch_partition(const PartPlan& plan, const PartDevice& d, double eps,
                            hipStream_t stream);

}  // namespace gefen
