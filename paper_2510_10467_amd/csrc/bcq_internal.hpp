// Internal launch descriptor shared by the dispatcher and the kernel files.
// Nothing here is part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bcq.h"

namespace bcq {

// One product call, uniform or per-request precision.
struct GemmArgs {
    const uint32_t *planes;                          // [>= p_max][m][n/32]
    const _Float16 *scales[BCQ_MAX_PLANES + 1];      // [q] = scale set of precision q, or nullptr
    const _Float16 *offsets[BCQ_MAX_PLANES + 1];     // [q] = offsets [m][n/group] of precision q, or nullptr (none)
    const int32_t *p_req;                            // device int32[batch], nullptr when uniform
    int uniform_p;                                   // > 0: every request runs at this precision
    int p_max;                                       // planes stored / upper bound of any p_req
    const _Float16 *x;                               // [batch][n]
    _Float16 *y;                                     // [batch][m]
    int64_t m, n;
    int batch;
    int group;
};

// Precision of request b: the uniform one, or p_req[b] clamped to [1, p_max];
// 0 when that precision has no scale set (the request then yields zeros).
__device__ __forceinline__ int request_precision(const GemmArgs &a, int b)
{
    int p = a.uniform_p;
    if (p == 0) {
        p = a.p_req[b];
        p = p < 1 ? 1 : (p > a.p_max ? a.p_max : p);
    }
    return a.scales[p] ? p : 0;
}

// The requests of precision q (after clamping to [1, p_max]) in the order of the batch: those of rank b0 .. b0 + TB - 1
// get their numbers written to req_of[0 .. TB - 1] by the workgroup's first wave; returns how many of these ranks
// exist (0 or less: none), the same number in every wave, each of which runs the whole ranking itself.  Sixteen
// independent loads at a time (1024 requests), so that a batch costs one memory latency, not one per 64 requests.
template <int TB>
__device__ __forceinline__ int rank_requests(const int32_t *p_req, const int batch, const int p_max, const int q, const int b0, uint32_t *req_of)
{
    const int lane = threadIdx.x & 63;
    int seen = 0;                               // requests of precision q so far
    for (int blk = 0; blk < batch && seen < b0 + TB; blk += 1024) {
        int pv[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int b = blk + 64 * j + lane;
            pv[j] = b < batch ? p_req[b] : 0;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int b = blk + 64 * j + lane;
            const int pc = pv[j] < 1 ? 1 : (pv[j] > p_max ? p_max : pv[j]);
            const bool is = b < batch && pc == q;
            const unsigned long long mask = __ballot(is);
            const int rank = seen + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (is && rank >= b0 && rank < b0 + TB && threadIdx.x < 64) req_of[rank - b0] = (uint32_t)b;
            seen += __popcll(mask);
        }
    }
    return seen - b0 > TB ? TB : seen - b0;
}

// More than 64 KiB of dynamic LDS needs a per-function attribute.  It sticks to the function, so it is set once per
// kernel instance and device (and again only if a later launch asks for more); defined in bcq_api.hip.
hipError_t allow_dynamic_lds(const void *kernel, int bytes);

// Kernel families.  *_supports tells whether the family can run the problem;
// *_launch enqueues it on `stream` and returns the HIP launch status.
bool sign_select_supports(const GemmArgs &a);
hipError_t sign_select_launch(const GemmArgs &a, hipStream_t stream);

// table look-ups (section 3.3's LUT formulation): any legal shape; the fallback ahead of sign_select
bool lut_supports(const GemmArgs &a);
hipError_t lut_launch(const GemmArgs &a, hipStream_t stream);

bool plane_mfma_supports(const GemmArgs &a);
bool plane_mfma_streams(const GemmArgs &a);     // tall matrix, 2 to 8 requests: the row-streaming form takes it
hipError_t plane_mfma_launch(const GemmArgs &a, hipStream_t stream);

// `count` matrices that share n, precision, batch and activations as ONE launch
bool plane_mfma_supports_multi(const GemmArgs *mats, int count);
bool plane_mfma_streams_multi(const GemmArgs *mats, int count);   // ... and the row-streaming form takes them together
hipError_t plane_mfma_launch_multi(const GemmArgs *mats, int count, hipStream_t stream);

bool dequant_mfma_supports(const GemmArgs &a);
// benchmarks and tests: force the workgroup shape (request tiles of 64, or 0 for one tile of 16; blocks of 16 rows); (0, 0) = automatic
bool dequant_mfma_force_shape(int request_tiles, int row_blocks);
// whether the forced shape, if there is one, can run the problem (the level form takes whole pairs of column groups only)
bool dequant_mfma_shape_fits(const GemmArgs &a);
// the shape that a product at one precision runs with, forced or automatic, as the pair bcq_select_dequant_shape takes
void dequant_mfma_shape(const GemmArgs &a, int &request_tiles, int &row_blocks);
// per-request precision: the shape of the level form that runs the call, forced or automatic ((1, 96): 128 x 96), (0, 0) where it does not
void dequant_mfma_mixed_shape(const GemmArgs &a, int &request_tiles, int &row_blocks);
// planewise: the variant that multiplies the +-1 planes themselves and scales the group sums (groups of 128 or 256)
hipError_t dequant_mfma_launch(const GemmArgs &a, hipStream_t stream, bool planewise = false, const GemmArgs *mats = nullptr, int count = 0);
// several matrices (same n, precision, batch, activations, group size; no offsets) in one launch of the large-batch kernels
bool dequant_mfma_supports_multi(const GemmArgs *mats, int count);
hipError_t dequant_mfma_launch_multi(const GemmArgs *mats, int count, hipStream_t stream, bool planewise);

// The level form of the large-batch kernels: weights rebuilt by look-ups, tiles of 32 x 32 (dequant_mfma_launch picks it).
constexpr int kLevelShapeCount = 6;
bool level_mfma_supports(const GemmArgs &a);
// its cheapest shape for a product, and what that one is expected to take in microseconds
int level_mfma_cheapest(const GemmArgs &a, float &us);
// Per-request precision: the same body per precision, each workgroup on the requests of one precision.  a: the call, with uniform_p the
// deepest precision and batch the requests that a precision is expected to have; nsets: that many precisions.
int level_mfma_cheapest_classes(const GemmArgs &a, int nsets, float &us);
// What a workgroup keeps and asks for (bcq_level_layout)
struct LevelLayout {
    int lds_bytes, window_columns, window_loads, word_columns;
};
LevelLayout level_mfma_layout(const GemmArgs &a, int shape);
hipError_t level_mfma_launch_classes(const GemmArgs &a, uint32_t class_order, int shape, hipStream_t stream);
// The estimate of both large-batch forms: `at_4096` is what a product of 4096 columns takes, of which `start` does not depend
// on the width (beyond 4096 columns it no longer counts).
inline float large_batch_us(float at_4096, float start, int64_t n)
{
    return n < 4096 ? start + (at_4096 - start) * ((float)n / 4096.f) : at_4096 * ((float)n / 4096.f);
}
hipError_t level_mfma_launch(const GemmArgs &a, int shape, hipStream_t stream, const GemmArgs *mats, int count);

// Offline quantiser (Algorithm 1): group must be 32, 64, 128 or 256; 1 <= p_low <= p_high <= 4.
bool quantize_supports(int64_t m, int64_t n, int group);
hipError_t quantize_launch(const _Float16 *w, int p_low, int p_high, int cycles, uint32_t *planes, _Float16 *const *scales_by_p,
                           _Float16 *const *offsets_by_p, int64_t m, int64_t n, int group, bool listing_residual, hipStream_t stream);

hipError_t pack_launch(const int8_t *codes, uint32_t *planes, int n_planes, int64_t m, int64_t n, hipStream_t stream);
hipError_t unpack_launch(const uint32_t *planes, int8_t *codes, int n_planes, int64_t m, int64_t n, hipStream_t stream);

}  // namespace bcq
