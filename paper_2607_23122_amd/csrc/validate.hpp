// Shared by the first-hit validation kernels (trace.hip, shaft.hip): the
// candidate lists, a pair's receiver and the run bookkeeping.
#pragma once
#include "density.hpp"
#include "lights.hpp"
#include "ocr_common.hpp"
#include "trace_pixel.hpp"

namespace ocr {

constexpr int kCountStride = 32;  // uint32 per list counter: one 128-byte line
constexpr int kMaxPairs = 33 * 33;             // (4r+1)^2 at r = 8
constexpr int kMaxWords = (kMaxPairs + 31) / 32;

// receiver k of candidate j at pair index q, its offset point and the segment
// vector w = z_j - o_k; false if k is outside the image or background
__device__ inline bool pair_receiver(const GBufView &g, int jx, int jy, int side, float inv_side, int D, int q,
                                     int64_t &k, uint32_t &primk, float ok[3], float nk[3]) {
    const int qy = small_div(q, inv_side);
    const int kx = jx + (q - qy * side) - D, ky = jy + qy - D;
    if (kx < 0 || kx >= g.w || ky < 0 || ky >= g.h) return false;
    k = (int64_t)ky * g.w + kx;
    // the three loads issue together; background is decided afterwards
    float xk[3];
    primk = g.prim[k];
    load3(g.pos, k, xk);
    load3(g.nrm, k, nk);
    if (primk == OCR_HIT_MISS) return false;
    offset_point(xk, nk, ok);
    return true;
}

// Consecutive runs of candidates an XCD takes at a time.
constexpr uint32_t kRunBlock = 256;
constexpr int kRunWords = 128;  // validation words of a run in LDS
static_assert(kRunWords >= kMaxWords, "a run holds at least one candidate's words");

// Position in the workspace of candidate c of the 8 lists taken one after the
// other (scalar).
__device__ inline uint32_t list_at(const uint32_t *lists, uint32_t per_xcd, uint32_t c) {
    uint32_t off = c, base = 8 * kCountStride;
#pragma unroll
    for (int x = 0; x < 7; ++x) {
        const uint32_t n = lists[x * kCountStride];
        if (off >= n) {
            off -= n;
            base += per_xcd;
        } else {
            break;
        }
    }
    return base + off;
}

// A candidate of the current run, as its walks need it.
struct RunCand {
    float oj[3], dzj[3];
    int32_t jx, jy;
    uint32_t hj;
    int32_t pad;
};

// shaft.hip: the validation of AO windows
hipError_t launch_validate_shaft(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, float R, int D, int words,
                                 uint32_t *bits, const uint32_t *lists, uint32_t per_xcd, hipStream_t st);

// validate_light.hip: the validation of the light effects' windows of radius 1
// to 3; the candidates it leaves are appended to the lists
hipError_t launch_validate_light(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, const LightF &L, int radius,
                                 uint32_t *bits, uint32_t *lists, uint32_t per_xcd, hipStream_t st);
hipError_t launch_validate_light(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, const LightSetF &L, int radius,
                                 uint32_t *bits, uint32_t *lists, uint32_t per_xcd, hipStream_t st);

}  // namespace ocr
