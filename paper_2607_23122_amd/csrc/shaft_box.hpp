// The shaft of a candidate (shaft.hip) and its box test; plain C++ besides, so
// that a host program can include it.
#pragma once
#include <math.h>

#include <stdint.h>

#ifdef __HIPCC__
#define OCR_SHAFT_FN __host__ __device__ inline
#else
#define OCR_SHAFT_FN inline
#endif

namespace ocr {

// Interval shaft of a candidate: z + s w with w in [lo, hi] and s in [0, 1]
// (wave-uniform).
struct Shaft {
    float lo[3], hi[3], rlo[3], rhi[3];  // the box of w and its reciprocals
    float zlo[3], zhi[3];                // -z times the reciprocals, for boxes wider by the pad
    uint32_t below;                      // bit a: lo[a] < 0; bit 3 + a: hi[a] > 0
};

// What a shaft is padded by, for the largest coordinates cz of its points and W
// of its w: 2^-20 of the one and 2^-18 of the other, above the 2^-21 and 2^-20
// that the walks' slabs allow and the roundings of z, w and the test itself.
OCR_SHAFT_FN float shaft_pad(float cz, float W) { return 0x1p-20f * cz + 0x1p-18f * W; }

// The shaft of S.lo, S.hi (w's least and largest) about z, padded.  The planes
// move as well, outwards: w's padding leaves a plane only s times the pad,
// nothing near z, where the plane's rounding (2^-24 |z / w| of s, without a bound
// as w's interval closes on 0) is as large as anywhere.  Folded into the
// constants, it costs a box nothing.  rcp: the reciprocal to use (1 ulp); uni: a
// value that all lanes hold, as a scalar.
template <class Rcp, class Uni>
OCR_SHAFT_FN void shaft_set(Shaft &S, const float z[3], float cz, float W, const Rcp &rcp, const Uni &uni) {
    const float pad = shaft_pad(cz, W);
    S.below = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float l = S.lo[a] - pad, h = S.hi[a] + pad;
        S.lo[a] = uni(fabsf(l) < 1e-20f ? 1e-20f : l);  // (it is divided by)
        S.hi[a] = uni(fabsf(h) < 1e-20f ? 1e-20f : h);
        S.rlo[a] = uni(rcp(S.lo[a]));
        S.rhi[a] = uni(rcp(S.hi[a]));
        S.zlo[a] = uni(-(z[a] - pad) * S.rlo[a]);
        S.zhi[a] = uni(-(z[a] + pad) * S.rhi[a]);
        S.below |= (S.lo[a] < 0.0f ? 1u << a : 0u) | (S.hi[a] > 0.0f ? 8u << a : 0u);
    }
}

// keeps the compiler from computing both sides of a branch and selecting
#ifdef __HIP_DEVICE_COMPILE__
#define OCR_SHAFT_KEEP(v) asm volatile("" : "+v"(v))
#else
#define OCR_SHAFT_KEEP(v) (void)(v)
#endif

// Whether the box [bl, bh] meets the shaft: per axis some s has s hi >= bl - z
// and s lo <= bh - z, each a bound on s; the shaft meets the box only if the
// bounds of all axes leave an s in [0, 1].  Which side a bound is on is the
// wave's, so it branches (selecting takes two more instructions per bound).
// The quotients err by 2^-22 of themselves besides, which the upper bounds' 1e-5
// is for.
OCR_SHAFT_FN bool shaft_meets(const Shaft &S, const float bl[3], const float bh[3]) {
    float s0 = 0.0f, s1 = 1.0f + 1e-5f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float p = fmaf(bl[a], S.rhi[a], S.zhi[a]), q = fmaf(bh[a], S.rlo[a], S.zlo[a]);
        if (S.below & (8u << a)) {
            s0 = fmaxf(s0, p);
            OCR_SHAFT_KEEP(s0);
        } else {
            s1 = fminf(s1, p + 1e-5f);
            OCR_SHAFT_KEEP(s1);
        }
        if (S.below & (1u << a)) {
            s0 = fmaxf(s0, q);
            OCR_SHAFT_KEEP(s0);
        } else {
            s1 = fminf(s1, q + 1e-5f);
            OCR_SHAFT_KEEP(s1);
        }
    }
    return s0 <= s1;
}

}  // namespace ocr
