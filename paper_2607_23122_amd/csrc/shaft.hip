// First-hit validation (Eq. occ-first-hit) of AO windows on the matrix cores.
//
// All segments of a candidate j end at its hit point z_j, and nearly all of
// them are free (of ~120 at 1080p, R = 2 m, one is blocked), so what has to be
// fast is to show that a triangle blocks none of them.  With w = o_k - z_j,
// the segment z_j + s w, 0 < s <= 1, meets the triangle (a, b, c) only where
// four functions linear in w have one sign: the edge volumes
// ((a - z) x (b - z)) . w, ((b - z) x (c - z)) . w, ((c - z) x (a - z)) . w and
// the plane distance n . w + n . (z - a) of o_k, the last as seen from z's
// side.  Four rows per triangle times the segments' (w, 1) is a matrix
// product, done 32 triangles by 32 segments at a time.
//
// The product only filters.  Each row carries a slack above every rounding of
// the row, of the product and of the exact test, so no blocked segment is
// dropped, and each pair left is decided by the watertight test in FP32
// (tri_hit), as in the walk of the other validations: the same bits.  The
// operands are split into two halves of 11 bits (x = hi + lo): the product's
// depth of 16 takes (hi, lo) of a row twice, against hi of w in the lanes of
// one half of the wave and lo of w in the other, all four partial products of
// three components and the constant.
//
// A wave takes runs of kShaftRun consecutive candidates (the lists of
// compact_kernel, dealt to the XCDs as to the walk's blocks).  Per candidate:
//   list     the receivers with positive density, their w as halves, their box;
//   gather   the leaves whose boxes the candidate's shaft (the hull of z_j and
//            the receivers' box) meets: up to ten nodes are opened at a time, a
//            child box per lane;
//   filter   64 triangles' rows, a triangle per lane, then the products with
//            all segments.
// The pairs left are decided 64 at a time, across the run's candidates.  A
// table that fills up is worked off before its producer goes on, so every
// scene, radius and leaf size takes this path.
//
// Against the walk it replaces (one any-hit walk of the hierarchy per 64
// segments: per walk 27 nodes at 58 VALU instructions and 43 triangles at 40),
// a filtered pair costs 1/20 of a triangle test: 1080p AO, 7x7 window, 26.7M
// segments, 2.18 -> 1.16 ms (1.46e9 -> 5.4e8 VALU instructions).  Bound by VALU
// issue (0.87 ms of it) and, at 4 waves per SIMD (128 registers, 10 KB of LDS),
// by the latency of the gather's dependent loads.
#include "ocr_common.hpp"
#include "shaft_box.hpp"
#include "traverse.hpp"
#include "validate.hpp"

namespace ocr {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kShaftRun = 2;      // candidates per run (of 1, 2, 3, 4 and 8 the fastest: 1.24, 1.21, 1.24, 1.30, 1.48 ms)
constexpr int kShaftRays = 192;   // segments of a candidate tested together
constexpr int kShaftStack = 128;  // nodes to open
constexpr int kShaftRefs = 160;   // leaves found, in pairs of their triangles
constexpr int kShaftPairs = 128;  // pairs to decide
constexpr int kShaftWords = 96;   // validation words of a run
static_assert(kShaftWords >= kMaxWords, "a run holds at least one candidate's words");
// Of sp waiting nodes as many are opened at a time as leave the stack no higher
// than kShaftWide (opening one adds up to three; one at a time, the rest of a
// walk adds at most 3 kMaxDepth) and as the leaf table has room for the
// children of.
constexpr int kShaftWide = kShaftStack - kStackTotal;
constexpr int kNodeRefs = 4 * kMaxLeaf / 2;  // leaf pairs below one node
static_assert(kShaftRefs / kNodeRefs <= 16 && (kShaftRefs - 31) / kNodeRefs >= 1, "a round's children fit the wave");

// A candidate of the run, as its pairs' decisions need it.
struct ShaftCand {
    float oj[3], dzj[3], nzj[3];
    int32_t jx, jy;
    uint32_t hj;
};

struct ShaftLds {
    half8 rows[4][64];                 // 64 triangles' rows: three edges, plane
    alignas(16) uint2 rays[kShaftRays][2];  // listed: w; in test: (w, 256) hi, (w, 0) lo
    uint16_t ray_q[kShaftRays];        // their receivers' offsets
    uint32_t stack[kShaftStack];
    uint32_t refs[kShaftRefs];         // first triangle | kLeafBit if a second follows
    uint32_t pair_tri[kShaftPairs];
    uint16_t pair_at[kShaftPairs];     // (place in the run << 11) | q
    uint32_t bits[kShaftWords];
    ShaftCand cand[kShaftRun];
};

__device__ inline float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
__device__ inline float min3f(float a, float b, float c) { return fminf(fminf(a, b), c); }

// Lanes of the mask before this one.
__device__ inline int rank_in(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ inline void cross3(const float a[3], const float b[3], float c[3]) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ inline uint32_t pack_rtz(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
__device__ inline float half_lo(uint32_t p) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(p & 0xFFFFu));
}
__device__ inline float half_hi(uint32_t p) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(p >> 16)); }

// (x, y, z, c) as hi and lo halves: hi truncates, so lo is exact in FP32 and
// loses 2^-10 of itself, 2^-20 of the value, when truncated in turn.
__device__ inline void split4(float x, float y, float z, float c, uint2 &hi, uint2 &lo) {
    hi.x = pack_rtz(x, y);
    hi.y = pack_rtz(z, c);
    lo.x = pack_rtz(x - half_lo(hi.x), y - half_hi(hi.x));
    lo.y = pack_rtz(z - half_lo(hi.y), c - half_hi(hi.y));
}

// A row (x, y, z, c) as halves, all scaled already.
__device__ inline half8 make_row(float x, float y, float z, float c) {
    uint2 hi, lo;
    split4(x, y, z, c, hi, lo);
    return __builtin_bit_cast(half8, make_uint4(hi.x, hi.y, lo.x, lo.y));
}

// The constant of a row scaled by 2^e, for w scaled by 2^ew and the 256 of w's
// fourth component.  Beyond +-30000 it decides alone (|n . w| < 256 * 1536).
__device__ inline float row_const(float c, int e) {
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_ldexpf(c, e - 8), -30000.0f, 30000.0f);
}

__global__ __launch_bounds__(64, 4) void validate_shaft_kernel(DeviceBVH bvh, GBufView g, OccView occ, float R2, int D,
                                                               int words, uint32_t *bits, const uint32_t *lists,
                                                               uint32_t per_xcd) {
    __shared__ ShaftLds s;
    const int lane = threadIdx.x;
    const int col = lane & 31, half = lane >> 5;
    const int side = 2 * D + 1, npairs = side * side;
    const float inv_side = 1.0f / (float)side;
    const int qself = D * side + D;
    const int run = min(kShaftRun, kShaftWords / words);
    uint32_t total = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) total += lists[x * kCountStride];
    const uint32_t nruns = (total + (uint32_t)run - 1) / (uint32_t)run;
    const uint32_t xcd = blockIdx.x & 7, stride = gridDim.x / 8;
    int npair = 0;

    // Decide the collected pairs: the watertight test of the walk.
    auto decide = [&]() {
        wave_sync();
        for (int p0 = 0; p0 < npair; p0 += 64) {
            if (p0 + lane < npair) {
                const uint32_t tri = s.pair_tri[p0 + lane], code = s.pair_at[p0 + lane];
                const int b = (int)(code >> 11), q = (int)(code & 2047u);
                const ShaftCand &c = s.cand[b];
                int64_t k;
                uint32_t primk;
                float ok[3], nk[3], w[3];
                pair_receiver(g, c.jx, c.jy, side, inv_side, D, q, k, primk, ok, nk);
                rel_vec(c.oj, ok, c.dzj, w);
                TRay r;
                ray_shear(ok, w, c.hj, primk, r);
                const float4 *tp = bvh.tris + 3 * (size_t)tri;
                const float4 v0 = tp[0], v1 = tp[1], v2 = tp[2];
                const uint32_t id = __float_as_uint(v0.w);
                if (id != r.ign0 && id != r.ign1) {
                    const float t = tri_hit(r, v0, v1, v2);
                    if (t > 0.0f && t < 1.0f - 1e-4f) atomicAnd(&s.bits[b * words + (q >> 5)], ~(1u << (q & 31)));
                }
            }
        }
        npair = 0;
        wave_sync();
    };

    for (uint32_t u = blockIdx.x >> 3;; u += stride) {
        const uint32_t ri = (u / kRunBlock) * (8u * kRunBlock) + xcd * kRunBlock + (u % kRunBlock);
        if (ri >= nruns) {
            if ((u / kRunBlock) * (8u * kRunBlock) >= nruns) break;
            continue;
        }
        const uint32_t c0 = ri * (uint32_t)run;
        const int nrun = (int)min((uint32_t)run, total - c0);
        for (int w = lane; w < nrun * words; w += 64) s.bits[w] = 0u;
        wave_sync();
        for (int b = 0; b < nrun; ++b) {
            const int64_t j = __builtin_amdgcn_readfirstlane((int)lists[list_at(lists, per_xcd, c0 + (uint32_t)b)]);
            const int jy = (int)((uint32_t)j / (uint32_t)g.w), jx = (int)j - jy * g.w;
            const uint32_t hj = occ.hit[j];
            float z[3];
            {
                float xj[3], nj[3], oj[3], dzj[3], nzj[3];
                load3(g.pos, j, xj);
                load3(g.nrm, j, nj);
                load3(occ.dz, j, dzj);
                load3(occ.nz, j, nzj);
                offset_point(xj, nj, oj);
                for (int a = 0; a < 3; ++a) z[a] = uniform_f(oj[a] + dzj[a]);
                if (lane == 0) {
                    ShaftCand &c = s.cand[b];
                    for (int a = 0; a < 3; ++a) {
                        c.oj[a] = oj[a];
                        c.dzj[a] = dzj[a];
                        c.nzj[a] = nzj[a];
                    }
                    c.jx = jx;
                    c.jy = jy;
                    c.hj = hj;
                    // z_j is its own first hit
                    s.bits[b * words + (qself >> 5)] |= 1u << (qself & 31);
                }
                wave_sync();
            }
            int nray = 0;                                // segments listed
            uint32_t prim0 = OCR_HIT_MISS;               // the first one's receiver triangle
            bool same = true;                            // ... and whether all have it
            int clo[3], chi[3];                          // the least w and -w (per lane, as ordered integers)

            // The listed segments against all triangles their shaft meets.
            auto test = [&]() {
                Shaft S;
                float cz = 0.0f, W = 0.0f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    S.lo[a] = from_ordered(wave_min_i(clo[a]));
                    S.hi[a] = -from_ordered(wave_min_i(chi[a]));
                    cz = fmaxf(cz, fabsf(z[a]));
                    W = max3f(W, fabsf(S.lo[a]), fabsf(S.hi[a]));
                }
                // the shaft padded by the rounding of its coordinates
                cz = uniform_f(cz + W);
                W = uniform_f(W);
                shaft_set(S, z, cz, W, [](float v) { return __builtin_amdgcn_rcpf(v); }, uniform_f);
                // The segments as halves, scaled by 2^ew to components below
                // 2^8.  The scale is their own (of R it would be far from theirs
                // where R is meant as no limit, and every pair would pass).
                const int ew = 8 - __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(W));
                const float scale = __builtin_amdgcn_ldexpf(1.0f, 8 - ew);
                for (int i = lane; i < nray; i += 64) {
                    const float4 w = *reinterpret_cast<const float4 *>(s.rays[i]);
                    uint2 hi, lo;
                    split4(__builtin_amdgcn_ldexpf(w.x, ew), __builtin_amdgcn_ldexpf(w.y, ew),
                           __builtin_amdgcn_ldexpf(w.z, ew), 256.0f, hi, lo);
                    *reinterpret_cast<uint4 *>(s.rays[i]) = make_uint4(hi.x, hi.y, lo.x, lo.y);
                }
                S.below = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.below);
                // (a row of the receivers' common triangle is no use: it is
                // never hit)
                const uint32_t own = same ? prim0 : OCR_HIT_MISS;

                // The triangles of s.refs[base, base + nref), nref <= 32, times
                // all the segments.
                auto block = [&](int base, int nref) {
                    {
                        const uint32_t ref = s.refs[base + ((lane >> 1) < nref ? lane >> 1 : 0)];
                        bool real = (lane >> 1) < nref && ((lane & 1) == 0 || (ref & kLeafBit) != 0u);
                        const uint32_t tri = (ref & 0x07FFFFFFu) + (real ? lane & 1 : 0);
                        const float4 *tp = bvh.tris + 3 * (size_t)tri;
                        const float4 v0 = tp[0], v1 = tp[1], v2 = tp[2];
                        const uint32_t id = __float_as_uint(v0.w);
                        real = real & (id != hj) & (id != own);  // (no branch: the load goes with the others)
                        float A[3] = {v0.x - z[0], v0.y - z[1], v0.z - z[2]};
                        float B[3] = {v1.x - z[0], v1.y - z[1], v1.z - z[2]};
                        float C[3] = {v2.x - z[0], v2.y - z[1], v2.z - z[2]};
                        float E1[3] = {v1.x - v0.x, v1.y - v0.y, v1.z - v0.z};
                        float E2[3] = {v2.x - v0.x, v2.y - v0.y, v2.z - v0.z};
                        float La = 0.0f, Lo = 0.0f, Ed = 0.0f;
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            const float bl = min3f(A[a], B[a], C[a]), bh = max3f(A[a], B[a], C[a]);
                            La = max3f(La, fabsf(bl), fabsf(bh));
                            Lo = max3f(Lo, bh - S.lo[a], S.hi[a] - bl);
                            Ed = max3f(Ed, fabsf(E1[a]), fabsf(E2[a]));
                        }
                        // vertices that are not finite, or too large to
                        // multiply: rows of zeros, which always pass (a pair
                        // passes where all four functions are positive)
                        if (!(La < 1e9f)) {
                            for (int a = 0; a < 3; ++a) A[a] = B[a] = C[a] = E1[a] = E2[a] = 0.0f;
                            La = Lo = Ed = 1.0f;
                        }
                        float n[3];
                        cross3(E1, E2, n);
                        const float dz = -(n[0] * A[0] + n[1] * A[1] + n[2] * A[2]);  // z's plane distance times |n|
                        const float n1 = fabsf(n[0]) + fabsf(n[1]) + fabsf(n[2]);
                        // Slacks, in the units of the functions.  The exact
                        // test rounds vertices relative to o_k (Lo) and forms
                        // edge functions and their weighted sum from them; the
                        // rows round vertices relative to z (La, with z itself
                        // rounded, cz), edges (Ed) and the halves (2^-17 of
                        // |n| |w|, and 2^-20 of w's scale where a half is
                        // subnormal).
                        const float half_ulp = 0x1p-17f * W + 0x1p-20f * scale;
                        const float edge = W * (0x1p-17f * Lo * Lo + 0x1p-18f * La * (cz + La)) + half_ulp * La * La;
                        const float side_z = 0x1p-20f * n1 * (cz + La) + 0x1p-19f * La * Ed * Ed;
                        const float plane = n1 * (0x1p-20f * cz + 0x1p-19f * (W + La) + half_ulp) +
                                            0x1p-19f * Lo * (Lo * Lo + Ed * Ed);
                        const bool flat = !(fabsf(dz) > side_z);  // z's side is not certain
                        const float sg = dz < 0.0f ? 1.0f : -1.0f;
                        const half8 never = {0, 0, 0, -1, 0, 0, 0, 0};
                        // The edges' rows share a scale (their halves err by
                        // 2^-20 of La^2, a part of `edge`) and the constant.
                        const int ee = 8 - 2 * __builtin_amdgcn_frexp_expf(La);
                        const float se = flat ? 0.0f : __builtin_amdgcn_ldexpf(sg, ee), ce = row_const(edge, ee + ew);
                        float X[3];
                        wave_sync();
                        cross3(A, B, X);
                        s.rows[0][lane] = make_row(X[0] * se, X[1] * se, X[2] * se, ce);
                        cross3(B, C, X);
                        s.rows[1][lane] = make_row(X[0] * se, X[1] * se, X[2] * se, ce);
                        cross3(C, A, X);
                        s.rows[2][lane] = make_row(X[0] * se, X[1] * se, X[2] * se, ce);
                        float sp = sg, c = plane - fabsf(dz);
                        if (flat) {
                            // z in the triangle's plane, as far as FP32 can
                            // tell: a hit at t < 1 - 1e-4 then needs |n . w| <=
                            // 1e4 times z's distance.  Of its two sides the one
                            // is tested that the middle of the receivers is
                            // beyond.
                            const float mid = n[0] * (S.lo[0] + S.hi[0]) + n[1] * (S.lo[1] + S.hi[1]) + n[2] * (S.lo[2] + S.hi[2]);
                            sp = mid > 0.0f ? -1.0f : 1.0f;
                            c = 1.1e4f * (fabsf(dz) + side_z) + plane;
                        }
                        const int en = 8 - __builtin_amdgcn_frexp_expf(n1);
                        sp = __builtin_amdgcn_ldexpf(sp, en);
                        const half8 r3 = make_row(n[0] * sp, n[1] * sp, n[2] * sp, row_const(c, en + ew));
                        s.rows[3][lane] = real ? r3 : never;
                        wave_sync();
                    }
                    for (int r0 = 0; r0 < 2 * nref; r0 += 32) {
                        const half8 a0 = s.rows[0][r0 + col], a1 = s.rows[1][r0 + col], a2 = s.rows[2][r0 + col],
                                    a3 = s.rows[3][r0 + col];
                        for (int i0 = 0; i0 < nray; i0 += 32) {
                            const uint2 bw = s.rays[i0 + col][half];
                            const half8 bf = __builtin_bit_cast(half8, make_uint4(bw.x, bw.y, bw.x, bw.y));
                            const float16v zero = {};
                            // lane (col, half) holds segment i0 + col and rows
                            // (i & 3) + 8 (i >> 2) + 4 half, whose sign bits go
                            // to bit 15 - i: set where one of the four functions
                            // rules the pair out.  (Two products at a time: all
                            // four's results do not fit the registers.)
                            const float16v f0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bf, zero, 0, 0, 0);
                            const float16v f1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, bf, zero, 0, 0, 0);
                            uint32_t v[16], mask = 0;
#pragma unroll
                            for (int i = 0; i < 16; ++i) v[i] = __float_as_uint(f0[i]) | __float_as_uint(f1[i]);
                            __builtin_amdgcn_sched_barrier(0);
                            const float16v f2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, bf, zero, 0, 0, 0);
                            const float16v f3 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a3, bf, zero, 0, 0, 0);
#pragma unroll
                            for (int i = 0; i < 16; ++i)
                                mask = __builtin_amdgcn_alignbit(mask, v[i] | __float_as_uint(f2[i]) | __float_as_uint(f3[i]), 31);
                            const int ray = i0 + col;
                            mask = ray < nray ? mask ^ 0xFFFFu : 0u;
                            if (wave_ballot(mask != 0u) == 0ull) continue;
                            int q = 0;
                            uint32_t prim = OCR_HIT_MISS;
                            if (mask != 0u) {
                                q = (int)s.ray_q[ray];
                                const int qy = small_div(q, inv_side);
                                prim = g.prim[(int64_t)(jy + qy - D) * g.w + (jx + (q - qy * side) - D)];
                            }
                            while (wave_ballot(mask != 0u) != 0ull) {
                                const int i = __clz((int)mask) - 16;  // (mask 0: 16, unused)
                                const int row = mask != 0u ? r0 + (i & 3) + 8 * (i >> 2) + 4 * half : 0;
                                const uint32_t tri = (s.refs[base + (row >> 1)] & 0x07FFFFFFu) + (uint32_t)(mask != 0u ? row & 1 : 0);
                                const bool want = (mask != 0u) & (__float_as_uint(bvh.tris[3 * (size_t)tri].w) != prim);
                                mask &= ~(0x8000u >> (i & 15));
                                const unsigned long long m = wave_ballot(want);
                                if (want) {
                                    const int at = npair + rank_in(m);
                                    s.pair_tri[at] = tri;
                                    s.pair_at[at] = (uint16_t)((b << 11) | q);
                                }
                                npair += __popcll(m);
                                if (npair > kShaftPairs - 64) decide();
                            }
                        }
                    }
                };

                // A child's link; returns the lanes whose child the shaft meets.
                auto child = [&](const float *f, uint32_t &link) {
                    link = __float_as_uint(f[24]);
                    const float bl[3] = {f[0], f[8], f[16]}, bh[3] = {f[4], f[12], f[20]};
                    return wave_ballot(shaft_meets(S, bl, bh)) & wave_ballot(link != kEmpty);
                };
                // Gather, from the first node of which the shaft meets more
                // than one child or a leaf.
                uint32_t node = 0;
                for (;;) {
                    uint32_t link;
                    const uint32_t m = (uint32_t)child(reinterpret_cast<const float *>(bvh.nodes + node) + (lane & 3), link) & 0xFu;
                    if (__builtin_popcount(m) != 1) break;
                    const uint32_t next = (uint32_t)__builtin_amdgcn_readlane((int)link, (int)__builtin_ctz(m));
                    if (next & kLeafBit) break;
                    node = next;
                }
                if (lane == 0) s.stack[0] = node;
                wave_sync();
                int sp = 1, nref = 0;
                for (;;) {
                  while (sp > 0 && nref < 32) {
                    const int n = min(min(sp, (kShaftRefs - nref) / kNodeRefs), max((kShaftWide - sp) / 3, 1));
                    // (lanes without a node read the first one's)
                    uint32_t link;
                    const int at = (lane >> 2) < n ? lane >> 2 : 0;
                    const unsigned long long met =
                        child(reinterpret_cast<const float *>(bvh.nodes + s.stack[sp - 1 - at]) + (lane & 3), link) &
                        (n < 16 ? (1ull << (4 * n)) - 1ull : ~0ull);
                    const bool leaf = (int32_t)link < 0;
                    const unsigned long long lf = wave_ballot(leaf), mi = met & ~lf;
                    const bool mine = (met >> lane) & 1ull;
                    wave_sync();
                    sp -= n;
                    if (mine && !leaf) s.stack[sp + rank_in(mi)] = link;
                    sp += __popcll(mi);
                    // a leaf in pairs of its triangles (most hold one pair)
                    int left = mine && leaf ? (int)((link >> 27) & 0xFu) + 1 : 0;
                    uint32_t tri = link & 0x07FFFFFFu;
                    for (;;) {
                        const unsigned long long ml = wave_ballot(left > 0);
                        if (ml == 0ull) break;
                        if (left > 0) s.refs[nref + rank_in(ml)] = tri | (left > 1 ? kLeafBit : 0u);
                        nref += __popcll(ml);
                        left -= 2;
                        tri += 2u;
                    }
                    wave_sync();
                  }
                  if (nref == 0) break;
                  const int take = min(nref, 32);
                  nref -= take;
                  block(nref, take);
                }
                wave_sync();
            };

            // A receiver's loads: a lane without one reads the nearest pixel.
            struct Recv {
                uint32_t prim;
                float x[3], n[3];
                bool in;
            };
            auto load = [&](int q, Recv &r) {
                const int qy = small_div(q, inv_side);
                const int kx = jx + (q - qy * side) - D, ky = jy + qy - D;
                r.in = q < npairs && q != qself && (uint32_t)kx < (uint32_t)g.w && (uint32_t)ky < (uint32_t)g.h;
                const int64_t k = (int64_t)min(max(ky, 0), g.h - 1) * g.w + min(max(kx, 0), g.w - 1);
                r.prim = g.prim[k];
                load3(g.pos, k, r.x);
                load3(g.nrm, k, r.n);
            };
            // the receivers with positive density, in q order; the next round's
            // loads are issued ahead of this one's densities
            Recv next;
            load(lane, next);
            for (int qb = 0; qb < npairs; qb += 64) {
                if (nray == 0) {
                    for (int a = 0; a < 3; ++a) {
                        clo[a] = 0x7FFFFFFF;
                        chi[a] = 0x7FFFFFFF;
                    }
                }
                const int q = qb + lane;
                const Recv r = next;
                if (qb + 64 < npairs) load(q + 64, next);
                const uint32_t primk = r.prim;
                float ok[3], w[3];
                bool want;
                {
                    // (the candidate from LDS: no registers across a test)
                    const ShaftCand &c = s.cand[b];
                    offset_point(r.x, r.n, ok);
                    rel_vec(c.oj, ok, c.dzj, w);
                    want = r.in && primk != OCR_HIT_MISS && dens_ao(w, r.n, c.nzj, R2) > 0.0f;
                }
                const unsigned long long m = wave_ballot(want);
                if (m != 0ull) {
                    if (nray == 0) prim0 = (uint32_t)__builtin_amdgcn_readlane((int)primk, (int)__builtin_ctzll(m));
                    same = (nray == 0 || same) && wave_ballot(want && primk != prim0) == 0ull;
                    if (want) {
                        for (int a = 0; a < 3; ++a) {
                            // (-x as an ordered integer is that of x, inverted)
                            const int i = ordered_int(w[a]);
                            w[a] = -w[a];
                            clo[a] = min(clo[a], ~i);
                            chi[a] = min(chi[a], i);
                        }
                        const int at = nray + rank_in(m);
                        *reinterpret_cast<float4 *>(s.rays[at]) = make_float4(w[0], w[1], w[2], 0.0f);
                        s.ray_q[at] = (uint16_t)q;
                        // free until found blocked
                        atomicOr(&s.bits[b * words + (q >> 5)], 1u << (q & 31));
                    }
                    nray += __popcll(m);
                }
                if (nray > 0 && (nray > kShaftRays - 64 || qb + 64 >= npairs)) {
                    wave_sync();
                    test();
                    nray = 0;
                }
            }
        }
        if (npair > 0) decide();
        wave_sync();
        for (int b = 0; b < nrun; ++b) {
            const int64_t j = (int64_t)s.cand[b].jy * g.w + s.cand[b].jx;
            for (int w = lane; w < words; w += 64) bits[j * words + w] = s.bits[b * words + w];
        }
        wave_sync();
    }
}

hipError_t launch_validate_shaft(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, float R, int D, int words,
                                 uint32_t *bits, const uint32_t *lists, uint32_t per_xcd, hipStream_t st) {
    // a wave per run, as many as the frame can need, up to 192 per CU (of 24576,
    // 49152 and 98304 waves within 1% of the fastest for small frames and large)
    const int64_t runs = ((int64_t)g.w * g.h + kShaftRun - 1) / kShaftRun;
    const int grid = 8 * (int)((runs < 49152 ? runs + 7 : 49152) / 8);
    hipLaunchKernelGGL(validate_shaft_kernel, dim3(grid), dim3(64), 0, st, bvh, g, occ, R * R, D, words, bits, lists,
                       per_xcd);
    return hipGetLastError();
}

}  // namespace ocr
