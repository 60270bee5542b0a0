// Sliding-window occluder-domain MIS reuse of one target tile (Sec. 4.2-4.4;
// steps 2-3 of App. D / App. H), shared by the per-frame reuse kernel and the
// batched schedule.
//
// For a target i with reuse set S(i):
//   B_i = sum_{j in S(i), hit_j} [p_i(j) > 0 and P_i(j) > 0] p_i(j) / P_i(j),
//   P_i(j) = sum_{k in S(i)} p_k(j),
// p = the pair density (validated by the first-hit bits when unbiased).
//
// P_i(j) depends on both i and j, but only through the pair densities p_k(j)
// with k - j in [-2R, 2R]^2, each needed by every target whose window holds
// both.  So each candidate j's (4R+1)^2 densities are evaluated once, every
// P_i(j) for the (2R+1)^2 targets around j is formed as box sums (row sums,
// then column sums), and p_i(j)/P_i(j) is scattered to the targets.  A block
// owns a 16x16 target tile and stages the receivers of the tile plus an
// R-pixel halo in LDS; the scattered terms are summed in LDS as 32.32
// fixed-point integers, which makes the sum independent of the order in which
// waves arrive (bitwise reproducible) at ~2^-33 absolute error per term.
// For R = 1..3 a lane takes one receiver row of one candidate (its densities
// in registers, its row sums to LDS) and then one (candidate, target) pair;
// other radii take one wave per candidate.  Both sum in the same order, so
// they give the same bits.
#pragma once
#include "density.hpp"
#include "lights.hpp"
#include "ocr_common.hpp"
#include "solid_angle.hpp"

namespace ocr {

constexpr int kRBlock = 256;     // lanes of a group or per-pixel block, and of a window tile's block
constexpr int kWinMost = 512;    // most lanes of a window tile's block
// A candidate with at most this many positive densities in its rectangle takes
// the sparse path of the scatter.
constexpr int kSparse = 8;
// Row-task radii, light effects: a candidate with at most this many receivers
// that may have a positive density is summed pair by pair.  (A pair's sum grows
// with the candidate's pairs, a row task's cost with the rows of the square:
// radius 1 / 2 / 3 unbiased shadows at 1080p 59 / 79 / 135 us with 10 pairs for
// all, 76 / 92 / 137 with 16, 92 / 126 / 164 with 24.)
__host__ __device__ constexpr int few_pairs(int R) { return 4 * R; }
// Which kernels have the pair body and at which radii: the light effects, of one
// light or with validation bits that mark the pairs (several lights' marks cost
// nearly their densities: two lights biased at 1080p 0.50 ms by row tasks, 0.58
// by pairs), and not the biased ones of radius 1, whose 25 densities are cheap
// (1280x720 boxes 30 us by row tasks, 37 by pairs).
template <int MODE, bool UNB, class LT>
constexpr bool kPairBody = MODE != OCR_AO && (UNB || !std::is_same<LT, LightSetF>::value);
template <int MODE, bool UNB, class LT>
__host__ __device__ constexpr bool pair_radius(int R) {
    return kPairBody<MODE, UNB, LT> && R <= 3 && R >= (UNB ? 1 : 2);
}
// Biased: a tile with at most this many candidates leaves them to the row tasks,
// which need no marks first: a batch of marks costs about as much as the rows of
// 13 candidates at radius 3 (five candidates in a 48x36 frame 9 us, 17 by pairs).
// In the small frames that kWinMost lanes are for, as many as one round of the
// waves takes.
__host__ __device__ constexpr int few_candidates(int R, int block) {
    return block > kRBlock ? block / 64 * (64 / (4 * R + 1)) : 16;
}
// The radii a window kernel is compiled for: one of the row-task radii, all others
// (at run time), or any (the batched schedule).  Apart, each has the registers it
// needs: with all in one kernel, the pair body's cost the others 3 to 9%.
constexpr int kAnyRadius = -1, kOtherRadii = 0;
// Counters ahead of the candidate list: candidates, their cursor, largest
// term_size (as its bits), whether the row tasks have candidates of the pair
// body's, and their cursor.
constexpr int kListHead = 8;

__device__ inline void ld3(const float *p, int64_t i, float v[3]) {
    v[0] = p[3 * i];
    v[1] = p[3 * i + 1];
    v[2] = p[3 * i + 2];
}

__device__ inline float finish(int mode, bool valid, float B, float F, bool dark, float prev, int accumulate) {
    float v;
    if (mode == OCR_AO) v = valid ? 1.0f - B : 1.0f;
    else v = valid ? (dark ? 0.0f : F - B) : 0.0f;
    return accumulate ? prev + v : v;
}

// The no-reuse estimate of pixel gi (S(i) = {i}).  AO: 1 - [hit]; area
// shadows of a uniformly sampled light: [unblocked].  The solid-angle and
// direct-illumination quantities, and any light sampled from the bilinear
// density, take the N = 1 case of their MIS estimators: the unshadowed term
// minus C(x_i, z_i) for a hit whose own density is positive (the ratio p/p
// is 1).
template <int MODE, class LT>
__device__ inline float noreuse_value(const GBufView &g, const OccView &occ, const LT &L, int64_t gi, float scale) {
    // (both ids read together; a background pixel's hit id is never used)
    const uint32_t prim = g.prim[gi], hit0 = occ.hit[gi];
    const bool valid = prim != OCR_HIT_MISS;
    if constexpr (MODE == OCR_AO) {
        return (!valid || hit0 == OCR_HIT_MISS) ? 1.0f : 0.0f;
    } else if constexpr (MODE == OCR_SHADOW && !kBilinear<LT>) {
        return (valid && hit0 == OCR_HIT_MISS) ? 1.0f : 0.0f;
    } else {
        if (!valid) return 0.0f;
        float x[3], n[3], o[3];
        ld3(g.pos, gi, x);
        ld3(g.nrm, gi, n);
        offset_point(x, n, o);
        float Bg = 0.0f;
        const uint32_t hit = hit0;
        if (hit < OCR_HIT_SELF) {
            float dz[3], nz[3];
            ld3(occ.dz, gi, dz);
            ld3(occ.nz, gi, nz);
            const auto rk = recv_of(o, L);
            if (dens_light(dz, n, rk, nz, L) > 0.0f) {
                Bg = 1.0f;
                if constexpr (MODE == kDI) Bg = di_pair_g(dz, n, rk.hk, L);
                else if constexpr (MODE == kShadowSA) Bg = sa_pair_g(dz, rk.hk, L);
                if constexpr (kBilinear<LT>) Bg *= inv_bilinear_q(dz, rk, L);
            }
        }
        if constexpr (MODE == kDI) return di_estimate(o, n, L, Bg, scale);
        else if constexpr (MODE == kShadowSA) return sa_estimate(o, n, L, Bg);
        else return front_light(o, n, L) - Bg;
    }
}

// Radii the row-task body handles (compiled per radius); others take the
// per-candidate body.
__host__ __device__ constexpr bool row_body_radius(int R) { return R >= 1 && R <= 3; }

// LDS layout of the window kernel for radius R (dynamic shared memory).
struct WinLayout {
    int RWX, RWY, cells, side, dens, hsum, words;
    size_t o_off, n_off, sh_off, flag_off, row_off, list_off, left_off, B_off, wave_off, total;
};

__host__ __device__ constexpr size_t lds_take(size_t &off, size_t bytes) {
    size_t at = off;
    off += (bytes + 15) & ~(size_t)15;
    return at;
}

// nrecv: floats of a receiver's light terms (kRecvFloats of the light type);
// waves: of the block; pairs: pair_radius of the kernel.
__host__ __device__ constexpr WinLayout win_layout(int R, int mode, bool pairs, int words, int nrecv = 3,
                                                   int waves = kRBlock / 64) {
    WinLayout l{};
    l.RWX = kWTX + 2 * R;
    l.RWY = kWTY + 2 * R;
    l.cells = l.RWX * l.RWY;
    l.side = 4 * R + 1;
    l.dens = l.side * l.side;
    l.hsum = l.side * (2 * R + 1) > 2 * kSparse ? l.side * (2 * R + 1) : 2 * kSparse;
    l.words = words;
    size_t off = 0;
    l.B_off = lds_take(off, sizeof(unsigned long long) * kWTX * kWTY);
    l.o_off = lds_take(off, sizeof(float) * 3 * l.cells);
    l.n_off = lds_take(off, sizeof(float) * 3 * l.cells);
    l.sh_off = lds_take(off, mode != OCR_AO ? sizeof(float) * nrecv * l.cells : 0);
    l.flag_off = lds_take(off, l.cells);
    l.row_off = lds_take(off, mode != OCR_AO ? sizeof(uint32_t) * l.RWY : 0);
    l.list_off = lds_take(off, kListHead * sizeof(int) + sizeof(uint16_t) * l.cells);
    // the candidates that the pair lanes leave to the row tasks, a bit each
    l.left_off = lds_take(off, pairs ? (l.cells + 63) / 64 * sizeof(unsigned long long) : 0);
    // per-wave scratch: the per-candidate body's densities and box sums (the
    // row-task body keeps its sums in registers), the pair lanes' candidates
    const int per_wave = !row_body_radius(R) ? (int)sizeof(float) * (l.dens + l.hsum) : (pairs ? 64 : 0);
    l.wave_off = lds_take(off, (size_t)waves * per_wave);
    l.total = off;
    return l;
}

// The scattered term of target cell kc: p_i(j) / P_i(j) times the factor
// C(x_i, z_j) of the estimator, g_ij under the solid-angle definition
// (kShadowSA), gd_ij for direct illumination (kDI), and divided by q_i(y'_ij)
// for a light sampled from the bilinear density; clamped below 2^31 so that
// the 32.32 fixed-point sum cannot overflow (the factor reaches that size only
// within ~1e-5 of the light).
template <int MODE, class LT>
__device__ inline float weighted_term(float ratio, const float *s_o, const float *s_n, const float *s_sh, int CELLS,
                                      int kc, const float oj[3], const float dzj[3], const LT &L) {
    const float oi[3] = {s_o[kc], s_o[CELLS + kc], s_o[2 * CELLS + kc]};
    float w[3];
    rel_vec(oj, oi, dzj, w);
    float gf = 1.0f;
    if constexpr (MODE == kDI) {
        const float ni[3] = {s_n[kc], s_n[CELLS + kc], s_n[2 * CELLS + kc]};
        gf = di_pair_g(w, ni, s_sh[kc], L);
    } else if constexpr (MODE == kShadowSA) {
        gf = sa_pair_g(w, s_sh[kc], L);
    }
    if constexpr (kBilinear<LT>) {
        float v[6];
        for (int a = 0; a < 6; ++a) v[a] = s_sh[a * CELLS + kc];
        gf *= inv_bilinear_q(w, recv_load(v, L), L);
    }
    return fminf(ratio * gf, 0x1p31f);
}

// The targets of tile cells [R, R + kWTX) x [R, R + kWTY) (staged
// coordinates) that candidate cell (cx, cy) reaches, [tx0, tx0 + ntx) x
// [ty0, ty0 + nty), and the receivers they need, [tx0 - R, tx0 + ntx + R) x
// [ty0 - R, ty0 + nty + R).
struct CandRect {
    int tx0, ty0, ntx, nty;
};
__device__ inline CandRect cand_rect(int cx, int cy, int R) {
    CandRect q;
    q.tx0 = max(cx - R, R);
    q.ty0 = max(cy - R, R);
    q.ntx = min(cx + R, R + kWTX - 1) - q.tx0 + 1;
    q.nty = min(cy + R, R + kWTY - 1) - q.ty0 + 1;
    return q;
}

// DPP control of the whole-wave shift that gives each lane the value of the
// previous lane (wave_shr:1).
constexpr int kDppPrevLane = 0x138;

// v of lane - 1 (whole-wave DPP shift; lane 0, which has no source lane, gets
// 0 through bound_ctrl).  With full row and bank masks and bound_ctrl set, the
// compiler folds the move into the instruction that uses it.
__device__ inline float from_prev_lane(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kDppPrevLane, 0xF, 0xF, true));
}

// Candidates of a staged tile with the row-task body (window radius R = 1..3,
// a template parameter so that a receiver row's 4R + 1 densities stay in
// registers).  The waves of the block claim batches of consecutive entries of
// the tile's candidate list in turn from one shared cursor (a compare-and-swap
// in LDS), a batch being the leading candidates whose receiver rows fit in 64
// lanes, the rows of a candidate on consecutive lanes; so only the tile's last
// batch is partly empty, not one per wave.  A lane takes one receiver row of one
// candidate j: the densities p_k(j) of the row's receivers, then the row's
// box sums over each window of 2R + 1 of them, H[t] = sum_e p(t + e) in e
// order, all in registers.  For each target column t, the window sums over
// rows, P_i(j) = sum of H over the 2R + 1 rows of target row r's window in
// row order, are folded through the lanes by cross-lane moves (no memory) and
// end on the lane of the window's last row, r + 2R, which takes p_i(j) from
// lane r + R and scatters p_i(j) / P_i(j) as the per-candidate body does.
// The sums run in the same order as that body's, so the estimates are the
// same bits.
//
// MARKED: of the candidates listed, those whose bits are set in s_left (what the
// pair body left); a batch then spans the others.
template <int MODE, bool UNB, class LT, int R, bool MARKED>
__device__ inline void tile_row_candidates(const WinLayout &lay, unsigned char *smem, const GBufView &g,
                                           const OccView &occ, float R2, const LT &L,
                                           const uint32_t *__restrict__ bits, int words, int tx, int ty) {
    constexpr int TW = 2 * R + 1, SIDE = 4 * R + 1, D = 2 * R;
    constexpr int TX = kWTX, TY = kWTY, RW = kWTX + 2 * R, CELLS = RW * (kWTY + 2 * R);
    // The staged normals and light terms follow the positions directly
    // (3 * CELLS floats each, a multiple of 16 bytes), so all the receiver
    // values a density reads sit at constant offsets from one LDS address.
    constexpr WinLayout kLay = win_layout(R, MODE, MARKED, 1, kRecvFloats<LT>);
    static_assert(kLay.cells == CELLS && kLay.n_off == kLay.o_off + 3 * CELLS * sizeof(float) &&
                      (MODE == OCR_AO || kLay.sh_off == kLay.n_off + 3 * CELLS * sizeof(float)),
                  "receiver arrays are contiguous");
    const float inv_rw = 1.0f / (float)RW;
    unsigned long long *s_B = reinterpret_cast<unsigned long long *>(smem + lay.B_off);
    const float *s_o = reinterpret_cast<const float *>(smem + lay.o_off);
    const float *s_n = s_o + 3 * CELLS;
    const float *s_sh = s_n + 3 * CELLS;
    const int lane = threadIdx.x & 63;
    const int x0 = tx * TX - R, y0 = ty * TY - R;
    // s_count[0] candidates listed; the shared cursor counts the entries claimed,
    // zero at the tile's start
    int *s_count = reinterpret_cast<int *>(smem + lay.list_off);
    const uint16_t *s_list = reinterpret_cast<const uint16_t *>(smem + lay.list_off + kListHead * sizeof(int));
    const unsigned long long *s_left = reinterpret_cast<const unsigned long long *>(smem + lay.left_off);
    int *s_cursor = &s_count[MARKED ? 4 : 1];
    const int end = s_count[0];
    for (;;) {
        const int cur = __builtin_amdgcn_readfirstlane(__atomic_load_n(s_cursor, __ATOMIC_RELAXED));
        if (cur >= end) break;
        // candidate lanes: lane k holds candidate cur + k and its receiver
        // rows; the batch is the leading candidates whose rows fit
        const int ci = cur + lane;
        int c = 0, hd = 0;
        if (ci < end) {
            c = s_list[ci];
            const int cy = small_div(c, inv_rw), cx = c - __mul24(cy, RW);
            hd = cand_rect(cx, cy, R).nty + 2 * R;
            if (MARKED && !((s_left[ci >> 6] >> (ci & 63)) & 1ull)) hd = 0;
        }
        const int rows_inc = wave_incl_scan(hd);
        const int nb = __popcll(wave_ballot(ci < end && rows_inc <= 64));
        const int rows_total = __builtin_amdgcn_readlane(rows_inc, nb - 1);
        const int rows_exc = rows_inc - hd;
        // claim the batch; if another wave moved the cursor first, form the
        // next batch from where it now stands (some wave succeeds each round)
        int won = 0;
        if (lane == 0) won = atomicCAS(s_cursor, cur, cur + nb) == cur;
        if (!__builtin_amdgcn_readfirstlane(won)) continue;

        // this lane's candidate and receiver row
        int k = 0;
        if constexpr (MARKED) {
            if (rows_total == 0) continue;
            const unsigned long long have = wave_ballot(hd > 0 && rows_inc <= 64);
            for (unsigned long long m = have; m != 0ull; m &= m - 1ull) {
                const int i = (int)__builtin_ctzll(m);
                k = lane >= __builtin_amdgcn_readlane(rows_exc, i) ? i : k;
            }
        } else {
            for (int m = 0; m < nb; ++m) k += lane >= __builtin_amdgcn_readlane(rows_inc, m) ? 1 : 0;
            k = min(k, nb - 1);
        }
        const int cl = __shfl(c, k), rs = __shfl(rows_exc, k);
        const int cy = small_div(cl, inv_rw), cx = cl - __mul24(cy, RW);
        const CandRect q = cand_rect(cx, cy, R);
        const int row = lane - rs;
        const bool has_row = lane < rows_total;
        const int64_t gj = (int64_t)(y0 + cy) * g.w + (x0 + cx);
        const float oj[3] = {s_o[cl], s_o[CELLS + cl], s_o[2 * CELLS + cl]};
        float dzj[3] = {0.f, 0.f, 0.f};
        float p[SIDE];
#pragma unroll
        for (int e = 0; e < SIDE; ++e) p[e] = 0.0f;
        if (has_row) {
            const int WD = q.ntx + 2 * R;
            const int kx0 = q.tx0 - R, ky = q.ty0 - R + row;
            float nzj[3];
            ld3(occ.dz, gj, dzj);
            ld3(occ.nz, gj, nzj);
            // unbiased: the row's validation bits, bit e for receiver kx0 + e
            uint32_t rowbits = 0xFFFFFFFFu;
            if (UNB) {
                const int qb = __mul24(ky - cy + D, SIDE) + (kx0 - cx + D);
                const int w0 = qb >> 5;
                const uint32_t lo = bits[gj * words + w0];
                const uint32_t hi = w0 + 1 < words ? bits[gj * words + w0 + 1] : 0u;
                rowbits = (uint32_t)((((unsigned long long)hi << 32) | lo) >> (qb & 31));
            }
            const int kcb = __mul24(ky, RW) + kx0;
            // Several lights: one at a time, its constants in scalar registers
            // (all lights' do not fit; the sums keep their order).  Unbiased
            // window 2, two lights, 1080p 141 -> 114 us, biased 143 -> 139, window 1
            // 54 -> 46; only the biased window 3, 226 -> 232, is better all at once.
            constexpr bool kByLight = std::is_same<LT, LightSetF>::value && (R < 3 || UNB);
            if constexpr (kByLight) {
#pragma unroll 1
                for (int l = 0; l < L.n; ++l) {
                    const LightF Ll = L.l[l];
#pragma unroll
                    for (int e = 0; e < SIDE; ++e) {
                        if (e < WD && ((rowbits >> e) & 1u)) {
                            const int kc = kcb + e;
                            const float ok[3] = {s_o[kc], s_o[CELLS + kc], s_o[2 * CELLS + kc]};
                            const float nk[3] = {s_n[kc], s_n[CELLS + kc], s_n[2 * CELLS + kc]};
                            float w[3];
                            rel_vec(oj, ok, dzj, w);
                            p[e] += dens_shadow(w, nk, recv_shadow(ok, Ll), nzj, Ll);
                        }
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < SIDE && !kByLight; ++e) {
                if (e < WD && ((rowbits >> e) & 1u)) {
                    const int kc = kcb + e;
                    const float ok[3] = {s_o[kc], s_o[CELLS + kc], s_o[2 * CELLS + kc]};
                    const float nk[3] = {s_n[kc], s_n[CELLS + kc], s_n[2 * CELLS + kc]};
                    float w[3];
                    rel_vec(oj, ok, dzj, w);
                    if constexpr (MODE == OCR_AO) {
                        p[e] = dens_ao(w, nk, nzj, R2);
                    } else {
                        float v[kRecvFloats<LT>];
                        for (int a = 0; a < kRecvFloats<LT>; ++a) v[a] = s_sh[a * CELLS + kc];
                        p[e] = dens_light(w, nk, recv_load(v, L), nzj, L);
                    }
                }
            }
        }
        // P_i(j) for target row tr = row - 2R, column t: the box sums of rows
        // tr .. row (lanes lane - 2R .. lane, all of this candidate when
        // row >= 2R), summed in row order.  The fold runs upwards through the
        // lanes, G_e(lane) = G_(e-1)(lane - 1) + H(lane), so that after 2R
        // steps the lane of row `row` holds the window that ends at it, and
        // each step is one add with a shifted operand; p_i(j) comes from row
        // tr + R.  Every lane takes part in the moves; the lanes of rows
        // 2R .. 2R + nty - 1 scatter for the candidate's nty target rows.
        const int tr = row - D;
        const bool target_row = has_row && tr >= 0;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            // (the sums start from their first term rather than from 0: the
            // same values, since no density is -0)
            float h = p[t];
#pragma unroll
            for (int e = 1; e < TW; ++e) h += p[t + e];
            float P = h;
#pragma unroll
            for (int e = 1; e < TW; ++e) P = from_prev_lane(P) + h;
            float pij = p[t + R];
#pragma unroll
            for (int e = 0; e < R; ++e) pij = from_prev_lane(pij);
            if (target_row && t < q.ntx && pij > 0.0f && P > 0.0f) {
                float term = pij * __builtin_amdgcn_rcpf(P);
                if constexpr (MODE >= kShadowSA || kBilinear<LT>) {
                    term = weighted_term<MODE>(term, s_o, s_n, s_sh, CELLS,
                                               __mul24(q.ty0 + tr, RW) + (q.tx0 + t), oj, dzj, L);
                }
                atomicAdd(&s_B[(q.ty0 + tr - R) * TX + (q.tx0 + t - R)],
                          (unsigned long long)rintf(term * 4294967296.0f));
            }
        }
    }
    (void)TY;
}

// The light effects' candidates with few positive densities, row-task radii.
// The light subtends a narrow cone at z_j, so most candidates have one or two
// among their (4R + 1)^2 densities, and only those receivers are targets with a
// term.  First a lane takes a candidate and marks the receivers that may have a
// positive density (unbiased: the validation bits; biased: may_support, 10 VALU
// instructions and 3 LDS values a receiver instead of 45 and 9).  Then a lane
// takes a marked pair, the pairs of a candidate on consecutive lanes in row and
// column order: it evaluates the density and sums P_i(j) over the candidate's
// pairs in the target's window, row by row, by cross-lane reads: the box sums
// without their zeros, so the same bits.  Candidates with more than few_pairs(R)
// marks are left to the row tasks (s_left, all ones at the tile's start).
// 1080p, window 3, one light, rows / pairs: biased 0.285 / 0.190 ms, unbiased
// 0.216 / 0.121 (1.16M triangles), 0.199 / 0.199 and 0.198 / 0.185 where a 24 m
// light leaves most candidates to the rows.  What is left is the tail:
// without the few tiles that hold hundreds of candidates for the row tasks
// (9500 of 882000), which take 100 us each, the unbiased launch would end after
// 40 us.
template <int MODE, bool UNB, class LT, int R>
__device__ inline void tile_pair_candidates(const WinLayout &lay, unsigned char *smem, const GBufView &g,
                                            const OccView &occ, const LT &L, const uint32_t *__restrict__ bits,
                                            int words, int tx, int ty) {
    constexpr int SIDE = 4 * R + 1, D = 2 * R, NW = (SIDE * SIDE + 31) / 32;
    constexpr int TX = kWTX, TY = kWTY, RW = kWTX + 2 * R, RH = kWTY + 2 * R, CELLS = RW * RH;
    constexpr float kInvRw = 1.0f / (float)RW, kInvSide = 1.0f / (float)SIDE;
    unsigned long long *s_B = reinterpret_cast<unsigned long long *>(smem + lay.B_off);
    const float *s_o = reinterpret_cast<const float *>(smem + lay.o_off);
    const float *s_n = reinterpret_cast<const float *>(smem + lay.n_off);
    const float *s_sh = reinterpret_cast<const float *>(smem + lay.sh_off);
    int *s_count = reinterpret_cast<int *>(smem + lay.list_off);
    const uint16_t *s_list = reinterpret_cast<const uint16_t *>(smem + lay.list_off + kListHead * sizeof(int));
    unsigned long long *s_left = reinterpret_cast<unsigned long long *>(smem + lay.left_off);
    uint8_t *l_own = smem + lay.wave_off + (threadIdx.x >> 6) * 64;
    const int lane = threadIdx.x & 63;
    const int x0 = tx * TX - R, y0 = ty * TY - R;
    const int ncand = __builtin_amdgcn_readfirstlane(s_count[0]);
    const float qmax = __int_as_float(s_count[2]);
    for (;;) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_count[1], 64);
        base = __builtin_amdgcn_readfirstlane(base);
        if (base >= ncand) break;
        const bool has = base + lane < ncand;
        const int c = s_list[has ? base + lane : base];
        const int cy = small_div(c, kInvRw), cx = c - __mul24(cy, RW);
        const int64_t gj = (int64_t)(y0 + cy) * g.w + (x0 + cx);
        // marked receivers: bit q for cell (cx - D + q % SIDE, cy - D + q / SIDE)
        uint32_t w[NW];
        bool dense = false;  // wave-uniform
        if constexpr (UNB) {
#pragma unroll
            for (int i = 0; i < NW; ++i) w[i] = bits[gj * words + i];
        } else {
            uint32_t v[NW];
#pragma unroll
            for (int i = 0; i < NW; ++i) v[i] = 0u;
            float dzj[3];
            ld3(occ.dz, gj, dzj);
            const CandTerms t = cell_terms(s_sh, CELLS, c, dzj, L, qmax);
            const int here = min(ncand - base, 64), most = here - here / 8;
            int marks = 0;
#pragma unroll 1
            for (int i0 = 0; i0 < SIDE; ++i0) {
                // the candidate's own row, where a large light's marks are, and
                // those below it first.  (A row outside the staged cells is read
                // from the nearest one and masked below; a column beyond them
                // reads a neighbour row.)
                const int y = i0 <= D ? D + i0 : i0 - D - 1;
                const int k0 = __mul24(min(max(cy - D + y, 0), RH - 1), RW) + (cx - D);
                uint32_t m = 0;
#pragma unroll
                for (int e = 0; e < SIDE; ++e) m |= cell_support(s_sh, CELLS, k0 + e, t) ? 1u << e : 0u;
                // under a large light most candidates have many pairs: once seven
                // in eight of a batch have, it and those not claimed yet are left
                // to the row tasks
                marks += __popc(m);
                if (__popcll(wave_ballot(has && marks > few_pairs(R))) > most) {
                    dense = true;
                    break;
                }
                // the row's bits enter above the earlier ones
#pragma unroll
                for (int i = 0; i < NW - 1; ++i) v[i] = __builtin_amdgcn_alignbit(v[i + 1], v[i], SIDE);
                v[NW - 1] = (v[NW - 1] >> SIDE) | (m << (32 - SIDE));
            }
            if (!dense) {
                // down to bit 0, and the rows in order: the last D come first
                constexpr int kRest = 32 * NW - SIDE * SIDE;
                uint32_t hi[NW], lo[NW];
                words_right<kRest + (D + 1) * SIDE>(v, hi);
                words_right<kRest>(v, lo);
                words_left<D * SIDE>(lo, w);
#pragma unroll
                for (int i = 0; i < NW; ++i) w[i] |= hi[i];
            }
        }
        if (dense) {
            // (Its bits of s_left stay set, and no entry is left to claim.  By
            // every lane: after a branch on lane 0 the compiler may send the
            // others past the claim's, and they would not wait for lane 0's.)
            s_count[3] = 1;
            s_count[1] = ncand;
            wave_sync();
            continue;
        }
        // the receivers that the candidate's targets of this tile need
        const CandRect q = cand_rect(cx, cy, R);
        const int ra = q.ty0 - R - (cy - D), rb = ra + q.nty + 2 * R;  // rows [ra, rb) of the square
        const uint32_t cols = ((1u << (q.ntx + 2 * R)) - 1u) << (q.tx0 - R - (cx - D));
        uint32_t keep[NW + 1];
#pragma unroll
        for (int i = 0; i <= NW; ++i) keep[i] = 0u;
#pragma unroll
        for (int y = 0; y < SIDE; ++y) {
            const uint32_t row = y >= ra && y < rb ? cols : 0u;
            const int i = (y * SIDE) >> 5, sh = (y * SIDE) & 31;
            keep[i] |= row << sh;
            if (sh + SIDE > 32) keep[i + 1] |= row >> ((32 - sh) & 31);
        }
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            w[i] = has ? w[i] & keep[i] : 0u;
            cnt += __popc(w[i]);
        }
        const bool many = has && cnt > few_pairs(R);
        const unsigned long long mm = wave_ballot(many);
        if (lane == 0) {
            s_left[base >> 6] = mm;
            if (mm != 0ull) s_count[3] = 1;
        }
        if (many) cnt = 0;
        const int incl = wave_incl_scan(cnt), excl = incl - cnt, total = __builtin_amdgcn_readlane(incl, 63);
        // lanes for the pairs of as many candidates at a time as 64 hold
        for (int done = 0; done < total;) {
            const bool take = cnt > 0 && excl >= done && incl <= done + 64;
            const unsigned long long tm = wave_ballot(take);
            const int upto = __builtin_amdgcn_readlane(incl, 63 - (int)__builtin_clzll(tm));
            // this lane's pair: the candidate's lane (each candidate's lane
            // number at its first pair, then the largest so far), and its place
            // among that one's pairs
            l_own[lane] = 0;
            if (take) l_own[excl - done] = (uint8_t)lane;
            wave_sync();
            const int own = wave_incl_max((int)l_own[lane]);
            wave_sync();
            const bool pair = lane < upto - done;
            const int first = __shfl(excl, own) - done, n = __shfl(cnt, own);
            int rank = lane - first;
            const int cc = __shfl(c, own), pcx = __shfl(cx, own), pcy = __shfl(cy, own);
            uint32_t b = 0;
            int qq = 0;
            bool found = false;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const uint32_t v = (uint32_t)__shfl((int)w[i], own);
                const int m = __popc(v);
                if (!found && rank < m) {
                    found = true;
                    b = v;
                    qq = 32 * i;
                }
                rank -= found ? 0 : m;
            }
            qq += nth_bit(b, rank);
            const int qy = small_div(qq, kInvSide);
            const int kx = pcx - D + (qq - __mul24(qy, SIDE)), ky = pcy - D + qy;
            const int kc = pair ? __mul24(ky, RW) + kx : 0;
            float p = 0.0f;
            float oj[3], dzj[3];
            if (pair) {
                const int64_t pj = (int64_t)(y0 + pcy) * g.w + (x0 + pcx);
                float nzj[3], wv[3], v[kRecvFloats<LT>];
                ld3(occ.dz, pj, dzj);
                ld3(occ.nz, pj, nzj);
                for (int a = 0; a < 3; ++a) oj[a] = s_o[a * CELLS + cc];
                const float ok[3] = {s_o[kc], s_o[CELLS + kc], s_o[2 * CELLS + kc]};
                const float nk[3] = {s_n[kc], s_n[CELLS + kc], s_n[2 * CELLS + kc]};
                rel_vec(oj, ok, dzj, wv);
                for (int a = 0; a < kRecvFloats<LT>; ++a) v[a] = s_sh[a * CELLS + kc];
                p = dens_light(wv, nk, recv_load(v, L), nzj, L);
            }
            // targets: pixels of the tile within R of the candidate
            const bool target = pair && p > 0.0f && (uint32_t)(kx - R) < (uint32_t)TX && (uint32_t)(ky - R) < (uint32_t)TY &&
                                abs(kx - pcx) <= R && abs(ky - pcy) <= R;
            if (wave_ballot(target) != 0ull) {
                const int at = (ky << 8) | kx;
                float P = 0.0f, h = 0.0f;
                int last = -1;
                // (four pairs' values read ahead of their sums; every lane
                // takes part, those with fewer pairs read their last one)
                for (int m0 = 0; wave_ballot(target && m0 < n) != 0ull; m0 += 4) {
                    int am[4];
                    float pm[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int src = first + min(m0 + e, n - 1);
                        am[e] = __shfl(at, src);
                        pm[e] = __shfl(p, src);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (m0 + e < n) {
                            const int ym = am[e] >> 8, xm = am[e] & 255;
                            if (ym != last) {
                                P += h;
                                h = 0.0f;
                                last = ym;
                            }
                            if (abs(ym - ky) <= R && abs(xm - kx) <= R) h += pm[e];
                        }
                    }
                }
                P += h;
                if (target) {
                    float term = p * __builtin_amdgcn_rcpf(P);
                    if constexpr (MODE >= kShadowSA || kBilinear<LT>)
                        term = weighted_term<MODE>(term, s_o, s_n, s_sh, CELLS, kc, oj, dzj, L);
                    atomicAdd(&s_B[(ky - R) * TX + (kx - R)], (unsigned long long)rintf(term * 4294967296.0f));
                }
            }
            done = upto;
        }
    }
}

// All candidates of a staged tile, row-task radii; BLOCK lanes call it.
template <int MODE, bool UNB, class LT, int R, int BLOCK>
__device__ inline void tile_candidates(const WinLayout &lay, unsigned char *smem, const GBufView &g,
                                       const OccView &occ, float R2, const LT &L,
                                       const uint32_t *__restrict__ bits, int words, int tx, int ty) {
    if constexpr (pair_radius<MODE, UNB, LT>(R)) {
        int *s_count = reinterpret_cast<int *>(smem + lay.list_off);
        bool rows = !UNB && __builtin_amdgcn_readfirstlane(s_count[0]) <= few_candidates(R, BLOCK);
        if (!rows) {
            if constexpr (!UNB) {
                // the largest term_size of the receivers (1 for cells without one;
                // floats from 0 up order as integers)
                constexpr int CELLS = (kWTX + 2 * R) * (kWTY + 2 * R);
                const float *s_sh = reinterpret_cast<const float *>(smem + lay.sh_off);
                const LightScale sc = light_scale(L);
                float q = 0.0f;
                for (int c = threadIdx.x; c < CELLS; c += BLOCK)
                    q = fmaxf(q, term_size(s_sh[c], s_sh[CELLS + c], s_sh[2 * CELLS + c], sc));
                const int m = ~wave_min_i(~__float_as_int(q));
                if ((threadIdx.x & 63) == 0) atomicMax(&s_count[2], m);
                __syncthreads();
            }
            tile_pair_candidates<MODE, UNB, LT, R>(lay, smem, g, occ, L, bits, words, tx, ty);
            __syncthreads();
            rows = __builtin_amdgcn_readfirstlane(s_count[3]) != 0;
        }
        if (rows) tile_row_candidates<MODE, UNB, LT, R, true>(lay, smem, g, occ, R2, L, bits, words, tx, ty);
    } else {
        tile_row_candidates<MODE, UNB, LT, R, false>(lay, smem, g, occ, R2, L, bits, words, tx, ty);
    }
}

// One kWTX x kWTY target tile (tx, ty) of the sliding-window estimator; every
// thread of the block calls it.  `smem` holds win_layout(radius, ...).total bytes.
// RT: the radius it is compiled for.
template <int MODE, bool UNB, class LT = LightF, int RT = kAnyRadius, int BLOCK = kRBlock>
__device__ inline void reuse_window_tile(unsigned char *smem, const GBufView &g, const OccView &occ, float R2,
                                         const LT &L, const uint32_t *__restrict__ bits, int words, int radius,
                                         int dark_guard, int accumulate, float *out, int tx, int ty,
                                         float scale = 1.0f) {
    const int R = RT > 0 ? RT : radius;
    const bool pairs = pair_radius<MODE, UNB, LT>(R);
    const WinLayout lay = win_layout(R, MODE, pairs, words, kRecvFloats<LT>, BLOCK / 64);
    const int TX = kWTX, TY = kWTY, RW = lay.RWX, CELLS = lay.cells, D = 2 * R, SIDE = lay.side, TW = 2 * R + 1;
    const float inv_rw = 1.0f / (float)RW;
    unsigned long long *s_B = reinterpret_cast<unsigned long long *>(smem + lay.B_off);
    float *s_o = reinterpret_cast<float *>(smem + lay.o_off);    // [3][cells]
    float *s_n = reinterpret_cast<float *>(smem + lay.n_off);    // [3][cells]
    float *s_sh = reinterpret_cast<float *>(smem + lay.sh_off);  // [kRecvFloats][cells]
    uint8_t *s_flag = smem + lay.flag_off;  // bit 0: a receiver, bit 1: whose ray hit nothing
    // the latter as a mask per row, for the dark-region guard (at most 32 columns)
    uint32_t *s_row = reinterpret_cast<uint32_t *>(smem + lay.row_off);
    int *s_count = reinterpret_cast<int *>(smem + lay.list_off);
    uint16_t *s_list = reinterpret_cast<uint16_t *>(smem + lay.list_off + kListHead * sizeof(int));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float *w_dens = reinterpret_cast<float *>(smem + lay.wave_off) + wave * (lay.dens + lay.hsum);
    float *w_h = w_dens + lay.dens;

    const int x0 = tx * TX - R, y0 = ty * TY - R;
    const int tid = threadIdx.x;
    if (tid < kListHead) s_count[tid] = 0;
    if (pairs && tid < 8) reinterpret_cast<unsigned long long *>(smem + lay.left_off)[min(tid, (CELLS - 1) / 64)] = ~0ull;
    for (int t = tid; t < TX * TY; t += BLOCK) s_B[t] = 0ull;
    __syncthreads();

    // Stage receivers (o, n, shadow terms), validity, misses, validation
    // bits, and compact the cells whose ray found an occluder.
    for (int c = tid; c < CELLS; c += BLOCK) {
        const int cyy = small_div(c, inv_rw);
        int gx = x0 + (c - __mul24(cyy, RW)), gy = y0 + cyy;
        bool inside = gx >= 0 && gx < g.w && gy >= 0 && gy < g.h;
        int64_t gi = inside ? (int64_t)gy * g.w + gx : 0;
        bool valid = inside && g.prim[gi] != OCR_HIT_MISS;
        float o[3] = {0.f, 0.f, 0.f}, n[3] = {0.f, 0.f, 0.f};
        uint32_t hit = OCR_HIT_MISS;
        if (valid) {
            float x[3];
            ld3(g.pos, gi, x);
            ld3(g.nrm, gi, n);
            offset_point(x, n, o);
            hit = occ.hit[gi];
        }
        for (int a = 0; a < 3; ++a) {
            s_o[a * CELLS + c] = o[a];
            s_n[a * CELLS + c] = n[a];
        }
        if (MODE != OCR_AO) {
            // the receiver's light terms (its point, for several lights)
            float v[kRecvFloats<LT>] = {};
            if (valid) recv_store(recv_of(o, L), v);
            for (int a = 0; a < kRecvFloats<LT>; ++a) s_sh[a * CELLS + c] = v[a];
        }
        s_flag[c] = (uint8_t)((valid ? 1 : 0) | (valid && hit == OCR_HIT_MISS ? 2 : 0));
        if (valid && hit < OCR_HIT_SELF) s_list[atomicAdd(s_count, 1)] = (uint16_t)c;
    }
    __syncthreads();

    // (read after the candidates' barrier; the window byte by byte, 49 reads a
    // target at radius 3, was a fifth of the biased shadows' time)
    if (MODE != OCR_AO && dark_guard && tid < lay.RWY) {
        uint32_t m = 0;
        for (int x = 0; x < RW; ++x) m |= (uint32_t)(s_flag[tid * RW + x] >> 1) << x;
        s_row[tid] = m;
    }

#define OCR_TILE_RADIUS(r)                                                                                   \
    if constexpr (RT == kAnyRadius || RT == r) {                                                             \
        if (R == r) tile_candidates<MODE, UNB, LT, r, BLOCK>(lay, smem, g, occ, R2, L, bits, words, tx, ty); \
    }
    OCR_TILE_RADIUS(1)
    OCR_TILE_RADIUS(2)
    OCR_TILE_RADIUS(3)
#undef OCR_TILE_RADIUS
    if ((RT == kAnyRadius || RT == kOtherRadii) && !row_body_radius(R)) {
        // Other radii: one wave per candidate j.
        const int ncand = *s_count;
        for (int li = wave; li < ncand; li += kRBlock >> 6) {
            const int c = __builtin_amdgcn_readfirstlane((int)s_list[li]);
            const int cy = small_div(c, inv_rw), cx = c - __mul24(cy, RW);
            const int64_t gj = (int64_t)(y0 + cy) * g.w + (x0 + cx);
            float oj[3] = {s_o[c], s_o[CELLS + c], s_o[2 * CELLS + c]};
            float dzj[3], nzj[3];
            ld3(occ.dz, gj, dzj);
            ld3(occ.nz, gj, nzj);
            // The targets of this tile that j reaches are the cells [tx0, tx1] x
            // [ty0, ty1] (staged coordinates; the tile is [R, R + TX) x [R, R + TY));
            // they need the receivers [tx0 - R, tx1 + R] x [ty0 - R, ty1 + R], a
            // WD x HD rectangle inside the staged region (13 x 13 at R = 3 for a
            // candidate whose targets are all in the tile, less in the halo).
            const int tx0 = max(cx - R, R), tx1 = min(cx + R, R + TX - 1);
            const int ty0 = max(cy - R, R), ty1 = min(cy + R, R + TY - 1);
            const int ntx = tx1 - tx0 + 1, nty = ty1 - ty0 + 1;
            const int WD = ntx + 2 * R, HD = nty + 2 * R;
            const int kx0 = tx0 - R, ky0 = ty0 - R;
            // (hardware reciprocals: small_div stays exact with a 1-ulp inverse
            // for the quotients below, all < 2^12)
            const float inv_wd = __builtin_amdgcn_rcpf((float)WD), inv_ntx = __builtin_amdgcn_rcpf((float)ntx);
            const int nq = WD * HD;
            // (1) densities p_k(j) over the rectangle, row stride SIDE; every lane
            // runs every pass so that the count of positive densities is uniform.
            // Shadow candidates have a few positive densities at most (the light
            // subtends a narrow cone); AO candidates most often have dozens.
            constexpr bool kSparsePath = MODE != OCR_AO;
            int npos = 0;
            int *e_code = reinterpret_cast<int *>(w_h);  // positive entries, q order
            float *e_p = w_h + kSparse;
            for (int q0 = 0; q0 < nq; q0 += 64) {
                const int q = q0 + lane;
                float p = 0.0f;
                int qy = 0, qx = 0;
                if (q < nq) {
                    // (index products by 24-bit multiplies: full rate, all operands < 2^23)
                    qy = small_div(q, inv_wd);
                    qx = q - __mul24(qy, WD);
                    const int kx = kx0 + qx, ky = ky0 + qy;
                    const int kc = __mul24(ky, RW) + kx;
                    // unbiased: candidate j's validation bit for the receiver at
                    // offset k - j first.  It is set only where the validation
                    // found the same density positive (and the segment free), so
                    // a pair without it contributes 0 whatever its density, and a
                    // round with no bit set skips the densities altogether
                    // (shadow candidates have a few positive pairs, clustered).
                    bool need = true;
                    if (UNB) {
                        const int qb = __mul24(ky - cy + D, SIDE) + (kx - cx + D);
                        const uint32_t wv = bits[gj * words + (qb >> 5)];
                        need = (wv >> (qb & 31)) & 1u;
                    }
                    if (need) {
                        float ok[3] = {s_o[kc], s_o[CELLS + kc], s_o[2 * CELLS + kc]};
                        float nk[3] = {s_n[kc], s_n[CELLS + kc], s_n[2 * CELLS + kc]};
                        float w[3];
                        rel_vec(oj, ok, dzj, w);
                        if (MODE == OCR_AO) {
                            p = dens_ao(w, nk, nzj, R2);
                        } else {
                            float v[kRecvFloats<LT>];
                            for (int a = 0; a < kRecvFloats<LT>; ++a) v[a] = s_sh[a * CELLS + kc];
                            p = dens_light(w, nk, recv_load(v, L), nzj, L);
                        }
                    }
                    w_dens[__mul24(qy, SIDE) + qx] = p;
                }
                if (!kSparsePath) continue;
                const unsigned long long pm = __ballot(p > 0.0f);
                if (npos < kSparse) {
                    // keep the first kSparse positive entries for the sparse path
                    const int at = npos + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(pm >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)pm, 0u));
                    if (p > 0.0f && at < kSparse) {
                        e_code[at] = (qy << 8) | qx;
                        e_p[at] = p;
                    }
                }
                npos += (int)__popcll(pm);
            }
            wave_sync();
            if (kSparsePath && npos <= kSparse) {
                // (2') Few positive densities (most shadow candidates): P_i(j) from
                // the positive entries alone.  Lane e takes entry e; the sums run
                // over the rows in order and within a row over the columns in
                // order, the grouping of the box sums below, which only add zeros
                // besides (exact), so both paths give the same bits.
                int my_code = 0;
                float my_p = 0.0f;
                if (lane < npos) {
                    my_code = e_code[lane];
                    my_p = e_p[lane];
                }
                const int my_y = my_code >> 8, my_x = my_code & 255;
                const bool tgt = lane < npos && my_x >= R && my_x < R + ntx && my_y >= R && my_y < R + nty;
                if (__ballot(tgt) != 0ull) {
                    float P = 0.0f, h = 0.0f;
                    int row = -1;
                    for (int m = 0; m < npos; ++m) {
                        const int cm = __builtin_amdgcn_readlane(my_code, m);
                        const float pv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_p), m));
                        const int ym = cm >> 8, xm = cm & 255;
                        if (ym != row) {
                            P += h;
                            h = 0.0f;
                            row = ym;
                        }
                        if (abs(ym - my_y) <= R && abs(xm - my_x) <= R) h += pv;
                    }
                    P += h;
                    if (tgt) {
                        float term = my_p * __builtin_amdgcn_rcpf(P);
                        if constexpr (MODE >= kShadowSA || kBilinear<LT>)
                            term = weighted_term<MODE>(term, s_o, s_n, s_sh, CELLS, __mul24(ky0 + my_y, RW) + (kx0 + my_x),
                                                       oj, dzj, L);
                        atomicAdd(&s_B[(ky0 + my_y - R) * TX + (kx0 + my_x - R)],
                                  (unsigned long long)rintf(term * 4294967296.0f));
                    }
                }
            } else {
                // (2) row box sums H[row][t] = sum_{e < 2R+1} p(row, t + e), t < ntx
                for (int q = lane; q < HD * ntx; q += 64) {
                    const int row = small_div(q, inv_ntx), t2 = q - __mul24(row, ntx);
                    const float *pr = w_dens + __mul24(row, SIDE) + t2;
                    float h = 0.0f;
                    // unrolled so the LDS reads issue together; the additions keep their order (by
                    // 8 instead of 4: window 8 at 1280x720 AO 1550 -> 1480 us)
    #pragma unroll 8
                    for (int e = 0; e < TW; ++e) h += pr[e];
                    w_h[__mul24(row, TW) + t2] = h;
                }
                wave_sync();
                // (3) target i = (tx0 + t2, ty0 + r2): P_i(j) is the column box sum of H
                for (int q = lane; q < nty * ntx; q += 64) {
                    const int r2 = small_div(q, inv_ntx), t2 = q - __mul24(r2, ntx);
                    const float *ph = w_h + __mul24(r2, TW) + t2;
                    float P = 0.0f;
    #pragma unroll 8
                    for (int e = 0; e < TW; ++e) P += ph[__mul24(e, TW)];
                    const float pij = w_dens[__mul24(r2 + R, SIDE) + (t2 + R)];
                    if (pij > 0.0f && P > 0.0f) {
                        float term = pij * __builtin_amdgcn_rcpf(P);
                        if constexpr (MODE >= kShadowSA || kBilinear<LT>)
                            term = weighted_term<MODE>(term, s_o, s_n, s_sh, CELLS, __mul24(ty0 + r2, RW) + (tx0 + t2), oj,
                                                       dzj, L);
                        atomicAdd(&s_B[(ty0 + r2 - R) * TX + (tx0 + t2 - R)],
                                  (unsigned long long)rintf(term * 4294967296.0f));
                    }
                }
            }
            wave_sync();
        }
    }
    __syncthreads();

    // one lane per target
    for (int t = tid; t < TX * TY; t += BLOCK) {
        const int ix = t % TX, iy = t / TX;
        const int px = tx * TX + ix, py = ty * TY + iy;
        if (px >= g.w || py >= g.h) continue;
        const int c = __mul24(iy + R, RW) + (ix + R);
        const bool valid = s_flag[c] & 1;
        float B = (float)((double)s_B[t] * 0x1p-32);
        float F = 1.0f;
        bool dark = false;
        if (MODE != OCR_AO && valid) {
            float o[3] = {s_o[c], s_o[CELLS + c], s_o[2 * CELLS + c]};
            float n[3] = {s_n[c], s_n[CELLS + c], s_n[2 * CELLS + c]};
            if constexpr (MODE == kShadowSA) {
                // F_Omega - (Area / Omega_A) B, as F - B below
                F = sa_estimate(o, n, L, B);
                B = 0.0f;
            } else if constexpr (MODE == kDI) {
                // (rho L_e / pi) (E - Area B), as F - B below
                F = di_estimate(o, n, L, B, scale);
                B = 0.0f;
            } else {
                F = front_light(o, n, L);
            }
            if (dark_guard) {
                uint32_t seen = 0;
                for (int dy = 0; dy < TW; ++dy) seen |= s_row[iy + dy];
                dark = ((seen >> ix) & ((1u << TW) - 1u)) == 0u;
            }
        }
        const int64_t gi = (int64_t)py * g.w + px;
        out[gi] = finish(MODE, valid, B, F, dark, accumulate ? out[gi] : 0.0f, accumulate);
    }
}


}  // namespace ocr
