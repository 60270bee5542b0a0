// First-hit validation (Eq. occ-first-hit) of the light effects' windows of
// radius 1 to 3: the pairs that may have a positive density are marked tile by
// tile, and the marked ones walked.
//
// The light subtends a narrow cone at z_j, so a candidate has one or two pairs
// among its (4R + 1)^2.  Listing them by their densities (the walk over
// candidate lists of trace.hip, which other radii take) was two thirds of its
// VALU instructions, which bound it.  1080p, 1.16M triangles, lists / marks:
// window 3 0.482 / 0.249 ms (marking 0.06 ms), window 2 0.411 / 0.233, window 1
// 0.347 / 0.218; 333x197 0.060 / 0.043; boxes 1920x1080 0.189 / 0.161, 333x197
// 0.031 / 0.028.  Under a light that marks half of the square, 24 m wide, 1.442 /
// 1.322 (131000 triangles).  Slower only where the marks say little: a light of
// 20 m by 1 m over a small frame, 0.029 / 0.031, and one of 100 m at 9.5 km, whose
// distance widens the marks' slack, 0.053 / 0.061.
#include "lights.hpp"
#include "ocr_common.hpp"
#include "traverse.hpp"
#include "validate.hpp"

namespace ocr {

constexpr int kLBlock = 256;
constexpr int kLTile = 16;    // 16 x 16 candidates per block
constexpr int kLTileRun = 8;  // consecutive tiles an XCD takes at a time

__host__ __device__ constexpr int light_cells(int R) { return (kLTile + 4 * R) * (kLTile + 4 * R); }
__device__ inline int lights_of(const LightF &) { return 1; }
__device__ inline int lights_of(const LightSetF &S) { return S.n; }
__device__ inline const LightF &light_at(const LightF &L, int) { return L; }
__device__ inline const LightF &light_at(const LightSetF &S, int l) { return S.l[l]; }

// Most marks of a candidate listed with those of few.  Those of more are walked
// first and in shorter runs: their runs take up to 20 walks, and one that starts
// late is the launch's end (1080p window 3 by one list and runs of 8: 0.47 ms).
constexpr int kFewMarks = 8;
// Most candidates of a run (8 of few marks measured 2% faster at 1080p and 6%
// slower at 720p).
constexpr int kMarkRun = 6;
// Candidates of many marks per further one in a run (2 to 6): a run's walks are
// fuller with more, once every wave has several runs (1920x1080 boxes window 3,
// 119000 candidates, runs of 1 / 2 / 4: 0.230 / 0.185 / 0.176 ms; 1280x720 terrain
// with few such candidates 0.195 / 0.209 / 0.253).
constexpr uint32_t kManyStep = 16384;
// Candidates of few marks per further one in a run (1 to 6).  Neighbours in the
// list may lie far apart in the frame, and a wave walks the union of their paths:
// in a large mesh, where those are long, a wave for each is the shorter way as
// long as there are waves (1.16M triangles 333x197, 73 candidates: 69 us by sixes,
// 37 alone; 291000 triangles 1280x720, 10000 candidates: 104 / 83); in a small one
// they share most of theirs (1154 triangles 333x197: 24 us by sixes, 33 alone).
constexpr uint32_t kFewStep = 8192, kFewStepSmall = 256;
constexpr int64_t kSmallMesh = 16384;

// Appends the wave's lanes that have something to a counted list (every lane
// calls it).
template <class F>
__device__ inline void list_append(uint32_t *count, bool want, const F &put) {
    const unsigned long long m = wave_ballot(want);
    if (m == 0ull) return;
    uint32_t at = 0;
    if ((threadIdx.x & 63) == 0) at = atomicAdd(count, (uint32_t)__popcll(m));
    at = __builtin_amdgcn_readfirstlane(at);
    if (want) put(at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)));
}

// The pairs (candidate j, receiver k) whose density may be positive are marked
// from the light terms of the tile's receivers (the tile and 2R pixels around
// it), staged in LDS: a lane takes a candidate and tests its (4R + 1)^2
// receivers by may_support, 10 VALU instructions and 3 LDS values each.  The
// marks are left in the candidates' validation words, and the candidates that
// have any are listed for the walks.
template <class LT, int R>
__global__ __launch_bounds__(kLBlock) void mark_pairs_kernel(GBufView g, OccView occ, LT L, uint32_t *bits,
                                                             uint32_t *lists, uint32_t per_xcd, int tiles_x,
                                                             int ntiles) {
    constexpr int D = 2 * R, SIDE = 4 * R + 1, NW = (SIDE * SIDE + 31) / 32, RW = kLTile + 2 * D, CELLS = RW * RW;
    constexpr int kNL = std::is_same<LT, LightSetF>::value ? kMaxLights : 1;
    constexpr int kSelf = D * SIDE + D;
    constexpr float kInvRw = 1.0f / (float)RW;
    extern __shared__ float s_t[];  // [lights][3][CELLS]
    __shared__ uint8_t s_list[kLBlock];
    __shared__ int s_count[kLBlock / 64];
    __shared__ int s_size[kMaxLights];  // largest term_size (its bits: floats from 0 up order as integers)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x, local = blk >> 3;
    const int t = (local / kLTileRun) * (8 * kLTileRun) + (blk & 7) * kLTileRun + local % kLTileRun;
    if (t >= ntiles) return;
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    const int nl = lights_of(L);

    // the tile's candidates, in the order of the threads (8 x 8 pixels a wave)
    {
        const int px = tx * kLTile + (wave & 1) * 8 + (lane & 7), py = ty * kLTile + (wave >> 1) * 8 + (lane >> 3);
        const bool inside = px < g.w && py < g.h;
        const bool cand = inside && occ.hit[inside ? (int64_t)py * g.w + px : 0] < OCR_HIT_SELF;
        const unsigned long long m = wave_ballot(cand);
        if (lane == 0) s_count[wave] = (int)__popcll(m);
        if (tid < kMaxLights) s_size[tid] = 0;
        __syncthreads();
        int at = 0;
        for (int v = 0; v < wave; ++v) at += s_count[v];
        at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (cand) s_list[at] = (uint8_t)tid;
    }
    const int ncand = s_count[0] + s_count[1] + s_count[2] + s_count[3];
    if (ncand == 0) return;

    // the receivers' light terms; those that no pair can have (outside the image,
    // background) get terms that no test passes
    const int x0 = tx * kLTile - D, y0 = ty * kLTile - D;
    float size[kNL] = {};
#pragma unroll
    for (int it = 0; it < (CELLS + kLBlock - 1) / kLBlock; ++it) {
        const int c = it * kLBlock + tid;
        const int cy = small_div(c, kInvRw), cx = c - __mul24(cy, RW);
        const int gx = x0 + cx, gy = y0 + cy;
        const bool inside = gx >= 0 && gx < g.w && gy >= 0 && gy < g.h;
        const int64_t gi = inside ? (int64_t)gy * g.w + gx : 0;
        float x[3], n[3], o[3];
        const bool valid = (g.prim[gi] != OCR_HIT_MISS) & inside;
        load3(g.pos, gi, x);
        load3(g.nrm, gi, n);
        offset_point(x, n, o);
        if (c < CELLS) {
#pragma unroll
            for (int l = 0; l < kNL; ++l) {
                if (l >= nl) break;
                const RecvShadow r = recv_shadow(o, light_at(L, l));
                float *p = s_t + l * 3 * CELLS + c;
                p[0] = valid ? r.hk : 0.0f;
                p[CELLS] = valid ? r.ak : INFINITY;
                p[2 * CELLS] = valid ? r.bk : INFINITY;
                if (valid) size[l] = fmaxf(size[l], term_size(r.hk, r.ak, r.bk, light_scale(light_at(L, l))));
            }
        }
    }
#pragma unroll
    for (int l = 0; l < kNL; ++l) {
        const int m = ~wave_min_i(~__float_as_int(size[l]));
        if (lane == 0) atomicMax(&s_size[l], m);
    }
    __syncthreads();

    // a wave per 64 candidates; of few, the rows of the square are shared by all
    // four waves (48x36 boxes, two lights, window 3 42 -> 35 us; 1080p
    // terrain under a light 950 m away 52 -> 47)
    const int parts = ncand <= 64 ? 4 : ncand <= 128 ? 2 : 1, part = wave & (parts - 1);
    const int base = (wave / parts) * 64;
    if (base >= ncand) return;  // (parts is 1: no barrier follows)
    const int row0 = part * SIDE / parts, row1 = (part + 1) * SIDE / parts;
    const bool has = base + lane < ncand;
    const int id = s_list[has ? base + lane : base];
    // the candidate's pixel in the tile and on the image
    const int lx = ((id >> 6) & 1) * 8 + (id & 7), ly = (id >> 7) * 8 + ((id >> 3) & 7);
    const int jx = tx * kLTile + lx, jy = ty * kLTile + ly;
    const int64_t j = (int64_t)jy * g.w + jx;
    float oj[3], dzj[3];
    {
        float x[3], n[3];
        load3(g.pos, j, x);
        load3(g.nrm, j, n);
        load3(occ.dz, j, dzj);
        offset_point(x, n, oj);
    }
    // marked receivers: bit q for pixel j + (q % SIDE - D, q / SIDE - D)
    uint32_t w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = 0u;
#pragma unroll 1
    for (int l = 0; l < nl; ++l) {
        const float *p = s_t + l * 3 * CELLS;
        const CandTerms ct = cell_terms(p, CELLS, __mul24(ly + D, RW) + lx + D, dzj, light_at(L, l), __int_as_float(s_size[l]));
        uint32_t v[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) v[i] = 0u;
#pragma unroll 1
        for (int y = 0; y < SIDE; ++y) {
            const int k0 = __mul24(ly + y, RW) + lx;
            uint32_t m = 0;
            if (y >= row0 && y < row1) {
#pragma unroll
                for (int e = 0; e < SIDE; ++e) m |= cell_support(p, CELLS, k0 + e, ct) ? 1u << e : 0u;
            }
            // the row's bits enter above the earlier ones
#pragma unroll
            for (int i = 0; i < NW - 1; ++i) v[i] = __builtin_amdgcn_alignbit(v[i + 1], v[i], SIDE);
            v[NW - 1] = (v[NW - 1] >> SIDE) | (m << (32 - SIDE));
        }
        // down to bit 0
        constexpr int kRest = 32 * NW - SIDE * SIDE;
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] |= i < NW - 1 ? __builtin_amdgcn_alignbit(v[i < NW - 1 ? i + 1 : i], v[i], kRest) : v[i] >> kRest;
    }
    if (parts > 1) {
        // the other waves' rows, through the light terms' LDS
        static_assert(256 * NW <= 3 * CELLS, "room for the words");
        uint32_t *s_w = reinterpret_cast<uint32_t *>(s_t);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NW; ++i) s_w[i * kLBlock + tid] = w[i];
        __syncthreads();
        if (part > 0) return;
        for (int o = 1; o < parts; ++o) {
#pragma unroll
            for (int i = 0; i < NW; ++i) w[i] |= s_w[i * kLBlock + tid + 64 * o];
        }
    }
    w[kSelf >> 5] &= ~(1u << (kSelf & 31));  // z_j is its own first hit
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) cnt += __popc(w[i]);
    // (a list holds the candidates of ceil(ntiles / 8) tiles: those of few
    // marks from its start, the others from its end)
    const bool marked = has && cnt > 0;
    const uint32_t list = (uint32_t)t / (uint32_t)((ntiles + 7) / 8);
    uint32_t *const entries = lists + 8 * kCountStride + list * per_xcd;
    list_append(lists + list * kCountStride, marked && cnt <= kFewMarks, [&](uint32_t at) { entries[at] = (uint32_t)j; });
    list_append(lists + list * kCountStride + 1, marked && cnt > kFewMarks,
                [&](uint32_t at) { entries[per_xcd - 1u - at] = (uint32_t)j; });
    if (has) {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const uint32_t self = i == (kSelf >> 5) ? 1u << (kSelf & 31) : 0u;
            bits[j * NW + i] = marked ? w[i] : self;
        }
    }
}

// A candidate of the current run.
struct MarkCand {
    float oj[3], dzj[3], nzj[3];
    int32_t jx, jy;
    uint32_t hj;
};

// The walks of the marked pairs: a wave takes a run of listed candidates,
// lists their marks (lane = word), and each 64 of them take a lane each: the
// density decides whether the pair is one, and a shared any-hit walk of the
// segments its bit.  Bounded to 7 waves per SIMD (a few words spill; 6 and 8
// measured up to 3% slower).
template <class LT, int R>
__global__ __launch_bounds__(kLBlock, 7) void walk_marked_kernel(DeviceBVH bvh, GBufView g, OccView occ, LT L,
                                                                 uint32_t *bits, const uint32_t *lists,
                                                                 uint32_t per_xcd, uint32_t few_step) {
    constexpr int D = 2 * R, SIDE = 4 * R + 1, NW = (SIDE * SIDE + 31) / 32;
    constexpr int kSelf = D * SIDE + D;
    constexpr float kInvSide = 1.0f / (float)SIDE;
    static_assert(kMarkRun * NW <= 64, "a lane per word");
    constexpr int kPairs = kMarkRun * SIDE * SIDE;
    __shared__ uint32_t s_stack[kLBlock / 64][kStackTotal];
    __shared__ uint16_t s_pair[kLBlock / 64][kPairs];
    __shared__ uint32_t s_bits[kLBlock / 64][kMarkRun * NW];
    __shared__ MarkCand s_cand[kLBlock / 64][kMarkRun];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint16_t *pairs = s_pair[wave];
    uint32_t *out = s_bits[wave];
    MarkCand *cands = s_cand[wave];
    uint32_t nfew = 0, nmany = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        nfew += lists[x * kCountStride];
        nmany += lists[x * kCountStride + 1];
    }
    const uint32_t per_many = min(max(nmany / kManyStep, 2u), (uint32_t)kMarkRun);
    const uint32_t per_few = min(max(nfew / few_step, 1u), (uint32_t)kMarkRun);
    const uint32_t few_runs = (nfew + per_few - 1) / per_few, many_runs = (nmany + per_many - 1) / per_many;
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t stride = (gridDim.x / 8) * (kLBlock / 64);
    const int b = lane / NW, wi = lane - b * NW;  // this lane's word of the run
    // first the candidates of many marks, whose runs take longest, then the others
    bool many = true;
    uint32_t u = (blockIdx.x >> 3) * (kLBlock / 64) + wave;
    for (;; u += stride) {
        // runs in blocks, dealt to the XCDs in turn
        const uint32_t nruns = many ? many_runs : few_runs, blk = many && per_many == 2u ? 4u : 64u;
        const uint32_t r0 = (u / blk) * (8u * blk), ri = r0 + xcd * blk + (u % blk);
        if (ri >= nruns) {
            if (r0 >= nruns) {
                if (!many) break;
                many = false;
                u = (blockIdx.x >> 3) * (kLBlock / 64) + wave - stride;
            }
            continue;
        }
        const uint32_t per = many ? per_many : per_few, all = many ? nmany : nfew;
        const uint32_t c0 = ri * per;
        const int nrun = (int)min(per, all - c0);
        uint32_t j = 0;
        if (lane < nrun) {
            // candidate c0 + lane of the 8 lists taken one after the other
            uint32_t off = c0 + (uint32_t)lane, base = 8 * kCountStride;
#pragma unroll
            for (int x = 0; x < 7; ++x) {
                const uint32_t n = lists[x * kCountStride + (many ? 1 : 0)];
                if (off < n) break;
                off -= n;
                base += per_xcd;
            }
            j = lists[many ? base + per_xcd - 1u - off : base + off];
            MarkCand &c = cands[lane];
            float x[3], n[3], o[3], v[3];
            load3(g.pos, j, x);
            load3(g.nrm, j, n);
            offset_point(x, n, o);
            for (int a = 0; a < 3; ++a) c.oj[a] = o[a];
            load3(occ.dz, j, v);
            for (int a = 0; a < 3; ++a) c.dzj[a] = v[a];
            load3(occ.nz, j, v);
            for (int a = 0; a < 3; ++a) c.nzj[a] = v[a];
            c.hj = occ.hit[j];
            c.jy = (int)(j / (uint32_t)g.w);
            c.jx = (int)j - c.jy * g.w;
        }
        const bool word = b < nrun;
        const int64_t at_word = (int64_t)(uint32_t)__shfl((int)j, word ? b : 0) * NW + wi;
        const uint32_t marks = word ? bits[at_word] : 0u;
        const int n = __popc(marks), incl = wave_incl_scan(n);
        int count = __builtin_amdgcn_readlane(incl, 63);
        if (word) out[lane] = wi == (kSelf >> 5) ? 1u << (kSelf & 31) : 0u;
        int at = incl - n;
        for (uint32_t v = marks; v != 0u; v &= v - 1u) pairs[at++] = (uint16_t)((b << 8) | (32 * wi + __builtin_ctz(v)));
        wave_sync();
        // the listed pair of a lane: receiver, w and whether its density is positive
        auto pair_of = [&](int idx, int &own, int &q, uint32_t &primk, float ok[3], float wv[3], bool sure) -> bool {
            own = q = 0;
            if (idx >= count) return false;
            const uint32_t e = pairs[idx];
            own = (int)(e >> 8);
            q = (int)(e & 255u);
            const MarkCand &c = cands[own];
            int64_t k;
            float nk[3];
            if (!pair_receiver(g, c.jx, c.jy, SIDE, kInvSide, D, q, k, primk, ok, nk)) return false;
            rel_vec(c.oj, ok, c.dzj, wv);
            return sure || dens_light(wv, nk, recv_of(ok, L), c.nzj, L) > 0.0f;
        };
        // more than a walk holds: the pairs with a positive density first
        const bool sure = count > 64;
        if (sure) {
            int kept = 0;
            for (int e0 = 0; e0 < count; e0 += 64) {
                int own, q;
                uint32_t primk;
                float ok[3], wv[3];
                const bool keep = pair_of(e0 + lane, own, q, primk, ok, wv, false);
                const unsigned long long m = wave_ballot(keep);
                wave_sync();  // read before they are overwritten
                if (keep)
                    pairs[kept + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                        (uint16_t)((own << 8) | q);
                kept += (int)__popcll(m);
            }
            count = kept;
            wave_sync();
        }
        for (int e0 = 0; e0 < count; e0 += 64) {
            TRay ray;
            ray.ign0 = ray.ign1 = OCR_HIT_MISS;
            int own, q;
            uint32_t primk;
            float ok[3], wv[3];
            const bool want = pair_of(e0 + lane, own, q, primk, ok, wv, sure);
            if (want) make_ray(ok, wv, cands[own].hj, primk, 1.0f - 1e-4f, ray);
            const bool blocked = traverse_wave_any(bvh, ray, 1.0f - 1e-4f, want, s_stack[wave]);
            if (want && !blocked) atomicOr(&out[own * NW + (q >> 5)], 1u << (q & 31));
        }
        wave_sync();
        if (word) bits[at_word] = out[lane];
        wave_sync();  // read before the next run refills it
    }
}

template <class LT>
static hipError_t launch_t(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, const LT &L, int nl, int radius,
                           uint32_t *bits, uint32_t *lists, uint32_t per_xcd, hipStream_t st) {
    const int tiles_x = (g.w + kLTile - 1) / kLTile, nt = tiles_x * ((g.h + kLTile - 1) / kLTile);
    const int per = (nt + 7) / 8;
    const dim3 grid(8 * ((per + kLTileRun - 1) / kLTileRun) * kLTileRun), block(kLBlock);
    const size_t lds = (size_t)nl * 3 * sizeof(float) * light_cells(radius);
    const uint32_t few_step = bvh.ntris >= kSmallMesh ? kFewStep : kFewStepSmall;
    // (no more than the frame's pixels could fill)
    const int blocks = min(12288, 8 * (per + 1));
#define OCR_VL(R_)                                                                                       \
    do {                                                                                                          \
        hipLaunchKernelGGL((mark_pairs_kernel<LT, R_>), grid, block, lds, st, g, occ, L, bits, lists, per_xcd,     \
                           tiles_x, nt);                                                                          \
        hipLaunchKernelGGL((walk_marked_kernel<LT, R_>), dim3(blocks), block, 0, st, bvh, g, occ, L, bits,    \
                           lists, per_xcd, few_step);                                                                       \
    } while (0)
    if (radius == 1) OCR_VL(1);
    else if (radius == 2) OCR_VL(2);
    else OCR_VL(3);
#undef OCR_VL
    return hipGetLastError();
}

hipError_t launch_validate_light(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, const LightF &L, int radius,
                                 uint32_t *bits, uint32_t *lists, uint32_t per_xcd, hipStream_t st) {
    return launch_t(bvh, g, occ, L, 1, radius, bits, lists, per_xcd, st);
}
hipError_t launch_validate_light(const DeviceBVH &bvh, const GBufView &g, const OccView &occ, const LightSetF &L, int radius,
                                 uint32_t *bits, uint32_t *lists, uint32_t per_xcd, hipStream_t st) {
    return launch_t(bvh, g, occ, L, L.n, radius, bits, lists, per_xcd, st);
}

}  // namespace ocr
