// Front-to-back alpha compositing of surfels per tile, its recompute-based
// backward, and the occlusion statistics of the pruning pass.
//
// Section 4.3: a pixel blends its assigned Gaussians front to back,
// accumulating colour and opacity, and stops once the accumulated opacity
// reaches a threshold close to one or the list is exhausted; a Gaussian that
// takes part in the blending of a pixel is "used" (visible).  Section 4.2
// (Eq. 1) consumes the accumulated alpha; Eq. 3's 2DGS regularisers consume
// depth, normal and distortion.
//
// One workgroup per (view, tile) over all views of the batch in a single
// launch; one thread per pixel; the entries of a tile are gathered in batches
// in LDS, their records read per wave from LDS or through the scalar cache
// (EntryRec); every pair is evaluated with the shared
// eval_test()/eval_finish() so that forward, backward and pruning take identical
// decisions.
#include <mutex>

#include <type_traits>

#include "common.h"
#include "launch.h"

namespace sr {

namespace {

constexpr int kWaveBlock = 8;   // side of the square block of pixels one wave covers

// Square root and reciprocal for the culling bounds: the hardware estimates
// refined by one Newton step, far more accurate than the culling's 1e-3
// margins need and a fraction of the instructions of the correctly rounded
// operations.  x >= 0 for the root: below 1e-300 it is taken as 0 (an error
// under 1e-150 px), an infinite x stays infinite; the reciprocal is taken of
// positive normal numbers.
__device__ __forceinline__ double cull_sqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);                 // 1/sqrt(x), refined as y (3 - x y^2) / 2
    const double r = x * (y * (1.5 - 0.5 * x * y * y));
    return x > 1e-300 ? (x <= 1.7e308 ? r : x) : 0.0;
}
__device__ __forceinline__ double cull_rcp(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return r * (2.0 - x * r);
}

// Global tile id of this workgroup; pixel coordinates of this thread; the
// run [start, start + n) of the tile's binning group.
struct TileCtx {
    int tile, v, W, H, ix, iy;
    int tx0, ty0;    // first pixel column and row of the tile
    int sx, sy;      // tile coordinates inside its binning group
    bool inside;
    int64_t pix_off;
    uint32_t start;
    int n;           // runs hold at most one entry per surfel of the view: below 2^SR_INST_ID_BITS
    float bg[3];
};

template <int TW, int TH>
// order (optional): the tile of each workgroup, a permutation of the tile ids
// (heaviest first); an id beyond the grid marks the workgroup idle
// (t.n = 0, nothing inside).
__device__ __forceinline__ void tile_ctx(const sr_camera* __restrict__ cams, int V,
                                         const uint2* __restrict__ ranges, TileCtx& t,
                                         const uint32_t* __restrict__ order = nullptr) {
    int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    bool idle = false;
    if (order) {
        const uint32_t o = order[blockIdx.x];
        idle = o >= gridDim.x;
        tile = idle ? 0 : (int)o;
    }
    t.tile = tile;
    t.v = view_of_tile(cams, V, tile);
    const sr_camera& c = cams[t.v];
    const int local = tile - c.tile_offset;
    const int ty = local / c.tiles_x, tx = local - ty * c.tiles_x;
    t.W = c.width;
    t.H = c.height;
    // wave w covers the 8x8 block (w % (TW / 8), w / (TW / 8)) of the tile
    constexpr int WB = kWaveBlock;
    const int w = (int)threadIdx.x >> 6, l = (int)threadIdx.x & 63;
    t.ix = tx * TW + (w % (TW / WB)) * WB + (l % WB);
    t.iy = ty * TH + (w / (TW / WB)) * WB + l / WB;
    t.tx0 = tx * TW;
    t.ty0 = ty * TH;
    t.sx = tx % SR_TILE_GROUP;
    t.sy = ty % SR_TILE_GROUP;
    t.inside = !idle && t.ix < t.W && t.iy < t.H;
    t.pix_off = c.pix_offset;
    t.bg[0] = c.bg[0]; t.bg[1] = c.bg[1]; t.bg[2] = c.bg[2];
    const uint2 rg = ranges[tile];
    t.start = rg.x;
    t.n = idle ? 0 : (int)(rg.y - rg.x);
}

constexpr int kMaxWaves = 8;    // waves per workgroup (tiles of up to 512 pixels)

// Waves per SIMD the kernels are compiled for (the register budget: 96 VGPRs
// at five, 80 at six, 72 at seven).  The walks themselves fit all three; the
// float64 culling bounds of the staging spill a few registers below 96, once
// per staged entry.  Measured with scalar records (compositing kernel; 1M
// surfels x 16 views / 3M x 8 / one 800x800 view of 100k): training step 6.64 /
// 5.47 / 0.372 ms at five, 6.13 / 5.13 / 0.369 at six, 5.93 / 4.97 / 0.381 at
// seven; backward with the depth terms of four 1559x1039 views 2.33 / 2.29 ms
// but 0.42 / 0.45 on one 800x600 view; the pruning pass of 100 views 50.5 /
// 50.5 / 49.7 ms.  With records in LDS (the forward, and where tiles are few)
// four and five measure the same.
#define SR_OCCUPANCY(waves) __attribute__((amdgpu_waves_per_eu(waves)))
constexpr int kPruneWaves = 7, kBwdWaves = 5, kTrainWaves = 6, kLdsWaves = 5, kAheadWaves = 4;

// MODE bits: 1 shade (colour, depth, normal, distortion outputs), 2 occlusion
// statistics, 4 count reached/blended pairs (work accounting), 8 median depth
// (the 2DGS surface depth: the depth of the last blended entry that starts
// with transmittance above 1/2) with the 1-based list index of that entry,
// 16 pixel rectangles read from the rectangle array (statistics without
// shading: no appearance records to take them from).
constexpr int kShade = 1, kStats = 2, kCount = 4, kMedian = 8, kRect = 16, kHits = 32;

// Per-wave culling.  Every wave of a tile covers an 8x8 block of its pixels
// (wave w: block column w % (TW / 8), block row w / (TW / 8)); a square
// footprint has the shortest boundary for its 64 pixels, so fewer of a
// wave's lanes sit outside the splats it works through than with a strip of
// rows.  When an entry is staged, its thread works out which blocks it can
// reach, one bit per wave; each wave then tests 64 staged entries at once
// with one ballot of its bit and walks only the set bits of that mask, so
// skipped entries cost no per-entry instructions.  A block is reached when
// the entry's pixel rectangle (packed in the last two slots of the appearance
// record) meets it and the y-range, within the block's columns that the
// rectangle meets, of the entry's cutoff conic or of its low-pass disc meets
// the block's rows:
//   surface  Q = (1 - tau)(w0^2 + w1^2) - 2 L (1 + tau) w2^2 <= 0 with
//            w = A dx + B dy + C' (the pass test of eval_test with a relative
//            slack tau): for an ellipse, Q(x, .) <= 0 is the interval between
//            the roots of a quadratic in y, whose lower end is convex and
//            upper end concave in x, so their extremes over the columns are
//            at the ellipse's lowest and highest points clamped to the
//            columns; any other conic reaches every block;
//   disc     dx^2 + dy^2 <= L (1 + tau).
// Float64, with a 1e-3 pixel margin on the columns and rows: an entry is
// skipped only where the exact test fails by a relative margin, and forward
// and backward skip the same entries.
template <int TW, int NW>
__device__ __forceinline__ uint32_t wave_bits(const float4& g0, const float4& g1, const float4& g2, float Lf,
                                              uint2 rr, int tx0, int ty0) {
    constexpr int WB = kWaveBlock;
    static_assert(TW % WB == 0 && NW % (TW / WB) == 0, "waves cover whole 8x8 blocks of the tile");
    constexpr int BX = TW / WB, BY = NW / BX;     // blocks per tile row and column
    constexpr double tau = 1e-3, mg = 1e-3;
    const uint32_t rx = rr.x, ry = rr.y;     // x_lo | x_hi << 16, y_lo | y_hi << 16
    const int ilo = (int)(rx & 0xffffu), ihi = (int)(rx >> 16), jlo = (int)(ry & 0xffffu), jhi = (int)(ry >> 16);
    const double cx = g2.y, cy = g2.z, L = Lf;
    // the conic's coefficients, independent of the columns
    const double s01 = 1.0 - tau, s2 = -2.0 * L * (1.0 + tau);
    const double a0 = g0.x, a1x = g0.y, a2 = g0.z, b0 = g0.w, b1 = g1.x, b2 = g1.y, c0 = g1.z, c1 = g1.w,
                 c2 = g2.x;
    // Q = P x^2 + 2 R x y + S y^2 + 2 U x + 2 W y + K
    const double P = s01 * (a0 * a0 + a1x * a1x) + s2 * (a2 * a2);
    const double R = s01 * (a0 * b0 + a1x * b1) + s2 * (a2 * b2);
    const double S = s01 * (b0 * b0 + b1 * b1) + s2 * (b2 * b2);
    const double U = s01 * (a0 * c0 + a1x * c1) + s2 * (a2 * c2);
    const double W = s01 * (b0 * c0 + b1 * c1) + s2 * (b2 * c2);
    const double K = s01 * (c0 * c0 + c1 * c1) + s2 * (c2 * c2);
    const double al = P * S - R * R;
    const bool ellipse = P > 0.0 && S > 0.0 && al > 0.0;
    // discriminant in y of Q(x, .): D(x) = -al x^2 + 2 be x + ga, >= 0 on the ellipse's columns
    const double be = R * W - S * U, ga = W * W - S * K;
    const double ex = be * be + al * ga;
    // the ellipse's columns [xl, xr] (empty unless ex >= 0) and the x of its
    // lowest and highest points (on P x + R y + U = 0, y roots of the
    // discriminant in x)
    double xl = 1.0, xr = -1.0, xb0 = 0.0, xt0 = 0.0, iS = 0.0;
    if (ellipse && ex >= 0.0) {
        const double ia = cull_rcp(al), sx = cull_sqrt(ex);
        xl = (be - sx) * ia;
        xr = (be + sx) * ia;
        const double bp = R * U - P * W, gp = U * U - P * K;
        const double sy = cull_sqrt(fmax(bp * bp + al * gp, 0.0));
        const double iP = cull_rcp(P);
        iS = cull_rcp(S);
        xb0 = -(R * ((bp - sy) * ia) + U) * iP;
        xt0 = -(R * ((bp + sy) * ia) + U) * iP;
    }
    uint32_t bits = 0u;
#pragma unroll 1
    for (int bx = 0; bx < BX; ++bx) {
        const int k0 = tx0 + bx * WB, k1 = k0 + WB - 1;
        const int clo = ilo > k0 ? ilo : k0, chi = ihi < k1 ? ihi : k1;
        if (clo > chi) continue;
        const double X0 = (clo + 0.5) - cx - mg, X1 = (chi + 0.5) - cx + mg;
        // disc: |dy| <= hd
        const double xd = fmin(fmax(0.0, X0), X1);
        const double hd2 = L * (1.0 + tau) - xd * xd;
        const double hd = hd2 >= 0.0 ? cull_sqrt(hd2) : -1.0;
        // surface: y-range [ylo, yhi] over these columns (empty when ylo > yhi)
        double ylo = -1e300, yhi = 1e300;
        if (ellipse) {
            ylo = 1.0;
            yhi = -1.0;
            const double xa = fmax(X0, xl), xb = fmin(X1, xr);
            if (xa <= xb) {
                const double xbot = fmin(fmax(xb0, xa), xb);
                const double xtop = fmin(fmax(xt0, xa), xb);
                const double db = fmax((-al * xbot + 2.0 * be) * xbot + ga, 0.0);
                const double dt = fmax((-al * xtop + 2.0 * be) * xtop + ga, 0.0);
                ylo = (-(R * xbot + W) - cull_sqrt(db)) * iS;
                yhi = (-(R * xtop + W) + cull_sqrt(dt)) * iS;
            }
        }
#pragma unroll
        for (int by = 0; by < BY; ++by) {
            const int r0 = ty0 + by * WB, r1 = r0 + WB - 1;
            const int lo = jlo > r0 ? jlo : r0, hi = jhi < r1 ? jhi : r1;
            if (lo > hi) continue;
            const double Y0 = (lo + 0.5) - cy - mg, Y1 = (hi + 0.5) - cy + mg;
            const bool disc = hd >= 0.0 && Y0 <= hd && Y1 >= -hd;
            const bool surf = ylo <= Y1 && yhi >= Y0;
            if (disc || surf) bits |= 1u << (by * BX + bx);
        }
    }
    return bits;
}

// A staged entry's record, read by the whole wave (the wave's entry is
// uniform), from one of two places:
//
// SCALAR: through the scalar cache into scalar registers, 18 to 24 words in
//   two or three loads, fetched one entry ahead.  Read as broadcasts from LDS
//   (six 16-byte reads) the records kept the LDS unit busy for two thirds of
//   the kernel's time.  (The price: an instruction with a scalar operand issues
//   at little over half the rate.)  A vector instruction takes one, so the
//   addends C, which meet a second one, come from LDS (staged in c, with
//   twice the cutoff in the fourth slot).
// else: broadcasts from LDS.  Where the launch holds few waves, nothing hides
//   a scalar load that misses its cache, and a wave's own latency per entry is
//   the kernel's time; the LDS unit is then idle.  The forward with outputs
//   measures faster so at every size.
//
// The rule is on the waves of the launch (scalar_records).
typedef float F16v __attribute__((ext_vector_type(16)));
typedef float F4v __attribute__((ext_vector_type(4)));
typedef float F2v __attribute__((ext_vector_type(2)));
template <typename T>
using ConstMem = const T __attribute__((address_space(4)));

template <bool SCALAR, int NB, bool APP>
struct RecStage;
template <int NB, bool APP>
struct RecStage<true, NB, APP> {
    float4 c[NB];                 // C0, C1, C2, 2 L
    __device__ __forceinline__ void put(int k, const float4 (&g)[kGeomF4], const float4*) {
        c[k] = make_float4(g[1].z, g[1].w, g[2].x, 2.0f * g[3].w);
    }
};
template <int NB, bool APP>
struct RecStage<false, NB, APP> {
    float4 g[kGeomF4][NB];
    float4 a[APP ? kAppF4 : 1][APP ? NB : 1];
    __device__ __forceinline__ void put(int k, const float4 (&gq)[kGeomF4], const float4* app) {
#pragma unroll
        for (int q = 0; q < kGeomF4; ++q) g[q][k] = gq[q];
        if (APP) {
            a[0][k] = app[0];
            a[1][k] = app[1];
        }
    }
};

struct EntryRec {
    F16v g;
    F4v a0;     // colour, normal x
    F2v a1;     // normal y, z
    float4 c;   // SCALAR: C0, C1, C2, 2 L
};

// geom_v, app_v: the view's records; g: uniform surfel id.
template <bool APP, bool NORMAL>
__device__ __forceinline__ void load_scalar(const float4* __restrict__ geom_v, const float4* __restrict__ app_v,
                                            uint32_t g, EntryRec& r) {
    r.g = *(ConstMem<F16v>*)(uintptr_t)((const char*)geom_v + (size_t)(g * (uint32_t)(16 * kGeomF4)));
    if (APP) {
        const char* a = (const char*)app_v + (size_t)(g * (uint32_t)(16 * kAppF4));
        r.a0 = *(ConstMem<F4v>*)(uintptr_t)a;
        if (NORMAL) r.a1 = *(ConstMem<F2v>*)(uintptr_t)(a + 16);
    }
}

// The parts of a staged record that eval_test reads, and the rest.
template <typename Stage>
__device__ __forceinline__ void load_lds_test(const Stage& st, int k, EntryRec& r) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float4 v = st.g[q][k];
        r.g[4 * q] = v.x;
        r.g[4 * q + 1] = v.y;
        r.g[4 * q + 2] = v.z;
        r.g[4 * q + 3] = v.w;
    }
    r.g[8] = st.g[2][k].x;
    r.g[9] = st.g[2][k].y;
    r.g[10] = st.g[2][k].z;
    r.g[15] = st.g[3][k].w;
}

template <bool APP, typename Stage>
__device__ __forceinline__ void load_lds_rest(const Stage& st, int k, EntryRec& r) {
    r.g[11] = st.g[2][k].w;
    r.g[12] = st.g[3][k].x;
    r.g[13] = st.g[3][k].y;
    r.g[14] = st.g[3][k].z;
    if (APP) {
        const float4 a0 = st.a[0][k];
        const float2 a1 = *reinterpret_cast<const float2*>(&st.a[1][k]);
        r.a0 = F4v{a0.x, a0.y, a0.z, a0.w};
        r.a1 = F2v{a1.x, a1.y};
    }
}

template <bool SCALAR>
__device__ __forceinline__ SurfelGeom geom_of(const EntryRec& r) {
    return SurfelGeom{r.g[0],  r.g[1],  r.g[2],  r.g[3],  r.g[4],  r.g[5],
                      SCALAR ? r.c.x : r.g[6], SCALAR ? r.c.y : r.g[7], SCALAR ? r.c.z : r.g[8],
                      r.g[9],  r.g[10], r.g[11], r.g[12], r.g[13], r.g[14], r.g[15],
                      SCALAR ? r.c.w : 2.0f * r.g[15]};
}

// Staged entries: the surfel id with the wave bits above it (ids hold
// SR_INST_ID_BITS bits), and the run position.
static_assert(SR_INST_ID_BITS + 4 <= 32, "wave bits above the surfel id");

// This wave's index in its workgroup.
__device__ __forceinline__ int wave_index() { return (int)__builtin_amdgcn_readfirstlane(threadIdx.x) >> 6; }

// Wave bits of the staged entries kept from the forward to the backward of
// the fused step (LDS, 4 bits per run position, 16 bytes per thread of the
// workgroup: positions below 32 per thread; the backward recomputes the bits
// of later positions).  The backward stages only positions the forward
// staged (below the largest last contributor), so every cached position it
// reads was written.
template <int NT>
struct BitCache {
    static constexpr int kWords = 4 * NT;
    static constexpr uint32_t kPos = 8u * kWords;
};

template <int NT>
__device__ __forceinline__ void bitcache_put(uint32_t* c, uint32_t jpos, uint32_t bits) {
    if (jpos < BitCache<NT>::kPos) atomicOr(&c[jpos >> 3], bits << ((jpos & 7u) << 2));
}

// Per-pixel state at the end of the forward pass.
struct PixFwd {
    float T, C0, C1, C2, N0, N1, N2, S0, S1, S2, zref, zmed;
    uint32_t last, kmed;
};

// LDS staging of the forward: NT entries per batch.
template <int NT, int MODE, bool SCALAR>
struct FwdSmem {
    RecStage<SCALAR, NT, (MODE & kShade) != 0> rec;
    uint32_t id[NT];          // surfel id | wave bits << SR_INST_ID_BITS
    uint32_t pos[NT];         // list index: run position + 1
    // occlusion statistics of the batch's entries over the workgroup's waves
    // (hits, then with kStats the max alpha and max weight bits), added to
    // the global ones once per (tile, entry) at the end of the batch
    uint32_t st[(MODE & kStats) ? 3 : 1][(MODE & (kStats | kHits)) ? NT : 1];
    uint32_t wcnt[NT / 64 + 1];   // gathering: members per wave, then the resume position
    uint32_t alive[NT / 64];      // waves with a pixel that has not terminated
};

// LDS staging and per-record accumulators of the backward.  acc[k] holds the
// sums over the workgroup's pixels of entry k (wave_contract); the padding to an
// odd stride keeps the per-thread reads of the flush free of bank conflicts.
template <int NT, int BATCH, bool GEO, bool HITS, bool SCALAR>
struct BwdSmem {
    static constexpr int kAcc = GEO ? 23 : 17;
    RecStage<SCALAR, BATCH, true> rec;
    uint32_t id[BATCH];           // surfel id | wave bits << SR_INST_ID_BITS
    uint32_t pos[BATCH];          // run position
    float4 xp[NT];                // transposition scratch, 64 slots per wave
    float acc[BATCH][kAcc];
    uint32_t hit[HITS ? BATCH : 1];
    uint64_t touched[(BATCH + 63) / 64];     // entries some pixel of the tile blends
    uint32_t maxn;
    uint32_t wcnt[kMaxWaves + 1];
};

// Gathering of a batch from the tile's group run: the NT threads examine NT
// run positions at once, keep the entries whose sub-rectangle covers the
// tile, and place them in consecutive batch slots by a block-wide rank
// (wave ballots, per-wave counts in LDS).  With ASC the slots [fill, cap)
// receive the members of [pos, pos + NT) in run order; otherwise slots
// (cap - 1 - fill) downwards receive the members of [pos - NT, pos), highest
// position first.  A round that overfills the batch stops after the last
// member placed and reports where the next batch resumes.  Returns the
// number of members placed in this round; block-uniform.
template <int NT, bool ASC>
__device__ __forceinline__ int gather_round(const TileCtx& t, const uint32_t* __restrict__ vals, int pos,
                                            int fill, int cap, uint32_t* __restrict__ id, uint32_t* __restrict__ rpos,
                                            uint32_t* wcnt, int& next) {
    const int tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const int j = ASC ? pos + tid : pos - NT + tid;
    const bool in = ASC ? j < t.n : j >= 0;
    const uint32_t gv = in ? vals[t.start + (uint32_t)j] : 0u;
    const bool mem = in && inst_covers(gv, t.sx, t.sy);
    const uint64_t bm = ballot64(mem);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (lane == 0) wcnt[w] = (uint32_t)__popcll(bm);
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        const int c = (int)wcnt[i];
        before += i < w ? c : 0;
        tot += c;
    }
    const int r_asc = before + __popcll(bm & lt);
    const int rank = ASC ? r_asc : tot - 1 - r_asc;          // order of placement
    const int taken = fill + rank;
    if (mem && taken < cap) {
        const int slot = ASC ? taken : cap - 1 - taken;
        id[slot] = gv;
        rpos[slot] = (uint32_t)j;
        if (taken == cap - 1 && fill + tot > cap) wcnt[NT / 64] = (uint32_t)(ASC ? j + 1 : j);
    }
    __syncthreads();
    if (fill + tot <= cap) {
        next = ASC ? pos + NT : (pos - NT > 0 ? pos - NT : 0);
    } else {
        next = (int)wcnt[NT / 64];
        tot = cap - fill;
    }
    __syncthreads();                                          // wcnt is reused by the next round
    // uniform, and known to be: the batch loops stay scalar
    next = __builtin_amdgcn_readfirstlane(next);
    return __builtin_amdgcn_readfirstlane(tot);
}

// Front to back over the tile list; every thread owns one pixel.
template <int TW, int NT, int MODE, bool SCALAR>
__device__ __forceinline__ void fwd_tile(const TileCtx& t, float px, float py, int N, const float4* __restrict__ geom,
                                         const float4* __restrict__ app, const uint2* __restrict__ rect,
                                         const uint32_t* __restrict__ vals, const RasterConsts& rc,
                                         FwdSmem<NT, MODE, SCALAR>& sm, PixFwd& st,
                                         uint32_t* __restrict__ hits, float* __restrict__ max_alpha,
                                         float* __restrict__ max_weight, uint64_t& n_reached, uint64_t& n_blended,
                                         uint64_t& n_witer, uint64_t& n_wblend, uint64_t& n_upto_last,
                                         uint32_t* bitcache = nullptr) {
    static_assert(NT / 64 <= 4, "four wave bits per cached entry");
    constexpr bool SHADE = (MODE & kShade) != 0;
    constexpr bool STATS = (MODE & kStats) != 0;              // hits and the two maxima
    constexpr bool HITS = STATS || (MODE & kHits) != 0;       // hits (blended pixels per surfel)
    constexpr bool COUNT = (MODE & kCount) != 0;
    constexpr bool MEDIAN = (MODE & kMedian) != 0;
    // the pixel rectangles are staged (with the appearance records, or from
    // the rectangle array): cull per wave
    constexpr bool RECT = (MODE & kRect) != 0 && !SHADE && !COUNT;
    constexpr bool CULL = SHADE || COUNT || RECT;
    uint32_t n_eval = 0, n_eval_last = 0;     // COUNT: entries tested by this pixel, up to its last blend
    const int tid = threadIdx.x;
    const int lane = __lane_id();
    st.T = 1.0f;
    st.C0 = st.C1 = st.C2 = st.N0 = st.N1 = st.N2 = st.S0 = st.S1 = st.S2 = st.zref = st.zmed = 0.f;
    st.last = st.kmed = 0;
    uint64_t px_live = ballot64(t.inside);    // the wave's pixels inside the image that have not terminated
    constexpr bool PLAIN = !COUNT && !HITS;
    const int wv = wave_index();
    const float4* geom_v = geom + kGeomF4 * (size_t)t.v * N;
    const float4* app_v = SHADE || (CULL && !RECT) ? app + kAppF4 * (size_t)t.v * N : nullptr;
    // statistics of the previous batch's entries: every thread adds its own
    // slot to the global arrays (after a barrier), before the slot is reused
    int prev_cnt = 0;
    auto flush = [&]() {
        if (tid < prev_cnt && sm.st[0][tid] != 0u) {
            const uint32_t g = sm.id[tid] & kInstIdMask;
            atomicAdd(&hits[g], sm.st[0][tid]);
            if (STATS) {
                atomicMax((uint32_t*)&max_alpha[g], sm.st[1][tid]);
                atomicMax((uint32_t*)&max_weight[g], sm.st[2][tid]);
            }
        }
    };
    // batches of up to NT entries of the tile, gathered from its group's run
    int pos = 0;
    while (pos < t.n) {
        // (gathering's barriers lie between this read and the next write)
        if (lane == 0) sm.alive[wv] = px_live != 0ull ? 1u : 0u;
        __syncthreads();
        uint32_t alive = 0u;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) alive |= sm.alive[i];
        if (__builtin_amdgcn_readfirstlane(alive) == 0u) break;
        if (HITS) flush();
        int cnt = 0;
        while (cnt < NT && pos < t.n) {
            int next;
            cnt += gather_round<NT, true>(t, vals, pos, cnt, NT, sm.id, sm.pos, sm.wcnt, next);
            pos = next;
        }
        if (tid < cnt) {
            const uint32_t g = sm.id[tid] & kInstIdMask;
            const uint32_t jpos = sm.pos[tid];
            float4 gq[kGeomF4];
#pragma unroll
            for (int q = 0; q < kGeomF4; ++q) gq[q] = geom_v[kGeomF4 * (size_t)g + q];
            sm.rec.put(tid, gq, SHADE ? app_v + kAppF4 * (size_t)g : nullptr);
            uint32_t bits = (1u << (NT / 64)) - 1u;
            if (CULL) {
                // the pixel rectangle as two packed ranges: from the rectangle
                // array, or the last two slots of the appearance record
                const uint2 rr = RECT ? rect[(size_t)t.v * N + g]
                                      : reinterpret_cast<const uint2*>(app_v + kAppF4 * (size_t)g)[3];
                bits = wave_bits<TW, NT / 64>(gq[0], gq[1], gq[2], gq[3].w, rr, t.tx0, t.ty0);
                if (!RECT && bitcache) bitcache_put<NT>(bitcache, jpos, bits);
            }
            sm.id[tid] = g | (bits << SR_INST_ID_BITS);
            sm.pos[tid] = jpos + 1u;
            if (HITS) sm.st[0][tid] = 0u;
            if (STATS) {
                sm.st[1][tid] = 0u;
                sm.st[2][tid] = 0u;
            }
        }
        __syncthreads();
        bool wave_done = px_live == 0ull;
        for (int c = 0; c * 64 < cnt && !wave_done; ++c) {
          const int slot = c * 64 + lane;
          const uint32_t my_id = slot < cnt ? sm.id[slot] : 0u, my_pos = sm.pos[slot];
          uint64_t live = ballot64((my_id >> (SR_INST_ID_BITS + wv)) & 1u);
          if (live == 0ull) continue;
          // SCALAR: the records of the wave's entries, one ahead of the evaluation
          int nbit = (int)__builtin_ctzll(live);
          EntryRec next_rec;
          if constexpr (SCALAR) {
            load_scalar<SHADE, SHADE>(geom_v, app_v, __builtin_amdgcn_readlane(my_id, nbit) & kInstIdMask, next_rec);
            next_rec.c = sm.rec.c[c * 64 + nbit];
          }
          // HITS: this wave's blended pixels of entry c * 64 + lane
          uint32_t my_hits = 0;
          while (live != 0ull) {
            const int bit = nbit, k = c * 64 + bit;
            EntryRec rec = next_rec;
            live &= live - 1ull;
            nbit = live != 0ull ? (int)__builtin_ctzll(live) : bit;
            const uint32_t jidx = __builtin_amdgcn_readlane(my_pos, bit);    // run position + 1
            if constexpr (SCALAR) {
                load_scalar<SHADE, SHADE>(geom_v, app_v, __builtin_amdgcn_readlane(my_id, nbit) & kInstIdMask, next_rec);
            } else {
                load_lds_test(sm.rec, k, rec);
                load_lds_rest<SHADE>(sm.rec, k, rec);
            }
            const SurfelGeom sg = geom_of<SCALAR>(rec);
            PairEval e;
            eval_test<SCALAR>(sg, px, py, e);
            // behind the last use of this entry's: the same registers
            if constexpr (SCALAR) next_rec.c = sm.rec.c[c * 64 + nbit];
            // blends entry k into the pixel state (before the transmittance update)
            auto accumulate = [&](float wgt) {
                // the depth reference of the distortion sums is the depth of
                // the pixel's first blended entry: T is exactly 1 until then
                // (every blended alpha is at least alpha_min)
                st.zref = st.T == 1.0f ? e.z : st.zref;
                const float zs = e.z - st.zref;
                if (SHADE) {
                    st.C0 = __builtin_fmaf(wgt, rec.a0.x, st.C0);
                    st.C1 = __builtin_fmaf(wgt, rec.a0.y, st.C1);
                    st.C2 = __builtin_fmaf(wgt, rec.a0.z, st.C2);
                    st.N0 = __builtin_fmaf(wgt, rec.a0.w, st.N0);
                    st.N1 = __builtin_fmaf(wgt, rec.a1.x, st.N1);
                    st.N2 = __builtin_fmaf(wgt, rec.a1.y, st.N2);
                }
                st.S0 += wgt;
                st.S1 = __builtin_fmaf(wgt, zs, st.S1);
                st.S2 = __builtin_fmaf(wgt * zs, zs, st.S2);
                if (MEDIAN && st.T > 0.5f) {         // T before this entry
                    st.zmed = e.z;
                    st.kmed = jidx;
                }
                st.last = jidx;
            };
            if (PLAIN) {
                // no per-wave bookkeeping: the lanes that do not blend skip the
                // block, and the wave skips it when none does
                float Tn = st.T;
                if (in_mask(pass_mask(e) & px_live)) {
                    eval_finish(sg, rc.alpha_max, e);
                    Tn = st.T * (1.0f - e.a);
                    if (!(Tn < rc.t_min)) accumulate(e.a * st.T);
                }
                const uint64_t ended = ballot64(Tn < rc.t_min);
                if (ended != 0ull) {
                    Tn = in_mask(ended) ? st.T : Tn;
                    px_live &= ~ended;
                }
                st.T = Tn;
                if (px_live == 0ull) {
                    wave_done = true;
                    break;
                }
                continue;
            }
            if (COUNT) {
                n_reached += (uint64_t)__popcll(px_live);
                n_witer += 1;
                n_eval += in_mask(px_live) ? 1u : 0u;
            }
            uint64_t bm = pass_mask(e) & px_live;
            // no pixel of this wave takes the entry: nothing changes
            if (bm == 0ull) continue;
            if (COUNT) n_wblend += 1;
            eval_finish(sg, rc.alpha_max, e);
            const float Tn = st.T * (1.0f - e.a);
            const uint64_t ended = bm & ballot64(Tn < rc.t_min);
            px_live &= ~ended;
            bm &= ~ended;
            const bool blend = in_mask(bm);
            float wgt = 0.f;
            if (blend) {
                wgt = e.a * st.T;
                accumulate(wgt);
                st.T = Tn;
                if (COUNT) n_eval_last = n_eval;
            }
            if (COUNT) n_blended += (uint64_t)__popcll(bm);
            if (HITS) {
                if (bm != 0ull) {
                    my_hits = (uint32_t)lane_write((int)__popcll(bm), bit, (int)my_hits);
                    if (STATS) {
                        // lane 0 holds the wave's max alpha, lane 32 its max weight
                        const uint32_t mx = wave_max2_bits(blend ? e.a : 0.f, wgt);
                        if ((lane & 31) == 0) atomicMax(&sm.st[lane == 0 ? 1 : 2][k], mx);
                    }
                }
            }
            if (px_live == 0ull) {
                wave_done = true;
                break;
            }
          }
          if (HITS && my_hits != 0u) atomicAdd(&sm.st[0][c * 64 + lane], my_hits);
        }
        prev_cnt = cnt;
    }
    if (HITS) {
        __syncthreads();
        flush();
    }
    if (COUNT) n_upto_last += n_eval_last;
}

// The final state of a pixel of a tile that computed nothing because the
// status word was set: every output NaN, no blended entry.
__device__ __forceinline__ void poison(PixFwd& st) {
    const float q = __builtin_nanf("");
    st.T = st.C0 = st.C1 = st.C2 = st.N0 = st.N1 = st.N2 = st.S0 = st.S1 = st.S2 = st.zref = st.zmed = q;
    st.last = st.kmed = 0u;
}

// Forward outputs of one pixel from its final state.
struct PixOut {
    float C0, C1, C2, A, D, Dist;
};

__device__ __forceinline__ PixOut pix_outputs(const PixFwd& st, const TileCtx& t) {
#pragma clang fp contract(off)
    PixOut o;
    o.C0 = st.C0 + st.T * t.bg[0];
    o.C1 = st.C1 + st.T * t.bg[1];
    o.C2 = st.C2 + st.T * t.bg[2];
    o.A = 1.0f - st.T;
    // depth = sum w z = S1 + zref S0 ; dist = 2 (S0 S2 - S1^2) with z shifted by zref
    o.D = __builtin_fmaf(st.zref, st.S0, st.S1);
    const float dd = 2.0f * (st.S0 * st.S2 - st.S1 * st.S1);
    o.Dist = (dd > 0.f || dd != dd) ? dd : 0.f;      // a NaN state stays NaN
    return o;
}

__device__ __forceinline__ void write_outputs(const PixFwd& st, const PixOut& o, const TileCtx& t,
                                              float* __restrict__ color, float* __restrict__ alpha,
                                              float* __restrict__ depth, float* __restrict__ normal,
                                              float* __restrict__ dist, float* __restrict__ T_final,
                                              uint32_t* __restrict__ n_contrib) {
    const int64_t HW = (int64_t)t.W * t.H;
    const int64_t p = (int64_t)t.iy * t.W + t.ix;
    const int64_t o1 = t.pix_off + p;
    const int64_t o3 = 3 * t.pix_off + p;
    color[o3] = o.C0;
    color[o3 + HW] = o.C1;
    color[o3 + 2 * HW] = o.C2;
    normal[o3] = st.N0;
    normal[o3 + HW] = st.N1;
    normal[o3 + 2 * HW] = st.N2;
    alpha[o1] = o.A;
    depth[o1] = o.D;
    dist[o1] = o.Dist;
    T_final[o1] = st.T;
    n_contrib[o1] = st.last;
}

template <int TW, int TH, int MODE, bool SCALAR>
__global__ void __launch_bounds__(TW * TH) SR_OCCUPANCY(SCALAR ? kPruneWaves : kLdsWaves)
k_render_fwd(const sr_camera* __restrict__ cams, int V, int N, const float4* __restrict__ geom,
             const float4* __restrict__ app, const uint2* __restrict__ rect, const uint32_t* __restrict__ vals,
             const uint2* __restrict__ ranges,
             RasterConsts rc, float* __restrict__ color, float* __restrict__ alpha, float* __restrict__ depth,
             float* __restrict__ normal, float* __restrict__ dist, float* __restrict__ T_final,
             uint32_t* __restrict__ n_contrib, uint32_t* __restrict__ hits, float* __restrict__ max_alpha,
             float* __restrict__ max_weight, unsigned long long* __restrict__ counts,
             float* __restrict__ median_depth, uint32_t* __restrict__ median_contrib,
             const uint32_t* __restrict__ tile_order, uint32_t* __restrict__ tile_cost) {
    constexpr int NT = TW * TH;
    __shared__ FwdSmem<NT, MODE, SCALAR> sm;
    __shared__ uint32_t s_cost;
    // an order entry beyond the grid leaves the workgroup idle
    if (tile_order && tile_order[blockIdx.x] >= gridDim.x) return;
    TileCtx t;
    tile_ctx<TW, TH>(cams, V, ranges, t, tile_order);
    const bool failed = status_failed(rc);
    if (failed) t.n = 0;
    const float px = (float)t.ix + 0.5f, py = (float)t.iy + 0.5f;
    PixFwd st;
    uint64_t n_reached = 0, n_blended = 0, n_witer = 0, n_wblend = 0, n_upto = 0;
    fwd_tile<TW, NT, MODE, SCALAR>(t, px, py, N, geom, app, rect, vals, rc, sm, st, hits, max_alpha, max_weight, n_reached,
                           n_blended,
                       n_witer, n_wblend, n_upto);
    if (failed) poison(st);
    if (MODE & kCount) {
        // per-pixel tally of the backward's pairs: summed over the wave first
        uint64_t up = n_upto;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) up += (uint64_t)__shfl_xor((long long)up, off, 64);
        if (__lane_id() == 0) {
            atomicAdd(&counts[0], (unsigned long long)n_reached);
            atomicAdd(&counts[1], (unsigned long long)n_blended);
            atomicAdd(&counts[2], (unsigned long long)n_witer);
            atomicAdd(&counts[3], (unsigned long long)n_wblend);
            atomicAdd(&counts[4], (unsigned long long)up);
        }
    }
    if ((MODE & kShade) && t.inside) write_outputs(st, pix_outputs(st, t), t, color, alpha, depth, normal, dist,
                                                   T_final, n_contrib);
    if ((MODE & kMedian) && t.inside) {
        const int64_t o1 = t.pix_off + (int64_t)t.iy * t.W + t.ix;
        median_depth[o1] = st.zmed;
        median_contrib[o1] = st.kmed;
    }
    if (tile_cost) {
        // the tile's cost for a later launch's order: its largest n_contrib
        if (threadIdx.x == 0) s_cost = 0u;
        __syncthreads();
        if (t.inside) atomicMax(&s_cost, st.last);
        __syncthreads();
        if (threadIdx.x == 0) tile_cost[t.tile] = s_cost;
    }
}

// Per-pixel inputs of the backward.
struct PixBwd {
    uint32_t ncon, kmed;
    float T, gC0, gC1, gC2, gA, gD, gN0, gN1, gN2, gS, gMed, S0, rmean, Q, Wacc;
};

__device__ __forceinline__ void pix_bwd_init(PixBwd& pb, const TileCtx& t, float Tf, uint32_t ncon, float S0,
                                             float D, float Dist) {
#pragma clang fp contract(off)
    pb.ncon = ncon;
    pb.T = Tf;
    pb.S0 = S0;
    pb.rmean = 0.f;
    pb.Q = 0.f;
    if (S0 > 0.f) {
        pb.rmean = D / S0;
        pb.Q = Dist / (2.0f * S0);
    }
    pb.Wacc = (pb.gC0 * t.bg[0] + pb.gC1 * t.bg[1] + pb.gC2 * t.bg[2]) * Tf;
}

// A lane's part in wave_contract: quarter wave (lane & 3) holds one of four
// values, b = lane >> 2 is its column of pixels 16 t + b (t = 0..3) of the
// wave's 8x8 block, i.e. x = b % 8, y = 2 t + b / 8.
struct ContractLane {
    float x, y;         // image coordinates of the column and of its first pixel (t = 0)
    int slot;           // of the accumulator this lane adds to, or -1
    int slot6;          // the same for wave_sum6, from slot 16 on
};

template <int TW>
__device__ __forceinline__ ContractLane contract_lane(const TileCtx& t) {
    constexpr int WB = kWaveBlock;
    const int lane = __lane_id(), b = lane >> 2, row = lane >> 4;
    const int w = wave_index();
    const int bx = (w % (TW / WB)) * WB, by = (w / (TW / WB)) * WB;
    ContractLane c;
    c.x = (float)(t.tx0 + bx + (b & 7)) + 0.5f;
    c.y = (float)(t.ty0 + by + (b >> 3)) + 0.5f;
    c.slot = (lane & 12) == 0 ? 4 * row + (lane & 3) : -1;
    c.slot6 = (lane & 28) == 0 ? ((lane >> 5) == 0 ? (lane & 3) : ((lane & 2) == 0 ? 4 + (lane & 1) : -1)) : -1;
    return c;
}

// Orders this wave's LDS accesses for the compiler (the LDS unit executes a
// wave's accesses in order, so no wait is needed between its lanes).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The four values p of every lane, transposed in quarter waves: register t of
// a lane is value lane & 3 of pixel 16 t + lane / 4.
__device__ __forceinline__ float4 wave_transpose4(float* scr, const float4& p) {
    const int lane = __lane_id();
    wave_lds_order();
    reinterpret_cast<float4*>(scr)[lane] = p;
    wave_lds_order();
    const float4 r = make_float4(scr[lane], scr[64 + lane], scr[128 + lane], scr[192 + lane]);
    wave_lds_order();
    return r;
}

// Sums over a wave of four values p, of each times dy, of each times dx (the
// pixel relative to the projected centre), and of four values u, given
// transposed as a and b: 16 sums, slots p 0..3, dy p 4..7, dx p 8..11, u 12..15
// of acc.  Every lane sums four pixels of one value after the transposition
// in LDS, so the product with dx is formed once per four pixels and the
// cross-lane stages (permlane swaps, row rotations) carry four registers: 24
// VALU instructions, where 11 products and a transposed reduction of 15
// registers took 46.  The offsets are those from the splat's own centre: about
// a point of the tile and shifted afterwards, the sums of a splat small
// against its distance from that point cancel (19 instructions, but 16 times
// the rounding at half a pixel).
__device__ __forceinline__ float wave_contract(const ContractLane& c, float2 centre, const float4& a,
                                               const float4& b) {
#pragma clang fp contract(off)
    const float S = (a.x + a.w) + (a.y + a.z);
    // rows 2 t + b / 8; the offsets of two rows differ by a whole number, so
    // that every one is as exact as its own difference from the centre
    const float dy = c.y - centre.y;
    const float Y = __builtin_fmaf(a.x, dy, __builtin_fmaf(a.y, dy + 2.0f,
                                   __builtin_fmaf(a.z, dy + 4.0f, a.w * (dy + 6.0f))));
    const float X = (c.x - centre.x) * S;
    const float U = (b.x + b.w) + (b.y + b.z);
    const auto r0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(S), __float_as_uint(X), false, false);
    const auto r1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(Y), __float_as_uint(U), false, false);
    const float s0 = __uint_as_float(r0[0]) + __uint_as_float(r0[1]);     // halves: S, X
    const float s1 = __uint_as_float(r1[0]) + __uint_as_float(r1[1]);     // halves: Y, U
    const auto r2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(s0), __float_as_uint(s1), false, false);
    float w = __uint_as_float(r2[0]) + __uint_as_float(r2[1]);            // rows: S, Y, X, U
    w += dpp_f<0x124, 0xF>(w);                  // row_ror:4
    w += dpp_f<0x128, 0xF>(w);                  // row_ror:8
    return w;
}

// The same for plain sums of six values: four transposed (a), two as the
// sum q of two pixels of value lane & 1.
__device__ __forceinline__ float wave_sum6(const float4& a, float q) {
    const float P = (a.x + a.w) + (a.y + a.z);
    q += dpp_f<0x4E, 0xF>(q);                   // quad_perm [2,3,0,1]
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(P), __float_as_uint(q), false, false);
    const uint32_t h = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));    // halves: P, q
    const auto r2 = __builtin_amdgcn_permlane16_swap(h, h, false, false);
    float w = __uint_as_float(r2[0]) + __uint_as_float(r2[1]);
    w += dpp_f<0x124, 0xF>(w);                  // row_ror:4
    w += dpp_f<0x128, 0xF>(w);                  // row_ror:8
    return w;
}

// The component of a gradient record that flush lane l adds: scale * acc[at]
// of the sums of an entry (the slots of wave_contract and, 16 on, of wave_sum6).
struct GradTerm {
    int comp, at;      // comp < 0: none
    float scale;
};

template <bool GEO>
__device__ __forceinline__ GradTerm grad_term(int l) {
    GradTerm t{-1, 0, 1.0f};
    if (l < 9) {
        const int i = l % 3, kind = l / 3;               // dA: dx sums, dB: dy sums, dC'
        t = GradTerm{l, kind == 0 ? 8 + i : (kind == 1 ? 4 + i : i), i == 2 ? -1.0f : 1.0f};   // the walk sums -dL/dw2
    } else if (l < 11) {
        t = GradTerm{l, l == 9 ? 11 : 7, -2.0f};                      // and -1/2 of the centre's
    } else if (l == 11) {
        t = GradTerm{11, 12, 1.0f};
    } else if (!GEO) {
        if (l < 15) t = GradTerm{l + 3, l + 1, 1.0f};                 // colour
    } else if (l < 21) {
        t = GradTerm{l, l < 15 ? l + 4 : (l < 18 ? l - 2 : l + 1), 1.0f};     // m_z, colour, normal
    }
    return t;
}

// Backward: per pixel, walk the tile list back to front from the last
// blended entry, recovering T_k = T_{k+1} / (1 - a_k).  With g_k the
// derivative of the loss by the blending weight w_k = a_k T_k of entry k and
// W_k = sum_{j>k} g_j w_j (+ the background term), dL/da_k = T_k g_k -
// W_k / (1 - a_k).  Per-record gradients are summed over each wave
// (wave_contract), over the workgroup in LDS, then added to grad_rec with one
// atomic per (tile, record, component); with grad_marks (the projection's
// tiles_touched) bit 31 of every record given a gradient is set.
// GEO: the loss has depth, normal or distortion terms (their upstream
// gradients are read); without them the depth path and six of the per-record
// components are identically zero and are not computed or reduced.
// HITS (without GEO): the backward also counts, per entry, the pixels that
// blend it (the forward's blend decisions, recomputed: positions below the
// pixel's last contributor that pass the cutoff): the wave's count of an
// entry is kept by the lane of the entry's position in its 64-entry chunk,
// added to the workgroup's once per chunk and to hits[g] at the flush.
//
// On many tiles VALU issue takes most of this walk (independent FP32
// instructions issue at 1.6 wave64 ones per CU and cycle with vector operands,
// 0.9 with a scalar one), and the sums over the wave's 64 pixels were a third
// of its instructions.  They are a contraction: the columns A, B, C' of dL/dw
// and the low-pass centre are the sums of {dw0, dw1, dw2, f2} times
// {dx, dy, 1}, and dx and dy depend on the pixel's column and row alone, so
// only those four values and four plain sums (opacity, colour) go through the
// reduction, not 15 products.
template <int TW, int NT, int BATCH, bool GEO, bool SCALAR, bool HITS>
__device__ __forceinline__ void bwd_tile(const TileCtx& t, float px, float py, int N, const float4* __restrict__ geom,
                                         const float4* __restrict__ app, const uint32_t* __restrict__ vals,
                                         const RasterConsts& rc, BwdSmem<NT, BATCH, GEO, HITS, SCALAR>& sm, PixBwd pb,
                                         float* __restrict__ grad_rec, uint32_t* __restrict__ grad_marks,
                                         uint32_t* __restrict__ hits = nullptr,
                                         uint32_t* __restrict__ cost_out = nullptr,
                                         const uint32_t* bitcache = nullptr) {
    static_assert(BATCH <= NT, "one record per thread and batch");
    static_assert(!(HITS && GEO), "the count is taken by the training step alone");
    // The depth terms from LDS (few tiles, often less than a wave per SIMD): the
    // next entry's test is read a whole entry ahead, for 4 waves per SIMD
    // instead of 5.  56 tiles of 40,000 entries: k_render_bwd 12.7 -> 11.7 ms.
    // The training step has no registers left for it (14.0 -> 14.2 ms on two
    // 165x153 views of 700k surfels), nor has the forward anything to hide it
    // behind (2M surfels, 1237x822: 0.554 -> 0.559 ms).
    constexpr bool AHEAD = !SCALAR && GEO;
    const int tid = threadIdx.x;
    const int lane = __lane_id();
    __syncthreads();
    if (tid == 0) sm.maxn = 0u;
    __syncthreads();
    atomicMax(&sm.maxn, pb.ncon);
    __syncthreads();
    const uint32_t maxn = __builtin_amdgcn_readfirstlane(sm.maxn);
    // the tile's cost for the next launch's order: the run positions it works through
    if (cost_out && tid == 0) *cost_out = maxn;
    if (maxn == 0u) return;
    // entries at or beyond the wave's own last contributor concern no lane
    uint32_t wave_maxn = pb.ncon;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)wave_maxn, off, 64);
        wave_maxn = o > wave_maxn ? o : wave_maxn;
    }
    wave_maxn = __builtin_amdgcn_readfirstlane(wave_maxn);   // uniform: keep the loop control scalar
    constexpr int TH = NT / TW;
    float T = pb.T, Wacc = pb.Wacc;
    const int wv = wave_index();
    const float4* geom_v = geom + kGeomF4 * (size_t)t.v * N;
    const float4* app_v = app + kAppF4 * (size_t)t.v * N;
    float* scr = reinterpret_cast<float*>(&sm.xp[64 * wv]);
    const ContractLane cr = contract_lane<TW>(t);
    static_assert(NT / 64 <= kMaxWaves, "gathering counts");
    // batches of up to BATCH entries of the tile below run position hi,
    // gathered from its group's run highest first into slots [lo, BATCH)
    int hi = (int)maxn;
    while (hi > 0) {
        __syncthreads();
        int fill = 0;
        while (fill < BATCH && hi > 0) {
            int next;
            fill += gather_round<NT, false>(t, vals, hi, fill, BATCH, sm.id, sm.pos, sm.wcnt, next);
            hi = next;
        }
        const int lo = BATCH - fill;
        if (tid < BATCH) {
            if (tid >= lo) {
                const uint32_t g = sm.id[tid] & kInstIdMask;
                const uint32_t jpos = sm.pos[tid];
                float4 gq[kGeomF4];
#pragma unroll
                for (int q = 0; q < kGeomF4; ++q) gq[q] = geom_v[kGeomF4 * (size_t)g + q];
                sm.rec.put(tid, gq, app_v + kAppF4 * (size_t)g);
                // the forward's wave bits of this position when cached
                const uint32_t bits = (bitcache && jpos < BitCache<NT>::kPos)
                                          ? (bitcache[jpos >> 3] >> ((jpos & 7u) << 2)) & 0xFu
                                          : wave_bits<TW, NT / 64>(gq[0], gq[1], gq[2], gq[3].w,
                                                                   reinterpret_cast<const uint2*>(app_v + kAppF4 * (size_t)g)[3],
                                                                   t.tx0, t.ty0);
                sm.id[tid] = g | (bits << SR_INST_ID_BITS);
            }
#pragma unroll
            for (int i = 0; i < (GEO ? 22 : 16); ++i) sm.acc[tid][i] = 0.f;
            if (HITS) sm.hit[tid] = 0u;
            if (tid < (BATCH + 63) / 64) sm.touched[tid] = 0ull;
        }
        __syncthreads();
        // entries skipped by the forward for this wave are skipped here too
        for (int c = (BATCH - 1) >> 6; c >= (lo >> 6); --c) {
          // entries at or beyond the wave's last contributor concern no lane of it
          const int slot = c * 64 + lane;
          const bool in = slot >= lo && slot < BATCH;
          const uint32_t my_id = in ? sm.id[slot] : 0u, my_pos = in ? sm.pos[slot] : 0u;
          uint64_t live = ballot64(((my_id >> (SR_INST_ID_BITS + wv)) & 1u) && my_pos < wave_maxn);
          if (live == 0ull) continue;
          int nbit = 63 - (int)__builtin_clzll(live);
          EntryRec next_rec;
          if constexpr (SCALAR) {
            load_scalar<true, GEO>(geom_v, app_v, __builtin_amdgcn_readlane(my_id, nbit) & kInstIdMask, next_rec);
            next_rec.c = sm.rec.c[c * 64 + nbit];
          } else if constexpr (AHEAD) {
            load_lds_test(sm.rec, c * 64 + nbit, next_rec);
          }
          uint32_t my_hits = 0;       // HITS: this wave's blended pixels of entry c * 64 + lane
          uint64_t blended = 0ull;    // the chunk's entries that a pixel of the wave blends
          while (live != 0ull) {
            const int hb = nbit, k = c * 64 + hb;
            EntryRec rec = next_rec;
            live &= ~(1ull << hb);
            nbit = live != 0ull ? 63 - (int)__builtin_clzll(live) : hb;
            uint32_t jj;                           // run position
            if constexpr (SCALAR || AHEAD) jj = __builtin_amdgcn_readlane(my_pos, hb);
            else jj = sm.pos[k];
            if constexpr (SCALAR) {
                load_scalar<true, GEO>(geom_v, app_v, __builtin_amdgcn_readlane(my_id, nbit) & kInstIdMask, next_rec);
            } else {
                if constexpr (!AHEAD) load_lds_test(sm.rec, k, rec);
                load_lds_rest<true>(sm.rec, k, rec);
            }
            // AHEAD: the centre is read again with the opacity, so that the next
            // entry's test takes the registers of this one's (kept for the sums
            // it cost nine moves an entry)
            float2 centre;
            if constexpr (AHEAD) {
                const float4 g2 = sm.rec.g[2][k];
                rec.g[11] = g2.w;
                centre = make_float2(g2.y, g2.z);
            } else {
                centre = make_float2(rec.g[9], rec.g[10]);
            }
            const SurfelGeom sg = geom_of<SCALAR>(rec);
            PairEval e;
            eval_test<SCALAR>(sg, px, py, e);
            // behind the last use of this entry's: the same registers
            if constexpr (SCALAR) next_rec.c = sm.rec.c[c * 64 + nbit];
            else if constexpr (AHEAD) load_lds_test(sm.rec, c * 64 + nbit, next_rec);
            const uint64_t blm = ballot64(jj < pb.ncon) & pass_mask(e);
            if (blm == 0ull) continue;
            blended |= 1ull << hb;
            const bool bl = in_mask(blm);
            eval_finish(sg, rc.alpha_max, e);
            // Gradients of this entry, branch-free: lanes that do not blend it
            // produce exact zeros (alpha, dL/do and the intersection terms are
            // selected to 0, and W only steps where they blend).
            const F4v a0 = rec.a0;
            const float o = sg.o;
            const float ae = bl ? e.a : 0.f;
            const float rin = __builtin_amdgcn_rcpf(1.0f - ae);
            T = T * rin;                                  // T before this entry; unchanged where ae = 0
            const float wgt = ae * T;
            float gk = pb.gC0 * a0.x + pb.gC1 * a0.y + pb.gC2 * a0.z + pb.gA;
            float dLdz = 0.f;
            if (GEO) {
                const float zr = e.z - pb.rmean;
                gk += pb.gD * e.z + pb.gN0 * a0.w + pb.gN1 * rec.a1.x + pb.gN2 * rec.a1.y +
                      pb.gS * 2.0f * (pb.Q + pb.S0 * zr * zr);
                // the median depth is the depth of entry kmed - 1 (0-based)
                const float gmed = jj + 1u == pb.kmed ? pb.gMed : 0.f;
                dLdz = bl ? __builtin_fmaf(wgt, pb.gD + 4.0f * pb.gS * pb.S0 * zr, gmed) : 0.f;
            }
            const float dLda = T * gk - Wacc * rin;
            Wacc = bl ? __builtin_fmaf(gk, wgt, Wacc) : Wacc;
            const float dLdo = bl && !e.clamped ? dLda * e.G : 0.f;
            const float dLdrho = -(o * dLdo);
            const float us = e.surf ? e.u : 0.f, vs = e.surf ? e.v : 0.f, rs = e.surf ? e.r : 0.f;
            float dw0, dw1, dw2, dzs = 0.f;
            if (GEO) {
                dzs = e.surf ? dLdz : 0.f;
                const float du = __builtin_fmaf(dzs, sg.m30, dLdrho * us), dv = __builtin_fmaf(dzs, sg.m31, dLdrho * vs);
                dw0 = du * rs;
                dw1 = dv * rs;
            } else {
                const float m = dLdrho * rs;
                dw0 = m * us;
                dw1 = m * vs;
            }
            dw2 = __builtin_fmaf(dw0, us, dw1 * vs);          // -dL/dw2
            const float f2 = e.surf ? 0.f : dLdrho;           // -1/2 of the centre's
            const float4 ta = wave_transpose4(scr, make_float4(dw0, dw1, dw2, f2));
            const float4 tb = wave_transpose4(scr, make_float4(dLdo, pb.gC0 * wgt, pb.gC1 * wgt, pb.gC2 * wgt));
            float4 tc;
            float q0 = 0.f, q1 = 0.f;
            if (GEO) {
                tc = wave_transpose4(scr, make_float4(dzs * us, dzs * vs, dLdz, pb.gN0 * wgt));
                reinterpret_cast<float2*>(scr)[lane] = make_float2(pb.gN1 * wgt, pb.gN2 * wgt);
                wave_lds_order();
                q0 = scr[lane];                                  // value lane & 1 of two pixels
                q1 = scr[64 + lane];
                wave_lds_order();
            }
            float w16 = wave_contract(cr, centre, ta, tb);
            // a lone wave: not before the contraction, whose values were read first
            if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
            float w6 = GEO ? wave_sum6(tc, q0 + q1) : 0.f;
            // summed before the branches: sunk below them, the last adds need moves of their own
            asm volatile("" : "+v"(w16), "+v"(w6));
            if (cr.slot >= 0) atomicAdd(&sm.acc[k][cr.slot], w16);
            if (GEO && cr.slot6 >= 0) atomicAdd(&sm.acc[k][16 + cr.slot6], w6);
            if (HITS) my_hits = (uint32_t)lane_write((int)__popcll(blm), hb, (int)my_hits);
          }
          if (HITS && my_hits != 0u) atomicAdd(&sm.hit[c * 64 + lane], my_hits);
          if (lane == 0 && blended != 0ull) atomicOr((unsigned long long*)&sm.touched[c], (unsigned long long)blended);
        }
        __syncthreads();
        // The batch's sums to memory.  The lanes of a quarter (half with GEO)
        // wave hold the components of one record, so its atomics leave as two
        // requests of adjacent words: with a lane per record every component
        // was a request of its own, and their rate bounded the backward (k_render_bwd
        // with the depth terms, four 1559x1039 views of 1M surfels: 2.3 ms
        // without any atomics, 3.5 ms with 21 requests a record).
        constexpr int LPR = GEO ? 32 : 16;              // lanes per record
        // the entries that were blended at all, listed by every wave for itself
        int* list = reinterpret_cast<int*>(scr);
        int touched = 0;
        wave_lds_order();
#pragma unroll
        for (int c = 0; c < (BATCH + 63) / 64; ++c) {
            const uint64_t m = sm.touched[c];
            if (in_mask(m)) list[touched + __popcll(m & (lane == 0 ? 0ull : ~0ull >> (64 - lane)))] = c * 64 + lane;
            touched += (int)__popcll(m);
        }
        wave_lds_order();
        int fl = tid & (LPR - 1);
        asm volatile("" : "+v"(fl));      // the term is formed here, not kept in registers through the walk
        const GradTerm term = grad_term<GEO>(fl);
        for (int n = tid / LPR; n < touched; n += NT / LPR) {
            const int e = list[n];
            const uint32_t g = sm.id[e] & kInstIdMask;
            const size_t r = (size_t)t.v * N + g;
            float v = 0.f;
            if (term.comp >= 0) {
                v = sm.acc[e][term.at] * term.scale;
                if (v != 0.f) atomicAdd(&grad_rec[r * SR_GRAD_STRIDE + term.comp], v);
            }
            // mark the record for the projection backward (bit 31)
            const uint64_t any = ballot64(v != 0.f) & ((LPR == 32 ? 0xFFFFFFFFull : 0xFFFFull) << (lane & ~(LPR - 1)));
            if (fl == 0) {
                if (grad_marks && any != 0ull) atomicOr(&grad_marks[r], 0x80000000u);
                if (HITS) {
                    const uint32_t n = sm.hit[e];
                    if (n != 0u) atomicAdd(&hits[g], n);
                }
            }
        }
    }
}

template <int TW, int TH, int BATCH, bool GEO, bool SCALAR>
__global__ void __launch_bounds__(TW * TH) SR_OCCUPANCY(SCALAR ? kBwdWaves : GEO ? kAheadWaves : kLdsWaves)
k_render_bwd(const sr_camera* __restrict__ cams, int V, int N, const float4* __restrict__ geom,
             const float4* __restrict__ app, const uint32_t* __restrict__ vals, const uint2* __restrict__ ranges,
             RasterConsts rc, const float* __restrict__ alpha, const float* __restrict__ depth,
             const float* __restrict__ dist, const float* __restrict__ T_final, const uint32_t* __restrict__ n_contrib,
             const float* __restrict__ dC, const float* __restrict__ dA, const float* __restrict__ dD,
             const float* __restrict__ dNrm, const float* __restrict__ dDist,
             const uint32_t* __restrict__ median_contrib, const float* __restrict__ dMed,
             float* __restrict__ grad_rec, uint32_t* __restrict__ grad_marks,
             const uint32_t* __restrict__ tile_order) {
    __shared__ BwdSmem<TW * TH, BATCH, GEO, false, SCALAR> sm;
    // an order entry beyond the grid leaves the workgroup idle; so does a set
    // status word (no gradients)
    if (tile_order && tile_order[blockIdx.x] >= gridDim.x) return;
    if (status_failed(rc)) return;
    TileCtx t;
    tile_ctx<TW, TH>(cams, V, ranges, t, tile_order);
    const float px = (float)t.ix + 0.5f, py = (float)t.iy + 0.5f;
    PixBwd pb;
    pb.gC0 = pb.gC1 = pb.gC2 = pb.gA = pb.gD = pb.gN0 = pb.gN1 = pb.gN2 = pb.gS = pb.gMed = 0.f;
    pb.ncon = pb.kmed = 0;
    pb.T = 1.f;
    pb.S0 = pb.rmean = pb.Q = pb.Wacc = 0.f;
    if (t.inside) {
        const int64_t HW = (int64_t)t.W * t.H;
        const int64_t p = (int64_t)t.iy * t.W + t.ix;
        const int64_t o1 = t.pix_off + p, o3 = 3 * t.pix_off + p;
        if (dC) { pb.gC0 = dC[o3]; pb.gC1 = dC[o3 + HW]; pb.gC2 = dC[o3 + 2 * HW]; }
        if (dA) pb.gA = dA[o1];
        if (dD) pb.gD = dD[o1];
        if (dNrm) { pb.gN0 = dNrm[o3]; pb.gN1 = dNrm[o3 + HW]; pb.gN2 = dNrm[o3 + 2 * HW]; }
        if (dDist) pb.gS = dDist[o1];
        if (dMed) { pb.gMed = dMed[o1]; pb.kmed = median_contrib[o1]; }
        pix_bwd_init(pb, t, T_final[o1], n_contrib[o1], alpha[o1], depth[o1], dist[o1]);
    }
    bwd_tile<TW, TW * TH, BATCH, GEO, SCALAR, false>(t, px, py, N, geom, app, vals, rc, sm, pb, grad_rec, grad_marks);
}

// One training step of the compositing for a tile: forward, the masked L1 +
// background loss gradients of every pixel (Eq. 1, Eq. 2) and the backward,
// with the per-pixel state kept in registers between the phases.  STATS = 1
// counts the blended pixels of every surfel (the usage record of Section
// 4.3), taken by the backward, which recomputes the same blend decisions;
// STATS = 2 has the forward take the count and the maximum alpha and weight;
// 0 records nothing.  Per-tile loss partial sums go to tile_loss[2*tile]
// (L_b numerator, L1 numerator).
template <int TW, int TH, int BATCH, int STATS, bool SCALAR>
__global__ void __launch_bounds__(TW * TH) SR_OCCUPANCY(SCALAR ? kTrainWaves : kLdsWaves)
k_train_raster(const sr_camera* __restrict__ cams, int V, int N, const float4* __restrict__ geom,
               const float4* __restrict__ app, const uint32_t* __restrict__ vals, const uint2* __restrict__ ranges,
               RasterConsts rc, const uint8_t* __restrict__ mask, const float* __restrict__ target, float gamma,
               float w_c, float* __restrict__ color, float* __restrict__ alpha, float* __restrict__ depth,
               float* __restrict__ normal, float* __restrict__ dist, float* __restrict__ T_final,
               uint32_t* __restrict__ n_contrib, uint32_t* __restrict__ hits, float* __restrict__ max_alpha,
               float* __restrict__ max_weight, float* __restrict__ tile_loss, float* __restrict__ grad_rec,
               uint32_t* __restrict__ grad_marks,
               const uint32_t* __restrict__ tile_order, uint32_t* __restrict__ tile_cost) {
    constexpr int NT = TW * TH;
    constexpr int MODE = kShade | (STATS == 2 ? kStats : 0);
    using FSmem = FwdSmem<NT, MODE, SCALAR>;
    using BSmem = BwdSmem<NT, BATCH, false, STATS == 1, SCALAR>;
    constexpr size_t kF = sizeof(FSmem), kB = sizeof(BSmem);
    __shared__ __align__(16) unsigned char smem[kF > kB ? kF : kB];
    __shared__ float s_red[NT / 64][2];
    // the wave-bit cache, except with the full statistics (whose larger
    // forward staging would lose a workgroup per CU to the extra LDS)
    constexpr bool CACHE = STATS != 2;
    __shared__ uint32_t s_bits[CACHE ? BitCache<NT>::kWords : 1];
    TileCtx t;
    // an order entry beyond the grid leaves the workgroup idle (not a valid
    // permutation: nothing of it is written)
    if (tile_order && tile_order[blockIdx.x] >= gridDim.x) return;
    tile_ctx<TW, TH>(cams, V, ranges, t, tile_order);
    // a set status word: nothing blended, NaN outputs and losses, no gradients
    const bool failed = status_failed(rc);
    if (failed) t.n = 0;
    const float px = (float)t.ix + 0.5f, py = (float)t.iy + 0.5f;
    PixFwd st;
    uint64_t n0 = 0, n1 = 0, n2 = 0, n3 = 0, n4 = 0;
    if (CACHE) {
        for (int i = threadIdx.x; i < BitCache<NT>::kWords; i += NT) s_bits[i] = 0u;
        __syncthreads();
    }
    fwd_tile<TW, NT, MODE, SCALAR>(t, px, py, N, geom, app, nullptr, vals, rc, *reinterpret_cast<FSmem*>(smem), st,
                           hits, max_alpha, max_weight, n0, n1, n2, n3, n4, CACHE ? s_bits : nullptr);
    if (failed) poison(st);
    const PixOut o = pix_outputs(st, t);
    PixBwd pb;
    pb.gC0 = pb.gC1 = pb.gC2 = pb.gA = pb.gD = pb.gN0 = pb.gN1 = pb.gN2 = pb.gS = pb.gMed = 0.f;
    pb.ncon = pb.kmed = 0;
    pb.T = 1.f;
    pb.S0 = pb.rmean = pb.Q = pb.Wacc = 0.f;
    float lb = 0.f, l1 = 0.f;
    if (t.inside) {
        write_outputs(st, o, t, color, alpha, depth, normal, dist, T_final, n_contrib);
        // the same per-pixel loss terms and gradients as sr_background_loss
        const int64_t HW = (int64_t)t.W * t.H;
        const int64_t p = (int64_t)t.iy * t.W + t.ix;
        const int64_t o1 = t.pix_off + p, o3 = 3 * t.pix_off + p;
        const float Cv[3] = {o.C0, o.C1, o.C2};
        const float Iv[3] = {target[o3], target[o3 + HW], target[o3 + 2 * HW]};
        float gC[3];
        pixel_loss_grad(mask[o1], o.A, Cv, Iv, gamma, w_c, (float)HW, (float)V, lb, l1, pb.gA, gC);
        pb.gC0 = gC[0]; pb.gC1 = gC[1]; pb.gC2 = gC[2];
        pix_bwd_init(pb, t, st.T, st.last, o.A, o.D, o.Dist);
    }
    // per-tile loss partials, in a fixed order: over the wave, then the waves
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lb += __shfl_xor(lb, off, 64);
        l1 += __shfl_xor(l1, off, 64);
    }
    if (__lane_id() == 0) {
        s_red[threadIdx.x >> 6][0] = lb;
        s_red[threadIdx.x >> 6][1] = l1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) sum += s_red[i][threadIdx.x];
        tile_loss[2 * (size_t)t.tile + threadIdx.x] = sum;
    }
    bwd_tile<TW, NT, BATCH, false, SCALAR, STATS == 1>(t, px, py, N, geom, app, vals, rc,
                                               *reinterpret_cast<BSmem*>(smem), pb, grad_rec, grad_marks, hits,
                                               tile_cost ? tile_cost + t.tile : nullptr, CACHE ? s_bits : nullptr);
}

__global__ void k_fill_f32(float* __restrict__ p, float v, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// A set status word (statistics incomplete) prunes nothing.
__global__ void k_prune_mask(int N, const float* __restrict__ max_alpha, float tau, const uint32_t* __restrict__ status,
                             uint8_t* __restrict__ mask) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const bool failed = status != nullptr && *status != 0u;
    if (g < N) mask[g] = (!failed && max_alpha[g] < tau) ? 1 : 0;
}

// Records per LDS batch of the backward: compiled for 32, 64, 128 and 256,
// each at most the tile's pixel count (one staging thread per record).  The
// default, min(128, pixels), keeps the separate backward's LDS footprint and
// hence its occupancy in check; in the fused kernel the forward's staging
// area is as large, so only 256 costs occupancy there.
constexpr int kBwdBatch = 128;

constexpr int resolve_batch(int pixels, int batch) {
    return batch != 0 ? batch : (pixels < kBwdBatch ? pixels : kBwdBatch);
}

// Calls f(integral_constant<int, B>) for the compiled batch B == batch (a
// value of resolve_batch); false when it is not compiled for this tile.
template <int PIX, typename F>
bool with_batch(int batch, F&& f) {
    switch (batch) {
        case 32: if constexpr (32 <= PIX) { f(std::integral_constant<int, 32>{}); return true; } break;
        case 64: if constexpr (64 <= PIX) { f(std::integral_constant<int, 64>{}); return true; } break;
        case 128: if constexpr (128 <= PIX) { f(std::integral_constant<int, 128>{}); return true; } break;
        case 256: if constexpr (256 <= PIX) { f(std::integral_constant<int, 256>{}); return true; } break;
        default: break;
    }
    return false;
}

// Where the entries' records are read from (EntryRec): through the scalar
// cache from so many waves per SIMD of the device on (all waves of the launch
// over all SIMDs), from LDS below.  A SIMD holds five to seven at a time; with
// few rounds of them the launch ends with the chains of its longest tiles,
// each wave alone with the latency of its loads, with many the other waves
// cover it and the LDS reads would fill the LDS unit.  The limits are the
// crossovers of a sweep (5 thousand to 1.5 million surfels, 1 to 16 views, 0.06
// to 256 waves per SIMD, the four tile shapes; LDS / scalar time, geometric
// means by waves per SIMD):
//   backward with depth terms  0.98 at 5, 1.00 at 8, 1.01 at 10, 1.06 at 13, 1.21 at 100
//   backward, colour and alpha 0.96 at 6, 0.98 at 10, 1.02 at 13, 1.04 at 16, 1.18 at 100
//   training step              0.96 at 10, 0.98 at 13, 0.99 at 16, 1.04 at 20, 1.17 at 100
//   pruning statistics         0.93 at 10, 0.97 at 20, 0.99 at 25, 1.01 at 32, 1.05 at 250
//   forward with outputs       0.98 at 6, 0.96 at 12, 0.97 at 28 and at 100: from LDS always
constexpr int kScalarGeoWaves = 10, kScalarBwdWaves = 14, kScalarTrainWaves = 18, kScalarPruneWaves = 28;
inline bool scalar_records(int tiles, int tile_pixels, int simds, int waves) {
    return (int64_t)tiles * (tile_pixels / 64) >= (int64_t)waves * simds;
}

template <int TW, int TH, int MODE>
void fwd_launch(int total_tiles, hipStream_t s, const sr_camera* cams, int V, int N, const float4* geom,
                const float4* app, const uint2* rect, const uint32_t* vals, const uint2* ranges, RasterConsts rc,
                float* color,
                float* alpha, float* depth, float* normal, float* dist, float* T_final, uint32_t* n_contrib,
                uint32_t* hits, float* max_alpha, float* max_weight, unsigned long long* counts,
                float* median_depth, uint32_t* median_contrib, const uint32_t* tile_order, uint32_t* tile_cost,
                int simds) {
    auto k = k_render_fwd<TW, TH, MODE, false>;
    if constexpr ((MODE & kStats) != 0 && (MODE & kShade) == 0) {
        if (scalar_records(total_tiles, TW * TH, simds, kScalarPruneWaves)) k = k_render_fwd<TW, TH, MODE, true>;
    }
    hipLaunchKernelGGL(k, dim3(total_tiles), dim3(TW * TH), 0, s, cams, V, N, geom, app,
                       rect, vals, ranges, rc, color, alpha, depth, normal, dist, T_final, n_contrib, hits, max_alpha,
                       max_weight, counts, median_depth, median_contrib, tile_order, tile_cost);
}

template <int TW, int TH>
bool fwd_dispatch(int mode, int total_tiles, hipStream_t s, const sr_camera* cams, int V, int N,
                  const float4* geom, const float4* app, const uint2* rect, const uint32_t* vals, const uint2* ranges,
                  RasterConsts rc, float* color, float* alpha, float* depth, float* normal, float* dist,
                  float* T_final, uint32_t* n_contrib, uint32_t* hits, float* max_alpha, float* max_weight,
                  unsigned long long* counts, float* median_depth, uint32_t* median_contrib,
                  const uint32_t* tile_order, uint32_t* tile_cost, int simds) {
#define SR_FWD(M)                                                                                        \
    fwd_launch<TW, TH, M>(total_tiles, s, cams, V, N, geom, app, rect, vals, ranges, rc, color, alpha, depth, \
                          normal, dist, T_final, n_contrib, hits, max_alpha, max_weight, counts,          \
                          median_depth, median_contrib, tile_order, tile_cost, simds)
    switch (mode) {
        case kShade: SR_FWD(kShade); return true;
        case kShade | kHits: SR_FWD(kShade | kHits); return true;
        case kShade | kStats: SR_FWD(kShade | kStats); return true;
        case kShade | kMedian: SR_FWD(kShade | kMedian); return true;
        case kShade | kHits | kMedian: SR_FWD(kShade | kHits | kMedian); return true;
        case kShade | kStats | kMedian: SR_FWD(kShade | kStats | kMedian); return true;
        case kStats: SR_FWD(kStats); return true;
        case kStats | kRect: SR_FWD(kStats | kRect); return true;
        case kCount: SR_FWD(kCount); return true;
        default: return false;       // not compiled
    }
#undef SR_FWD
}

template <int TW, int TH>
bool bwd_launch(int batch, int total_tiles, hipStream_t s, const sr_camera* cams, int V, int N, const float4* geom,
                const float4* app, const uint32_t* vals, const uint2* ranges, RasterConsts rc, const float* alpha,
                const float* depth, const float* dist, const float* T_final, const uint32_t* n_contrib,
                const float* dC, const float* dA, const float* dD, const float* dN, const float* dS,
                const uint32_t* median_contrib, const float* dMed, float* grad_rec, uint32_t* grad_marks,
                const uint32_t* tile_order, int simds) {
    const bool geo = dD || dN || dS || dMed;
    return with_batch<TW * TH>(resolve_batch(TW * TH, batch), [&](auto bc) {
        constexpr int B = decltype(bc)::value;
        const bool sc = scalar_records(total_tiles, TW * TH, simds, geo ? kScalarGeoWaves : kScalarBwdWaves);
        auto k = geo ? (sc ? k_render_bwd<TW, TH, B, true, true> : k_render_bwd<TW, TH, B, true, false>)
                     : (sc ? k_render_bwd<TW, TH, B, false, true> : k_render_bwd<TW, TH, B, false, false>);
        hipLaunchKernelGGL(k, dim3(total_tiles), dim3(TW * TH), 0, s, cams, V, N, geom, app, vals, ranges, rc, alpha,
                           depth, dist, T_final, n_contrib, dC, dA, dD, dN, dS, median_contrib, dMed, grad_rec,
                           grad_marks, tile_order);
    });
}

template <int TW, int TH>
bool train_launch(int stats, int batch, int total_tiles, hipStream_t s, const sr_camera* cams, int V, int N,
                  const float4* geom, const float4* app, const uint32_t* vals, const uint2* ranges, RasterConsts rc,
                  const uint8_t* mask, const float* target, float gamma, float w_c, float* color, float* alpha,
                  float* depth, float* normal, float* dist, float* T_final, uint32_t* n_contrib, uint32_t* hits,
                  float* max_alpha, float* max_weight, float* tile_loss, float* grad_rec, uint32_t* grad_marks,
                  const uint32_t* tile_order,
                  uint32_t* tile_cost, int simds) {
    return with_batch<TW * TH>(resolve_batch(TW * TH, batch), [&](auto bc) {
        constexpr int B = decltype(bc)::value;
        const bool sc = scalar_records(total_tiles, TW * TH, simds, kScalarTrainWaves);
#define SR_TRAIN(S)                                                                                              \
    hipLaunchKernelGGL((sc ? k_train_raster<TW, TH, B, S, true> : k_train_raster<TW, TH, B, S, false>),         \
                       dim3(total_tiles), dim3(TW * TH), 0, s, cams, V, N, geom, app, vals, ranges, rc, mask,    \
                       target, gamma, w_c, color, alpha, depth, normal, dist, T_final, n_contrib, hits, max_alpha, \
                       max_weight, tile_loss, grad_rec, grad_marks, tile_order, tile_cost)
        if (stats == 2)
            SR_TRAIN(2);
        else if (stats == 1)
            SR_TRAIN(1);
        else
            SR_TRAIN(0);
#undef SR_TRAIN
    });
}

// Compiled tile shapes (the binning takes any shape; the raster kernels are
// instantiated for these).
#define SR_TILE_SHAPES(X) X(16, 16) X(16, 8) X(8, 8) X(32, 8)

}  // namespace

bool tile_shape_supported(int tw, int th) {
#define SR_TS(W, H) if (tw == W && th == H) return true;
    SR_TILE_SHAPES(SR_TS)
#undef SR_TS
    return false;
}

bool bwd_batch_supported(int tw, int th, int batch) {
    if (!tile_shape_supported(tw, th)) return false;
    const int b = resolve_batch(tw * th, batch);
    return (b == 32 || b == 64 || b == 128 || b == 256) && b <= tw * th;
}

hipError_t fill_f32(float* p, float v, uint64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3(1024), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_render_fwd(const sr_config& cfg, int N, int V, int total_tiles, const sr_camera* cams,
                             const float* geom, const float* app, const uint16_t* rect, const uint32_t* vals,
                             const uint32_t* ranges, float* color, float* alpha, float* depth, float* normal,
                             float* dist, float* T_final, uint32_t* n_contrib, uint32_t* hits, float* max_alpha,
                             float* max_weight, unsigned long long* counts, float* median_depth,
                             uint32_t* median_contrib, const uint32_t* tile_order, uint32_t* tile_cost,
                             const uint32_t* status, int simds, hipStream_t s) {
    if (total_tiles == 0) return hipSuccess;
    RasterConsts rc{cfg.alpha_min, cfg.alpha_max, cfg.t_min, cfg.flags, status};
    const int stats = hits ? (max_alpha ? kStats : kHits) : 0;
    int mode = counts ? kCount
                      : ((color ? kShade : 0) | stats | (color && median_depth ? kMedian : 0) |
                         (!color && hits && rect ? kRect : 0));
#define SR_TS(W, H)                                                                                              \
    if (cfg.tile_w == W && cfg.tile_h == H) {                                                                   \
        if (!fwd_dispatch<W, H>(mode, total_tiles, s, cams, V, N, (const float4*)geom, (const float4*)app,     \
                                (const uint2*)rect, vals, (const uint2*)ranges, rc, color, alpha, depth, normal, \
                                dist, T_final, n_contrib, hits, max_alpha, max_weight, counts, median_depth,     \
                                median_contrib, tile_order, tile_cost, simds))                                     \
            return hipErrorInvalidValue;                                                                        \
        return hipGetLastError();                                                                               \
    }
    SR_TILE_SHAPES(SR_TS)
#undef SR_TS
    return hipErrorInvalidValue;
}

hipError_t launch_render_bwd(const sr_config& cfg, int N, int V, int total_tiles, const sr_camera* cams,
                             const float* geom, const float* app, const uint32_t* vals, const uint32_t* ranges,
                             const float* alpha, const float* depth, const float* dist, const float* T_final,
                             const uint32_t* n_contrib, const float* dC, const float* dA, const float* dD,
                             const float* dN, const float* dS, const uint32_t* median_contrib, const float* dMed,
                             float* grad_rec, uint32_t* grad_marks, const uint32_t* tile_order,
                             const uint32_t* status, int simds, hipStream_t s) {
    if (total_tiles == 0) return hipSuccess;
    RasterConsts rc{cfg.alpha_min, cfg.alpha_max, cfg.t_min, cfg.flags, status};
#define SR_TS(W, H)                                                                                            \
    if (cfg.tile_w == W && cfg.tile_h == H) {                                                                 \
        if (!bwd_launch<W, H>(cfg.bwd_batch, total_tiles, s, cams, V, N, (const float4*)geom,                 \
                              (const float4*)app, vals, (const uint2*)ranges, rc, alpha, depth, dist, T_final,  \
                              n_contrib, dC, dA, dD, dN, dS, median_contrib, dMed, grad_rec, grad_marks,       \
                              tile_order, simds))                                                               \
            return hipErrorInvalidValue;                                                                      \
        return hipGetLastError();                                                                             \
    }
    SR_TILE_SHAPES(SR_TS)
#undef SR_TS
    return hipErrorInvalidValue;
}

hipError_t launch_train_raster(const sr_config& cfg, int N, int V, int total_tiles, const sr_camera* cams,
                               const float* geom, const float* app, const uint32_t* vals, const uint32_t* ranges,
                               const uint8_t* mask, const float* target, float gamma, float w_c, float* color,
                               float* alpha, float* depth, float* normal, float* dist, float* T_final,
                               uint32_t* n_contrib, uint32_t* hits, float* max_alpha, float* max_weight,
                               float* tile_loss, float* grad_rec, uint32_t* grad_marks, const uint32_t* tile_order,
                               uint32_t* tile_cost,
                               const uint32_t* status, int simds, hipStream_t s) {
    if (total_tiles == 0) return hipSuccess;
    RasterConsts rc{cfg.alpha_min, cfg.alpha_max, cfg.t_min, cfg.flags, status};
#define SR_TS(W, H)                                                                                               \
    if (cfg.tile_w == W && cfg.tile_h == H) {                                                                    \
        if (!train_launch<W, H>(hits ? (max_alpha ? 2 : 1) : 0, cfg.bwd_batch, total_tiles, s, cams, V, N,      \
                                (const float4*)geom, (const float4*)app, vals, (const uint2*)ranges, rc, mask,   \
                                target, gamma, w_c, color, alpha, depth, normal, dist, T_final, n_contrib, hits, \
                                max_alpha, max_weight, tile_loss, grad_rec, grad_marks, tile_order, tile_cost,  \
                                simds))                                                                          \
            return hipErrorInvalidValue;                                                                         \
        return hipGetLastError();                                                                                \
    }
    SR_TILE_SHAPES(SR_TS)
#undef SR_TS
    return hipErrorInvalidValue;
}

// ---- the allocation-free training step ------------------------------------------
//
// The per-tile loss partials of sr_train_step_raster_noalloc live in this
// file-scope device array (one copy per GPU, held until the process ends)
// instead of a caller buffer.  On the host its name is a stand-in symbol, not
// a device address: host code uses only the address hipGetSymbolAddress
// returns, taken once per device with that device current.
__device__ __align__(256) float scratch[2 * SR_NOALLOC_MAX_TILES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t scratch_address(int device, float** out) {
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_dev[device] = static_cast<float*>(p);
    }
    *out = g_scratch_dev[device];
    return hipSuccess;
}

hipError_t launch_prune_mask(int N, const float* max_alpha, float tau, const uint32_t* status, uint8_t* mask,
                             hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_prune_mask, dim3((N + 255) / 256), dim3(256), 0, s, N, max_alpha, tau, status, mask);
    return hipGetLastError();
}

}  // namespace sr
