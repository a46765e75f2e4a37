// Internal device helpers shared by the surfel rasterizer kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "surfelrast.h"

namespace sr {

constexpr int kGeomF4 = SR_GEOM_STRIDE / 4;   // float4 per geometry record
constexpr int kAppF4 = SR_APP_STRIDE / 4;     // float4 per appearance record
constexpr int kNumGrad = 21;                  // gradient floats per record

// Constants of the compositing rule, passed by value to the raster kernels.
struct RasterConsts {
    float alpha_min;
    float alpha_max;
    float t_min;
    uint32_t flags;
    // the context's device status word (NULL: none); while it is set the
    // instance lists are truncated and the compositing kernels compute nothing
    const uint32_t* status;
};

// The status word's verdict, read once per workgroup (uniform).
__device__ __forceinline__ bool status_failed(const RasterConsts& rc) {
    return rc.status != nullptr && *rc.status != 0u;
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.
// Neighbouring tiles read mostly the same surfel records, so give every XCD a
// contiguous run of tiles: block b of round r = b / 8 on XCD x = b % 8 takes
// tile x * (G / 8) + r.  The last G % 8 blocks keep their own id (bijection).
__device__ __forceinline__ int xcd_tile(int b, int G) {
    const int full = G >> 3;
    if (b >= (full << 3)) return b;
    return (b & 7) * full + (b >> 3);
}

// View that owns a global tile id (views are stored in tile order).
__device__ __forceinline__ int view_of_tile(const sr_camera* __restrict__ cams, int V, int tile) {
    int lo = 0, hi = V - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (cams[mid].tile_offset <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int view_of_group(const sr_camera* __restrict__ cams, int V, int group) {
    int lo = 0, hi = V - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (cams[mid].group_offset <= group) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Sorted instance values: surfel id in the low SR_INST_ID_BITS bits, the
// surfel's tile rectangle clipped to the group (2-bit tile coordinates
// x_lo, x_hi, y_lo, y_hi inside the group) above.
constexpr uint32_t kInstIdMask = (1u << SR_INST_ID_BITS) - 1u;
__device__ __forceinline__ bool inst_covers(uint32_t v, int sx, int sy) {
    const uint32_t sub = v >> SR_INST_ID_BITS;
    // no short circuit: four compares, no branches
    return ((int)(sub & 3u) <= sx) & (sx <= (int)((sub >> 2) & 3u)) & ((int)((sub >> 4) & 3u) <= sy) &
           (sy <= (int)((sub >> 6) & 3u));
}

// ---------------------------------------------------------------------------
// Wavefront (64 lanes) reductions with DPP row operations.  Results land in
// lane 63.  Must be called with all 64 lanes active.
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// Wave maxima of two non-negative floats, compared as their bit patterns
// (which order like the values): the halves of the wave exchange a and b, the
// row pairs exchange again, then each row reduces with DPP.  On return lanes
// 0..31 hold the bits of max(a) over the wave and lanes 32..63 those of max(b).
__device__ __forceinline__ uint32_t wave_max2_bits(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    uint32_t m = r[0] > r[1] ? r[0] : r[1];
    const auto q = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    m = q[0] > q[1] ? q[0] : q[1];
    uint32_t d;
    d = dpp_u<0xB1>(m); m = m > d ? m : d;    // quad_perm [1,0,3,2]
    d = dpp_u<0x4E>(m); m = m > d ? m : d;    // quad_perm [2,3,0,1]
    d = dpp_u<0x141>(m); m = m > d ? m : d;   // row_half_mirror
    d = dpp_u<0x140>(m); m = m > d ? m : d;   // row_mirror
    return m;
}

__device__ __forceinline__ uint64_t ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// old with lane `lane` (uniform) replaced by v (uniform).
__device__ int lane_write(int v, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// ---------------------------------------------------------------------------
// Evaluation of one (pixel, surfel) pair.  Shared verbatim by the forward,
// backward and pruning kernels so that they take identical decisions: every
// operation is written explicitly and contraction is disabled.
//
// Geometry record (16 floats), for pixel centre x and dx = x - c:
//   w = A dx + B dy + C  (w ~ (u, v, 1): inverse of the splat homography),
//   c = projected centre, o = opacity, m3 = (a_u.z, a_v.z, p_z) so that the
//   surface depth is m3 . (u, v, 1), L = ln(o / alpha_min).
//   [A0 A1 A2 B0 | B1 B2 C0 C1 | C2 cx cy o | m30 m31 m32 L]
// An entry passes the alpha cutoff when min(rho_s/2, rho_f) <= L with
// rho_s = u^2 + v^2 and rho_f = |x - c|^2, i.e. o exp(-rho) >= alpha_min.
// ---------------------------------------------------------------------------
struct PairEval {
    float dx, dy, w0, w1, w2, rho_f;
    bool q_ok, w_ok, f_ok, s_ok;
    float r, u, v, rho, G, a, z;   // r = 1/w2
    bool surf, clamped;
};

// A geometry record as the evaluation reads it.
struct SurfelGeom {
    float A0, A1, A2, B0, B1, B2, C0, C1, C2, cx, cy, o, m30, m31, m32, L, L2;   // L2 = 2 L
};

// a b + c.  With a in a scalar register (SCALAR) the result takes a register
// of its own: the compiler would accumulate into c's, which the next record's
// load takes, and copy it out.
template <bool SCALAR>
__device__ __forceinline__ float fma_rec(float a, float b, float c) {
    if (!SCALAR) return __builtin_fmaf(a, b, c);
    float d;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "s"(a), "v"(b), "v"(c));
    return d;
}

// Stage 1: the cutoff test (no division, no exponential).
template <bool SCALAR>
__device__ __forceinline__ void eval_test(const SurfelGeom& s, float px, float py, PairEval& e) {
#pragma clang fp contract(off)
    e.dx = px - s.cx;
    e.dy = py - s.cy;
    e.w0 = __builtin_fmaf(s.A0, e.dx, fma_rec<SCALAR>(s.B0, e.dy, s.C0));
    e.w1 = __builtin_fmaf(s.A1, e.dx, fma_rec<SCALAR>(s.B1, e.dy, s.C1));
    e.w2 = __builtin_fmaf(s.A2, e.dx, fma_rec<SCALAR>(s.B2, e.dy, s.C2));
    e.rho_f = __builtin_fmaf(e.dx, e.dx, e.dy * e.dy);
    const float q = __builtin_fmaf(e.w0, e.w0, e.w1 * e.w1);
    const float w22 = e.w2 * e.w2;
    e.q_ok = q <= s.L2 * w22;
    e.w_ok = e.w2 != 0.0f;
    e.s_ok = e.q_ok && e.w_ok;
    e.f_ok = e.rho_f <= s.L;
}

// The lanes whose pair passes the cutoff, and a lane's own bit of a mask (no
// vector instruction: the mask itself is the condition).
__device__ __forceinline__ uint64_t pass_mask(const PairEval& e) {
    return (ballot64(e.q_ok) & ballot64(e.w_ok)) | ballot64(e.f_ok);
}
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Stage 2: intersection, Gaussian value, alpha and depth of a passing pair.
__device__ __forceinline__ void eval_finish(const SurfelGeom& s, float alpha_max, PairEval& e) {
#pragma clang fp contract(off)
    e.r = __builtin_amdgcn_rcpf(e.w2);
    e.u = e.w0 * e.r;
    e.v = e.w1 * e.r;
    const float rho_s = 0.5f * __builtin_fmaf(e.u, e.u, e.v * e.v);
    e.surf = e.s_ok && (rho_s <= e.rho_f);
    e.rho = e.surf ? rho_s : e.rho_f;
    // exp(-rho) = 2^(-rho log2 e)
    e.G = __builtin_amdgcn_exp2f(-1.4426950408889634f * e.rho);
    const float oG = s.o * e.G;
    e.clamped = oG > alpha_max;
    // min(oG, alpha_max) as the median of (oG, 0, alpha_max): oG >= 0, and
    // one instruction where the select needs the bound in a vector register
    e.a = __builtin_amdgcn_fmed3f(oG, 0.0f, alpha_max);
    e.z = e.surf ? __builtin_fmaf(s.m30, e.u, __builtin_fmaf(s.m31, e.v, s.m32)) : s.m32;
}

// Per-pixel terms of the masked losses (Eq. 1 and the L1 part of Eq. 2) and
// their gradients for L = (1/V) sum_v (w_c L1_v + gamma L_b,v); shared by the
// loss kernel and the fused training step so both round identically.
__device__ __forceinline__ void pixel_loss_grad(uint8_t mask, float A, const float* C, const float* I, float gamma,
                                                float w_c, float HW, float V, float& lb, float& l1, float& gA,
                                                float* gC) {
#pragma clang fp contract(off)
    const float ga = gamma / (HW * V);
    const float gc = w_c / (3.0f * HW * V);
    const float m = mask ? 1.0f : 0.0f;
    lb += A * (1.0f - m);
    gA = ga * (1.0f - m);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float d = m * C[ch] - m * I[ch];
        l1 += fabsf(d);
        gC[ch] = d > 0.f ? gc * m : (d < 0.f ? -gc * m : 0.f);
    }
}

}  // namespace sr
