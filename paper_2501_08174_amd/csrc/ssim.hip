// Masked structural similarity of the rendered and target views: the D-SSIM
// part of the photometric loss of Eq. 2 (the 3DGS loss on M*R and M*I) with
// its gradient, and the masked SSIM / PSNR metrics.
//
//   x = M R, y = M I per colour channel; G = 11x11 Gaussian (sigma 1.5,
//   normalised, separable), correlation with zero padding
//   S(p) = (2 mu_x mu_y + C1)(2 s_xy + C2) / ((mu_x^2 + mu_y^2 + C1)(s_x + s_y + C2))
//   SSIM_v = mean of S over channels and pixels; L = (1/V) sum_v w_s (1 - SSIM_v)
//   PSNR_v = -10 log10(mean (x - y)^2)
//
// Forward: per 32x32 tile and channel, x and y with a five-pixel halo go to
// LDS, a horizontal then a vertical 11-tap pass give the five filtered
// moments, and each pixel forms S and dL/d{mu_x, E[x^2], E[xy]}.  Backward:
// those three maps are filtered the same way (the window is symmetric, so
// the adjoint of the correlation is the same correlation) and combined with
// x and y into dL/dR = M dL/dx.  One flat grid over the (view, channel,
// tile) slots of all views.  A thread forms four neighbouring outputs of
// the horizontal pass (two of the vertical) from a window of values held in
// registers: 8 LDS reads of 16 bytes a quadruple (88 single ones before), the
// products x^2, y^2 and xy once per value; the larger tile filters 1.3 halo
// rows per row instead of 1.6, and the tile's loads are all issued before the
// first is used (one by one, their latency was half of the kernels' time).
// 16 views, 14.6 Mpx: forward 785 -> 530 us, backward 401 -> 313 us, totals
// (a block per view) 177 -> 13 us.  The forward is bound by VALU issue (245M
// wave instructions, most with the tap in a scalar register; such issue at 0.9
// per CU and cycle: 0.44 ms), the backward by the traffic of the
// three gradient maps (36 bytes a pixel written and read) and its latency
// between two barriers (105M, 0.19 ms).
// Per-tile sums are reduced per view in a fixed order.
#include <cmath>

#include "common.h"
#include "launch.h"

namespace sr {

namespace {

constexpr int kNT = 512;
constexpr int kTX = 32, kTY = 32;                     // output tile (two rows per thread)
constexpr int kR = 5;                                 // window radius
constexpr int kHX = kTX + 2 * kR, kHY = kTY + 2 * kR; // tile with halo
constexpr int kSX = (kHX + 3) / 4 * 4;                // row stride in LDS: 16-byte rows
constexpr int kQ = 4, kV = 2;                         // outputs a thread forms in a horizontal / vertical pass
constexpr int kWin = kQ + 2 * kR;                     // the window of values four outputs need
static_assert(kTX * kTY == kV * kNT && kTX == 32, "one column of kV outputs per thread");
static_assert(kHY * (kTX / kQ) <= kNT, "one horizontal quadruple per thread");
constexpr float kC1 = 0.01f * 0.01f, kC2 = 0.03f * 0.03f;

struct Taps {
    float g[2 * kR + 1];
};

__host__ __device__ inline int tiles_of(int W, int H) { return ((W + kTX - 1) / kTX) * ((H + kTY - 1) / kTY); }

// Sums of two values over the block, in a fixed order (wave, then waves);
// valid in thread 0.
__device__ __forceinline__ float2 block_sum2(float a, float b, float2* s) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if (__lane_id() == 0) s[threadIdx.x >> 6] = make_float2(a, b);
    __syncthreads();
    float2 r = s[0];
#pragma unroll
    for (int w = 1; w < kNT / 64; ++w) {
        r.x += s[w].x;
        r.y += s[w].y;
    }
    return r;
}

// The window of values from p on (16-byte aligned, readable to the next
// multiple of four).
__device__ __forceinline__ void load_window(const float* p, float (&v)[kWin]) {
    static_assert(kWin == 14, "three whole quadruples and a half");
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const float4 t = reinterpret_cast<const float4*>(p)[q];
        v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
    }
    const float2 t = reinterpret_cast<const float2*>(p)[6];
    v[12] = t.x; v[13] = t.y;
}

// The n outputs of a window of n + 2 kR values.
template <int n>
__device__ __forceinline__ void filter(const Taps& taps, const float (&v)[n + 2 * kR], float (&o)[n]) {
#pragma unroll
    for (int k = 0; k < n; ++k) {
        o[k] = 0.f;
#pragma unroll
        for (int d = 0; d <= 2 * kR; ++d) o[k] = __builtin_fmaf(taps.g[d], v[k + d], o[k]);
    }
}

__device__ __forceinline__ void store4(float* p, const float (&o)[kQ]) {
    *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
}

// The kV vertical outputs from row r on of column x.
__device__ __forceinline__ void filter_column(const Taps& taps, const float (&m)[kHY][kTX], int r, int x,
                                              float (&o)[kV]) {
    float v[kV + 2 * kR];
#pragma unroll
    for (int d = 0; d < kV + 2 * kR; ++d) v[d] = m[r + d][x];
    filter<kV>(taps, v, o);
}

// Tile, channel and view of this workgroup (slot = its index among the
// view's 3 * tiles slots); false past the last view.
struct SsimTile {
    int v, ch, x0, y0, W, H, slot;
    int64_t HW, off;
};

__device__ __forceinline__ bool ssim_tile(const sr_camera* cams, int V, SsimTile& t) {
    int b = (int)blockIdx.x, v = 0;
    for (; v < V; ++v) {
        const int ns = 3 * tiles_of(cams[v].width, cams[v].height);
        if (b < ns) break;
        b -= ns;
    }
    if (v >= V) return false;
    t.v = v;
    const sr_camera& c = cams[t.v];
    t.W = c.width;
    t.H = c.height;
    const int nt = tiles_of(t.W, t.H);
    t.ch = b / nt;
    const int tile = b - t.ch * nt;
    const int ntx = (t.W + kTX - 1) / kTX;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    t.x0 = tx * kTX;
    t.y0 = ty * kTY;
    t.HW = (int64_t)t.W * t.H;
    t.off = c.pix_offset;
    t.slot = b;
    return true;
}

// Calls f(k, inside, p) for this thread's values of the tile with halo: k is
// the position in an LDS array, p the pixel (clamped to the image; 64 bits, a
// view may hold more than 2^31 pixels).  Unrolled: every load of a pass over
// the values is issued before the first is used.
constexpr int kLoads = (kHX * kHY + kNT - 1) / kNT;
template <typename F>
__device__ __forceinline__ void for_halo(const SsimTile& t, F&& f) {
#pragma unroll
    for (int r = 0; r < kLoads; ++r) {
        const int k = r * kNT + (int)threadIdx.x;
        const int ly = k / kHX, lx = k - ly * kHX;
        const int i = t.x0 - kR + lx, j = t.y0 - kR + ly;
        const bool in = k < kHX * kHY && i >= 0 && i < t.W && j >= 0 && j < t.H;
        f(r, k < kHX * kHY ? ly * kSX + lx : -1, in, in ? (int64_t)j * t.W + i : (int64_t)0);
    }
}

// Masked inputs of the tile and its halo (zero outside the image).
__device__ __forceinline__ void load_xy(const SsimTile& t, const float* __restrict__ C, const float* __restrict__ I,
                                        const uint8_t* __restrict__ M, float (&sx)[kHY][kSX],
                                        float (&sy)[kHY][kSX]) {
    float xv[kLoads], yv[kLoads];
    uint8_t mv[kLoads];
    for_halo(t, [&](int r, int, bool, int64_t p) {
        xv[r] = C[p];
        yv[r] = I[p];
        mv[r] = M[p];
    });
    for_halo(t, [&](int r, int k, bool in, int64_t) {
        const float m = mv[r] ? 1.0f : 0.0f;
        if (k >= 0) {
            (&sx[0][0])[k] = in ? m * xv[r] : 0.f;
            (&sy[0][0])[k] = in ? m * yv[r] : 0.f;
        }
    });
}

__global__ void __launch_bounds__(kNT)
k_ssim_fwd(const sr_camera* __restrict__ cams, int V, const float* __restrict__ color,
           const float* __restrict__ target, const uint8_t* __restrict__ mask, Taps taps, float w_s, int nslot,
           int64_t P3, float* __restrict__ partial, float* __restrict__ gmaps) {
#pragma clang fp contract(off)
    __shared__ __align__(16) float sx[kHY][kSX], sy[kHY][kSX];
    __shared__ __align__(16) float sh[5][kHY][kTX];
    __shared__ float2 s_red[kNT / 64];
    SsimTile t;
    if (!ssim_tile(cams, V, t)) return;               // uniform: the whole block leaves
    const int64_t base = 3 * t.off + t.ch * t.HW;     // this channel of this view in [3P] arrays
    load_xy(t, color + base, target + base, mask + t.off, sx, sy);
    __syncthreads();
    if ((int)threadIdx.x < kHY * (kTX / kQ)) {
        const int ly = (int)threadIdx.x / (kTX / kQ), x0 = kQ * ((int)threadIdx.x % (kTX / kQ));
        float xv[kWin], yv[kWin], p[kWin], o[kQ];
        load_window(&sx[ly][x0], xv);
        load_window(&sy[ly][x0], yv);
        filter<kQ>(taps, xv, o);
        store4(&sh[0][ly][x0], o);
        filter<kQ>(taps, yv, o);
        store4(&sh[1][ly][x0], o);
#pragma unroll
        for (int d = 0; d < kWin; ++d) p[d] = xv[d] * xv[d];
        filter<kQ>(taps, p, o);
        store4(&sh[2][ly][x0], o);
#pragma unroll
        for (int d = 0; d < kWin; ++d) p[d] = yv[d] * yv[d];
        filter<kQ>(taps, p, o);
        store4(&sh[3][ly][x0], o);
#pragma unroll
        for (int d = 0; d < kWin; ++d) p[d] = xv[d] * yv[d];
        filter<kQ>(taps, p, o);
        store4(&sh[4][ly][x0], o);
    }
    __syncthreads();
    const int lx = (int)threadIdx.x % kTX, r0 = (int)threadIdx.x / kTX * kV;
    float mom[5][kV];
#pragma unroll
    for (int m = 0; m < 5; ++m) filter_column(taps, sh[m], r0, lx, mom[m]);
    float ssum = 0.f, se = 0.f;
#pragma unroll
    for (int k = 0; k < kV; ++k) {
      const int ly = r0 + k;
      const int i = t.x0 + lx, j = t.y0 + ly;
      if (i < t.W && j < t.H) {
        const float mx = mom[0][k], my = mom[1][k], ex2 = mom[2][k], ey2 = mom[3][k], exy = mom[4][k];
        const float vx = ex2 - mx * mx, vy = ey2 - my * my, cxy = exy - mx * my;
        const float A1 = 2.0f * mx * my + kC1, A2 = 2.0f * cxy + kC2;
        const float B1 = mx * mx + my * my + kC1, B2 = (vx + vy) + kC2;
        const float inv = 1.0f / (B1 * B2);            // the one division: 1 / B1 = B2 inv, 1 / B2 = B1 inv
        const float S = (A1 * A2) * inv;
        ssum += S;
        const float xv = sx[ly + kR][lx + kR], yv = sy[ly + kR][lx + kR];
        se += (xv - yv) * (xv - yv);
        if (gmaps) {
            // dL/dS = -w_s / (3 H W V); chain through A1, A2, B1, B2
            const float dS = -w_s / (3.0f * (float)t.HW * (float)V);
            const float sa1 = A2 * inv, sa2 = A1 * inv;              // S / A1, S / A2
            const float sb1 = S * (B2 * inv), sb2 = S * (B1 * inv);  // S / B1, S / B2
            const float d_mx = ((sa1 * (2.0f * my) - sa2 * (2.0f * my)) - sb1 * (2.0f * mx)) + sb2 * (2.0f * mx);
            const float d_ex2 = -sb2;
            const float d_exy = 2.0f * sa2;
            const int64_t p = base + (int64_t)j * t.W + i;
            gmaps[p] = dS * d_mx;
            gmaps[P3 + p] = dS * d_ex2;
            gmaps[2 * P3 + p] = dS * d_exy;
        }
      }
    }
    const float2 sum = block_sum2(ssum, se, s_red);
    if (threadIdx.x == 0) {
        partial[2 * ((size_t)t.v * nslot + t.slot)] = sum.x;
        partial[2 * ((size_t)t.v * nslot + t.slot) + 1] = sum.y;
    }
}

// dL/dx = G*g1 + 2 x G*g2 + y G*g3; dL/dR += M dL/dx
__global__ void __launch_bounds__(kNT)
k_ssim_bwd(const sr_camera* __restrict__ cams, int V, const float* __restrict__ color,
           const float* __restrict__ target,
           const uint8_t* __restrict__ mask, Taps taps, int64_t P3, const float* __restrict__ gmaps,
           float* __restrict__ dL_dcolor) {
#pragma clang fp contract(off)
    __shared__ __align__(16) float sg[3][kHY][kSX];
    __shared__ __align__(16) float sh[3][kHY][kTX];
    SsimTile t;
    if (!ssim_tile(cams, V, t)) return;
    const int64_t base = 3 * t.off + t.ch * t.HW;
    {
        const float* g = gmaps + base;
        float v[3][kLoads];
        for_halo(t, [&](int r, int, bool, int64_t p) {
            v[0][r] = g[p];
            v[1][r] = g[P3 + p];
            v[2][r] = g[2 * P3 + p];
        });
        for_halo(t, [&](int r, int k, bool in, int64_t) {
#pragma unroll
            for (int m = 0; m < 3; ++m)
                if (k >= 0) (&sg[m][0][0])[k] = in ? v[m][r] : 0.f;
        });
    }
    __syncthreads();
    if ((int)threadIdx.x < kHY * (kTX / kQ)) {
        const int ly = (int)threadIdx.x / (kTX / kQ), x0 = kQ * ((int)threadIdx.x % (kTX / kQ));
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float v[kWin], o[kQ];
            load_window(&sg[m][ly][x0], v);
            filter<kQ>(taps, v, o);
            store4(&sh[m][ly][x0], o);
        }
    }
    __syncthreads();
    const int lx = (int)threadIdx.x % kTX, r0 = (int)threadIdx.x / kTX * kV;
    float f[3][kV];
#pragma unroll
    for (int m = 0; m < 3; ++m) filter_column(taps, sh[m], r0, lx, f[m]);
#pragma unroll
    for (int k = 0; k < kV; ++k) {
      const int i = t.x0 + lx, j = t.y0 + r0 + k;
      if (i < t.W && j < t.H) {
        const int64_t q = (int64_t)j * t.W + i;
        if (mask[t.off + q]) {
            const float xv = color[base + q], yv = target[base + q];
            const float dx = (f[0][k] + 2.0f * xv * f[1][k]) + yv * f[2][k];
            dL_dcolor[base + q] += dx;
        }
      }
    }
}

// out[v] = SSIM_v, out[V+v] = PSNR_v (one block per view); the total of a
// single view, written with its terms (one launch less)
__global__ void __launch_bounds__(kNT)
k_ssim_final(const sr_camera* __restrict__ cams, int V, int nslot, const float* __restrict__ partial, float w_s,
             float* __restrict__ out) {
    __shared__ float2 s[kNT / 64];
    const int v = blockIdx.x;
    const int ns = 3 * tiles_of(cams[v].width, cams[v].height);
    float a = 0.f, b = 0.f;
    for (int i = threadIdx.x; i < ns; i += kNT) {
        a += partial[2 * ((size_t)v * nslot + i)];
        b += partial[2 * ((size_t)v * nslot + i) + 1];
    }
    const float2 sum = block_sum2(a, b, s);
    if (threadIdx.x == 0) {
        const float n = 3.0f * (float)cams[v].width * (float)cams[v].height;
        const float ssim = sum.x / n;
        out[v] = ssim;
        out[V + v] = -10.0f * log10f(sum.y / n);
        if (V == 1) out[2] = w_s * (1.0f - ssim);
    }
}

// out[2V] = (1/V) sum_v w_s (1 - SSIM_v), in a fixed order
__global__ void __launch_bounds__(kNT)
k_ssim_total(int V, float w_s, float* __restrict__ out) {
    __shared__ float2 s[kNT / 64];
    float t = 0.f;
    for (int v = threadIdx.x; v < V; v += kNT) t += w_s * (1.0f - out[v]);
    const float2 sum = block_sum2(t, 0.f, s);
    if (threadIdx.x == 0) out[2 * V] = sum.x / (float)V;
}

Taps make_taps() {
    Taps t;
    double g[2 * kR + 1], sum = 0.0;
    for (int k = 0; k <= 2 * kR; ++k) {
        const double d = (double)(k - kR);
        g[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
        sum += g[k];
    }
    for (int k = 0; k <= 2 * kR; ++k) t.g[k] = (float)(g[k] / sum);
    return t;
}

}  // namespace

int ssim_slots(int W, int H) { return 3 * tiles_of(W, H); }

size_t ssim_workspace_bytes(int V, int max_slots, int64_t P, bool with_grad) {
    size_t b = (size_t)V * (size_t)max_slots * 2 * sizeof(float);
    b = (b + 255) & ~size_t(255);
    if (with_grad) b += (size_t)3 * 3 * (size_t)P * sizeof(float);
    return b;
}

hipError_t launch_ssim(int V, int max_slots, int total_slots, int64_t P, const sr_camera* cams, const float* color,
                       const float* target, const uint8_t* mask, float w_s, void* ws, float* out,
                       float* dL_dcolor, hipStream_t s) {
    if (V == 0 || max_slots == 0) return hipSuccess;
    const Taps taps = make_taps();
    float* partial = (float*)ws;
    size_t pb = (size_t)V * (size_t)max_slots * 2 * sizeof(float);
    pb = (pb + 255) & ~size_t(255);
    float* gmaps = dL_dcolor ? (float*)((char*)ws + pb) : nullptr;
    const int64_t P3 = 3 * P;
    hipLaunchKernelGGL(k_ssim_fwd, dim3(total_slots), dim3(kNT), 0, s, cams, V, color, target, mask, taps, w_s,
                       max_slots, P3, partial, gmaps);
    if (dL_dcolor)
        hipLaunchKernelGGL(k_ssim_bwd, dim3(total_slots), dim3(kNT), 0, s, cams, V, color, target, mask, taps, P3,
                           (const float*)gmaps, dL_dcolor);
    hipLaunchKernelGGL(k_ssim_final, dim3(V), dim3(kNT), 0, s, cams, V, max_slots, (const float*)partial, w_s, out);
    if (V > 1) hipLaunchKernelGGL(k_ssim_total, dim3(1), dim3(kNT), 0, s, V, w_s, out);
    return hipGetLastError();
}

}  // namespace sr
