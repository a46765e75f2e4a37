// Masked losses on the rendered views (Section 4.2):
//   background loss (Eq. 1)   L_b,v = (1/(H W)) sum_p A(p) (1 - M(p))
//   masked photometric L1 (Eq. 2, L1 part)  L1_v = (1/(3 H W)) sum |M C - M I|
// and the gradients of L = (1/V) sum_v (w_c L1_v + gamma L_b,v).
// Per-view sums use a fixed two-stage reduction order (deterministic).
#include "common.h"
#include "launch.h"

namespace sr {

namespace {

constexpr int kNT = 256;
constexpr int kChunk = 8192;   // pixels per block of the first stage

__device__ __forceinline__ float block_sum(float v, float* s) {
    // fixed-order tree over the 256 threads
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = kNT / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    const float r = s[0];
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(kNT)
k_loss_partial(const sr_camera* __restrict__ cams, int V, const float* __restrict__ alpha,
               const uint8_t* __restrict__ mask, const float* __restrict__ color, const float* __restrict__ target,
               float gamma, float w_c, int nchunk, float* __restrict__ partial, float* __restrict__ dL_dalpha,
               float* __restrict__ dL_dcolor) {
    __shared__ float s[kNT];
    const int v = blockIdx.y;
    const sr_camera& c = cams[v];
    const int64_t HW = (int64_t)c.width * c.height;
    const int64_t b = (int64_t)blockIdx.x * kChunk;
    float lb = 0.f, l1 = 0.f;
    if (b < HW) {
        const int64_t e = b + kChunk < HW ? b + kChunk : HW;
        for (int64_t p = b + threadIdx.x; p < e; p += kNT) {
            const int64_t o1 = c.pix_offset + p;
            const int64_t o3 = 3 * c.pix_offset + p;
            float C[3] = {0.f, 0.f, 0.f}, I[3] = {0.f, 0.f, 0.f}, gC[3], gA;
            if (color) {
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    C[ch] = color[o3 + ch * HW];
                    I[ch] = target[o3 + ch * HW];
                }
            }
            float l1p = 0.f;
            pixel_loss_grad(mask[o1], alpha[o1], C, I, gamma, w_c, (float)HW, (float)V, lb, l1p, gA, gC);
            if (dL_dalpha) dL_dalpha[o1] = gA;
            if (color) {
                l1 += l1p;
                if (dL_dcolor) {
#pragma unroll
                    for (int ch = 0; ch < 3; ++ch) dL_dcolor[o3 + ch * HW] = gC[ch];
                }
            }
        }
    }
    lb = block_sum(lb, s);
    l1 = block_sum(l1, s);
    if (threadIdx.x == 0) {
        partial[2 * ((size_t)v * nchunk + blockIdx.x)] = lb;
        partial[2 * ((size_t)v * nchunk + blockIdx.x) + 1] = l1;
    }
}

// The total of a single view, written with its terms (one launch less).
__device__ __forceinline__ void one_view_total(float a, float wa, float b, float wb, float* __restrict__ loss) {
    loss[2] = wa * a + wb * b;
}

__global__ void __launch_bounds__(kNT)
k_loss_final(const sr_camera* __restrict__ cams, int V, int nchunk, const float* __restrict__ partial, float gamma,
             float w_c, float* __restrict__ loss) {
    __shared__ float s[kNT];
    const int v = blockIdx.x;
    float lb = 0.f, l1 = 0.f;
    for (int i = threadIdx.x; i < nchunk; i += kNT) {
        lb += partial[2 * ((size_t)v * nchunk + i)];
        l1 += partial[2 * ((size_t)v * nchunk + i) + 1];
    }
    lb = block_sum(lb, s);
    l1 = block_sum(l1, s);
    if (threadIdx.x == 0) {
        const float HW = (float)cams[v].width * (float)cams[v].height;
        loss[v] = lb / HW;
        loss[V + v] = l1 / (3.0f * HW);
        if (V == 1) one_view_total(loss[1], w_c, loss[0], gamma, loss);
    }
}

// loss[2V] = (1/V) sum_v (w_c L1_v + gamma L_b,v), summed in view order
__global__ void __launch_bounds__(kNT)
k_loss_total(int V, float gamma, float w_c, float* __restrict__ loss) {
    __shared__ float s[kNT];
    float t = 0.f;
    for (int v = threadIdx.x; v < V; v += kNT) t += w_c * loss[V + v] + gamma * loss[v];
    t = block_sum(t, s);
    if (threadIdx.x == 0) loss[2 * V] = t / (float)V;
}

// Per-view totals from the per-tile partial sums of the fused training step
// (tiles of a view are contiguous), summed in tile order.
__global__ void __launch_bounds__(kNT)
k_loss_tiles(const sr_camera* __restrict__ cams, int V, const float* __restrict__ tile_loss, float gamma, float w_c,
             float* __restrict__ loss) {
    __shared__ float s[kNT];
    const int v = blockIdx.x;
    const sr_camera& c = cams[v];
    const int T0 = c.tile_offset, nt = c.tiles_x * c.tiles_y;
    float lb = 0.f, l1 = 0.f;
    for (int i = threadIdx.x; i < nt; i += kNT) {
        lb += tile_loss[2 * (size_t)(T0 + i)];
        l1 += tile_loss[2 * (size_t)(T0 + i) + 1];
    }
    lb = block_sum(lb, s);
    l1 = block_sum(l1, s);
    if (threadIdx.x == 0) {
        const float HW = (float)c.width * (float)c.height;
        loss[v] = lb / HW;
        loss[V + v] = l1 / (3.0f * HW);
        if (V == 1) one_view_total(loss[1], w_c, loss[0], gamma, loss);
    }
}

// ---- 2DGS regularisers of the total loss (Eq. 3) ---------------------------
//   L_d,v = mean_p dist(p)
//   L_n,v = mean_p (A(p) - N(p) . N_d(p)),  N_d from central differences of
//           the camera-space points P = s ray, zero on the one-pixel border;
//           the surface depth s is D / A (0 where A = 0) or, when a median
//           depth map is given, the median depth (its gradient then goes to
//           that map and none to D)
//   L_reg = (1/V) sum_v (w_dist L_d,v + w_normal L_n,v)
// One workgroup per 32x16 pixel tile of a view: the camera-space points of
// the tile and a two-pixel halo are formed once in LDS, then the depth
// normals of the tile and a one-pixel halo with the two vectors every normal
// passes back to its neighbours' points (the gradient through n = a x b),
// then each pixel gathers its point's gradient from its four neighbours.
// Each pixel writes only its own gradients (no atomics); per-tile loss sums
// go to a per-(view, tile) slot and are reduced in a fixed order.

constexpr float kEpsNormal = 1e-12f;
constexpr int kRegTX = 32, kRegTY = 16;                // tile: two rows per thread
constexpr int kRegPX = kRegTX + 4, kRegPY = kRegTY + 4; // points: two-pixel halo
constexpr int kRegNX = kRegTX + 2, kRegNY = kRegTY + 2; // normals: one-pixel halo

__device__ __forceinline__ float3 f3sub(float3 a, float3 b) { return make_float3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ __forceinline__ float3 f3cross(float3 a, float3 b) {
#pragma clang fp contract(off)
    return make_float3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float f3dot(float3 a, float3 b) {
#pragma clang fp contract(off)
    return a.x * b.x + a.y * b.y + a.z * b.z;
}

// n / d from inv = 1 / d, d > 0: the product corrected by its remainder is the
// rounded quotient (Markstein), in four operations instead of a division's
// ten, where the reciprocal and the quotient are normal numbers (or the
// quotient is zero).  ok is cleared where they are not: reciprocals of d below
// 2.9e-39 overflow, those above 8.5e37 are subnormal, and infinities and NaNs
// have no remainder.
__device__ __forceinline__ float quotient(float n, float d, float inv, bool& ok) {
    constexpr int kNormal = 0x108, kZero = 0x60;      // of either sign, as v_cmp_class counts them
    const float q = n * inv, c = __builtin_fmaf(__builtin_fmaf(-q, d, n), inv, q);
    ok = ok && __builtin_amdgcn_classf(inv, kNormal) && __builtin_amdgcn_classf(c, kNormal | kZero);
    return c;
}

// The quotients of three numbers by d; the division itself, in a branch that
// ordinary maps do not enter, where the above does not hold for one of them.
__device__ __forceinline__ float3 quotient3(float3 n, float d, float inv) {
    bool ok = true;
    float3 c = make_float3(quotient(n.x, d, inv, ok), quotient(n.y, d, inv, ok), quotient(n.z, d, inv, ok));
    if (!ok) c = make_float3(n.x / d, n.y / d, n.z / d);
    return c;
}

__host__ __device__ inline int reg_tiles_of(int W, int H) {
    return ((W + kRegTX - 1) / kRegTX) * ((H + kRegTY - 1) / kRegTY);
}
__device__ __forceinline__ int reg_tiles(int W, int H) { return reg_tiles_of(W, H); }

__global__ void __launch_bounds__(kNT)
k_reg_partial(const sr_camera* __restrict__ cams, int V, const float* __restrict__ alpha,
              const float* __restrict__ depth, const float* __restrict__ normal, const float* __restrict__ dist,
              const float* __restrict__ median, float w_dist, float w_normal, int nslot, float* __restrict__ partial,
              float* __restrict__ dL_dalpha, float* __restrict__ dL_ddepth, float* __restrict__ dL_dnormal,
              float* __restrict__ dL_ddist, float* __restrict__ dL_dmedian) {
#pragma clang fp contract(off)
    // Bound by memory (52 bytes a pixel) and, before, by latency and IEEE
    // divisions (18 a pixel with the halo's): every load of the tile is now
    // issued at the start, the rays are formed once per column and row, and a
    // normal, its gradient and a pixel's depth gradient take one division each.
    // 8 views of 1237x822: 195 -> 145 us.
    constexpr int kPts = (kRegPX * kRegPY + kNT - 1) / kNT, kNrm = (kRegNX * kRegNY + kNT - 1) / kNT;
    constexpr int kPix = kRegTX * kRegTY / kNT, kStep = kNT / kRegTX;      // pixels of a thread, rows apart
    __shared__ float2 s_red[kNT / 64];
    __shared__ float sRx[kRegPX], sRy[kRegPY];
    __shared__ float3 sP[kRegPY][kRegPX];
    __shared__ float3 sGa[kRegNY][kRegNX], sGb[kRegNY][kRegNX], sNd[kRegNY][kRegNX];
    // one flat grid over the tiles of all views
    int v = 0, tile = (int)blockIdx.x;
    for (; v < V; ++v) {
        const int nt = reg_tiles(cams[v].width, cams[v].height);
        if (tile < nt) break;
        tile -= nt;
    }
    if (v >= V) return;                                     // uniform: the whole block leaves
    const sr_camera& c = cams[v];
    const int W = c.width, H = c.height;
    const int ntx = (W + kRegTX - 1) / kRegTX;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    const int x0 = tx * kRegTX, y0 = ty * kRegTY;
    const int64_t HW = (int64_t)W * H;
    const float* A = alpha + c.pix_offset;
    const float* D = depth + c.pix_offset;
    const float* Md = median ? median + c.pix_offset : nullptr;
    const float* Nr = normal + 3 * c.pix_offset;
    const float scale = 1.0f / ((float)HW * (float)V);
    const float gn = w_normal * scale;
    // loads, at clamped positions: nothing below waits for the one before it
    float ld_a[kPts], ld_d[kPts];
    float3 ld_n[kNrm];
    float px_dist[kPix], px_ga[kPix];
#pragma unroll
    for (int r = 0; r < kPts; ++r) {
        const int k = r * kNT + (int)threadIdx.x, ly = k / kRegPX, lx = k - ly * kRegPX;
        const int i = x0 - 2 + lx, j = y0 - 2 + ly;
        const bool in = k < kRegPX * kRegPY && i >= 0 && i < W && j >= 0 && j < H;
        const int64_t p = in ? (int64_t)j * W + i : 0;
        ld_a[r] = A[p];
        ld_d[r] = Md ? Md[p] : D[p];
    }
#pragma unroll
    for (int r = 0; r < kNrm; ++r) {
        const int k = r * kNT + (int)threadIdx.x, ly = k / kRegNX, lx = k - ly * kRegNX;
        const int i = x0 - 1 + lx, j = y0 - 1 + ly;
        const bool in = k < kRegNX * kRegNY && i >= 0 && i < W && j >= 0 && j < H;
        const int64_t p = in ? (int64_t)j * W + i : 0;
        ld_n[r] = make_float3(Nr[p], Nr[p + HW], Nr[p + 2 * HW]);
    }
    const int lx = (int)threadIdx.x % kRegTX, ly0 = (int)threadIdx.x / kRegTX;
#pragma unroll
    for (int q = 0; q < kPix; ++q) {
        const int i = x0 + lx, j = y0 + ly0 + q * kStep;
        const int64_t o1 = c.pix_offset + (i < W && j < H ? (int64_t)j * W + i : 0);
        px_dist[q] = dist[o1];
        px_ga[q] = dL_dalpha[o1];
    }
    if (threadIdx.x < kRegPX) sRx[threadIdx.x] = ((float)(x0 - 2 + (int)threadIdx.x) + 0.5f - c.cx) / c.fx;
    else if (threadIdx.x >= 64 && threadIdx.x < 64 + kRegPY)
        sRy[threadIdx.x - 64] = ((float)(y0 - 2 + (int)threadIdx.x - 64) + 0.5f - c.cy) / c.fy;
    __syncthreads();
    // points P = s ray of the tile and a two-pixel halo (0 outside)
#pragma unroll
    for (int r = 0; r < kPts; ++r) {
        const int k = r * kNT + (int)threadIdx.x, ly = k / kRegPX, lxx = k - ly * kRegPX;
        if (k >= kRegPX * kRegPY) continue;
        const int i = x0 - 2 + lxx, j = y0 - 2 + ly;
        float3 P = make_float3(0.f, 0.f, 0.f);
        if (i >= 0 && i < W && j >= 0 && j < H) {
            const float sd = Md ? ld_d[r] : (ld_a[r] > 0.f ? ld_d[r] / ld_a[r] : 0.f);
            P = make_float3(sd * sRx[lxx], sd * sRy[ly], sd);
        }
        sP[ly][lxx] = P;
    }
    __syncthreads();
    // depth normals of the tile and a one-pixel halo; the vectors b x dn and
    // dn x a that each normal sends to the points of its neighbours
#pragma unroll
    for (int r = 0; r < kNrm; ++r) {
        const int k = r * kNT + (int)threadIdx.x, ly = k / kRegNX, lxx = k - ly * kRegNX;
        if (k >= kRegNX * kRegNY) continue;
        const int i = x0 - 1 + lxx, j = y0 - 1 + ly;
        float3 nd = make_float3(0.f, 0.f, 0.f), ga = nd, gb = nd;
        if (i >= 1 && i <= W - 2 && j >= 1 && j <= H - 2) {
            const int px = lxx + 1, py = ly + 1;             // position in sP
            const float3 a = f3sub(sP[py + 1][px], sP[py - 1][px]);
            const float3 b = f3sub(sP[py][px + 1], sP[py][px - 1]);
            const float3 n = f3cross(a, b);
            const float len = sqrtf(f3dot(n, n));
            const bool some = len > kEpsNormal;
            const float den = some ? len : kEpsNormal, inv = 1.0f / den;
            nd = quotient3(n, den, inv);
            const float3 g = make_float3(-gn * ld_n[r].x, -gn * ld_n[r].y, -gn * ld_n[r].z);
            // dL/dn: the part across nd, or all of g where the length is the
            // constant (also that of a NaN normal, whose nd stays out of it)
            const float kk = f3dot(nd, g);
            const float3 along = some ? make_float3(nd.x * kk, nd.y * kk, nd.z * kk) : make_float3(0.f, 0.f, 0.f);
            const float3 dn = quotient3(f3sub(g, along), den, inv);
            ga = f3cross(b, dn);                             // dL/da
            gb = f3cross(dn, a);                             // dL/db
        }
        sNd[ly][lxx] = nd;
        sGa[ly][lxx] = ga;
        sGb[ly][lxx] = gb;
    }
    __syncthreads();
    float ld = 0.f, ln = 0.f;
#pragma unroll
    for (int q = 0; q < kPix; ++q) {
        const int ly = ly0 + q * kStep;
        const int i = x0 + lx, j = y0 + ly;
        if (i >= W || j >= H) continue;
        const int64_t p = (int64_t)j * W + i;
        const int64_t o1 = c.pix_offset + p, o3 = 3 * c.pix_offset + p;
        const int nx = lx + 1, ny = ly + 1;                  // position in the normal arrays
        const float3 nd = sNd[ny][nx];
        const float a = A[p];
        const float3 N = make_float3(Nr[p], Nr[p + HW], Nr[p + 2 * HW]);
        ld += px_dist[q];
        ln += a - f3dot(N, nd);
        // this point is P(i, j+1) of the normal above, P(i, j-1) of the one
        // below, P(i+1, j) of the left one and P(i-1, j) of the right one
        const float3 u = sGa[ny - 1][nx], dw = sGa[ny + 1][nx], l = sGb[ny][nx - 1], r = sGb[ny][nx + 1];
        const float3 dP = make_float3(((u.x - dw.x) + l.x) - r.x, ((u.y - dw.y) + l.y) - r.y,
                                      ((u.z - dw.z) + l.z) - r.z);
        const float ds = f3dot(dP, make_float3(sRx[lx + 2], sRy[ly + 2], 1.0f));
        float gA = gn, gD = 0.f;
        if (Md) {
            dL_dmedian[o1] = ds;
        } else if (a > 0.f) {
            const float inv = 1.0f / a, dz = ds * sP[ly + 2][lx + 2].z;      // the point's z is D / A
            bool ok = true;
            gD = quotient(ds, a, inv, ok);
            float gz = quotient(dz, a, inv, ok);
            if (!ok) {
                gD = ds / a;
                gz = dz / a;
            }
            gA = gA - gz;
        }
        dL_dalpha[o1] = px_ga[q] + gA;
        dL_ddepth[o1] = gD;
        dL_dnormal[o3] = -gn * nd.x;
        dL_dnormal[o3 + HW] = -gn * nd.y;
        dL_dnormal[o3 + 2 * HW] = -gn * nd.z;
        dL_ddist[o1] = w_dist * scale;
    }
    // per-tile sums in a fixed order: over the wave, then the waves
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        ld += __shfl_xor(ld, off, 64);
        ln += __shfl_xor(ln, off, 64);
    }
    if (__lane_id() == 0) s_red[threadIdx.x >> 6] = make_float2(ld, ln);
    __syncthreads();
    if (threadIdx.x == 0) {
        float2 sum = s_red[0];
#pragma unroll
        for (int w = 1; w < kNT / 64; ++w) {
            sum.x += s_red[w].x;
            sum.y += s_red[w].y;
        }
        partial[2 * ((size_t)v * nslot + tile)] = sum.x;
        partial[2 * ((size_t)v * nslot + tile) + 1] = sum.y;
    }
}

// loss[v] = L_d,v, loss[V+v] = L_n,v from the chunk partials; loss[2V] total
__global__ void __launch_bounds__(kNT)
k_reg_final(const sr_camera* __restrict__ cams, int V, int nslot, const float* __restrict__ partial, float w_dist,
            float w_normal, float* __restrict__ loss) {
    __shared__ float s[kNT];
    const int v = blockIdx.x;
    const int nt = reg_tiles(cams[v].width, cams[v].height);
    float ld = 0.f, ln = 0.f;
    for (int i = threadIdx.x; i < nt; i += kNT) {
        ld += partial[2 * ((size_t)v * nslot + i)];
        ln += partial[2 * ((size_t)v * nslot + i) + 1];
    }
    ld = block_sum(ld, s);
    ln = block_sum(ln, s);
    if (threadIdx.x == 0) {
        const float HW = (float)cams[v].width * (float)cams[v].height;
        loss[v] = ld / HW;
        loss[V + v] = ln / HW;
        if (V == 1) one_view_total(loss[0], w_dist, loss[1], w_normal, loss);
    }
}

__global__ void __launch_bounds__(kNT)
k_reg_total(int V, float w_dist, float w_normal, float* __restrict__ loss) {
    __shared__ float s[kNT];
    float t = 0.f;
    for (int v = threadIdx.x; v < V; v += kNT) t += w_dist * loss[v] + w_normal * loss[V + v];
    t = block_sum(t, s);
    if (threadIdx.x == 0) loss[2 * V] = t / (float)V;
}

}  // namespace

int reg_tile_count(int W, int H) { return reg_tiles_of(W, H); }

hipError_t launch_reg_loss(int V, int max_tiles, int total_tiles, const sr_camera* cams, const float* alpha,
                           const float* depth,
                           const float* normal, const float* dist, const float* median, float w_dist,
                           float w_normal, void* ws, float* loss, float* dL_dalpha, float* dL_ddepth,
                           float* dL_dnormal, float* dL_ddist, float* dL_dmedian, hipStream_t s) {
    if (V == 0 || max_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_reg_partial, dim3(total_tiles), dim3(kNT), 0, s, cams, V, alpha, depth, normal, dist,
                       median, w_dist, w_normal, max_tiles, (float*)ws, dL_dalpha, dL_ddepth, dL_dnormal, dL_ddist,
                       dL_dmedian);
    hipLaunchKernelGGL(k_reg_final, dim3(V), dim3(kNT), 0, s, cams, V, max_tiles, (const float*)ws, w_dist,
                       w_normal, loss);
    if (V > 1) hipLaunchKernelGGL(k_reg_total, dim3(1), dim3(kNT), 0, s, V, w_dist, w_normal, loss);
    return hipGetLastError();
}

hipError_t launch_loss_from_tiles(int V, const sr_camera* cams, const float* tile_loss, float gamma, float w_c,
                                  float* loss, hipStream_t s) {
    if (V == 0) return hipSuccess;
    hipLaunchKernelGGL(k_loss_tiles, dim3(V), dim3(kNT), 0, s, cams, V, tile_loss, gamma, w_c, loss);
    if (V > 1) hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(kNT), 0, s, V, gamma, w_c, loss);
    return hipGetLastError();
}

int loss_chunks(int64_t max_hw) { return (int)((max_hw + kChunk - 1) / kChunk); }

size_t loss_workspace_bytes(int V, int64_t max_hw, int max_reg_tiles) {
    const int64_t slots = loss_chunks(max_hw) > max_reg_tiles ? loss_chunks(max_hw) : max_reg_tiles;
    return (size_t)V * (size_t)slots * 2 * sizeof(float);
}

hipError_t launch_loss(int V, int64_t max_hw, const sr_camera* cams, const float* alpha, const uint8_t* mask,
                       const float* color, const float* target, float gamma, float w_c, void* ws, float* loss,
                       float* dL_dalpha, float* dL_dcolor, hipStream_t s) {
    if (V == 0) return hipSuccess;
    const int nchunk = loss_chunks(max_hw);
    hipLaunchKernelGGL(k_loss_partial, dim3(nchunk, V), dim3(kNT), 0, s, cams, V, alpha, mask, color, target, gamma,
                       w_c, nchunk, (float*)ws, dL_dalpha, dL_dcolor);
    hipLaunchKernelGGL(k_loss_final, dim3(V), dim3(kNT), 0, s, cams, V, nchunk, (const float*)ws, gamma,
                       color ? w_c : 0.f, loss);
    if (V > 1)
        hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(kNT), 0, s, V, gamma, color ? w_c : 0.f, loss);
    return hipGetLastError();
}

}  // namespace sr
