// Stream compaction of the per-surfel arrays: the pruning decided by the
// occlusion statistics (Section 4.3), optionally with a minimum opacity,
// applied to the parameters (and whatever else the caller keeps per surfel,
// such as optimiser moments).  Stable: kept surfels keep their order.
//
// Pass 1 counts the kept surfels of every chunk; a single block scans the
// chunk counts; pass 2 lists the kept surfels of its chunk in LDS and copies
// their rows array by array, the block's threads over consecutive words of
// the destination: bound by memory.  Chunks of 1024 surfels give a million
// surfels four blocks per CU (8192 left half of the CUs idle), and a thread
// copying its surfel's rows word by word touched 64 rows per access.  1M
// surfels, five arrays of 232 bytes, a fifth kept: passes 20 + 332 us before,
// 6 + 24 us now.
#include "common.h"
#include "launch.h"

namespace sr {

namespace {

constexpr int kNT = 256;
constexpr int kChunk = 1024;          // surfels per block
constexpr int kRounds = kChunk / kNT;
constexpr int kMaxArrays = SR_COMPACT_MAX_ARRAYS;

struct CompactArrays {
    const float* src[kMaxArrays];
    float* dst[kMaxArrays];
    int width[kMaxArrays];
    int n;
};

__device__ __forceinline__ bool kept(int64_t i, const uint8_t* __restrict__ prune, const float* __restrict__ opac,
                                     float min_opac) {
    return !prune[i] && (opac == nullptr || opac[i] >= min_opac);
}

__global__ void __launch_bounds__(kNT)
k_compact_count(int N, const uint8_t* __restrict__ prune, const float* __restrict__ opac, float min_opac,
                uint32_t* __restrict__ counts) {
    __shared__ uint32_t s[kNT];
    const int64_t b = (int64_t)blockIdx.x * kChunk;
    const int64_t e = b + kChunk < N ? b + kChunk : N;
    uint32_t c = 0;
    for (int64_t i = b + threadIdx.x; i < e; i += kNT) c += kept(i, prune, opac, min_opac) ? 1u : 0u;
    s[threadIdx.x] = c;
    __syncthreads();
    for (int off = kNT / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = s[0];
}

// exclusive scan of the chunk counts in place (one block); total to *n_kept
__global__ void __launch_bounds__(kNT)
k_compact_scan(int nchunk, uint32_t* __restrict__ counts, uint32_t* __restrict__ n_kept) {
    __shared__ uint32_t s[2][kNT / 64];
    const int lane = __lane_id(), w = (int)threadIdx.x >> 6;
    uint32_t carry = 0;
    int buf = 0;                                          // two sets of wave sums: one barrier a round
    for (int base = 0; base < nchunk; base += kNT, buf ^= 1) {
        const int i = base + (int)threadIdx.x;
        const uint32_t v = i < nchunk ? counts[i] : 0u;
        uint32_t incl = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t t = __shfl_up(incl, d, 64);
            incl += lane >= d ? t : 0u;
        }
        if (lane == 63) s[buf][w] = incl;
        __syncthreads();
        uint32_t before = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kNT / 64; ++q) {
            before += q < w ? s[buf][q] : 0u;
            tot += s[buf][q];
        }
        if (i < nchunk) counts[i] = carry + before + incl - v;
        carry += tot;
    }
    if (threadIdx.x == 0) *n_kept = carry;
}

// Rows list[0, kept) of src, each of w words of type T, to consecutive rows of dst.
template <typename T>
__device__ __forceinline__ void copy_rows(const T* __restrict__ src, T* __restrict__ dst, int w, int kept,
                                          const uint16_t* list) {
    // (row, column) of this thread's word, stepped by the block's threads without a division
    int row = (int)threadIdx.x / w, col = (int)threadIdx.x - row * w;
    const int drow = kNT / w, dcol = kNT - drow * w;
    const size_t words = (size_t)kept * (size_t)w;
    for (size_t e = threadIdx.x; e < words; e += kNT) {
        dst[e] = src[(size_t)list[row] * (size_t)w + (size_t)col];
        row += drow;
        col += dcol;
        if (col >= w) {
            col -= w;
            ++row;
        }
    }
}

__global__ void __launch_bounds__(kNT)
k_compact_copy(int N, const uint8_t* __restrict__ prune, const float* __restrict__ opac, float min_opac,
               const uint32_t* __restrict__ offs, CompactArrays arr) {
    __shared__ uint16_t list[kChunk];                      // kept surfels of the chunk, in order
    __shared__ uint32_t s_cnt[kRounds][kNT / 64];
    const int64_t b = (int64_t)blockIdx.x * kChunk;
    const int lane = __lane_id(), w = (int)threadIdx.x >> 6;
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
    uint64_t m[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t i = b + r * kNT + threadIdx.x;
        m[r] = ballot64(i < N && kept(i, prune, opac, min_opac));
        if (lane == 0) s_cnt[r][w] = (uint32_t)__popcll(m[r]);
    }
    __syncthreads();
    uint32_t run = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
#pragma unroll
        for (int q = 0; q < kNT / 64; ++q) {
            if (q == w && ((m[r] >> lane) & 1ull))
                list[run + (uint32_t)__popcll(m[r] & lt)] = (uint16_t)(r * kNT + (int)threadIdx.x);
            run += s_cnt[r][q];
        }
    }
    __syncthreads();
    if (run == 0u) return;
    for (int a = 0; a < arr.n; ++a) {
        const int wd = arr.width[a];
        const float* src = arr.src[a] + (size_t)b * wd;
        float* dst = arr.dst[a] + (size_t)offs[blockIdx.x] * wd;
        // whole rows of 16-byte words where the width and both pointers allow
        // it (b and the offset are then multiples of 16 bytes as well)
        const bool quad = (wd & 3) == 0 && ((((uintptr_t)arr.src[a]) | ((uintptr_t)arr.dst[a])) & 15u) == 0u;
        if (quad)
            copy_rows((const float4*)src, (float4*)dst, wd >> 2, (int)run, list);
        else
            copy_rows(src, dst, wd, (int)run, list);
    }
}

}  // namespace

size_t compact_workspace_bytes(int N) { return (size_t)((N + kChunk - 1) / kChunk + 1) * sizeof(uint32_t); }

hipError_t launch_compact(int N, const uint8_t* prune, const float* opac, float min_opac, int n_arrays,
                          const float* const* src, float* const* dst, const int* widths, void* ws,
                          uint32_t* n_kept, hipStream_t s) {
    CompactArrays arr{};
    arr.n = n_arrays;
    for (int a = 0; a < n_arrays; ++a) {
        arr.src[a] = src[a];
        arr.dst[a] = dst[a];
        arr.width[a] = widths[a];
    }
    const int nchunk = (N + kChunk - 1) / kChunk;
    uint32_t* counts = (uint32_t*)ws;
    if (N == 0) {
        hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(kNT), 0, s, 0, counts, n_kept);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_compact_count, dim3(nchunk), dim3(kNT), 0, s, N, prune, opac, min_opac, counts);
    hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(kNT), 0, s, nchunk, counts, n_kept);
    hipLaunchKernelGGL(k_compact_copy, dim3(nchunk), dim3(kNT), 0, s, N, prune, opac, min_opac,
                       (const uint32_t*)counts, arr);
    return hipGetLastError();
}

}  // namespace sr
