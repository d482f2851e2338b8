// Per-tile maximum of the statistic over a bank (paper Sec. "Results", false-alarm
// probabilities: the background distribution is built from the largest statistic a
// noise-only search returns in each parameter tile, realisation by realisation).
//
// Two passes over the bank after a fill: the maximum per tile on the IEEE bit pattern (monotone for the
// non-negative values the statistic takes), then the smallest index attaining it.  Every pass is a plain
// kernel, so the sequence can be captured into a HIP graph.
//
// What bounds it: reading stat and tile (12 bytes per template) twice, the second time from the Infinity
// Cache.  With many templates per tile, one global atomic per template serialises on the few addresses (4M
// templates on 64 tiles: 4122 us, about 1 ns per atomic).  The maximum pass then reduces in LDS first, where a
// running maximum is raised only by values above it (a few times per tile and block), and the block sends its
// tiles' maxima on with one comparison each: 4M templates, 64 tiles, 23 us for the maximum pass and 11 us for the
// index pass (4.4 TB/s).  With few templates per tile the atomics hardly meet and the blocks' tables would be the
// larger part: each template sends its own (launch_tile_max has the rule).
#include "tfsc_kernels.hpp"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tfsc {

namespace {

constexpr unsigned long long kNoIndex = ~0ull;  // int64 -1: the tile holds no template

// Tiles whose running maxima a block keeps in LDS at most: 8 bytes each, 64 KB, so that two blocks fit a CU.
constexpr int32_t kTilesLds = 8192;

// A value other blocks may raise or lower meanwhile, read past the CU's own cache; used only to skip an atomic
// that could not change it (both tables are monotone), never as the result.
__device__ __forceinline__ unsigned long long peek(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool tile_entry(const double *stat, const int32_t *tile, int64_t i, int32_t n_tiles,
                                           int32_t &t, unsigned long long &bits) {
    const double v = stat[i];
    t = tile[i];
    if (t < 0 || t >= n_tiles || !(v >= 0.0)) return false;  // excluded: no tile, negative or NaN
    bits = (unsigned long long)__double_as_longlong(v + 0.0);  // -0 counts as +0
    return true;
}

__global__ void k_tile_fill(int32_t n_tiles, unsigned long long *mx, unsigned long long *arg) {
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_tiles) {
        mx[t] = 0ull;
        arg[t] = kNoIndex;
    }
}

// The block's running maxima in LDS; kPer templates per thread whose loads are issued together.
template <int kPer>
__global__ __launch_bounds__(256) void k_tile_max(const double *__restrict__ stat, const int32_t *__restrict__ tile,
                                                  int64_t n, int32_t n_tiles, unsigned long long *mx) {
    extern __shared__ unsigned long long top[];
    for (int t = threadIdx.x; t < n_tiles; t += 256) top[t] = peek(mx + t);
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * 256 * kPer;
    for (int64_t base = (int64_t)blockIdx.x * 256 * kPer; base < n; base += step) {
        int32_t t[kPer];
        unsigned long long b[kPer];
        bool ok[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = base + q * 256 + threadIdx.x;
            ok[q] = i < n && tile_entry(stat, tile, i, n_tiles, t[q], b[q]);
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (ok[q] && b[q] > *(volatile unsigned long long *)(top + t[q])) atomicMax(top + t[q], b[q]);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < n_tiles; t += 256)
        if (top[t] > peek(mx + t)) atomicMax(mx + t, top[t]);
}

// One atomic per template, or per wave where all of its templates lie in one tile (a bank in the tiles' order).
__global__ __launch_bounds__(256) void k_tile_max_each(const double *__restrict__ stat, const int32_t *__restrict__ tile,
                                                       int64_t n, int32_t n_tiles, unsigned long long *mx) {
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t base = (int64_t)blockIdx.x * 256; base < n; base += step) {
        const int64_t i = base + threadIdx.x;
        int32_t t = -1;
        unsigned long long b = 0;
        const bool ok = i < n && tile_entry(stat, tile, i, n_tiles, t, b);
        const uint64_t act = __ballot(ok);
        if (!act) continue;
        const int first = __ffsll((unsigned long long)act) - 1, t0 = __shfl(t, first, 64);
        if (__ballot(ok && t == t0) != act) {
            if (ok) atomicMax(mx + t, b);
            continue;
        }
        if (!ok) b = 0;
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long other = __shfl_xor(b, o, 64);
            b = other > b ? other : b;
        }
        if (lane == first) atomicMax(mx + t, b);
    }
}

template <int kPer>
__global__ __launch_bounds__(256) void k_tile_arg(const double *__restrict__ stat, const int32_t *__restrict__ tile,
                                                  int64_t n, int32_t n_tiles,
                                                  const unsigned long long *__restrict__ mx, unsigned long long *arg) {
    const int64_t step = (int64_t)gridDim.x * 256 * kPer;
    for (int64_t base = (int64_t)blockIdx.x * 256 * kPer; base < n; base += step) {
        int32_t t[kPer];
        unsigned long long b[kPer];
        bool ok[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = base + q * 256 + threadIdx.x;
            ok[q] = i < n && tile_entry(stat, tile, i, n_tiles, t[q], b[q]);
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const unsigned long long i = (unsigned long long)(base + q * 256 + threadIdx.x);
            if (ok[q] && b[q] == mx[t[q]] && (kPer == 1 || i < peek(arg + t[q]))) atomicMin(arg + t[q], i);
        }
    }
}

template <int kPer>
void launch_tile_lds(const double *stat, const int32_t *tile, int64_t n, int32_t n_tiles, int64_t per,
                     unsigned long long *mx, unsigned long long *arg, hipStream_t st) {
    const int64_t want = (n + per - 1) / per, most = (n + 256 * kPer - 1) / (256 * kPer);
    const unsigned nb = (unsigned)(want < 1024 ? want : 1024), na = (unsigned)(most < 2048 ? most : 2048);
    hipLaunchKernelGGL(k_tile_max<kPer>, dim3(nb), dim3(256), sizeof(unsigned long long) * n_tiles, st, stat, tile, n,
                       n_tiles, mx);
    hipLaunchKernelGGL(k_tile_arg<kPer>, dim3(na), dim3(256), 0, st, stat, tile, n, n_tiles, mx, arg);
}

}  // namespace

hipError_t launch_tile_max(const double *stat, const int32_t *tile, int64_t n, int32_t n_tiles, double *tile_max,
                           int64_t *tile_arg, hipStream_t st) {
    auto *mx = reinterpret_cast<unsigned long long *>(tile_max);
    auto *arg = reinterpret_cast<unsigned long long *>(tile_arg);
    const unsigned tb = (unsigned)((n_tiles + 255) / 256);
    hipLaunchKernelGGL(k_tile_fill, dim3(tb), dim3(256), 0, st, n_tiles, mx, arg);
    if (n > 0) {
        // Tables in LDS from 48 templates a tile on, and, as the chip wants some hundred blocks, each with a table to load
        // and to send on, from n_tiles / 20 a tile on.  Both calls, tables against an atomic each, us, templates in any
        // order: 1024 tiles: 20,000 15.4 / 15.4; 50,000 15.2 / 15.2; 100,000 14.4 / 18.0; 1M 26.5 / 129; 4096 tiles:
        // 300,000 30 / 18; 1M 48 / 44; 4M 85 / 160; 8192 tiles: 1M 60 / 46; 4M 127 / 167.
        const int64_t a_tile = n_tiles / 20 > 48 ? n_tiles / 20 : 48;
        if (n_tiles <= kTilesLds && n >= a_tile * n_tiles) {
            // From 131,072 templates on eight at a time, and four per tile and block, so that loading and sending on
            // the tables stays the smaller part, else two and one, for more blocks (1024 tiles, 100,000 templates:
            // 20.4 / 14.4 us; 1M: 26.5 / 41).  The maximum pass takes at most 1024 blocks: each sends its maxima to
            // the same few addresses (64 tiles, 4M templates: 53 us with 1953 blocks, 23 with 1024, 24 with 512, 37
            // with 256).
            if (n >= 131072)
                launch_tile_lds<8>(stat, tile, n, n_tiles, 4 * (int64_t)n_tiles > 2048 ? 4 * (int64_t)n_tiles : 2048, mx, arg, st);
            else
                launch_tile_lds<2>(stat, tile, n, n_tiles, n_tiles > 512 ? n_tiles : 512, mx, arg, st);
        } else {
            const int64_t want = (n + 255) / 256;
            const unsigned nb = (unsigned)(want < 4096 ? want : 4096);
            hipLaunchKernelGGL(k_tile_max_each, dim3(nb), dim3(256), 0, st, stat, tile, n, n_tiles, mx);
            hipLaunchKernelGGL(k_tile_arg<1>, dim3(nb), dim3(256), 0, st, stat, tile, n, n_tiles, mx, arg);
        }
    }
    return hipGetLastError();
}

}  // namespace tfsc
