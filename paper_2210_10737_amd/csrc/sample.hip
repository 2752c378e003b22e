// Randomized column-row sampling (section 2.2, Eq. 2 with the probabilities
// of Eq. 3): k i.i.d. draws i_t ~ p, p_i proportional to sqrt(q_i), each
// drawn pair scaled by 1/(k p_{i_t}).
//
// Every decision is integer, so the draws are reproducible bit for bit:
//   * p is held as integer weights w_i = floor(sqrt(q_i) * 2^S / m),
//     m = max_j sqrt(q_j) (a max over the keys, order-free), with S = 38 up
//     to 2^24 pairs and 62 - ceil(log2 n) above, so the total stays <= 2^62;
//   * the CDF W_i = w_0 + ... + w_i is an exact int64 inclusive scan;
//   * draw t takes the t-th output z_t of the SplitMix64 generator seeded
//     with `seed`, u_t = floor(z_t * total / 2^64), and i_t = the smallest i
//     with W_i > u_t (binary search); counts are integer atomics;
//   * if some score is +Inf, the infinite ones share the mass uniformly;
//   * a column drawn c_i times enters once with scale
//     colw_i = c_i * total / (k * w_i) (fp64), i.e. c_i / (k p_i).
#include "rsc_internal.h"

namespace rsc {
namespace {

// Five launches: largest key, tile sums, CDF, draws, scales. For 358,000 draws
// from 716,847 columns they take 6.0 + 5.2 + 6.5 + 34.5 + 6.1 us; as eight
// launches, with the weights stored and the tile sums scanned by a launch of
// its own, they took 80 us.
//
// Weights and CDF in tiles of 1,024 columns (256 threads x 4): 716,847 columns
// make 701 tiles, enough blocks for every CU (175 tiles of 4,096: 9.3 and 9.4
// us in place of 5.2 and 6.5).
constexpr int kScanTile = 1024;
constexpr int kScanPer = kScanTile / 256;

// Up to here a tile adds the sums of the tiles before it up by itself (at
// most 32 loads a thread, out of L2); above, where all tiles together would
// read nt^2 / 2 sums (over 0.25 GB), one block scans them first.
constexpr int32_t kAddTilesMax = 8192;

constexpr int kMaxBlocks = 256;  // of max_key_kernel; max_root reads one maximum a thread

__device__ __forceinline__ double key_sqrt(uint64_t u) {
    return u == 0 ? 0.0 : sqrt(__longlong_as_double((long long)(u - 1)));
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t t) {
    uint64_t z = seed + (t + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// w_i of a key; m = sqrt of the largest key, scale = 2^S / m
__device__ __forceinline__ int64_t weight(uint64_t u, double m, double scale, int bits) {
    const double r = key_sqrt(u);
    // infinite scores share the mass uniformly
    return isinf(m) ? (isinf(r) ? ((int64_t)1 << bits) : 0) : (int64_t)(r * scale);
}

// the largest key out of the blocks' maxima (at most kMaxBlocks of them)
__device__ __forceinline__ double max_root(const uint64_t *__restrict__ block_max, int nb, unsigned long long *s) {
    unsigned long long m = (int)threadIdx.x < nb ? (unsigned long long)block_max[threadIdx.x] : 0ull;
    for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned long long)__shfl_down(m, off));
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    return key_sqrt(max(max(s[0], s[1]), max(s[2], s[3])));
}

// the largest key of each block's share; the draws' counters are cleared on
// the way
__global__ __launch_bounds__(256) void max_key_kernel(const uint64_t *__restrict__ key, int32_t n,
                                                      uint64_t *__restrict__ block_max, int32_t *__restrict__ count) {
    __shared__ unsigned long long s[4];
    unsigned long long m = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        m = max(m, (unsigned long long)key[i]);
        count[i] = 0;
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned long long)__shfl_down(m, off));
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) block_max[blockIdx.x] = max(max(s[0], s[1]), max(s[2], s[3]));
}

// per-tile sums of w. The weights themselves are not stored: reading the keys
// once more in prefix_kernel costs what reading the weights would, and w_i is
// W_i - W_{i-1} where a drawn column needs it.
__global__ __launch_bounds__(256) void tile_sum_kernel(const uint64_t *__restrict__ key, int32_t n, int bits,
                                                       const uint64_t *__restrict__ block_max, int nb,
                                                       int64_t *__restrict__ tile_sum) {
    __shared__ unsigned long long sm[4];
    __shared__ int64_t s[4];
    const double m = max_root(block_max, nb, sm);
    const double scale = m > 0.0 ? ldexp(1.0, bits) / m : 0.0;  // 2^S / m
    const int64_t ts = (int64_t)blockIdx.x * kScanTile;
    int64_t acc = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t i = ts + threadIdx.x + 256 * j;
        if (i < n) acc += weight(key[i], m, scale, bits);
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        tile_sum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
        // one value behind the tiles: the largest root, for prefix_kernel (the
        // blocks' maxima stand where it writes W)
        if (blockIdx.x == 0) tile_sum[gridDim.x] = __double_as_longlong(m);
    }
}

// exclusive scan of the tile sums, in place (one block of 1024 threads)
__global__ __launch_bounds__(1024) void tile_scan_kernel(int64_t *__restrict__ tile_sum, int32_t nt) {
    __shared__ int64_t sh[1024];
    const int t = threadIdx.x;
    const int32_t per = (nt + 1023) / 1024;
    const int32_t lo = min(nt, t * per), hi = min(nt, lo + per);
    int64_t s = 0;
    for (int32_t i = lo; i < hi; ++i) s += tile_sum[i];
    sh[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t x = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    int64_t run = sh[t] - s;
    for (int32_t i = lo; i < hi; ++i) {
        const int64_t c = tile_sum[i];
        tile_sum[i] = run;
        run += c;
    }
}

// inclusive prefix W: each thread sums 4 consecutive weights, a wave scans the
// threads' sums by shuffles, the waves' sums are added through LDS. kScanned:
// tile_sum holds exclusive offsets already.
template <bool kScanned>
__global__ __launch_bounds__(256) void prefix_kernel(const uint64_t *__restrict__ key, int32_t n, int bits,
                                                     const int64_t *__restrict__ tile_sum, int32_t nt,
                                                     int64_t *__restrict__ W) {
    __shared__ int64_t sh[8];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const double m = __longlong_as_double(tile_sum[nt]);
    const double scale = m > 0.0 ? ldexp(1.0, bits) / m : 0.0;
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)t * kScanPer;
    int64_t v[kScanPer];
    int64_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        v[j] = base + j < n ? weight(key[base + j], m, scale, bits) : 0;
        s += v[j];
    }
    int64_t before = 0;  // sums of earlier tiles
    if (!kScanned) {
        for (int32_t i = t; i < (int32_t)blockIdx.x; i += 256) before += tile_sum[i];
        for (int off = 32; off > 0; off >>= 1) before += __shfl_down(before, off);
    }
    int64_t x = s;
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[wv] = x;
    if (lane == 0) sh[4 + wv] = before;
    __syncthreads();
    int64_t run = kScanned ? tile_sum[blockIdx.x] : sh[4] + sh[5] + sh[6] + sh[7];
    for (int i = 0; i < wv; ++i) run += sh[i];
    run += x - s;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        run += v[j];
        if (base + j < n) W[base + j] = run;
    }
}

// One thread a draw. The counters' atomics bound it, about 12 of them a
// nanosecond: 358,000 draws from 716,847 columns take 34.5 us, and 36 us with
// all but the last 8 steps of the search in LDS.
__global__ __launch_bounds__(256) void draw_kernel(const int64_t *__restrict__ W, int32_t n, int32_t k,
                                                   uint64_t seed, int32_t *__restrict__ count) {
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= k) return;
    const uint64_t total = (uint64_t)W[n - 1];
    if (total == 0) return;
    const uint64_t u = __umul64hi(splitmix64(seed, (uint64_t)t), total);
    int32_t lo = 0, hi = n - 1;  // smallest i with W[i] > u
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if ((uint64_t)W[mid] > u) hi = mid; else lo = mid + 1;
    }
    atomicAdd(&count[lo], 1);
}

__global__ __launch_bounds__(256) void colw_kernel(const int32_t *__restrict__ count,
                                                   const int64_t *__restrict__ W, int32_t n, int32_t k,
                                                   double *__restrict__ colw, uint32_t *__restrict__ mask,
                                                   uint32_t *__restrict__ prev) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool in = i < n;
    const int32_t c = in ? count[i] : 0;
    if (in) {
        double v = 0.0;
        if (c) {
            const int64_t w = W[i] - (i ? W[i - 1] : 0);
            v = (double)c * (double)W[n - 1] / ((double)k * (double)w);
        }
        colw[i] = v;
    }
    const uint64_t bal = __ballot(c > 0);
    const int64_t word = (i - lane) / 32;
    const int64_t nwords = ((int64_t)n + 31) / 32;
    const int64_t at = word + (lane >> 5);
    if ((lane & 31) == 0 && at < nwords) {
        if (prev) prev[at] = mask[at];  // the selection this one replaces
        mask[at] = (uint32_t)(lane == 0 ? bal : bal >> 32);
    }
}

}  // namespace

size_t sample_ws_bytes(int32_t n) {
    const size_t nn = (size_t)std::max<int32_t>(n, 1);
    const size_t nt = (size_t)ceil_div((int64_t)nn, kScanTile);
    return align_up(nn * 8, 256) + align_up((nt + 1) * 8, 256);
}

hipError_t sample_launch(const uint64_t *key, int32_t n, int32_t k, uint64_t seed, int32_t *count,
                         double *colw, uint32_t *mask, void *ws, hipStream_t stream, uint32_t *prev) {
    if (n == 0) return hipSuccess;
    const size_t nn = (size_t)n;
    const int32_t nt = (int32_t)ceil_div(n, kScanTile);
    char *p = static_cast<char *>(ws);
    int64_t *W = reinterpret_cast<int64_t *>(p);
    p += align_up(nn * 8, 256);
    int64_t *tile = reinterpret_cast<int64_t *>(p);
    // at most ceil(n / 256) <= n of them, and no longer needed when W is written
    uint64_t *block_max = reinterpret_cast<uint64_t *>(W);
    const int nb = (int)std::min<int64_t>(ceil_div(n, 256), kMaxBlocks);
    int bits = 38;  // weight resolution S
    if (n > (1 << 24)) {
        int lg = 0;
        while ((int64_t{1} << lg) < (int64_t)n) ++lg;
        bits = 62 - lg;
    }
    max_key_kernel<<<nb, 256, 0, stream>>>(key, n, block_max, count);
    tile_sum_kernel<<<nt, 256, 0, stream>>>(key, n, bits, block_max, nb, tile);
    if (nt <= kAddTilesMax) {
        prefix_kernel<false><<<nt, 256, 0, stream>>>(key, n, bits, tile, nt, W);
    } else {
        tile_scan_kernel<<<1, 1024, 0, stream>>>(tile, nt);
        prefix_kernel<true><<<nt, 256, 0, stream>>>(key, n, bits, tile, nt, W);
    }
    if (k > 0) draw_kernel<<<(unsigned)ceil_div(k, 256), 256, 0, stream>>>(W, n, k, seed, count);
    colw_kernel<<<(unsigned)ceil_div(n, 256), 256, 0, stream>>>(count, W, n, k, colw, mask, prev);
    return hipGetLastError();
}

}  // namespace rsc
