// Top-k selection (section 2.2.1): the k largest uint64 keys, ties broken by
// the lower index, returned as ascending indices and an n-bit mask.
//
// 1. Radix select of the threshold T = the k-th largest key, most significant
//    digit first: 6 passes of 11/11/11/11/10/10 bits. Each pass builds a
//    grid-wide histogram of the digit over the keys that match the prefix
//    chosen so far (LDS histograms, then integer atomics into global bins).
//    The digit that holds the k-th key is picked at the start of the next
//    kernel: every block reads the finished histogram and makes the same
//    pick (a wave-shuffle scan over the bins), and its first block records
//    the state after it, one slot per pass, so no kernel of its own is
//    needed. After the last pass T is known, and r = the number of keys
//    equal to T that must be kept (G = k - r keys are strictly above T).
//    A pick whose bin is wanted whole (as many keys as remain to be taken,
//    a single one as a rule after three digits) ends the search: the digits
//    below are left out of every comparison, and the remaining passes return
//    without reading a key.
// 2. Tiles of keys count (== T) and (> T) (their kernel makes the last pick);
//    the next kernel adds the counts of the tiles before its own and keeps key
//    i iff key > T, or key == T and fewer than r equal keys precede it,
//    writing mask words from wave ballots and idx at the running count of kept
//    keys. Everything is integer, so the result is exact and deterministic.
// Up to 16,384 keys the whole selection runs in one block with the keys in
// registers (one launch; the small graphs are launch-bound).
//
// Bound by launches: 9 dependent ones of 2 to 10 us each. us, every pass over
// all keys and a scan of its own / this form: 2,449,029 keys 101 / 80; 132,534
// keys 61 / 45; 4,096 keys (one launch) 25.6 / 8.7.
#include "rsc_internal.h"

namespace rsc {
namespace {

constexpr int kBins = 2048;
constexpr int kPasses = 6;

// Of eq keys equal to the threshold, how many are taken when want more are
// still wanted: want clamped to [0, eq], in integers.
__device__ __forceinline__ int64_t clamp_take(int64_t want, int64_t eq) {
    return want < 0 ? 0 : (want < eq ? want : eq);
}

__constant__ const int kShift[kPasses] = {53, 42, 31, 20, 10, 0};
__constant__ const int kWidth[kPasses] = {11, 11, 11, 11, 10, 10};

struct TopkState {
    uint64_t prefix;  // digits of T fixed so far
    uint64_t pmask;   // which bits of prefix are fixed
    int64_t k_rem;    // how many keys among those matching prefix remain to be taken
    int64_t done;     // all of them: no further digit matters
};

// st[p] = the state after p picks (st[0] initial, st[kPasses] final: prefix
// = T, k_rem = r); the histogram of pass p is hist[p % 3] (pass p reads
// pass p - 1's and clears pass p + 1's, three distinct buffers).
struct TopkWs {
    TopkState st[kPasses + 1];
    uint32_t hist[3][kBins];
};

struct PickOut {
    uint64_t prefix, pmask;
    int64_t k_rem, done;
};

// One block of 256 threads picks the digit of `pass` from histogram h,
// starting from state *sp: thread t owns the bins nb-1-t*per .. nb-per-t*per
// (descending), and an exclusive scan over threads (within each wave by
// shuffles, then over the four wave totals) gives the count of keys in
// higher bins. Every thread gets the new state; a search that is done keeps
// its state. True if it is done.
__device__ bool block_pick_256(const TopkState *sp, const uint32_t *h, int pass, uint64_t &prefix, uint64_t &pmask,
                               int64_t &k_rem, int64_t *wsum, PickOut *s_out) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (sp->done) {  // uniform
        prefix = sp->prefix;
        pmask = sp->pmask;
        k_rem = sp->k_rem;
        return true;
    }
    const int shift = kShift[pass];
    const int nb = 1 << kWidth[pass];
    const int per = nb / 256;  // 8 or 4
    uint32_t hv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) hv[j] = j < per ? h[nb - 1 - (t * per + j)] : 0u;
    prefix = sp->prefix;
    pmask = sp->pmask;
    k_rem = sp->k_rem;
    int64_t s = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s += hv[j];
    int64_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t x = __shfl_up(incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int64_t run = incl - s;  // keys in bins above this thread's range
    for (int u = 0; u < w; ++u) run += wsum[u];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int64_t c = hv[j];
        if (j < per && run < k_rem && run + c >= k_rem) {  // exactly one (thread, bin) satisfies this
            const int b = nb - 1 - (t * per + j);
            s_out->prefix = prefix | ((uint64_t)b << shift);
            s_out->pmask = pmask | ((uint64_t)(nb - 1) << shift);
            s_out->k_rem = k_rem - run;
            s_out->done = c == k_rem - run;
        }
        run += c;
    }
    __syncthreads();
    prefix = s_out->prefix;
    pmask = s_out->pmask;
    k_rem = s_out->k_rem;
    return s_out->done != 0;
}

__global__ __launch_bounds__(256) void topk_init_kernel(TopkWs *h, int64_t k) {
    for (int b = threadIdx.x; b < kBins; b += blockDim.x) h->hist[0][b] = 0;
    if (threadIdx.x == 0) {
        h->st[0].prefix = 0;
        h->st[0].pmask = 0;
        h->st[0].k_rem = k;
        h->st[0].done = 0;
    }
}

// Pass p: the pick of pass p - 1 (from its finished histogram; the first
// block records the state in st[p]), the clearing of pass p + 1's histogram,
// then this pass's histogram over the keys that match the prefix.
__global__ __launch_bounds__(256) void topk_hist_kernel(const uint64_t *__restrict__ key, int32_t n, TopkWs *ws,
                                                        int pass) {
    __shared__ uint32_t lh[kBins];
    __shared__ int64_t wsum[4];
    __shared__ PickOut s_out;
    const int shift = kShift[pass];
    const uint64_t dmask = (1ull << kWidth[pass]) - 1ull;
    for (int b = threadIdx.x; b < kBins; b += blockDim.x) lh[b] = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // eight keys per thread loaded before any is counted (the first eight
    // before the pick, so the two waits overlap), then the rest one at a time
    uint64_t k[8];
    bool more = i + 7 * stride < n;
    if (more) {
#pragma unroll
        for (int u = 0; u < 8; ++u) k[u] = key[i + u * stride];
    }
    uint64_t prefix = ws->st[0].prefix, pmask = ws->st[0].pmask;
    if (pass > 0) {
        int64_t k_rem;
        const bool done = block_pick_256(&ws->st[pass - 1], ws->hist[(pass - 1) % 3], pass - 1, prefix, pmask, k_rem,
                                         wsum, &s_out);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ws->st[pass].prefix = prefix;
            ws->st[pass].pmask = pmask;
            ws->st[pass].k_rem = k_rem;
            ws->st[pass].done = done;
        }
        if (done) return;  // grid-uniform; no later pass reads a histogram
    }
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b < kBins; b += blockDim.x) ws->hist[(pass + 1) % 3][b] = 0;
    __syncthreads();  // lh cleared
    uint32_t *hist = ws->hist[pass % 3];
    while (more) {
        if (pass == 0) {  // block-uniform
            // the top digit is nearly constant over the keys: a wave whose
            // keys all share one digit adds them with one LDS atomic
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t dg = (uint32_t)((k[u] >> shift) & dmask);
                const uint32_t d0 = __shfl(dg, 0);
                if (__ballot(dg == d0) == ~0ull) {
                    if ((threadIdx.x & 63) == 0) atomicAdd(&lh[d0], 64u);
                } else {
                    atomicAdd(&lh[dg], 1u);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if ((k[u] & pmask) == prefix) atomicAdd(&lh[(k[u] >> shift) & dmask], 1u);
        }
        i += 8 * stride;
        more = i + 7 * stride < n;
        if (more) {
#pragma unroll
            for (int u = 0; u < 8; ++u) k[u] = key[i + u * stride];
        }
    }
    for (; i < n; i += stride) {
        const uint64_t kv = key[i];
        if ((kv & pmask) == prefix) atomicAdd(&lh[(kv >> shift) & dmask], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < (1 << kWidth[pass]); b += blockDim.x)
        if (lh[b]) atomicAdd(&hist[b], lh[b]);
}

// Also makes the last pass's pick (every block; the first records the final
// state, T and r, for the emit). kPer keys per thread, 256 kPer per tile.
template <int kPer>
__global__ __launch_bounds__(256) void topk_tile_count_kernel(const uint64_t *__restrict__ key,
                                                              int32_t n, TopkWs *ws,
                                                              uint32_t *__restrict__ tile_eq,
                                                              uint32_t *__restrict__ tile_gt) {
    __shared__ uint32_t s_eq[4], s_gt[4];
    __shared__ int64_t wsum[4];
    __shared__ PickOut s_out;
    // the tile's keys are loaded before the pick, so the two waits overlap
    const int64_t ts = (int64_t)blockIdx.x * 256 * kPer;
    uint64_t kv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) kv[j] = key[std::min<int64_t>(ts + threadIdx.x + 256 * j, n - 1)];
    uint64_t T, pmask;
    int64_t r;
    block_pick_256(&ws->st[kPasses - 1], ws->hist[(kPasses - 1) % 3], kPasses - 1, T, pmask, r, wsum, &s_out);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ws->st[kPasses].prefix = T;
        ws->st[kPasses].pmask = pmask;
        ws->st[kPasses].k_rem = r;
    }
    uint32_t eq = 0, gt = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const bool in = ts + threadIdx.x + 256 * j < n;
        eq += in && (kv[j] & pmask) == T;
        gt += in && (kv[j] & pmask) > T;
    }
    for (int off = 32; off > 0; off >>= 1) {
        eq += __shfl_down(eq, off);
        gt += __shfl_down(gt, off);
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) { s_eq[w] = eq; s_gt[w] = gt; }
    __syncthreads();
    if (threadIdx.x == 0) {
        tile_eq[blockIdx.x] = s_eq[0] + s_eq[1] + s_eq[2] + s_eq[3];
        tile_gt[blockIdx.x] = s_gt[0] + s_gt[1] + s_gt[2] + s_gt[3];
    }
}

// Sum of x[0 .. m) by a block of 256 threads; every thread gets it. sh holds
// four entries and may be reused after the caller's next barrier.
__device__ __forceinline__ int64_t block_sum_256(const uint32_t *__restrict__ x, int32_t m, int64_t *sh) {
    int64_t v = 0;
#pragma unroll 4
    for (int32_t i = threadIdx.x; i < m; i += 256) v += x[i];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

// Sums of the tile counts per kCoarse tiles, for selections of more tiles
// than the emit's blocks should add one by one.
constexpr int kCoarse = 1024;
constexpr int kDirectTiles = 8192;

__global__ __launch_bounds__(256) void topk_coarse_kernel(const uint32_t *__restrict__ tile_eq,
                                                          const uint32_t *__restrict__ tile_gt, int32_t nt,
                                                          uint32_t *__restrict__ coarse_eq,
                                                          uint32_t *__restrict__ coarse_gt) {
    __shared__ int64_t sh[2][4];
    const int32_t lo = blockIdx.x * kCoarse, m = min(kCoarse, nt - lo);
    const int64_t eq = block_sum_256(tile_eq + lo, m, sh[0]);
    const int64_t gt = block_sum_256(tile_gt + lo, m, sh[1]);
    if (threadIdx.x == 0) {
        coarse_eq[blockIdx.x] = (uint32_t)eq;
        coarse_gt[blockIdx.x] = (uint32_t)gt;
    }
}

// prev (nullable): receives each mask word's old value, the selection that
// this one replaces.
template <int kPer>
__global__ __launch_bounds__(256) void topk_emit_kernel(const uint64_t *__restrict__ key, int32_t n,
                                                        const TopkState *__restrict__ st,
                                                        const uint32_t *__restrict__ tile_eq,
                                                        const uint32_t *__restrict__ tile_gt,
                                                        const uint32_t *__restrict__ coarse_eq,
                                                        const uint32_t *__restrict__ coarse_gt,
                                                        int32_t *__restrict__ idx,
                                                        uint32_t *__restrict__ mask, uint32_t *__restrict__ prev,
                                                        int32_t k) {
    __shared__ uint32_t s_eq[4], s_gt[4];
    __shared__ int64_t s_sum[4][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int64_t wbase = ((int64_t)blockIdx.x * 4 + w) * (64 * kPer);
    const int64_t nwords = ((int64_t)n + 31) / 32;
    uint64_t kv[kPer];
#pragma unroll
    for (int g = 0; g < kPer; ++g) kv[g] = key[std::min<int64_t>(wbase + 64 * g + lane, n - 1)];
    const uint64_t T = st->prefix, pmask = st->pmask;
    const int64_t r = st->k_rem;
    // the equal and greater keys of the tiles before this one
    int64_t eq_base, gt_base;
    if (coarse_eq) {
        const int32_t c = blockIdx.x / kCoarse, lo = c * kCoarse, m = blockIdx.x - lo;
        eq_base = block_sum_256(coarse_eq, c, s_sum[0]) + block_sum_256(tile_eq + lo, m, s_sum[1]);
        gt_base = block_sum_256(coarse_gt, c, s_sum[2]) + block_sum_256(tile_gt + lo, m, s_sum[3]);
    } else {
        eq_base = block_sum_256(tile_eq, blockIdx.x, s_sum[0]);
        gt_base = block_sum_256(tile_gt, blockIdx.x, s_sum[1]);
    }
    uint32_t eq = 0, gt = 0;
#pragma unroll
    for (int g = 0; g < kPer; ++g) {
        const bool in = wbase + 64 * g + lane < n;
        kv[g] &= pmask;
        eq += __popcll(__ballot(in && kv[g] == T));
        gt += __popcll(__ballot(in && kv[g] > T));
    }
    if (lane == 0) { s_eq[w] = eq; s_gt[w] = gt; }
    __syncthreads();
    for (int v = 0; v < w; ++v) {
        gt_base += s_gt[v];
        eq_base += s_eq[v];
    }
    // of the equal keys the first r are kept
    int64_t sel_base = gt_base + clamp_take(r, eq_base);
#pragma unroll
    for (int g = 0; g < kPer; ++g) {
        const int64_t base = wbase + 64 * g;
        const int64_t i = base + lane;
        const bool in = i < n;
        const bool is_eq = in && kv[g] == T;
        const uint64_t eqbal = __ballot(is_eq);
        const bool sel = (in && kv[g] > T) || (is_eq && eq_base + __popcll(eqbal & lt_mask) < r);
        const uint64_t selbal = __ballot(sel);
        const int64_t pos = sel_base + __popcll(selbal & lt_mask);
        if (sel && pos < k) idx[pos] = (int32_t)i;
        const int64_t word = base / 32 + (lane >> 5);
        if ((lane & 31) == 0 && word < nwords) {
            if (prev) prev[word] = mask[word];
            mask[word] = (uint32_t)(lane == 0 ? selbal : selbal >> 32);
        }
        eq_base += __popcll(eqbal);
        sel_base += __popcll(selbal);
    }
}

// Small inputs (n <= kSmallN) in one block of 1024 threads: thread t holds
// keys [kPer t, kPer (t + 1)) in registers. The same radix passes (LDS
// histogram, a block scan picks the digit) until the picked bin is wanted
// whole, then block scans of each thread's (== T) count and of its kept count
// give the ranks; idx is written at the running kept count and the threads of
// 32 keys put their bits together into a mask word.
constexpr int kSmallN = 16384;
constexpr int kSmallThreads = 1024;

// Exclusive scan over the block (by shuffles within each wave, then over the
// 16 wave totals in sh). Ends with a barrier.
__device__ __forceinline__ uint32_t block_exclusive_scan_1024(uint32_t v, uint32_t *sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = __shfl_up(incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) sh[w] = incl;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int u = 0; u < 15; ++u) before += u < w ? sh[u] : 0;
    __syncthreads();  // sh may be rewritten by the next call
    return before + incl - v;
}

template <int kPer>
__global__ __launch_bounds__(kSmallThreads) void topk_small_kernel(const uint64_t *__restrict__ key, int32_t n,
                                                                   int32_t k, int32_t *__restrict__ idx,
                                                                   uint32_t *__restrict__ mask,
                                                                   uint32_t *__restrict__ prev) {
    __shared__ uint32_t s_hist[kBins];
    __shared__ uint32_t s_scan[kSmallThreads / 64];
    __shared__ PickOut s_out;
    const int t = threadIdx.x, lane = t & 63;
    const int lo = t * kPer, cnt = min(max(n - lo, 0), kPer);
    uint64_t kv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) kv[j] = key[min(lo + j, n - 1)];
    uint64_t prefix = 0, pmask = 0;
    uint32_t k_rem = (uint32_t)k;
    for (int pass = 0; pass < kPasses; ++pass) {
        const int shift = kShift[pass], nb = 1 << kWidth[pass];
        const uint64_t dmask = (uint64_t)(nb - 1);
        for (int b = t; b < kBins; b += kSmallThreads) s_hist[b] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const bool in = j < cnt && (kv[j] & pmask) == prefix;
            const uint32_t dg = (uint32_t)((kv[j] >> shift) & dmask);
            if (pass == 0) {  // the top digit is nearly constant: one atomic for a wave of one digit
                const uint32_t d0 = __shfl(dg, 0);
                const uint64_t same = __ballot(in && dg == d0);
                if (lane == 0 && same) atomicAdd(&s_hist[d0], (uint32_t)__popcll(same));
                if (in && dg != d0) atomicAdd(&s_hist[dg], 1u);
            } else if (in) {
                atomicAdd(&s_hist[dg], 1u);
            }
        }
        __syncthreads();
        // thread t owns the bins nb - 1 - t per .. downwards; the scan gives the keys in higher bins
        const int per = nb / kSmallThreads;  // 2 or 1
        uint32_t c[2] = {s_hist[nb - 1 - t * per], per == 2 ? s_hist[nb - 2 - t * per] : 0u};
        uint32_t run = block_exclusive_scan_1024(c[0] + c[1], s_scan);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (j < per && run < k_rem && run + c[j] >= k_rem) {  // exactly one (thread, bin)
                const uint64_t b = (uint64_t)(nb - 1 - t * per - j);
                s_out.prefix = prefix | (b << shift);
                s_out.pmask = pmask | (dmask << shift);
                s_out.k_rem = k_rem - run;
                s_out.done = c[j] == k_rem - run;
            }
            run += c[j];
        }
        __syncthreads();
        prefix = s_out.prefix;
        pmask = s_out.pmask;
        k_rem = (uint32_t)s_out.k_rem;
        if (s_out.done) break;  // block-uniform; s_out is rewritten two barriers later at the earliest
    }
    uint32_t eq = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        kv[j] &= pmask;
        eq += j < cnt && kv[j] == prefix;
    }
    uint32_t eq_before = block_exclusive_scan_1024(eq, s_scan);
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        bool sel = kv[j] > prefix;
        if (kv[j] == prefix) sel = eq_before++ < k_rem;
        if (sel && j < cnt) bits |= 1u << j;
    }
    uint32_t pos = block_exclusive_scan_1024(__popc(bits), s_scan);
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if ((bits >> j) & 1u) idx[pos++] = lo + j;
    constexpr int kLanes = 32 / kPer;  // threads per mask word
    uint32_t word = bits << (kPer * (t % kLanes));
#pragma unroll
    for (int m = 1; m < kLanes; m <<= 1) word |= __shfl_xor(word, m);
    const int at = t / kLanes;
    if (t % kLanes == 0 && at < (n + 31) / 32) {
        if (prev) prev[at] = mask[at];
        mask[at] = word;
    }
}

__global__ __launch_bounds__(256) void clear_mask_kernel(uint32_t *mask, uint32_t *prev, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (prev) prev[i] = mask[i];
        mask[i] = 0;
    }
}

// Keys per thread of the tile kernels: small tiles until they fill the chip.
constexpr int32_t kSmallTileN = 1 << 20;
int tile_per(int32_t n) { return n <= kSmallTileN ? 4 : 16; }

}  // namespace

size_t topk_ws_bytes(int32_t n) {
    n = std::max<int32_t>(n, 1);
    const size_t nt = (size_t)ceil_div(n, 256 * tile_per(n)), nc = (size_t)ceil_div((int64_t)nt, kCoarse);
    return align_up(sizeof(TopkWs), 256) + 2 * align_up(nt * sizeof(uint32_t), 256) +
           2 * align_up(nc * sizeof(uint32_t), 256);
}

hipError_t topk_launch(const uint64_t *key, int32_t n, int32_t k, int32_t *idx, uint32_t *mask,
                       void *ws, hipStream_t stream, uint32_t *prev) {
    if (n == 0) return hipSuccess;
    const int64_t nwords = ceil_div(n, 32);
    if (k == 0) {
        clear_mask_kernel<<<(unsigned)std::min<int64_t>(ceil_div(nwords, 256), 1024), 256, 0, stream>>>(mask, prev,
                                                                                                     nwords);
        return hipGetLastError();
    }
    if (n <= kSmallN) {
        if (n <= 4 * kSmallThreads)
            topk_small_kernel<4><<<1, kSmallThreads, 0, stream>>>(key, n, k, idx, mask, prev);
        else
            topk_small_kernel<16><<<1, kSmallThreads, 0, stream>>>(key, n, k, idx, mask, prev);
        return hipGetLastError();
    }
    TopkWs *h = static_cast<TopkWs *>(ws);
    const int per = tile_per(n);
    const int32_t nt = (int32_t)ceil_div(n, 256 * per), nc = (int32_t)ceil_div(nt, kCoarse);
    char *p = static_cast<char *>(ws) + align_up(sizeof(TopkWs), 256);
    const size_t tb = align_up((size_t)nt * sizeof(uint32_t), 256), cb = align_up((size_t)nc * sizeof(uint32_t), 256);
    uint32_t *tile_eq = reinterpret_cast<uint32_t *>(p);
    uint32_t *tile_gt = reinterpret_cast<uint32_t *>(p + tb);
    uint32_t *coarse_eq = nullptr, *coarse_gt = nullptr;

    topk_init_kernel<<<1, 256, 0, stream>>>(h, k);
    // Each block flushes its non-empty bins with one global atomic each. The
    // first two passes count every key, into a few bins (pass 0) or into
    // most of them (pass 1), so they run on 256 and 128 blocks to keep those
    // atomics few (measured on 2.45M keys: 12.4 and 9.5 us, against 18.9 and
    // 29.6 with eight keys per thread); later passes count only the keys
    // under the chosen prefix and take eight keys per thread, for more loads
    // in flight.
    const unsigned hgrid_wide = (unsigned)std::min<int64_t>(ceil_div(n, 256 * 8), 2048);
    const unsigned hgrid_pass[2] = {std::min(hgrid_wide, 256u), std::min(hgrid_wide, 128u)};
    for (int pass = 0; pass < kPasses; ++pass)
        topk_hist_kernel<<<pass < 2 ? hgrid_pass[pass] : hgrid_wide, 256, 0, stream>>>(key, n, h, pass);
    if (per == 4)
        topk_tile_count_kernel<4><<<nt, 256, 0, stream>>>(key, n, h, tile_eq, tile_gt);
    else
        topk_tile_count_kernel<16><<<nt, 256, 0, stream>>>(key, n, h, tile_eq, tile_gt);
    if (nt > kDirectTiles) {
        coarse_eq = reinterpret_cast<uint32_t *>(p + 2 * tb);
        coarse_gt = reinterpret_cast<uint32_t *>(p + 2 * tb + cb);
        topk_coarse_kernel<<<nc, 256, 0, stream>>>(tile_eq, tile_gt, nt, coarse_eq, coarse_gt);
    }
    if (per == 4)
        topk_emit_kernel<4><<<nt, 256, 0, stream>>>(key, n, &h->st[kPasses], tile_eq, tile_gt, coarse_eq, coarse_gt,
                                                    idx, mask, prev, k);
    else
        topk_emit_kernel<16><<<nt, 256, 0, stream>>>(key, n, &h->st[kPasses], tile_eq, tile_gt, coarse_eq, coarse_gt,
                                                     idx, mask, prev, k);
    return hipGetLastError();
}

}  // namespace rsc
