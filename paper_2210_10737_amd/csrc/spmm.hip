// Sparse-dense product Y = A * B for CSR A (the aggregation SpMM of the
// GCN layer, section 2.1; the same kernel runs on the column slice for the
// top-k approximation of section 2.2.1).
//
// Work mapping (gfx950, wave64):
//   * one wave per row; the feature dimension is spread over the lanes,
//     4 consecutive fp32 features per lane (one 128-bit load), 256 features
//     per wave, two such vectors per lane for widths up to 512;
//   * the row's (col, val) pairs are fetched 64 at a time with one
//     coalesced, non-temporal load and broadcast from the owning lane with
//     v_readlane into scalar registers, so each gathered B row is addressed
//     by a scalar base plus the lane offset;
//   * 4 to 8 gather instructions are in flight per wave (16 in long rows of
//     over 256 features);
//   * products are accumulated in fp32 over each run of <= 64 entries and the
//     run sum is folded into an fp64 accumulator; one fp32 rounding per output;
//   * rows with more than kLongRow entries are taken by a whole block: the
//     waves take interleaved runs of 64 entries and their fp64 sums are
//     combined in LDS in fixed wave order. No float atomics, so the result is
//     bitwise reproducible;
//   * features up to 128 wide take a layout of 16..128 floats (several
//     entries per load instruction), and B may be processed in several such
//     feature slices when the slice of the referenced B rows gets close to
//     cache size;
//   * on graphs with long rows on average, rows are taken longest length
//     class first (a scheduling order only);
//   * when the referenced B rows span a few L2-sized ranges, the columns are
//     cut into those ranges and processed one range at a time, with fp32
//     partial rows combined in fixed range order (column-blocked mode);
//   * bit 31 of a column index (set only in a plan's own copy of col) marks
//     hub columns; when the gathered rows far outgrow the caches, the other
//     columns' rows are loaded non-temporally so the hubs' stay in L2;
//   * the per-call preparation (long-row list or row order, split bounds)
//     can be done once by a plan or at a cache refresh and reused.
#include <cstdlib>
#include <utility>

#include "rsc_internal.h"

namespace rsc {

// Rows with more than kLongRow entries are processed by a whole block (its
// waves take interleaved runs of 64 entries, then a fixed-order LDS
// reduction); shorter rows by one wave.
constexpr int kLongRow = 1024;
constexpr int kSpmmWaves = 4;          // waves per block, and short rows
// Passes of 129 to 256 features (one entry per load) over rows of 32 entries
// and more take 8 waves per block from this many rows on: 2,449,029 rows, mean
// 51, d = 256: 16.48 ms against 16.60 with 4. On shorter rows (that graph's 30 %
// slice, 5 per row) 4 waves are 1.4 % faster; fewer rows would leave compute
// units without a block, and at 512 features 8 waves cost 13 %.
constexpr int32_t kWideBlockRows = 16384;
constexpr int32_t kWideBlockMean = 32;
constexpr int kCoopWindow = 1024;      // blocks that share out the long rows among theirs
constexpr int kSpmmLongBlocks = 1024;  // blocks that walk a long-row list of unknown length
constexpr int kSpmmLongBlocksMax = 8192;  // ... of known length (a row each up to here), or that look for them
constexpr int32_t kListedRows = 262144;  // from here on an unplanned product lists its long rows
static_assert(kListedRows <= kSpmmLongBlocksMax * kSpmmWaves * kWave, "a thread for each row that is looked at");

namespace {

constexpr int kUnroll = 8;
typedef float vf4 __attribute__((ext_vector_type(4)));
constexpr int32_t kColMask = 0x7FFFFFFF;  // bit 31 of a column index: cache hint

__device__ __forceinline__ float4 load_nt(const float4 *p) {
    const vf4 x = __builtin_nontemporal_load(reinterpret_cast<const vf4 *>(p));
    return make_float4(x.x, x.y, x.z, x.w);
}

__global__ void zero_count_kernel(int32_t *p) { *p = 0; }

// Appends every row longer than kLongRow to `list`. Each thread checks
// kCollectPerThread rows (coalesced reads); a block-wide scan gives each long
// row its place, and one atomic per block reserves the block's range, so the
// list costs a few hundred atomics rather than one per row. The list order
// only decides which block takes which row.
constexpr int kCollectThreads = 1024;
constexpr int kCollectPerThread = 4;

__global__ __launch_bounds__(kCollectThreads) void collect_long_rows_kernel(
    const int32_t *__restrict__ rowptr, int32_t n_rows, int32_t *count, int32_t *list) {
    __shared__ int32_t s_wave[kCollectThreads / 64];
    __shared__ int32_t s_base;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * kCollectThreads * kCollectPerThread;
    bool is_long[kCollectPerThread];
    int32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kCollectPerThread; ++i) {
        const int64_t r = base + t + (int64_t)kCollectThreads * i;
        is_long[i] = r < n_rows && rowptr[r + 1] - rowptr[r] > kLongRow;
        mine += is_long[i];
    }
    // exclusive scan of `mine` over the block: within the wave, then across waves
    int32_t incl = mine;
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t x = __shfl_up(incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int32_t before = incl - mine, total = 0;
    for (int w = 0; w < kCollectThreads / 64; ++w) {
        before += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    if (total == 0) return;  // block-uniform
    if (t == 0) s_base = atomicAdd(count, total);
    __syncthreads();
    int32_t pos = s_base + before;
#pragma unroll
    for (int i = 0; i < kCollectPerThread; ++i)
        if (is_long[i]) list[pos++] = (int32_t)(base + t + (int64_t)kCollectThreads * i);
}

// Lane layout: LPE lanes per gathered entry, G = 64 / LPE entries per load
// instruction. Lane L belongs to entry-group g = L / LPE and owns features
// 4 * (L % LPE) .. +3 of the current feature slice (plus +256 for NV = 2,
// which is only used with LPE = 64).

// ---- one entry per load instruction (LPE = 64) ----------------------------
// Accumulates runs of 64 entries starting at beg, beg + stride, ... (< end)
// into acc; d features, 4 a lane and vector q.
// (col, val) are broadcast into SGPRs, so each B row has a scalar base.
// Bit 31 of a column index is a cache hint (set by a plan or a cache on
// their own copies; a caller's indices are < 2^31): with kHint, gathers of
// columns without it bypass cache allocation (non-temporal), so the rows of
// the columns that carry half the entries stay in L2. Values are unchanged.
// kWin gathers are in flight. kAll: lanes past the last feature read the last
// vector again in place of being masked (their sums are never stored). Without
// the mask the two kinds of load are a uniform choice, where with it the
// compiler waits for each gather before the next. A long row, whose waits no
// other wave hides, takes a third of the time so (4,000 rows, one of 1,000,000
// entries, d = 512, hinted: 80.7 ms / 27.5); short rows gain or lose by their
// number and width (hinted, 1,500,000 rows of 3, d = 300: 1,641 us / 1,319;
// 400,000 of 6, d = 512: 748 / 782) and are left masked.
template <int NV, bool kHint, int kWin, bool kAll>
__device__ __forceinline__ void accumulate_runs(const int32_t *__restrict__ col,
                                                const float *__restrict__ val,
                                                const float *__restrict__ B, int64_t ldb,
                                                int64_t beg, int64_t end, int32_t stride,
                                                int32_t d, int lane, double (&acc)[NV][4]) {
    bool act[NV];  // this lane's q-th float4 lies inside d
    int32_t at[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        at[q] = lane + kWave * q;
        act[q] = 4 * at[q] < d;
        if (kAll) at[q] = min(at[q], (d - 1) / 4);
    }
    for (int64_t base = beg; base < end; base += stride) {  // int64: base + stride may pass 2^31 - 1
        const int32_t cnt = __builtin_amdgcn_readfirstlane((int32_t)min<int64_t>(kWave, end - base));
        int32_t my_c = 0;
        float my_v = 0.f;
        if (lane < cnt) {
            my_c = __builtin_nontemporal_load(col + base + lane);
            my_v = __builtin_nontemporal_load(val + base + lane);
        }
        float a[NV][4];
#pragma unroll
        for (int q = 0; q < NV; ++q) a[q][0] = a[q][1] = a[q][2] = a[q][3] = 0.f;
        for (int32_t t = 0; t < cnt; t += kWin) {
            float4 b[kWin][NV];
            float v[kWin];
#pragma unroll
            for (int u = 0; u < kWin; ++u) {
                if constexpr (!kAll) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) b[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
                v[u] = 0.f;
                if (t + u < cnt) {  // wave-uniform
                    const int32_t cf = __builtin_amdgcn_readlane(my_c, t + u);
                    v[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v), t + u));
                    const float4 *brow = reinterpret_cast<const float4 *>(B + (int64_t)(cf & kColMask) * ldb);
                    if (kHint && cf >= 0) {  // not a hub column: stream it past the caches
#pragma unroll
                        for (int q = 0; q < NV; ++q)
                            if (kAll || act[q]) b[u][q] = load_nt(brow + at[q]);
                    } else {
#pragma unroll
                        for (int q = 0; q < NV; ++q)
                            if (kAll || act[q]) b[u][q] = brow[at[q]];
                    }
                } else if constexpr (kAll) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) b[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
#pragma unroll
            for (int u = 0; u < kWin; ++u)
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    a[q][0] = fmaf(v[u], b[u][q].x, a[q][0]);
                    a[q][1] = fmaf(v[u], b[u][q].y, a[q][1]);
                    a[q][2] = fmaf(v[u], b[u][q].z, a[q][2]);
                    a[q][3] = fmaf(v[u], b[u][q].w, a[q][3]);
                }
        }
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[q][x] += (double)a[q][x];
    }
}

// ---- G = 64 / LPE entries per load instruction (LPE = 4, 8, 16, 32) --------
// Entry-group g (LPE lanes) takes entries g, g + G, g + 2G, ... of a 64-entry
// run; its fp32 sum over them is folded into the lane's fp64 acc, and the
// groups' sums are added when the row is done (sum_groups). Two forms give
// the same sums bit for bit: through a buffer descriptor (accumulate_groups),
// and with 64-bit addresses (accumulate_groups_wide) for operands that a
// descriptor cannot cover and for the hub hint, which needs a lane mask
// around two kinds of load (as two descriptor loads, each out of range for
// the other's lanes, the hint gained less or lost: 1.86M nodes of mean
// degree 26, d = 96, 2.89 ms against 2.52).
//
// The descriptor form: (col, val) are loaded in order and permuted once per
// run, so that the entry group g needs at step t sits in a lane of g's own
// row of 16 lanes and reaches the others by a DPP operand: entry t * G + g in
// lane t of each group for LPE <= 16; for LPE = 32 both rows of a group hold
// the same 16 entries, steps 0..15 in one register pair and 16..31 in a
// second. (Loading them permuted instead touches four times the lines per
// load.) The byte offset of an entry's B row is one multiply by the lane that
// loaded it, and the descriptor's range check returns zeros for the entries
// past the end of a run, so no step has a branch, a lane mask or 64-bit
// address arithmetic: 6 vector instructions per 1 KB gather, against about 25
// with a ds_bpermute broadcast per step, each of which the next gather waited
// for.
constexpr uint32_t kNoEntry = 0xFFFFF000u;  // offset past every operand the descriptor may cover
constexpr uint64_t kBufMax = kNoEntry;      // operands read through a descriptor are smaller than this

// lane T of the caller's entry-group (of its row of 16 for LPE = 32)
template <int LPE, int T>
__device__ __forceinline__ int32_t bcast(int32_t x) {
    if constexpr (LPE >= 16) {
        return __builtin_amdgcn_update_dpp(0, x, 0x150 + T, 0xf, 0xf, true);  // row_newbcast:T
    } else if constexpr (LPE == 8) {  // two groups per row: lanes 0-7, then lanes 8-15
        const int32_t lo = __builtin_amdgcn_update_dpp(0, x, 0x150 + T, 0xf, 0xf, true);
        return __builtin_amdgcn_update_dpp(lo, x, 0x150 + 8 + T, 0xf, 0xc, false);
    } else {
        static_assert(LPE == 4, "lane layouts");
        return __builtin_amdgcn_update_dpp(0, x, T * 0x55, 0xf, 0xf, true);  // quad_perm:[T,T,T,T]
    }
}

struct Operand {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t lane_off;  // byte offset of this lane's features within a row
};

// row: the byte offset of my entry's B row, kNoEntry if there is none
template <int LPE, int T>
__device__ __forceinline__ vf4 gather(const Operand &op, int32_t row) {
    const uint32_t at = (uint32_t)bcast<LPE, T>(row) + op.lane_off;
    return __builtin_bit_cast(vf4, __builtin_amdgcn_raw_buffer_load_b128(op.rsrc, at, 0, 0));
}

// The entries of one 64-entry run, as the lanes hold them: register pair q
// has the entries of steps 16 q .. 16 q + 15.
template <int LPE>
struct Run {
    static constexpr int kGroups = kWave / LPE;
    static constexpr int kSteps = kWave / kGroups;           // steps of a whole run
    static constexpr int kPairSteps = LPE < 16 ? LPE : 16;   // steps one register pair covers
    static constexpr int kPairs = kSteps / kPairSteps;
    static constexpr int kBlocks = kSteps / 4;               // steps are taken four at a time
    int32_t row[kPairs];
    float v[kPairs];
};

// Four steps' gathers, and their products.
template <int LPE, int BLK, int... U>
__device__ __forceinline__ void issue4(const Operand &op, const Run<LPE> &run, vf4 (&b)[4],
                                       std::integer_sequence<int, U...>) {
    constexpr int T0 = BLK * 4 % Run<LPE>::kPairSteps, q = BLK * 4 / Run<LPE>::kPairSteps;
    ((b[U] = gather<LPE, T0 + U>(op, run.row[q])), ...);
}
template <int LPE, int BLK, int... U>
__device__ __forceinline__ void add4(const Run<LPE> &run, const vf4 (&b)[4], float (&a)[4],
                                     std::integer_sequence<int, U...>) {
    constexpr int T0 = BLK * 4 % Run<LPE>::kPairSteps, q = BLK * 4 / Run<LPE>::kPairSteps;
    const auto add = [&](float v, const vf4 &x) {
        a[0] = fmaf(v, x.x, a[0]);
        a[1] = fmaf(v, x.y, a[1]);
        a[2] = fmaf(v, x.z, a[2]);
        a[3] = fmaf(v, x.w, a[3]);
    };
    (add(__int_as_float(bcast<LPE, T0 + U>(__float_as_int(run.v[q]))), b[U]), ...);
}

// Blocks 0 .. NB - 1 of a run in straight-line code, four to eight gathers in
// flight: block b + 2 is issued when block b has been added. `behind` (the
// load of the next run's entries) goes behind the first gathers, so that no
// gather waits for it.
template <int LPE, int NB, int BLK = 0, typename F>
__device__ __forceinline__ void run_blocks(const Operand &op, const Run<LPE> &run, vf4 (&b0)[4],
                                           vf4 (&b1)[4], float (&a)[4], F behind) {
    using four = std::make_integer_sequence<int, 4>;
    if constexpr (BLK == 0) {
        issue4<LPE, 0>(op, run, b0, four{});
        if constexpr (NB > 1) issue4<LPE, 1>(op, run, b1, four{});
        behind();
        __builtin_amdgcn_sched_barrier(0);  // all of them before the first wait
    }
    add4<LPE, BLK>(run, b0, a, four{});
    if constexpr (BLK + 2 < NB) issue4<LPE, BLK + 2>(op, run, b0, four{});
    if constexpr (BLK + 1 < NB) run_blocks<LPE, NB, BLK + 1>(op, run, b1, b0, a, behind);
}

__device__ __forceinline__ void fold(const float (&a)[4], double (&acc)[4]) {
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[x] += (double)a[x];
}

// The run's first nb blocks (1 <= nb <= kBlocks, wave-uniform).
template <int LPE, int NB = 1>
__device__ __forceinline__ void run_first(const Operand &op, const Run<LPE> &run, int32_t nb, float (&a)[4]) {
    if (NB == Run<LPE>::kBlocks || nb == NB) {
        vf4 b0[4], b1[4];
        run_blocks<LPE, NB>(op, run, b0, b1, a, [] {});
    } else if constexpr (NB < Run<LPE>::kBlocks) {
        run_first<LPE, NB + 1>(op, run, nb, a);
    }
}

// Sums the entries of runs beg, beg + stride, ... (< end; stride >= 64, beg <
// end): each group's fp32 sum over its share of a run is folded into the
// lane's fp64 acc, but for the last run's, which is left in `last`. Every run
// but the last is whole.
template <int LPE>
__device__ __forceinline__ void accumulate_groups(const int32_t *__restrict__ col, const float *__restrict__ val,
                                                  const Operand &op, uint32_t ldb_bytes, int64_t beg,
                                                  int64_t end, int32_t stride, int lane, double (&acc)[4],
                                                  float (&last)[4]) {
    using R = Run<LPE>;
    constexpr int kPairEntries = R::kPairSteps * R::kGroups;
    // lane that loaded this lane's entry of a run (pair q's is kPairEntries further on)
    const int32_t e0 = (lane % R::kPairSteps) * R::kGroups + lane / LPE;
    int32_t nc;
    float nv;
    const auto load = [&](int64_t base) {  // past the end: the row's last entry, masked by take()
        const int64_t p = min<int64_t>(base + lane, end - 1);
        nc = __builtin_nontemporal_load(col + p);
        nv = __builtin_nontemporal_load(val + p);
    };
    R run;
    const auto take = [&](int64_t base, bool whole) {
        const bool in = whole || base + lane < end;
        const int32_t r = in ? (int32_t)((uint32_t)(nc & kColMask) * ldb_bytes) : (int32_t)kNoEntry;
        const float v = in ? nv : 0.f;
#pragma unroll
        for (int q = 0; q < R::kPairs; ++q) {
            run.row[q] = __shfl(r, e0 + q * kPairEntries);
            run.v[q] = __shfl(v, e0 + q * kPairEntries);
        }
    };
    load(beg);
    int64_t base = beg;  // int64: base + stride may pass 2^31 - 1
    for (; base + stride < end; base += stride) {
        take(base, true);
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        vf4 b0[4], b1[4];
        run_blocks<LPE, R::kBlocks>(op, run, b0, b1, a, [&] { load(base + stride); });
        fold(a, acc);
    }
    take(base, false);
    const int32_t left = __builtin_amdgcn_readfirstlane((int32_t)min<int64_t>(kWave, end - base));
    run_first<LPE>(op, run, (left + 4 * R::kGroups - 1) / (4 * R::kGroups), last);
}

// The same sums with 64-bit addresses and a lane mask per step; kHint as in
// accumulate_runs.
template <int LPE, bool kHint, int kMaxWin>
__device__ __forceinline__ void accumulate_groups_wide(const int32_t *__restrict__ col,
                                                       const float *__restrict__ val, const float *__restrict__ B,
                                                       int64_t ldb, int64_t beg, int64_t end, int32_t stride,
                                                       bool act, int lane, double (&acc)[4], float (&last)[4]) {
    constexpr int G = kWave / LPE;
    constexpr int kSteps = kWave / G;           // steps that cover the 64-entry run
    constexpr int kWin = G >= 8 ? 4 : std::min(kMaxWin, kUnroll);  // steps per window (gathers in flight)
    const int g = lane / LPE, sl = lane % LPE;
    for (int64_t base = beg; base < end; base += stride) {
        if (base > beg) fold(last, acc);
        const int32_t cnt = __builtin_amdgcn_readfirstlane((int32_t)min<int64_t>(kWave, end - base));
        int32_t my_c = 0;
        float my_v = 0.f;
        if (lane < cnt) {
            my_c = __builtin_nontemporal_load(col + base + lane);
            my_v = __builtin_nontemporal_load(val + base + lane);
        }
        float a[4] = {0.f, 0.f, 0.f, 0.f};
        // one window at a time: unrolling the step loop too keeps every
        // window's (col, val) live at once (130 VGPRs for G = 2) and costs
        // occupancy
#pragma unroll 1
        for (int t0 = 0; t0 < kSteps; t0 += kWin) {
            if (t0 * G >= cnt) break;  // wave-uniform
            float4 b[kWin];
            float v[kWin];
#pragma unroll
            for (int u = 0; u < kWin; ++u) {
                const int j = (t0 + u) * G + g;  // entry of this group within the run
                const int32_t cf = __shfl(my_c, j & (kWave - 1));
                const int32_t c = cf & kColMask;
                const float vv = __shfl(my_v, j & (kWave - 1));
                const bool in = t0 + u < kSteps && j < cnt && act;
                // selected out here: set inside the branch, the compiler had
                // each window's first gather waited for before the others were
                // issued (1,500,000 rows of 3 entries, d = 96, hinted: 657 us
                // against 570)
                v[u] = in ? vv : 0.f;
                b[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (in) {
                    const float4 *brow = reinterpret_cast<const float4 *>(B + (int64_t)c * ldb) + sl;
                    b[u] = (kHint && cf >= 0) ? load_nt(brow) : *brow;
                }
            }
#pragma unroll
            for (int u = 0; u < kWin; ++u) {
                a[0] = fmaf(v[u], b[u].x, a[0]);
                a[1] = fmaf(v[u], b[u].y, a[1]);
                a[2] = fmaf(v[u], b[u].z, a[2]);
                a[3] = fmaf(v[u], b[u].w, a[3]);
            }
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) last[x] = a[x];
    }
}

// Adds the groups' sums; every lane of a group ends with the total of its
// features. Fixed order.
template <int LPE, typename T>
__device__ __forceinline__ void sum_groups(T (&a)[4]) {
#pragma unroll
    for (int m = LPE; m < kWave; m <<= 1)
#pragma unroll
        for (int x = 0; x < 4; ++x) a[x] += __shfl_xor(a[x], m);
}

// What a wave accumulates for one row with either kind of layout; in the
// sliced ones the last run's sums are left in `last`.
template <int LPE, int NV, bool kHint, bool kBuf, int kWin = kUnroll, bool kLong = false>
__device__ __forceinline__ void accumulate(const int32_t *__restrict__ col, const float *__restrict__ val,
                                           const float *__restrict__ B, int64_t ldb, uint32_t b_bytes, int64_t beg,
                                           int64_t end, int32_t stride, int32_t d, int lane, double (&acc)[NV][4],
                                           float (&last)[4]) {
    if constexpr (LPE == kWave) {
        accumulate_runs<NV, kHint, kWin, kLong>(col, val, B, ldb, beg, end, stride, d, lane, acc);
    } else {
        static_assert(NV == 1, "the sliced layouts hold one float4 per lane");
        if constexpr (kBuf) {
            static_assert(!kHint, "the hint takes the wide form");
            // a lane past the last feature reads the last one's vector again (no
            // further line is touched); its sums are never stored
            Operand op;
            op.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(B), 0, b_bytes, 0x00027000);
            op.lane_off = 16u * min(lane % LPE, (d - 1) / 4);
            if (beg < end)
                accumulate_groups<LPE>(col, val, op, (uint32_t)(4 * ldb), beg, end, stride, lane, acc[0], last);
        } else {
            accumulate_groups_wide<LPE, kHint, kWin>(col, val, B, ldb, beg, end, stride, 4 * (lane % LPE) < d, lane,
                                                     acc[0], last);
        }
    }
}

template <int LPE, int NV, typename T>
__device__ __forceinline__ void store_row(float *__restrict__ yrow, int32_t d, int lane, const T (&acc)[NV][4]) {
    if (lane >= LPE) return;  // every entry-group holds the same sums; group 0 stores
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int32_t f = 4 * lane + 4 * kWave * q;
        if (f + 4 <= d) {
            vf4 o = {(float)acc[q][0], (float)acc[q][1], (float)acc[q][2], (float)acc[q][3]};
            __builtin_nontemporal_store(o, reinterpret_cast<vf4 *>(yrow + f));
        } else if (f < d) {
            for (int x = 0; x < d - f; ++x) yrow[f + x] = (float)acc[q][x];
        }
    }
}

// A long row by the whole block: the waves' sums are added in wave order
// through LDS and the last wave stores the total. Reached by every wave. kWin
// gathers are in flight per wave (one entry per load).
template <int LPE, int NV, bool kHint, bool kBuf, int kWaves, int kWin>
__device__ __forceinline__ void take_long_row(const int32_t *__restrict__ col, const float *__restrict__ val,
                                              const float *__restrict__ B, int64_t ldb, uint32_t b_bytes,
                                              float *__restrict__ yrow, int32_t d, int32_t s, int32_t e, int lane,
                                              int wave, double (*red)[kWave]) {
    double acc[NV][4];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q][0] = acc[q][1] = acc[q][2] = acc[q][3] = 0.0;
    float last[4] = {0.f, 0.f, 0.f, 0.f};
    accumulate<LPE, NV, kHint, kBuf, kWin, true>(col, val, B, ldb, b_bytes, (int64_t)s + kWave * wave, e,
                                                 kWave * kWaves, d, lane, acc, last);
    if constexpr (LPE < kWave) fold(last, acc[0]);
    // opaque: what derives from the lane below is computed here and not kept
    // in registers through the gathers
    asm volatile("" : "+v"(lane));
    for (int w = 0; w < kWaves; ++w) {  // block-uniform
        if (w > 0) __syncthreads();
        if (wave != w) continue;
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (w > 0) acc[q][x] = red[q * 4 + x][lane] + acc[q][x];
                if (w < kWaves - 1) red[q * 4 + x][lane] = acc[q][x];
                __builtin_amdgcn_sched_barrier(0);  // one value at a time: registers, not latency
            }
    }
    if (wave == kWaves - 1) {
        if constexpr (LPE < kWave) sum_groups<LPE>(acc[0]);
        store_row<LPE, NV>(yrow, d, lane, acc);
    }
    __syncthreads();  // red is reused by the next row
}

// One launch takes all rows. Row r spans [ptr[r], ptr[r + off]) and is
// written to row r of Y; kCsr says off == 1 (a CSR row pointer). B and Y point
// at the first feature of the current slice; d is its width.
//
// Blocks from n_long on take kWaves consecutive rows, one wave each. Long
// rows are a block's work, by one of three ways:
//   * a list: the first n_long blocks walk the prepared list of long rows (or
//     the head of `order`), so that the heaviest rows start first;
//   * no list (NULL; nothing prepared): each of the first n_long blocks looks
//     through every n_long-th row and takes the long ones it finds. Long rows
//     side by side (nodes sorted by degree) so go to as many blocks;
//   * kCoop (column-blocked, n_long = 0): a block looks at every step-th row of
//     a window of kCoopWindow blocks' rows, and takes the long ones when its
//     short rows are done. A window is about what the chip holds at once, so a
//     long piece reads the range of B that its neighbours read.
// (Blocks that took the long ones of their own rows: 60,013 rows, mean 27,
// hubs of 30,000 entries in the first rows, d = 41: 426 us, against 129; d =
// 128: 758, against 246.)
// With `order`, the rows are taken in that order after its first *long_count
// entries (the long rows). Which block takes a row never changes its sum.
// (Long rows in a launch of their own before the others left the chip to its
// last few rows twice. us, two launches / one: 60,013 nodes, mean 27, d = 41
// 70 / 46; 716,847 nodes, mean 20, d = 512: 4,160 / 4,044; the 30 % slice of
// 232,965 nodes, mean 490, d = 256: 3,257 / 3,122.)
//
// A long row is a serial chain: with one entry per load, 4 waves have too few
// gathers in flight. Its features are halved over two blocks then (kParts;
// the n_long blocks are pairs), which have twice as many entries in flight:
// over 256 features as 16 gathers of 1 KB in place of 8 of 2 KB, fewer in the
// 128-float layout, two entries per load. 8-wave blocks take theirs whole. us,
// whole with 4 waves / so: 60,013 rows, mean 27, hubs of 30,000 entries, d =
// 256: 888 / 344; a row of 1,000,000 entries among 4,000, d = 256: 32,000 /
// 9,300, d = 512: 40,800 / 24,000.
constexpr int long_parts(int lpe, int nv, int waves) { return lpe == kWave && (nv == 2 || waves == 4) ? 2 : 1; }

template <int LPE, int NV, bool kCsr, bool kHint, bool kBuf, bool kCoop, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void spmm_kernel(
    const int32_t *__restrict__ ptr, int64_t off, const int32_t *__restrict__ col, const float *__restrict__ val,
    const float *__restrict__ B, int64_t ldb, uint32_t b_bytes, float *__restrict__ Y, int64_t ldy, int32_t n_rows,
    int32_t d, int32_t n_long, const int32_t *__restrict__ list, int32_t ordered,
    const int32_t *__restrict__ long_count) {
    __shared__ double red[4][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    constexpr int kParts = long_parts(LPE, NV, kWaves), kHalf = 2 * kWave * NV;  // of the features
    const auto take_long = [&](int32_t r) {
        const int32_t s = __builtin_amdgcn_readfirstlane(ptr[r]);
        const int32_t e = __builtin_amdgcn_readfirstlane(ptr[(int64_t)r + (kCsr ? 1 : off)]);
        int ln = lane;
        asm volatile("" : "+v"(ln));  // as in take_long_row
        if constexpr (kParts == 1) {
            take_long_row<LPE, 1, kHint, kBuf, kWaves, kUnroll>(col, val, B, ldb, b_bytes, Y + (int64_t)r * ldy, d, s, e,
                                                                ln, wave, red);
        } else {  // 6: the 64-bit form then keeps 64 registers, as the short rows do
            const int32_t f = blockIdx.x % 2 * kHalf;
            take_long_row<NV == 2 ? kWave : kWave / 2, 1, kHint, kBuf, kWaves, NV == 2 ? 2 * kUnroll : 6>(
                col, val, B + f, ldb, b_bytes - 4 * f, Y + (int64_t)r * ldy + f, min(d - f, kHalf), s, e, ln, wave, red);
        }
    };
    const int32_t bid = blockIdx.x;
    if constexpr (!kCoop) {
        if (bid < n_long) {
            if (kParts == 2 && bid % 2 * kHalf >= d) return;
            const int32_t me = bid / kParts, n_me = n_long / kParts;
            __shared__ uint64_t found[kWaves];
            if (!list) {  // thread t looks at row me + n_me t (n_me * kWaves * kWave >= n_rows)
                const int32_t q = me + n_me * threadIdx.x;
                const uint64_t mine = __ballot(q < n_rows && ptr[q + 1] - ptr[q] > kLongRow);
                if (lane == 0) found[wave] = mine;
                __syncthreads();
            }
            const int32_t n_list = list ? __builtin_amdgcn_readfirstlane(*long_count) : kWaves;
            uint64_t left = 0;  // of the 64 rows that wave j looked at
            for (int32_t j = list ? me : -1;;) {
                int32_t r;
                if (list) {
                    if (j >= n_list) return;
                    r = __builtin_amdgcn_readfirstlane(list[j]);
                    j += n_me;
                } else {
                    while (left == 0) {
                        if (++j == n_list) return;
                        left = (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(found[j] >> 32)) << 32 |
                               (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)found[j]);
                    }
                    r = me + n_me * (j * kWave + __builtin_ctzll(left));
                    left &= left - 1;
                }
                take_long(r);
            }
        }
    }
    const int32_t first = (kCoop ? bid : bid - n_long) * kWaves;  // the block's first row
    int32_t r = first + wave, s = 0, e = 0;
    if (!kCoop && ordered) {
        const int64_t i = (int64_t)__builtin_amdgcn_readfirstlane(*long_count) + r;
        if (i >= n_rows) return;
        r = __builtin_amdgcn_readfirstlane(list[i]);
    }
    const auto end_of = [&](int32_t row) { return ptr[(int64_t)row + (kCsr ? 1 : off)]; };
    // the block's share of its window's long rows: every wave finds the same
    uint32_t longs = 0;
    int32_t long0 = 0, step = 0;
    if constexpr (kCoop) {
        const int32_t w0 = bid / kCoopWindow * kCoopWindow;
        step = min(kCoopWindow, (int32_t)gridDim.x - w0);
        long0 = w0 * kWaves + (bid - w0);
        int32_t len[kWaves];  // in one round of scalar loads
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            const int32_t q = min(long0 + i * step, n_rows - 1);
            len[i] = end_of(q) - ptr[q];
        }
#pragma unroll
        for (int i = 0; i < kWaves; ++i)
            if (len[i] > kLongRow && long0 + i * step < n_rows) longs |= 1u << i;
    }
    if (r < n_rows) {
        s = __builtin_amdgcn_readfirstlane(ptr[r]);
        e = __builtin_amdgcn_readfirstlane(end_of(r));
    }
    if (r < n_rows && !((kCoop || n_long > 0) && e - s > kLongRow)) {
        double acc[NV][4];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q][0] = acc[q][1] = acc[q][2] = acc[q][3] = 0.0;
        float last[1][4] = {{0.f, 0.f, 0.f, 0.f}};
        accumulate<LPE, NV, kHint, kBuf>(col, val, B, ldb, b_bytes, s, e, kWave, d, lane, acc, last[0]);
        if constexpr (LPE < kWave) {
            // One run: its fp32 sums are added and stored as they are (through
            // fp64 and back, 1,500,000 rows of 3 entries, d = 32, took 415 us
            // in place of 400). A negative zero becomes the positive one that
            // the fp64 sums give.
            if (e - s <= kWave) {
                sum_groups<LPE>(last[0]);
#pragma unroll
                for (int x = 0; x < 4; ++x) last[0][x] += 0.f;
            } else {
                fold(last[0], acc[0]);
                sum_groups<LPE>(acc[0]);
#pragma unroll
                for (int x = 0; x < 4; ++x) last[0][x] = (float)acc[0][x];
            }
            store_row<LPE, 1>(Y + (int64_t)r * ldy, d, lane, last);
        } else {
            store_row<LPE, NV>(Y + (int64_t)r * ldy, d, lane, acc);
        }
    }
    if constexpr (kCoop)
        for (; longs; longs &= longs - 1) take_long(long0 + __builtin_ctz(longs) * step);  // block-uniform
}

// Bytes of B that a pass over dl features may read, counted from the first
// one (whole 16-byte vectors, ld % 4 == 0); 0 when they pass what
// a buffer descriptor's 32-bit offsets cover below kNoEntry.
inline uint32_t buffer_bytes(int32_t n_cols, int64_t ldb, int32_t dl) {
    if (n_cols <= 0) return 0;
    const __int128 bytes = 4 * ((__int128)(n_cols - 1) * ldb + (dl + 3) / 4 * 4);
    return bytes < (__int128)kBufMax ? (uint32_t)bytes : 0u;
}

constexpr int kClasses = 32;

struct SpmmWs {
    int32_t long_count;  // rows in the long-row list
    int32_t pad[31];
    int32_t cls_count[kClasses];   // rows per length class (ordered mode)
    int32_t cls_cursor[kClasses];  // next free slot of each class in the order
    int32_t pad2[32];
};

inline int64_t long_rows_bound(int32_t n_rows, int64_t nnz) {
    return std::min<int64_t>(n_rows, nnz / (kLongRow + 1));
}

// Length class of a row: 0 for at most one entry, else ceil(log2(len)), so
// rows longer than kLongRow = 1024 are exactly the classes >= 11.
__device__ __forceinline__ int row_class(int32_t len) { return len <= 1 ? 0 : 32 - __clz(len - 1); }
constexpr int kLongClass = 11;
static_assert(kLongRow == 1024, "class boundary of the long rows");

__global__ __launch_bounds__(128) void zero_header_kernel(SpmmWs *h) {
    reinterpret_cast<int32_t *>(h)[threadIdx.x] = 0;
}

// Rows per length class: an LDS histogram per block, one atomic per class.
__global__ __launch_bounds__(kCollectThreads) void class_hist_kernel(const int32_t *__restrict__ rowptr,
                                                                    int32_t n_rows, SpmmWs *h) {
    __shared__ int32_t hist[kClasses];
    if (threadIdx.x < kClasses) hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kCollectThreads * kCollectPerThread;
#pragma unroll
    for (int i = 0; i < kCollectPerThread; ++i) {
        const int64_t r = base + threadIdx.x + (int64_t)kCollectThreads * i;
        if (r < n_rows) atomicAdd(&hist[row_class(rowptr[r + 1] - rowptr[r])], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses && hist[threadIdx.x]) atomicAdd(&h->cls_count[threadIdx.x], hist[threadIdx.x]);
}

// Class start offsets with the longest class first; the long rows (classes
// >= kLongClass) come out as the first long_count entries of the order.
__global__ __launch_bounds__(64) void class_scan_kernel(SpmmWs *h) {
    const int c = threadIdx.x;
    if (c >= kClasses) return;
    int32_t start = 0, lng = 0;
    for (int k = c + 1; k < kClasses; ++k) start += h->cls_count[k];
    for (int k = kLongClass; k < kClasses; ++k) lng += h->cls_count[k];
    h->cls_cursor[c] = start;
    if (c == 0) {
        h->long_count = lng;
    }
}

// Places every row in its class's range (the order within a class follows
// the atomics and does not matter: it only decides which wave takes a row).
__global__ __launch_bounds__(kCollectThreads) void class_scatter_kernel(const int32_t *__restrict__ rowptr,
                                                                       int32_t n_rows, SpmmWs *h,
                                                                       int32_t *__restrict__ order) {
    __shared__ int32_t hist[kClasses];
    __shared__ int32_t slot[kClasses];
    if (threadIdx.x < kClasses) hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kCollectThreads * kCollectPerThread;
    int cls[kCollectPerThread];
#pragma unroll
    for (int i = 0; i < kCollectPerThread; ++i) {
        const int64_t r = base + threadIdx.x + (int64_t)kCollectThreads * i;
        cls[i] = r < n_rows ? row_class(rowptr[r + 1] - rowptr[r]) : -1;
        if (cls[i] >= 0) atomicAdd(&hist[cls[i]], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses)
        slot[threadIdx.x] = hist[threadIdx.x] ? atomicAdd(&h->cls_cursor[threadIdx.x], hist[threadIdx.x]) : 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCollectPerThread; ++i)
        if (cls[i] >= 0)
            order[atomicAdd(&slot[cls[i]], 1)] = (int32_t)(base + threadIdx.x + (int64_t)kCollectThreads * i);
}

// Rows are taken longest class first when rows are long on average: the
// heavy rows then start first and the kernels end on short rows. Results do
// not depend on it. RSC_SPMM_ORDER=0/1 overrides.
// Gathered rows beyond this many bytes per feature pass take the column
// cache hint (twice the 256 MB MALL).
constexpr double kHintBytes = 512.0 * 1024 * 1024;

inline bool use_hint() {
    if (const char *env = getenv("RSC_SPMM_HINT")) return atoi(env) != 0;
    return true;
}

inline bool use_order(int32_t n_rows, int64_t nnz) {
    if (const char *env = getenv("RSC_SPMM_ORDER")) return atoi(env) != 0;
    return n_rows > 0 && nnz >= 128LL * n_rows;
}

// ---- column-blocked mode ------------------------------------------------
// When the columns of B fit L2 in a few pieces, the product is taken one
// piece at a time: the columns are cut into P equal ranges, and "virtual row"
// (b, r) = the entries of row r whose column lies in range b (contiguous in
// the row, since columns are sorted). The virtual rows are processed
// block-major, so at any moment the whole GPU gathers from one range of B
// rows (a few MB, resident in each XCD's L2) instead of from all of them.
// Each virtual row writes a partial row; a combine pass adds the P partials
// of row r in fixed order b = 0..P-1 in fp64 and rounds once.
constexpr int kBlockW = 64;                         // features per blocked pass, the widest layout
constexpr double kBlockBytes = 4.5 * 1024 * 1024;   // B bytes per column range (~ one XCD's L2)
constexpr double kFineBytes = 3.0 * 1024 * 1024;    // and for 64-float passes when the pieces stay long
constexpr int kMaxBlocks = 12;                      // partial outputs at most 12 x Y per pass
constexpr int kCoarseBlocks = 8;                    // ... 8 x with ranges of kBlockBytes
constexpr int kPieceMin = 56;                       // mean entries per piece of a row for blocking

// Features per blocked pass for feature width d: the narrowest of the 16-,
// 32- and 64-float layouts that holds d (wider d in several 64-float
// passes), so no lane of a narrow product idles.
inline int32_t blocked_width(int32_t d) { return d <= 16 ? 16 : d <= 32 ? 32 : kBlockW; }

// the row list: the whole processing order, or the long rows
inline size_t list_bytes(int32_t n_rows) {
    return align_up(sizeof(int32_t) * (size_t)std::max(n_rows, 1), 256);
}
// bytes of the blocked mode's split points and partial rows for P ranges
inline size_t blocked_bytes(int32_t n_rows, int32_t P) {
    if (P <= 1) return 0;
    return align_up(sizeof(int32_t) * (size_t)n_rows * (P + 1), 256) +
           align_up(sizeof(float) * (size_t)P * n_rows * kBlockW, 256);
}

// Number of column ranges P for a product with n_rows rows, about nnz
// entries, n_src distinct B rows referenced and d features; 1 = not blocked.
// Blocked when the referenced slice of B one pass gathers from (the
// blocked_width(d) floats of each row) spans 2..16 L2-sized ranges and rows
// are long enough that each piece still fills about 14 load instructions on
// average: kPieceMin entries in the 64-float layout (4 entries per
// instruction), twice and four times that in the 32- and 16-float layouts
// (8 and 16 per instruction). Beyond 8 ranges P stays 8: ranges of up to two
// L2 sizes still keep most gathers on chip. 64-float passes over long rows
// take ranges of 3 MiB instead, up to 12 of them while a piece keeps
// kPieceMin entries: a range of 4.24 MB does not quite fit an L2 that col,
// val and the partial rows stream through as well. Shorter rows lose by it.
// us, by the number of ranges (1 = not blocked, * = the rule's):
//   132,534 nodes, 600 per row, uniform
//     d = 256, exact      1 9,508  6 4,823  8 4,640  10* 4,499  12 4,485  16 4,734
//     30 % of the columns 1 1,600  2 1,498  3* 1,389  4 1,409  6 1,557
//     d = 32, exact       1 1,175  3 682  4* 660  5 655  8 687
//     d = 16, exact       1 827  2* 603  3 587  4 597  8 635
//   232,965 nodes, 490 per row, power law
//     d = 256, exact      1 9,279  4 7,634  6 7,360  8* 7,482  10 7,701  16 8,632
//     30 % of the columns 1* 3,226  2 3,529  4 3,644  8 4,281
//     d = 32, exact       1* 1,107  3 1,037  8 1,123; d = 16: 1* 957  4 908  8 1,021
//   100,000 nodes, 260 per row, power law
//     d = 256, exact      1* 1,835  2 1,904  4 1,842  8 2,054
// Where the scratch of
// rsc_spmm_noalloc holds the buffers of the 4.5 MiB ranges, no more ranges
// than it holds, so that both calls give the same bits.
// RSC_SPMM_BLOCKED=0 switches the mode off, =2..8 forces that P.
inline int32_t column_blocks(int32_t n_rows, int64_t nnz, int64_t n_src, int32_t d) {
    if (n_rows <= 0 || (int64_t)(kMaxBlocks + 1) * n_rows > INT32_MAX) return 1;  // virtual rows are int32
    if (const char *env = getenv("RSC_SPMM_BLOCKED")) {
        const int v = atoi(env);
        if (v == 0) return 1;
        if (v >= 2 && v <= kCoarseBlocks) return v;
    }
    const int32_t W = blocked_width(d);
    int64_t P = (int64_t)std::ceil((double)n_src * W * 4 / kBlockBytes);
    if (P < 2 || P > 2 * kCoarseBlocks) return 1;
    P = std::min<int64_t>(P, kCoarseBlocks);
    if (nnz < (int64_t)kPieceMin * (kBlockW / W) * P * n_rows) return 1;
    if (W == kBlockW) {
        const int64_t r = (int64_t)std::ceil((double)n_src * W * 4 / kFineBytes);
        const int64_t fine = std::max(P, std::min<int64_t>({r, kMaxBlocks, nnz / ((int64_t)kPieceMin * n_rows)}));
        const auto in_scratch = [&](int64_t p) {
            return spmm_blocked_fits(n_rows, (int32_t)p) <= kNoallocScratchBytes;
        };
        const bool coarse_fits = in_scratch(P);
        while (P < fine && (!coarse_fits || in_scratch(P + 1))) ++P;
    }
    return (int32_t)P;
}

// S[b * n_rows + r] = first entry of row r with column >= b * n_cols / P
// (b = 0: rowptr[r]; b = P: rowptr[r + 1]); binary search in the sorted row.
// Piece b of row r ("virtual row" v = b * n_rows + r) is then
// [S[v], S[v + n_rows]): the row kernels take S with offset n_rows as their
// row pointer, and consecutive virtual rows run through one column range.
__global__ __launch_bounds__(256) void split_rows_kernel(const int32_t *__restrict__ rowptr,
                                                         const int32_t *__restrict__ col, int32_t n_rows,
                                                         int32_t n_cols, int32_t P, int32_t *__restrict__ S) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_rows * (P + 1)) return;
    const int32_t b = (int32_t)(t / n_rows);
    const int64_t r = t - (int64_t)b * n_rows;
    const int32_t s = rowptr[r], e = rowptr[r + 1];
    int32_t pos;
    if (b == 0) {
        pos = s;
    } else if (b == P) {
        pos = e;
    } else {
        const int64_t bound = (int64_t)b * n_cols / P;
        int32_t lo = s, hi = e;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if ((col[mid] & kColMask) < bound) lo = mid + 1; else hi = mid;
        }
        pos = lo;
    }
    S[t] = pos;
}

// Y[r][f] = fl32(sum over b = 0..P-1 of part[b * n_rows + r][f]) in fp64;
// one thread per 4 features of a row.
__global__ __launch_bounds__(256) void combine_blocks_kernel(const float *__restrict__ part, int64_t ldp,
                                                             int32_t n_rows, int32_t P, int32_t d,
                                                             float *__restrict__ Y, int64_t ldy) {
    const int32_t q = (d + 3) / 4;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_rows * q) return;
    const int64_t r = t / q;
    const int32_t f = 4 * (int32_t)(t - r * q);
    const int32_t m = min(4, d - f);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int32_t b = 0; b < P; ++b) {
        const float *p = part + ((int64_t)b * n_rows + r) * ldp + f;
        if (m == 4) {
            const vf4 x = __builtin_nontemporal_load(reinterpret_cast<const vf4 *>(p));
            acc[0] += (double)x.x;
            acc[1] += (double)x.y;
            acc[2] += (double)x.z;
            acc[3] += (double)x.w;
        } else {
            for (int i = 0; i < m; ++i) acc[i] += (double)p[i];
        }
    }
    float *y = Y + r * ldy + f;
    if (m == 4) {
        const vf4 o = {(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
        __builtin_nontemporal_store(o, reinterpret_cast<vf4 *>(y));
    } else {
        for (int i = 0; i < m; ++i) y[i] = (float)acc[i];
    }
}

}  // namespace

int32_t spmm_column_blocks(int32_t n_rows, int64_t nnz, int64_t n_src, int32_t d) {
    return column_blocks(n_rows, nnz, n_src, d);
}

hipError_t spmm_split_launch(int32_t n_rows, int32_t n_cols, const int32_t *rowptr, const int32_t *col, int32_t P,
                             int32_t *S, hipStream_t stream) {
    const int64_t ns = (int64_t)n_rows * (P + 1);
    if (ns > 0) split_rows_kernel<<<(unsigned)ceil_div(ns, 256), 256, 0, stream>>>(rowptr, col, n_rows, n_cols, P, S);
    return hipGetLastError();
}

size_t spmm_ws_bytes(int32_t n_rows, int64_t nnz, int32_t n_cols) {
    // header, the row list, then the blocked mode's buffers when the full
    // product would be blocked (a slice of it never needs more ranges)
    size_t blocked = 0;
    for (const int32_t d : {16, 32, kBlockW})  // the three blocked layouts' range counts
        blocked = std::max(blocked, blocked_bytes(n_rows, column_blocks(n_rows, nnz, n_cols, d)));
    return sizeof(SpmmWs) + list_bytes(n_rows) + blocked;
}

int32_t spmm_slice_width(int32_t n_rows, int64_t nnz, int64_t n_src, int32_t d) {
    // Feature-slice width (floats) of one pass. Slices of 16/32/64/128 use
    // 4/8/16/32 lanes per gathered entry; 256 (512 for d > 256) is one pass.
    // Features up to 128 wide take the narrowest layout that holds them in one
    // pass (several entries per load instruction instead of idle lanes).
    // Gathers are limited by the rate of L2-miss requests, so several narrower
    // passes pay off when the slice of the referenced B rows comes close to L2
    // size and rows are long enough to amortise the extra passes over
    // rowptr/col/val; only for widths of whole 128-byte lines (d % 32 == 0),
    // since a slice that straddles lines doubles the requests.
    if (const char *env = getenv("RSC_SPMM_SLICE")) {
        const int v = atoi(env);
        if (v == 16 || v == 32 || v == 64 || v == 128) return v;
        if (v == 256 || v == 512) return d > 256 ? 512 : 256;
    }
    const int32_t fit = d <= 16 ? 16 : d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : d <= 256 ? 256 : 512;
    if (d <= 32 || d % 32 != 0 || n_rows <= 0 || nnz < 128LL * n_rows) return fit;
    const double mib = 1024.0 * 1024.0;
    const double ws32 = (double)n_src * 32 * 4 / mib, ws64 = 2 * ws32;
    if (ws32 > 64.0) return fit;
    if (ws64 <= 30.0 && ws32 > 8.0) return std::min(64, fit);
    return 32;
}

bool spmm_use_order(int32_t n_rows, int64_t nnz) { return use_order(n_rows, nnz); }

bool spmm_hint_taken(int64_t n_src, int32_t d, int32_t slice) {
    return use_hint() && (double)n_src * std::min(d, slice) * sizeof(float) > kHintBytes;
}

hipError_t spmm_rows_prepare(int32_t n_rows, int64_t nnz_bound, const int32_t *rowptr, void *ws,
                             hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    SpmmWs *h = static_cast<SpmmWs *>(ws);
    int32_t *list = reinterpret_cast<int32_t *>(h + 1);
    const int64_t lbound = long_rows_bound(n_rows, nnz_bound);
    const unsigned cgrid = (unsigned)ceil_div(n_rows, kCollectThreads * kCollectPerThread);
    if (use_order(n_rows, nnz_bound)) {
        zero_header_kernel<<<1, 128, 0, stream>>>(h);
        class_hist_kernel<<<cgrid, kCollectThreads, 0, stream>>>(rowptr, n_rows, h);
        class_scan_kernel<<<1, 64, 0, stream>>>(h);
        class_scatter_kernel<<<cgrid, kCollectThreads, 0, stream>>>(rowptr, n_rows, h, list);
    } else if (lbound > 0) {
        zero_count_kernel<<<1, 1, 0, stream>>>(&h->long_count);
        collect_long_rows_kernel<<<cgrid, kCollectThreads, 0, stream>>>(rowptr, n_rows, &h->long_count, list);
    }
    return hipGetLastError();
}

size_t spmm_core_ws_bytes(int32_t n_rows) { return sizeof(SpmmWs) + list_bytes(n_rows); }

size_t spmm_blocked_fits(int32_t n_rows, int32_t P) {
    return sizeof(SpmmWs) + list_bytes(n_rows) + blocked_bytes(n_rows, P);
}

const int32_t *spmm_long_count_of(const void *ws) { return &static_cast<const SpmmWs *>(ws)->long_count; }

// Whether a product without a plan lists its long rows first (two launches,
// about 10 us) or leaves it to the first blocks to look for them.
// Looking costs a block a round trip, listing the launches (us, looked for /
// listed: 262,144 rows, mean 3, d = 23 84 / 89, mean 27, d = 256 1,058 / 1,055;
// 500,000 rows, mean 10, d = 64 196 / 200; 1,000,000 rows, mean 10, d = 256
// 1,726 / 1,696; 2,000,000 rows, mean 10, d = 256 3,940 / 3,876): level from
// about 500,000 rows on, and under 2 % apart but for short rows below that.
bool spmm_lists_long_rows(int32_t n_rows) { return n_rows >= kListedRows; }

hipError_t spmm_launch(int32_t n_rows, int32_t n_cols, int64_t nnz_bound, const int32_t *rowptr,
                       const int32_t *col, const float *val, const float *B, int32_t d, int64_t ldb, float *Y,
                       int64_t ldy, void *ws, size_t ws_bytes, hipStream_t stream, int64_t nnz_hint,
                       int64_t n_src_hint, bool hint_cols, const SpmmPrepared *prep, bool *listed_anew,
                       hipEvent_t stop) {
    if (listed_anew) *listed_anew = false;
    if (n_rows == 0) return hipSuccess;
    SpmmWs *h = static_cast<SpmmWs *>(ws);
    int32_t *list = reinterpret_cast<int32_t *>(h + 1);  // long-row list, or the whole processing order
    // The blocked mode is chosen from the expected entries and referenced B
    // rows (the same for the exact product and a full-budget slice of it);
    // it runs only when the workspace holds its buffers.
    const int32_t P = column_blocks(n_rows, nnz_hint, n_src_hint, d);
    const size_t head = sizeof(SpmmWs) + list_bytes(n_rows);
    if (P > 1 && head + blocked_bytes(n_rows, P) <= ws_bytes) {
        char *p = static_cast<char *>(ws) + head;
        float *part = reinterpret_cast<float *>(p + align_up(sizeof(int32_t) * (size_t)n_rows * (P + 1), 256));
        const int32_t nv = P * n_rows;  // virtual rows, block-major
        // split bounds: a plan's, prepared once, or this call's
        const bool pre = prep && prep->ready && prep->P == P && prep->split;
        const int32_t *S = pre ? prep->split : reinterpret_cast<const int32_t *>(p);
        if (!pre) {
            const hipError_t e = spmm_split_launch(n_rows, n_cols, rowptr, col, P, reinterpret_cast<int32_t *>(p),
                                                   stream);
            if (e != hipSuccess) return e;
        }
        // Long pieces (a piece of a row longer than kLongRow) are taken by
        // the block that holds them, so that they read the same range of B as
        // their neighbours (from a list, ahead of all ranges: 232,965 nodes,
        // 490 per row, d = 256: 8.75 ms against 7.53).
        const int32_t coop = long_rows_bound(n_rows, nnz_bound) > 0 && !(pre && prep->long_rows == 0) ? 1 : 0;
        const unsigned vgrid = (unsigned)ceil_div(nv, kSpmmWaves);
        // partial rows are W floats apart (the workspace holds kBlockW)
        const int32_t W = blocked_width(d);
        for (int32_t f0 = 0; f0 < d; f0 += W) {
            const int32_t dl = std::min<int32_t>(d - f0, W);
            const uint32_t bb = buffer_bytes(n_cols, ldb, dl);
#define RSC_SPMM_BLOCKED_LAUNCH_B(LPE_, BUF_, COOP_)                                                   \
    spmm_kernel<LPE_, 1, false, false, BUF_, COOP_, kSpmmWaves><<<vgrid, kSpmmWaves * 64, 0, stream>>>(\
        S, n_rows, col, val, B + f0, ldb, bb, part, W, nv, dl, 0, nullptr, 0, nullptr)
#define RSC_SPMM_BLOCKED_LAUNCH(LPE_)                        \
    do {                                                     \
        if (bb != 0 && coop)                                 \
            RSC_SPMM_BLOCKED_LAUNCH_B(LPE_, true, true);     \
        else if (bb != 0)                                    \
            RSC_SPMM_BLOCKED_LAUNCH_B(LPE_, true, false);    \
        else                                                 \
            RSC_SPMM_BLOCKED_LAUNCH_B(LPE_, false, true);    \
    } while (0)
            if (W == 16)
                RSC_SPMM_BLOCKED_LAUNCH(4);
            else if (W == 32)
                RSC_SPMM_BLOCKED_LAUNCH(8);
            else
                RSC_SPMM_BLOCKED_LAUNCH(16);
#undef RSC_SPMM_BLOCKED_LAUNCH_B
#undef RSC_SPMM_BLOCKED_LAUNCH
            const int64_t nc = (int64_t)n_rows * ((dl + 3) / 4);
            launch(combine_blocks_kernel, (unsigned)ceil_div(nc, 256), 256, stream, f0 + W >= d ? stop : nullptr,
                   (const float *)part, (int64_t)W, n_rows, P, dl, Y + f0, ldy);
        }
        return hipGetLastError();
    }
    const bool ordered = use_order(n_rows, nnz_bound);
    // a plan's row list (long rows, or the whole order) prepared once sits in
    // this workspace already; else it is built here, except over few rows
    const bool pre = prep && prep->ready && prep->P == 1 && prep->ordered == ordered;
    int32_t n_long = 0;  // blocks that take the long rows
    const int32_t *rows = nullptr;  // their list (or the order); NULL: they look for them
    if (ordered || (long_rows_bound(n_rows, nnz_bound) > 0 && !(pre && prep->long_rows == 0))) {
        const bool listed = ordered || (pre ? prep->list : spmm_lists_long_rows(n_rows));
        if (listed && !pre) {
            if (listed_anew) *listed_anew = true;
            const hipError_t e = spmm_rows_prepare(n_rows, nnz_bound, rowptr, ws, stream);
            if (e != hipSuccess) return e;
        }
        if (listed) rows = list;
        const int64_t bound = long_rows_bound(n_rows, nnz_bound);
        if (!listed)  // at least a thread for each row
            n_long = (int32_t)std::min<int64_t>(std::max(bound, ceil_div(n_rows, kSpmmWaves * kWave)),
                                                kSpmmLongBlocksMax);
        else if (pre && prep->long_rows >= 0)
            n_long = std::min(prep->long_rows, kSpmmLongBlocksMax);
        else
            n_long = (int32_t)std::min<int64_t>(bound, kSpmmLongBlocks);
    }
    const int32_t slice = spmm_slice_width(n_rows, nnz_hint, n_src_hint, d);
    // the hint pays off only when the gathered rows far outgrow the on-chip
    // caches (MALL included); below that, bypassing them loses reuse
    const bool hint = hint_cols && spmm_hint_taken(n_src_hint, d, slice);
    const bool wide_blocks = n_rows >= kWideBlockRows && nnz_hint >= (int64_t)kWideBlockMean * n_rows;
    for (int32_t f0 = 0; f0 < d;) {
        const int32_t dl = std::min<int32_t>(d - f0, slice);
        const uint32_t bb = buffer_bytes(n_cols, ldb, dl);
#define RSC_SPMM_LAUNCH_H(LPE_, NV_, H_, BUF_, W_)                                                       \
    launch(spmm_kernel<LPE_, NV_, true, H_, BUF_, false, W_>,                                            \
           (unsigned)(long_parts(LPE_, NV_, W_) * n_long + ceil_div(n_rows, W_)), W_ * 64, stream,       \
           f0 + dl >= d ? stop : nullptr, rowptr, (int64_t)1, col, val, B + f0, ldb, bb, Y + f0, ldy, n_rows, dl, \
           long_parts(LPE_, NV_, W_) * n_long, rows, (int32_t)(ordered ? 1 : 0), (const int32_t *)&h->long_count)
#define RSC_SPMM_LAUNCH_SLICED(LPE_)                                \
    do {                                                            \
        if (hint)                                                   \
            RSC_SPMM_LAUNCH_H(LPE_, 1, true, false, kSpmmWaves);    \
        else if (bb != 0)                                           \
            RSC_SPMM_LAUNCH_H(LPE_, 1, false, true, kSpmmWaves);    \
        else                                                        \
            RSC_SPMM_LAUNCH_H(LPE_, 1, false, false, kSpmmWaves);   \
    } while (0)
#define RSC_SPMM_LAUNCH_ROW(H_)                                     \
    do {                                                            \
        if (dl > 4 * kWave)                                         \
            RSC_SPMM_LAUNCH_H(64, 2, H_, false, kSpmmWaves);        \
        else if (wide_blocks)                                       \
            RSC_SPMM_LAUNCH_H(64, 1, H_, false, 8);                 \
        else if (!H_ && bb != 0)                                    \
            RSC_SPMM_LAUNCH_H(64, 1, false, true, kSpmmWaves);      \
        else                                                        \
            RSC_SPMM_LAUNCH_H(64, 1, H_, false, kSpmmWaves);        \
    } while (0)
        switch (slice) {
            case 16: RSC_SPMM_LAUNCH_SLICED(4); break;
            case 32: RSC_SPMM_LAUNCH_SLICED(8); break;
            case 64: RSC_SPMM_LAUNCH_SLICED(16); break;
            case 128: RSC_SPMM_LAUNCH_SLICED(32); break;
            default:
                if (hint) RSC_SPMM_LAUNCH_ROW(true); else RSC_SPMM_LAUNCH_ROW(false);
        }
#undef RSC_SPMM_LAUNCH_ROW
#undef RSC_SPMM_LAUNCH_SLICED
#undef RSC_SPMM_LAUNCH_H
        f0 += dl;
    }
    return hipGetLastError();
}

}  // namespace rsc
