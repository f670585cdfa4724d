// Internal declarations shared by the host side and the device kernels of
// libsline.  Not installed; the public interface is include/sline.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sl {

constexpr int kWave = 64;
constexpr int32_t kEmpty = -1;

// Error bits accumulated on the device while checking the input CSR.
enum : int32_t {
    kErrRowPtr0 = 1,      // row_ptr[0] != 0
    kErrRowPtrOrder = 2,  // row_ptr decreases
    kErrColRange = 4,     // a member outside [0, n_vertices)
    kErrColOrder = 8,     // a row that is not strictly increasing
    kErrInternal = 16,    // a table probe that found no room (never expected)
    // a replayed batch plan (fixed buffers): the input or the work outgrew it
    kErrPlanShape = 32,   // a graph's row_ptr[0] or row_ptr[m] differs from the plan's
    kErrPlanTasks = 64,   // more counting tasks than the plan's task arrays hold
    kErrPlanPairs = 128,  // more pairs than the plan's result arrays hold
};

// Tunable launch parameters of the counting kernels (the autotuner sets them).
struct Tuning {
    int32_t small_max_wedges = 512;  // items with W_a up to this go to the one-wave kernel
    int32_t task_wedges = 5000;      // wedges per workgroup task (j sub-range of an item)
    int32_t group_parts = 8;         // consecutive tasks of one item run by one workgroup
    int32_t light_len = 12;          // member runs up to this are walked by one lane
    int32_t small_grid_per_cu = 16;  // one-wave workgroups per CU for the small kernel
    int32_t task_grid_per_cu = 4;    // resident workgroups per CU for the task kernel
    int64_t stage_max_bytes = 96ll << 30;  // cap of the staging pool (one counting pass)
    int32_t dense_min_wedges = 4096;  // cut items into dense sub-ranges when each gets this many wedges
    int32_t small_slots = 1024;  // LDS table of the one-wave kernel: 512, 1024 or 2048 home slots
    int32_t task_slots = 8960;   // LDS table of the task kernel: 4480, 8960, 13440 or 17920 home slots
    int32_t tiny_max_wedges = 10;  // items of up to this many wedges go one per lane (0: off)
};

// Rows that each wave takes of n, where it looks at a row per lane and walks some of
// them one after the other: 64, or as few as keep kRowWaves waves at work.
constexpr int64_t kRowWaves = 8192;
inline int32_t lanes_per_wave(int64_t n) {
    int32_t per = kWave;
    while (per > 1 && n < per * kRowWaves) per /= 2;
    return per;
}

// Scan tile: 256 threads x 8 items.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// Table sizes (home slots) of the counting kernels are tuning values
// (Tuning::small_slots, Tuning::task_slots), each kernel built for the sizes
// listed there: 8960 home slots + 64 pad = 9024 packed 4-byte slots lets four
// 256-thread task workgroups share a CU, 13440 two; 17920 runs with 512
// threads, two workgroups per CU.
constexpr int kTaskThreads = 256;
// Tiny items (one lane each): at most kTinyCap members and kTinyCap wedges.
// With s > 2 few wedges make a pair, and up to three times tiny_max_wedges of them
// are taken, so tiny_max_wedges <= kTinyMaxCost keeps them within kTinyCap (by the
// exact W_a: a planning cost is not lowered to that many, see k_mark_lookup).
constexpr int kTinyCap = 32;
constexpr int kTinyMaxCost = 10;
constexpr int kTinyThreads = 256;

// Candidate numbers.  A build that filters by s may number its kept items 0, 1,
// ... in id order and let the member lists hold those ranks: the candidates
// of an item then lie in a range with no items that cannot be in a pair, so
// the range is cut into fewer tables.  The price is a look-up per pair to
// turn ranks back into items.  Build time without and with ranks: 10^6-item power
// law, s = 2 (99.98 % kept) 34.4 and 37.9 ms, s = 3 23.3 and 20.3, s = 8 (15 % kept)
// 11.0 and 6.0, its dual at s = 8 9.1 and 3.1; 10^6 items of even sizes, 95 %, 74 % and
// 47 % kept, 14.4 and 14.2, 11.5 and 11.1, 6.45 and 6.57.  Ranks are used when at
// most three in four items are kept (crank[N] counts them; every kernel derives the
// same answer from it): what more would bring rests on how sizes and wedges go
// together, and the line is on the safe side of it.  And in builds of one graph with
// kRankMinItems items or more, as a smaller one fits a few ranges anyhow (even
// sizes, 63 % kept: 131,072 items 1.30 and 1.23 ms, 100,000 items 0.968 and
// 0.972, 50,000 items 0.63 and 0.65), and so does each graph of a batch.
constexpr int64_t kRankMinItems = 1 << 17;
__host__ __device__ inline bool ranks_pay(int64_t kept, int64_t N) { return kept * 4 <= N * 3; }

// A kernel drops crank (and orig) at its start when the build does not use ranks;
// a candidate's number is then its item's id.
__device__ __forceinline__ const int32_t *ranks_or_null(const int32_t *crank, int32_t N) {
    return crank && ranks_pay(crank[N], N) ? crank : nullptr;
}

__device__ __forceinline__ int32_t cand_of(const int32_t *crank, int32_t item) {
    return crank ? crank[item] : item;
}

// First candidate of item a: the one after a (product mode: 0).
__device__ __forceinline__ int32_t cand_first(const int32_t *crank, int32_t full, int32_t a) {
    return full ? 0 : cand_of(crank, a) + 1;
}

// One past the last candidate of item a: the end of its graph (batches) or of
// all items.
__device__ __forceinline__ int32_t cand_end(const int32_t *crank, const int32_t *item_end,
                                            int32_t N, int32_t a) {
    return cand_of(crank, item_end ? item_end[a] : N);
}

// Direct counting (sline_flat.hip): an item's candidate range is cut into
// ranges of kFlatBlock << k candidates that fit kFlatWords words of counters
// wide enough for the item's size: 4 bits (k = 2), 8 (k = 1) or 16 (k = 0).
constexpr int32_t kFlatWords = 15360;
constexpr int32_t kFlatBlock = kFlatWords * 2;
constexpr int32_t kFlatMaxSize = 65535;      // members of an item at most
constexpr int32_t kFlatTaskWedges = 1 << 16; // a task's share of a heavy item
// With s = 1, items of at most kFlatKeep wedges and kFlatThreads members keep
// their wedges in registers and take one bit per candidate, in ranges of
// kKeepWidth.
constexpr int32_t kFlatThreads = 512;
constexpr int32_t kFlatKeep = 32 * kFlatThreads;
constexpr int32_t kKeepWidth = kFlatWords / 2 * 32;
constexpr int32_t kKeepRanks = kFlatWords / 4;  // pairs of a range counted at a time

// Flat-table counting by one workgroup per item (k_count_item): up to kMiniWedges
// wedges in one step of a wave; sieved, with s > 1, up to kSieveWedges * threads
// (kSieveSmall or kSieveLarge threads); with s = 1, where nothing can be
// sieved out, up to kOnesWedges.  A member per thread, in a wave per lane.
// Where the lines lie: a step of a wave is four chunks of 64; a sieve's two bit
// maps of 16 bits per wedge and its table fill a quarter of a CU's LDS at 8,192
// wedges, and a larger one would leave too few waves.  10^6 hyperedges, s = 2: 47.8 ms
// with the sieves, 55.5 with direct counters or hashed tasks for all items above 512
// wedges (the kernels as they were when the sieves came in).
constexpr int32_t kMiniWedges = 256;
constexpr int32_t kSieveSmall = 64, kSieveLarge = 256;
constexpr int32_t kSieveWedges = 32;
constexpr int32_t kOnesWedges = 480;
// An item whose candidates fit kSieveRanges ranges of direct counters is not sieved by
// four waves: a sieve's hash table holds its candidates in their order, and where
// they crowd in a part of the range, as with ids in the order of the sizes, it
// overflows and the range is split again and again.  Build time with every
// such item sieved, and with those of one, two and four ranges counted directly:
// 200,000 hyperedges by ascending size, s = 2: 14.9, 7.4, 5.3, 5.3 ms, s = 4: 9.4,
// 2.8, 2.7, 2.8; 10^6 in random order, s = 2: 34.3, 34.3, 34.0, 35.2, s = 8: 6.3,
// 5.9, 5.9, 5.9.
constexpr int32_t kSieveRanges = 2;

// The list positions of all these kernels fit a 32-bit byte offset: builds with
// this many incidences or more use the hashed kernels alone.
constexpr int64_t kDirectMaxNnz = (int64_t)1 << 30;

// Blocks that hold `cands` candidates.
__device__ __forceinline__ int32_t flat_blocks(int32_t cands) {
    return (int32_t)(((int64_t)cands + kFlatBlock - 1) / kFlatBlock);
}

struct FlatShape {
    int32_t base;    // first candidate of the first range
    int32_t width;   // candidates per range
    int32_t ranges;
    uint32_t lbits;  // 1 << lbits bits per counter
};

// Ranges of an item with candidates [first, nend) and `size` members: one
// that starts at its first candidate, or several that start at a block.
__device__ __forceinline__ FlatShape flat_shape(int32_t first, int32_t nend, int32_t size) {
    FlatShape f;
    f.lbits = size < 16 ? 2u : size < 256 ? 3u : 4u;
    f.width = kFlatBlock << (4u - f.lbits);
    f.base = first;
    f.ranges = 1;
    if ((int64_t)nend - first > f.width) {
        f.base = first / kFlatBlock * kFlatBlock;
        f.ranges = (int32_t)(((int64_t)nend - f.base + f.width - 1) / f.width);
    }
    return f;
}

// Whether an item keeps its wedges in registers, and its ranges then.
__device__ __forceinline__ bool flat_keeps(int32_t s, int64_t cost, int32_t size) {
    return s == 1 && cost <= kFlatKeep && size <= kFlatThreads;
}

__device__ __forceinline__ int32_t keep_ranges(int32_t first, int32_t nend) {
    return (int32_t)(((int64_t)nend - first + kKeepWidth - 1) / kKeepWidth);
}

// Ranges of a task of an item with `cost` wedges.
__device__ __forceinline__ int32_t flat_ranges_per_task(const FlatShape &f, int64_t cost) {
    const int64_t parts = (cost + kFlatTaskWedges - 1) / kFlatTaskWedges;
    return parts >= f.ranges ? 1 : (int32_t)((f.ranges + parts - 1) / parts);
}

// What the task planner needs to know about the items besides their cost.
struct PlanItems {
    const int32_t *ptrI;      // item lists (sizes)
    const int32_t *crank;     // candidate numbers of the items, or null: their ids
    const int32_t *item_end;  // per item: end of its graph's items (batches), or null
    const int32_t *s_item;    // per-item s (batches), or null: s
    int32_t N, s;
    int32_t full;             // product mode
    int32_t small_max;        // Tuning::small_max_wedges
    int32_t target;           // Tuning::task_wedges
    int32_t dense_min;        // Tuning::dense_min_wedges
    int32_t slots;            // Tuning::task_slots
};

// How an item is counted.  The lists of its tasks are counts[kind] long.
enum : int32_t {
    kKindSmall = 0,   // one wave, hash table
    kKindGroups = 1,  // workgroup task groups, hash table
    kKindTiny = 2,    // one lane
    kKindFlat = 3,    // direct counters
    kKindSieve1 = 4,  // sieved, kSieveSmall threads
    kKindSieve4 = 5,  // sieved, kSieveLarge threads
    kKindMini = 6,    // one wave, every wedge at once
    kKinds = 7,
};

// Tasks of item a when every wedge of it is counted by one of the kernels
// without hashed wedge lists (kind: which; ranges: those that stage their pairs
// by themselves), 0 when it is not.  Direct counters take an item with at
// least dense_min / 8 wedges per range (512; a sixteenth where it keeps its
// wedges, s = 1).  Fewer change little, as a range's fixed work is then about what
// hashing costs; with more, hashing is slower.  Build time with at least 64, 512,
// 2048 and 8192 wedges a range: 10^6 hyperedges, s = 2: 34.6, 34.6, 36.2, 52.9 ms;
// s = 8: 6.0, 6.0, 6.1, 7.1; 200,000, s = 1 (half as many): 5.5, 5.5, 5.8, 7.6.
// `cost` is W_a, or the lowered planning
// cost of an item that was not to be counted so by its W_a (and is not by less).
__device__ __forceinline__ int32_t direct_tasks(const PlanItems &I, int32_t a, int64_t cost,
                                                int32_t &kind, int32_t &ranges) {
    ranges = 0;
    if (cost <= 0 || I.dense_min <= 0 || I.full) return 0;
    const int32_t size = I.ptrI[a + 1] - I.ptrI[a];
    const int32_t s = I.s_item ? I.s_item[a] : I.s;
    if (size <= kSieveSmall) {
        kind = kKindMini;
        if (cost <= kMiniWedges) return 1;
        kind = kKindSieve1;
        if (cost <= (s > 1 ? kSieveWedges * kSieveSmall : kOnesWedges)) return 1;
    }
    kind = kKindSieve4;
    if (cost <= I.small_max) return 0;
    const int32_t first = cand_first(I.crank, 0, a), nend = cand_end(I.crank, I.item_end, I.N, a);
    if (s > 1 && cost <= kSieveWedges * kSieveLarge && size <= kSieveLarge) {
        const int32_t ranges = flat_shape(first, nend, size).ranges;
        if (ranges > kSieveRanges || cost * 8 < (int64_t)I.dense_min * ranges) return 1;
    }
    kind = kKindFlat;
    if (size > kFlatMaxSize) return 0;
    if (flat_keeps(s, cost, size)) {
        const int32_t n = keep_ranges(first, nend);
        if (cost * 16 < (int64_t)I.dense_min * n) return 0;
        ranges = n + (int32_t)(cost / kKeepRanks);
        return 1;
    }
    const FlatShape f = flat_shape(first, nend, size);
    if (cost * 8 < (int64_t)I.dense_min * f.ranges) return 0;
    const int32_t per = flat_ranges_per_task(f, cost);
    ranges = f.ranges;
    return (f.ranges + per - 1) / per;
}

// ------------------------------------------------------------ launchers
// Every launcher enqueues on `st` and returns the launch status.

// seen (host memory the device can write, seen[1] zeroed by the caller): [0]
// receives row_ptr[m], [1] becomes 1 if row_ptr[0] != 0 or row_ptr decreases.
hipError_t launch_check_rowptr(hipStream_t st, const int32_t *rp, int32_t m, int32_t *seen);

// Counters that every workgroup adds to are kept in kSumRows rows of a cache line
// or more, added up when they are read: atomics on one address take about 10 ns
// each, one after the other (12,000 of them at the end of a kernel: 0.1 ms).
constexpr int kSumRows = 64;
constexpr int kTotalCols = 16;  // cost totals [0..2], the planner's sums [3..]
constexpr int kStatCols = 8;    // table passes, task kernel incidences, wedges, pairs
constexpr int kCountStride = 16;  // words between two kinds' list lengths

// A read-back: up to kMost runs of 32-bit words copied to host memory by one
// launch (a copy per run would cost a launch each).
struct Report {
    static constexpr int kMost = 6;
    int32_t n = 0;
    const int32_t *src[kMost];
    int32_t *dst[kMost];
    int32_t words[kMost];
    // sums over kSumRows rows of int64: `vals` columns of rows of `cols`
    int n_sums = 0;
    const int64_t *rows[2];
    int64_t *sums[2];
    int32_t cols[2], vals[2];
    void add_rows(int64_t *to, const int64_t *from, int32_t row_cols, int32_t n_vals) {
        rows[n_sums] = from;
        sums[n_sums] = to;
        cols[n_sums] = row_cols;
        vals[n_sums++] = n_vals;
    }
    void add(void *to, const void *from, int32_t bytes) {
        src[n] = static_cast<const int32_t *>(from);
        dst[n] = static_cast<int32_t *>(to);
        words[n++] = bytes / 4;
    }
};
hipError_t launch_report(hipStream_t st, const Report &R);
// Checks of the rows, and the row of every incidence: rowid[k] = i, or -1 in rows
// of fewer than s entries (s_item[i] when given); with crank, the row's rank
// instead of i, where ranks pay.
hipError_t launch_rows(hipStream_t st, const int32_t *rp, const int32_t *col, int32_t m,
                       int32_t n, int64_t nnz, int check_order, int32_t *rowid, int32_t *err,
                       int32_t s = 0, const int32_t *s_item = nullptr,
                       const int32_t *crank = nullptr);
// crank[it] (N + 1 entries) = items of at least s members before it; kept: N
// entries of scratch, part32 the scan's partials.
hipError_t launch_ranks(hipStream_t st, const int32_t *ptrI, int32_t N, int32_t s, int32_t *kept,
                        int32_t *crank, int32_t *part32);
// orig[rank] = item, where ranks pay
hipError_t launch_rank_items(hipStream_t st, const int32_t *crank, int32_t N, int32_t *orig);

hipError_t launch_fill_i32(hipStream_t st, int32_t *p, int64_t n, int32_t v);
hipError_t launch_fill_i64(hipStream_t st, int64_t *p, int64_t n, int64_t v);
hipError_t launch_copy_i32(hipStream_t st, int32_t *dst, const int32_t *src, int64_t n);

// Exclusive scan: out[0..n] with out[n] = total.  `partial` needs
// scan_partials(n) entries of the accumulator type.
int64_t scan_partials(int64_t n);
hipError_t launch_scan_i32(hipStream_t st, const int32_t *in, int64_t n, int32_t *out,
                           int32_t *partial);
hipError_t launch_scan_i32_to_i64(hipStream_t st, const int32_t *in, int64_t n, int64_t *out,
                                  int64_t *partial);

// start[k] = map[k] + 1 (unfiltered member lists)
hipError_t launch_start_from_map(hipStream_t st, int64_t nnz, const int32_t *map, int32_t *start);

// Transpose of an nnz-entry CSR with members in [0, n): ptrT (n + 1), colT
// (the item rowid[k] of each incidence, grouped by member, items ascending),
// kT[q] = the incidence at transposed slot q and posT[k] = its slot (kT,
// posT may be null).  A stable least-significant-digit radix sort of the
// (member, incidence) pairs; rsK / rsV are two pairs of nnz-entry buffers,
// hist holds transpose_hist(nnz) counts and part32 the partials of their
// scan.
int64_t transpose_hist(int64_t nnz);
// Radix passes of a transpose over members in [0, n); its sorted members end
// in rsK[(passes - 1) & 1].
int transpose_passes(int32_t n);
hipError_t launch_transpose(hipStream_t st, const int32_t *col, int64_t nnz, int32_t n,
                            const int32_t *rowid, int32_t *const rsK[2], int32_t *const rsV[2],
                            int32_t *hist, int32_t *part32, int32_t *ptrT, int32_t *colT,
                            int32_t *kT, int32_t *posT);

// The filtered member lists of a primal build in one sort: of the nnz
// incidences (col[k], item[k]) those with item[k] >= 0, by member, items ascending:
// itm (their items), ptr (n + 1 list pointers) and start[k] = the position after
// k's own entry (the back-pointer of kept incidence k; start may be null).  item
// is used up; rsW: one more nnz-entry buffer; *n_dev receives their number.
hipError_t launch_member_lists(hipStream_t st, const int32_t *col, int32_t *item, int64_t nnz,
                               int32_t n, int32_t *const rsK[2], int32_t *const rsV[2],
                               int32_t *rsW, int32_t *hist, int32_t *part32, int32_t *n_dev,
                               int32_t *ptr, int32_t *itm, int32_t *start);

// The same sort of keys that carry a value v, and w if not null: with p =
// transpose_passes(n) - 1, the sorted values end in rsV[p & 1] and rsW[p & 1], and
// ptr[x] (n + 1 entries) is the first key >= x.
hipError_t launch_sort_values(hipStream_t st, const int32_t *key, const int32_t *v,
                              const int32_t *w, int64_t nnz, int32_t n, int32_t *const rsK[2],
                              int32_t *const rsV[2], int32_t *const rsW[2], int32_t *hist,
                              int32_t *part32, int32_t *ptr);

// s filter of a dual build: N_s(v) = the items of N(v) with |S| >= s, every list
// in its order, written to itmS with list pointers ptrS (M + 1 entries).  pos
// (nnz + 1 entries) receives the kept entries before each member-list entry;
// part32 holds the scan's partials.  The back-pointer of every kept entry is
// written as well: start[inv[p]] = (its position in itmS) + 1, inv mapping
// member-list positions to item incidences.
// Nothing is read while kErrColRange is set in *err.
// kept (N entries, scratch) receives each item's keep flag first.  With crank
// given (N + 1 entries), crank[it] = kept items before it, and where ranks pay
// (ranks_pay), itmS holds ranks and orig[rank] (up to N entries) their items.
hipError_t launch_filter(hipStream_t st, const int32_t *ptrM, const int32_t *itmM, int32_t M,
                         int64_t nnz, const int32_t *ptrI, int32_t N, int32_t s,
                         int32_t *kept, int32_t *pos, int32_t *part32, int32_t *ptrS,
                         int32_t *itmS, const int32_t *inv, int32_t *start, int32_t *crank,
                         int32_t *orig, const int32_t *err);

// Per-item exact wedge count W_a, the back-pointer start[k] (first item > a
// in N_s(v) for member incidence k of a kept item a) and the run totals:
// totals[0] = kept items, [1] = kept incidences, [2] = wedges.
// full != 0 (product mode): start[k] = the first entry of N_s(v) and W_a counts
// every b in the lists, a itself included.
// Nothing is read while *err (if given) is not 0.
hipError_t launch_cost(hipStream_t st, const int32_t *ptrI, const int32_t *memI, int32_t N,
                       int32_t s, const int32_t *s_item, const int32_t *ptrS, const int32_t *itmS,
                       int64_t *cost, int32_t *start, int64_t *totals, int32_t full = 0,
                       int32_t have_start = 0, const int32_t *err = nullptr);

// Keep the entries (a, b, w) with b > a and w >= s of a row-sorted product,
// in order: pass 1 (out_a == nullptr) counts per block into cnt, pass 2 writes
// at the exclusive scan off of those counts.  kFilterTile entries per block.
constexpr int kFilterTile = 4096;
hipError_t launch_product_filter(hipStream_t st, const int32_t *a, const int32_t *b, const int32_t *w,
                                 int64_t n, int32_t s, int32_t *cnt, const int64_t *off,
                                 int32_t *out_a, int32_t *out_b, int32_t *out_w);

// Lookup-only members (insertion cutoff, s > 1): a candidate b with
// |S_a & S_b| >= s lies in at least s of the lists N_s(v), v in S_a, so if up
// to s - 1 members of a only count candidates that the other members inserted
// before them, every such b is still counted exactly; the others stay below s
// and are dropped.  The longest lists (most wedges) are chosen; the choice is
// flagged in the sign bit of start[k], and cost[a] is lowered to the planning
// cost max(W_a - flagged wedges, W_a / 3), but not so far that a kernel would be
// given the item that has no room for W_a wedges.
constexpr int32_t kStartMask = 0x7fffffff;
constexpr int32_t kMaxLookup = 15;  // lookup-only members per item at most
// Only items that k_count_tasks counts are marked: every other kernel counts all
// wedges, and would gain nothing.  Nothing is done while *err (if given) is not 0.
hipError_t launch_mark_lookup(hipStream_t st, const PlanItems &I, const int32_t *memI,
                              const int32_t *ptrS, int32_t *start, int64_t *cost,
                              const int32_t *err = nullptr);

// Tasks: item a with W_a wedges becomes P_a tasks (sub-ranges of its
// candidate range); ntask[a] = P_a.  Task t of item a (t = tbase[a] + p) is
// listed in small_tasks, with its item in small_items (W_a <= small_max), or
// in big_tasks; counts[0] / [1]
// receive the list lengths.
// sums (kSumRows rows of kTotalCols, zeroed by the caller): [0] receives the ranges
// of the items counted directly, each of which stages its pairs by itself, [1 + kind] the items of
// each kind.
// bound != 0: instead of P_a, no fewer tasks than the item can come to have in a
// replay of the same lists at any larger s.
hipError_t launch_task_count(hipStream_t st, const int64_t *cost, const PlanItems &I,
                             int32_t tiny_max, int32_t *ntask, int64_t *sums,
                             int32_t bound = 0);
// big_tasks receives, per group of up to group_parts consecutive tasks of an
// item, the index of the group's first task; counts[1] = number of groups.
// With `abort` given, the kernel does nothing while *abort != 0.
// Tiny one-task items (Tuning::tiny_max_wedges) go to tiny_tasks /
// tiny_items instead of the small lists; counts[2] receives their number.
// Items of the other kinds go to the ends of the lists, each with `cap` entries,
// room for every task: big_tasks[cap - 1 - i] holds task i < counts[kKindFlat];
// small_tasks (kKindSieve1), tiny_tasks (kKindSieve4) and small_items
// (kKindMini) hold items in the same way.
hipError_t launch_task_fill(hipStream_t st, const int64_t *cost, const PlanItems &I,
                            int32_t tiny_max, int32_t group, const int64_t *tbase,
                            int32_t *task_item, int32_t *task_part, int32_t *small_tasks,
                            int32_t *small_items, int32_t *tiny_tasks, int32_t *tiny_items,
                            int32_t *big_tasks, int32_t cap, int32_t *counts,
                            const int32_t *abort = nullptr);

// Positions of the multiples of kFlatBlock candidates in the long lists (bnd:
// as many entries as itmS, nnz at most), for the items counted directly.  long_lists:
// scratch of as many; n_long: its length, zeroed by the caller; n_flat: the tasks
// of those items.  Nothing is done without any, or while *err (if given) is not 0.
hipError_t launch_flat_bounds(hipStream_t st, const int32_t *ptrS, const int32_t *itmS, int32_t M,
                              const int32_t *crank, int32_t N, int64_t nnz, int32_t *bnd,
                              int32_t *long_lists, int32_t *n_long, const int32_t *n_flat,
                              const int32_t *err = nullptr);

// Counting-kernel modes.
enum : int32_t {
    kModeCount = 0,  // pairs per task only
    kModeFill = 1,   // write (a, b, w) at task_off (only tasks flagged in `need`, if given)
    kModeStage = 2,  // pairs per task, and each extracted range's (b, w) into the pool
};

// One staged range: `n` pairs of task `t` at pool[off], destined for
// task_off[t] + rel.
struct StageRec {
    int64_t off;
    int32_t t, rel, n, pad;
};

struct CountArgs {
    int32_t mode;
    const int32_t *ptrI, *memI;  // item lists
    const int32_t *ptrS, *itmS;  // filtered membership lists, as candidate numbers
    // Candidate numbers: crank[item] (N + 1 entries) and orig[candidate], used
    // where ranks pay, or both null: a candidate is its item's id.
    // The pool holds candidates; what leaves the counting kernels or the copy
    // holds items.
    const int32_t *crank, *orig;
    int32_t N, s;
    const int32_t *s_item;       // per-item s (batches), or null: s for every item
    const int32_t *item_end;     // per item: one past the last item of its graph (batches), or null: N
    int32_t full;                // product mode: every candidate b (both triangles and b = a)
    const int64_t *cost;         // W_a per item
    const int32_t *start;        // back-pointers per item incidence (see launch_cost)
    const int32_t *task_item, *task_part;
    const int64_t *tbase;        // first task of each item
    int32_t n_tasks;
    const int32_t *small_tasks, *big_tasks;
    const int32_t *small_items;  // item of each small task
    const int32_t *tiny_tasks, *tiny_items;  // tiny tasks (one lane each) and their items
    const int32_t *task_counts;  // list lengths: task_counts[kind * kCountStride]
    int32_t grid[kKinds];        // workgroups per kind (0: no items)
    const int32_t *bnd;          // bounds table of the direct path (launch_flat_bounds)
    int32_t *queue;              // queue heads: task groups, direct tasks (reset by the launcher)
    int32_t *task_cnt;           // count mode: pairs per task
    const int64_t *task_off;     // fill mode: output offset per task (nullptr = count mode)
    int32_t *out_a, *out_b, *out_w;  // out_w null: weights not written (SLINE_NO_WEIGHTS)
    // stage mode: pool of (b, w) pairs and the range log; tasks that found no
    // room are flagged in need[] (need_count counts them) for a fill pass
    int32_t *pool_b, *pool_w;    // pool_w null: weights not staged
    int64_t pool_cap;
    // Pool pairs and log records a workgroup reserves at a time, by kind.  The
    // workgroups' first chunks lie at pool_first / log_first of their kind, one
    // after the other, pool_own pairs and log_own records in all (0: none are
    // set aside).
    int64_t pool_chunk[kKinds], pool_first[kKinds], pool_own;
    int32_t log_chunk[kKinds], log_first[kKinds], log_own;
    unsigned long long *pool_head;
    StageRec *log;
    int32_t log_cap;
    int32_t *log_head;
    int32_t *need;
    int32_t *need_count;
    int64_t *passes;             // kSumRows rows of kStatCols: [0] table passes; task kernel
                                 // work: [1] incidences, [2] wedges, [3] pairs (count and
                                 // stage modes)
    int32_t *err;
    Tuning tune;
    int32_t n_cu;
    // batches written straight to per-graph outputs (n_graphs > 0; fill and
    // stage-copy writes only): graph g owns the combined items
    // [g_ibase[g], g_ibase[g + 1]) and the pairs [g_off[g], g_off[g + 1]); its
    // arrays are g_out[g], g_out[G + g] and g_out[2G + g] (null without
    // weights), and both ids are written less g_ibase[g]
    // With g_out null, every pair goes to out_a/out_b/out_w at its combined
    // position, both ids less its graph's g_ibase (g_off unused).
    int32_t n_graphs;
    const int64_t *g_ibase, *g_off;
    int32_t *const *g_out;
    // Replayed plans: while *abort != 0 the counting and copy kernels do
    // nothing (the plan's bounds were exceeded, or its input is malformed).
    const int32_t *abort;
};
constexpr int64_t kPoolChunkMin = 256;   // pairs a workgroup reserves at least
// Workgroups per kind for `items` items of each; returns their number.  Needs tune
// and n_cu.
int32_t set_grids(CountArgs &a, const int64_t *items);
// Chunks of pool and log for the grids, pool_cap, log_cap and mode.
void set_chunks(CountArgs &a);
// `mid` (may be null) is recorded between the one-wave kernel and the task kernel.
hipError_t launch_count(hipStream_t st, const CountArgs &a, hipEvent_t mid = nullptr);
// The direct counting kernel alone (launch_count calls it).
hipError_t launch_count_flat(hipStream_t st, const CountArgs &a);

// ---------------------------------------------------------------- batches
// One graph of a batch (a device array of these drives the batch kernels).
struct BatchGraph {
    const int32_t *rp, *col;  // the caller's CSR
    int32_t m, n;             // edges, vertices
    int32_t dual, s;
    int64_t nnz;              // row_ptr[m]: every row must lie inside [0, nnz)
    int64_t ibase, mbase;     // first combined item id, first combined member id
    int64_t dbase, dzbase;    // dual graphs: first row and first entry in XD
    int64_t vdbase;           // dual graphs: first row of XD^T (vertex rows)
};

hipError_t launch_batch_nnz(hipStream_t st, const BatchGraph *gr, int32_t G, int64_t *nnz,
                            int32_t *err);
// XD = rows of the GD dual graphs (graph dual_ids[q] has rows [dbase[q], dbase[q+1])).
// ZD: its entries.  long_rows: scratch of ZD entries; n_long: its length, zeroed by
// the caller.
hipError_t launch_batch_concat(hipStream_t st, const BatchGraph *gr, const int32_t *dual_ids,
                               const int64_t *dbase, int32_t GD, int64_t E, int64_t ZD,
                               int32_t *xcol, int32_t *xrow, int32_t *long_rows, int32_t *n_long,
                               int32_t *err);
// Combined items: graph g owns [ibase[g], ibase[g + 1]); ptrT / colT = XD^T.
hipError_t launch_batch_len(hipStream_t st, const BatchGraph *gr, const int64_t *ibase, int32_t G,
                            int64_t NI, const int32_t *ptrT, int32_t *len, int32_t *s_item,
                            int32_t *item_end, int32_t *err);
// Combined member lists: zb (G + 1 entries) receives each graph's first
// combined incidence; memC[ZT] the member ids (one thread per incidence),
// members out of range reported in *err (kErrColRange).  The order of the
// members within a row is left to the row check of the combined lists.
// The concat, length and row kernels do nothing once kErrPlanShape is set in
// *err (a replayed plan then keeps the lists of its previous run).
hipError_t launch_batch_rows(hipStream_t st, const BatchGraph *gr, const int64_t *ibase, int32_t G,
                             int64_t ZT, const int32_t *ptrT, const int32_t *colT,
                             const int32_t *ptrC, int32_t *zb, int32_t *memC, int32_t *err);
hipError_t launch_batch_bounds(hipStream_t st, const int64_t *ibase, int32_t G, const int32_t *a,
                               int64_t P, int64_t *off);
hipError_t launch_batch_split(hipStream_t st, const int64_t *ibase, const int64_t *off, int32_t G,
                              const int32_t *a, const int32_t *b, const int32_t *w, int64_t P,
                              int32_t *const *oa, int32_t *const *ob, int32_t *const *ow);

// g_off[g] = task_off of the first task whose item is >= g_ibase[g], for
// g = 0..G (task_item is non-decreasing; task_off has n_tasks + 1 entries).
// n_tasks_dev (nullable): the task count on the device, read as
// min(*n_tasks_dev, n_tasks) (n_tasks is then the task arrays' capacity).
hipError_t launch_batch_graph_off(hipStream_t st, const int32_t *task_item, int32_t n_tasks,
                                  const int64_t *task_off, const int64_t *g_ibase, int32_t G,
                                  int64_t *g_off, const int64_t *n_tasks_dev = nullptr);

// Replayed plans.  Per graph: row_ptr[0] == 0 and row_ptr[m] == the planned
// nnz, else kErrPlanShape in *err.  And: *value > cap sets `bit` in *err.
hipError_t launch_plan_check_shape(hipStream_t st, const BatchGraph *gr, int32_t G, int32_t *err);
hipError_t launch_plan_guard(hipStream_t st, const int64_t *value, int64_t cap, int32_t bit,
                             int32_t *err);

// Copy staged ranges to their final place (skipping tasks flagged in need).
// n_rec < 0: the records are counted on the device (*log_head, at most
// log_cap), for launches whose sizes are fixed in advance.
hipError_t launch_stage_copy(hipStream_t st, const CountArgs &a, int32_t n_rec);

// ------------------------------------------------- stages (sline_stages.hip)
// Filter of a weighted edge list: pairs with w >= s, in order.  Pass 1
// (oa == nullptr) writes per-tile counts, pass 2 writes at the exclusive scan
// off of those counts.
int64_t wfilter_tiles(int64_t n);
hipError_t launch_wfilter(hipStream_t st, const int32_t *a, const int32_t *b, const int32_t *w,
                          int64_t n, int32_t s, int32_t *cnt, const int64_t *off, int32_t *oa,
                          int32_t *ob, int32_t *ow);
// flag[x] = 1 for items in a pair (flag zeroed by the caller); err gets
// kErrColRange for an id out of [0, N) or a >= b, kErrColOrder for pairs out
// of (a, b) order.
hipError_t launch_mark_present(hipStream_t st, const int32_t *a, const int32_t *b, int64_t n,
                               int32_t N, int32_t *flag, int32_t *err);
hipError_t launch_old_ids(hipStream_t st, const int32_t *flag, const int32_t *newid, int32_t N,
                          int32_t *old_id);
// ptr[x] (x = 0..N) = first pair with a >= x, for pairs sorted by a.
hipError_t launch_run_starts(hipStream_t st, const int32_t *a, int64_t n, int32_t N, int64_t *ptr);
hipError_t launch_degrees(hipStream_t st, const int64_t *fwd, const int32_t *ptrT, int32_t N,
                          int32_t *deg);
// Row pointers from off; then off[x] and fwd[x] (from launch_run_starts) are
// what launch_adj_fill adds to a pair's position for its slot: bwd and fwd there.
hipError_t launch_row_ptr(hipStream_t st, const int32_t *flag, const int32_t *newid, int64_t *off,
                          int64_t *fwd, const int32_t *ptrT, int32_t N, int32_t n_nodes,
                          int64_t *row_ptr);
// Neighbours (and weights, ow may be null) of all rows: n pairs (a, b, w), and
// the same sorted by second item as (y, c, v).
hipError_t launch_adj_fill(hipStream_t st, int64_t n, const int32_t *newid, const int64_t *bwd,
                           const int32_t *y, const int32_t *c, const int32_t *v, const int64_t *fwd,
                           const int32_t *a, const int32_t *b, const int32_t *w, int32_t *ocol,
                           int32_t *ow);
hipError_t launch_iota(hipStream_t st, int32_t *p, int64_t n);
// comp[x] = smallest item of x's component in the graph of the pairs; label: N
// entries of scratch.
hipError_t launch_components(hipStream_t st, const int32_t *a, const int32_t *b, int64_t n,
                             int32_t N, int32_t *comp, int32_t *label);
hipError_t launch_cc_count(hipStream_t st, const int32_t *comp, const int32_t *flag, int32_t N,
                           unsigned long long *count);
hipError_t launch_gather(hipStream_t st, const int32_t *src, const int32_t *idx, int64_t n,
                         int32_t *dst);
hipError_t launch_map_pairs(hipStream_t st, const int32_t *a, const int32_t *b, int64_t n,
                            const int32_t *perm, int32_t *oa, int32_t *ob);
hipError_t launch_sizes(hipStream_t st, const int32_t *ptr, int32_t N, int32_t *size,
                        int32_t *max_size);
hipError_t launch_size_keys(hipStream_t st, const int32_t *size, int32_t N, const int32_t *max_size,
                            int32_t descending, int32_t *key);
hipError_t launch_invert(hipStream_t st, const int32_t *perm, int32_t N, int32_t *inv);
// Rows of (rp, col) in the order perm: nrp (N + 1, len and part32 scratch), ncol.
hipError_t launch_perm_rows(hipStream_t st, const int32_t *rp, const int32_t *col,
                            const int32_t *perm, int32_t N, int32_t *len, int32_t *nrp,
                            int32_t *part32, int32_t *ncol);
hipError_t launch_row_ids(hipStream_t st, const int32_t *rp, int32_t m, int32_t *rowid);
// One set intersection per wedge (the variants without visited skipping):
// count mode (oa == nullptr) writes each item's accepted pairs to cnt, write
// mode appends them from off[a]; inters (nullable) adds the intersections.
hipError_t launch_wedge_intersect(hipStream_t st, const int32_t *ptrI, const int32_t *memI,
                                  const int32_t *ptrS, const int32_t *itmS, const int32_t *start,
                                  int32_t N, int32_t s, int32_t prune, int32_t shortcut,
                                  int32_t *cnt, const int64_t *off, int32_t *oa, int32_t *ob,
                                  int32_t *ow, unsigned long long *inters, int32_t n_cu);

}  // namespace sl
