// Preparation kernels of libsline for gfx950: CSR checks, device-wide
// exclusive scans, the transpose (a stable radix sort of the incidences by
// member), the s-filtered membership lists, the exact per-item wedge count
// W_a and the lookup-only members.
//
// The transpose turns the hyperedge -> vertex incidence lists into vertex ->
// hyperedge lists (the other side of the bipartite representation, Sec. III);
// with both adjacencies the counting kernels walk, for an item a, only the
// items that share a member with it (Sec. IV-B).  Item sizes |S_a| drive the
// degree-based pruning of Sec. IV-C.
#include <type_traits>

#include "sline_internal.h"

namespace sl {

namespace {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        T t = __shfl_up(v, d, kWave);
        if (lane >= d) v += t;
    }
    return v;
}

// Exclusive scan across a 256-thread block; returns the exclusive prefix of
// `v` and writes the block total to `total`.
template <typename T>
__device__ T block_excl_scan(T v, T *sh /* 4 + 1 */, T &total) {
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    T inc = wave_incl_scan(v);
    if (lane == kWave - 1) sh[wid] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int w = 0; w < kScanThreads / kWave; ++w) {
            T t = sh[w];
            sh[w] = run;
            run += t;
        }
        sh[kScanThreads / kWave] = run;
    }
    __syncthreads();
    T ex = sh[wid] + inc - v;
    total = sh[kScanThreads / kWave];
    __syncthreads();
    return ex;
}

// first index p in [lo, hi) with arr[p] > key (arr ascending), hi if none
__device__ __forceinline__ int32_t upper_bound(const int32_t *arr, int32_t lo, int32_t hi,
                                               int32_t key) {
    while (lo < hi) {
        int32_t mid = lo + ((hi - lo) >> 1);
        if (arr[mid] <= key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

inline int grid_for(int64_t work, int per_block, int cap = 1 << 20) {
    int64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// ------------------------------------------------------------- checks

// Short rows are walked by groups of kGroup lanes (eight rows per wave) or, with
// kLaneRows rows and more, by a lane each; longer rows by whole waves, in a
// second loop that looks at 64 rows at a time and takes the long ones in turn.
// Short means at most 32 entries, or kLaneShort for a lane.  What bounds such
// walks is the latency of their dependent loads: with rows enough for every
// lane, a lane per row has eight times the rows in flight; with fewer, it
// would only make the longest chain longer.  5*10^6 rows, 3.7*10^7 entries: k_rows
// 0.25 -> 0.17 ms, k_cost 0.45 -> 0.38 ms.
constexpr int kGroup = 8;
constexpr int kLaneShort = 16;
constexpr int64_t kLaneRows = 1 << 17;

template <int W, typename T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
    for (int d = W / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

template <int W>
__device__ __forceinline__ uint64_t group_max(uint64_t v) {
#pragma unroll
    for (int d = W / 2; d >= 1; d >>= 1) {
        const uint64_t o = __shfl_xor(v, d, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// Call body(a, gl) for the rows a of one kind: with W < kWave, every row of at
// most SHORT entries, by a group of W lanes (gl = lane in the group); with
// W == kWave, every longer row, by the whole wave.
template <int W, int SHORT, typename Body>
__device__ __forceinline__ void for_rows(const int32_t *ptrI, int64_t N, Body body) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    if (W < kWave) {
        constexpr int G = kWave / W;
        const int gl = lane & (W - 1);
        for (int64_t a = wave * G + lane / W; a < N; a += nwaves * G) {
            if (ptrI[a + 1] - ptrI[a] > SHORT) continue;  // the whole-wave loop takes it
            body(a, gl);
        }
    } else {
        for (int64_t base = wave * kWave; base < N; base += nwaves * kWave) {
            const int64_t r = base + lane;
            uint64_t m = __ballot(r < N && ptrI[r + 1] - ptrI[r] > SHORT);
            while (m) {
                const int64_t a = base + __builtin_ctzll(m);
                m &= m - 1;
                body(a, lane);
            }
        }
    }
}

// Every row in one launch: body(a, gl, W), W lanes to a row, gl this lane's
// place.  LANES: a lane per row where the rows are many.
template <int SHORT, bool LANES, typename Body>
__device__ __forceinline__ void for_all_rows(const int32_t *ptrI, int64_t N, Body body) {
    if (LANES && N >= kLaneRows) {
        for_rows<1, kLaneShort>(ptrI, N, [&](int64_t a, int gl) { body(a, gl, 1); });
        for_rows<kWave, kLaneShort>(ptrI, N, [&](int64_t a, int gl) { body(a, gl, kWave); });
        return;
    }
    for_rows<kGroup, SHORT>(ptrI, N, [&](int64_t a, int gl) { body(a, gl, kGroup); });
    for_rows<kWave, SHORT>(ptrI, N, [&](int64_t a, int gl) { body(a, gl, kWave); });
}

// row_ptr checks; seen (host memory): [0] = row_ptr[m], [1] = 1 if one failed.
__global__ void k_check_rowptr(const int32_t *rp, int32_t m, int32_t *seen) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) seen[0] = rp[m];
    if ((i == 0 && rp[0] != 0) || (i < m && rp[i] > rp[i + 1])) seen[1] = 1;
}

// Device words to host memory, one launch for all of a read-back.
__global__ __launch_bounds__(kWave) void k_report(Report R) {
    for (int i = 0; i < R.n; ++i)
        for (int32_t w = threadIdx.x; w < R.words[i]; w += kWave)
            R.dst[i][w] = R.src[i][w];
    for (int i = 0; i < R.n_sums; ++i) {
        static_assert(kSumRows == kWave, "a lane per row");
        const int64_t *row = R.rows[i] + (int64_t)threadIdx.x * R.cols[i];
        for (int32_t v = 0; v < R.vals[i]; ++v) {
            const int64_t s = wave_sum(row[v]);
            if (threadIdx.x == 0) R.sums[i][v] = s;
        }
    }
}

// Workgroups of such a launch: as many as rows need, at most `cap`.
inline int rows_grid(int64_t N, int cap) {
    return grid_for(N >= kLaneRows ? N : N * kGroup, 256, cap);
}

// Loads in flight per lane of a row walk.
constexpr int kRowLoads = 4;

// The row id of every incidence, member range checks and, when asked, the
// strictly-increasing check of each row.  Rows of fewer than s entries (s_item[i]
// when given) get -1; with crank, where ranks pay, the others get their rank.
__global__ __launch_bounds__(256) void k_rows(const int32_t *rp, const int32_t *col, int32_t m,
                                              int32_t n, int64_t nnz, int check_order, int32_t s,
                                              const int32_t *s_item, const int32_t *crank,
                                              int32_t *rowid, int32_t *err) {
    int32_t bad = 0;
    crank = ranks_or_null(crank, m);
    for_all_rows<32, true>(rp, m, [&](int64_t i, int gl, int W) {
        int64_t b = rp[i], e = rp[i + 1];
        if (b < 0) b = 0;
        if (e > nnz) e = nnz;
        const int32_t id = e - b < (s_item ? s_item[i] : s) ? -1 : crank ? crank[i] : (int32_t)i;
        for (int64_t k0 = b + gl; k0 < e; k0 += kRowLoads * W) {
            int32_t v[kRowLoads], next[kRowLoads];
#pragma unroll
            for (int q = 0; q < kRowLoads; ++q) {
                const int64_t k = min(k0 + q * W, e - 1);
                v[q] = col[k];
                next[q] = check_order ? col[min(k + 1, e - 1)] : 0;
            }
#pragma unroll
            for (int q = 0; q < kRowLoads; ++q) {
                const int64_t k = k0 + q * W;
                if (k >= e) break;
                rowid[k] = id;
                if (v[q] < 0 || v[q] >= n) bad |= kErrColRange;
                if (check_order && k + 1 < e && next[q] <= v[q]) bad |= kErrColOrder;
            }
        }
    });
    if (bad) atomicOr(err, bad);
}


template <typename T>
__global__ void k_fill(T *p, int64_t n, T v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_copy(int32_t *dst, const int32_t *src, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// --------------------------------------------------------------- scan
// Three phases: per-tile sums, one-block scan of the tile sums, per-tile
// scan plus tile offset.  out has n + 1 entries; out[n] is the total.

template <typename TI, typename TA>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const TI *in, int64_t n,
                                                              TA *partial) {
    __shared__ TA sh[kScanThreads / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    TA s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q)
        if (base + q < n) s += (TA)in[base + q];
    TA tot;
    block_excl_scan<TA>(s, sh, tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

template <typename TA>
__global__ __launch_bounds__(kScanThreads) void k_scan_partials(TA *partial, int64_t nb) {
    __shared__ TA sh[kScanThreads / kWave + 1];
    TA carry = 0;
    for (int64_t c = 0; c < nb; c += kScanTile) {
        const int64_t base = c + (int64_t)threadIdx.x * kScanItems;
        TA v[kScanItems];
        TA s = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            v[q] = (base + q < nb) ? partial[base + q] : (TA)0;
            s += v[q];
        }
        TA tot;
        TA ex = block_excl_scan<TA>(s, sh, tot);
        TA run = carry + ex;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (base + q < nb) partial[base + q] = run;
            run += v[q];
        }
        carry += tot;
    }
}

// SUMS: partial holds the tiles' sums, not yet scanned, and every workgroup adds
// up those before its own (few tiles: less than a launch to scan them costs).
constexpr int64_t kScanSumTiles = 1024;

template <typename TI, typename TO, bool SUMS>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const TI *in, int64_t n,
                                                            const TO *partial, TO *out) {
    __shared__ TO sh[kScanThreads / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    TO before = 0;
    if (SUMS) {
        TO s = 0;
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) s += partial[i];
        block_excl_scan<TO>(s, sh, before);
    } else {
        before = partial[blockIdx.x];
    }
    TO v[kScanItems];
    TO s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        v[q] = (base + q < n) ? (TO)in[base + q] : (TO)0;
        s += v[q];
    }
    TO tot;
    TO ex = block_excl_scan<TO>(s, sh, tot);
    TO run = before + ex;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        if (base + q < n) out[base + q] = run;
        run += v[q];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = before + tot;
}

// Short scans: one workgroup, one launch instead of three (which cost about
// 2.5 us each, as much as 20,000 entries take here).
constexpr int kScanOneThreads = 1024;
constexpr int64_t kScanOneMax = 16384;

template <typename TI, typename TO>
__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const TI *in, int64_t n, TO *out) {
    constexpr int NW = kScanOneThreads / kWave;
    __shared__ TO sh[NW];
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    TO carry = 0;
    for (int64_t c = 0; c < n; c += kScanOneThreads * kScanItems) {
        const int64_t base = c + (int64_t)threadIdx.x * kScanItems;
        TO v[kScanItems];
        TO s = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            v[q] = base + q < n ? (TO)in[base + q] : (TO)0;
            s += v[q];
        }
        const TO incl = wave_incl_scan(s);
        if (lane == kWave - 1) sh[wid] = incl;
        __syncthreads();
        TO run = carry + incl - s;
        for (int w = 0; w < NW; ++w) {
            const TO x = sh[w];
            if (w < wid) run += x;
            carry += x;
        }
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (base + q < n) out[base + q] = run;
            run += v[q];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

template <typename TO>
__global__ void k_zero_total(TO *out) { out[0] = 0; }

// ---------------------------------------------------------- transpose



// start[k] = map[k] + 1 for every item incidence k (lists not filtered: the
// first item after a in N(v) follows a's own position in the list).
__global__ void k_start_from_map(int64_t nnz, const int32_t *map, int32_t *start) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz;
         k += (int64_t)gridDim.x * blockDim.x)
        start[k] = map[k] + 1;
}






// ------------------------------------------------ transpose by radix sort
// The transpose is a stable sort of the incidences (v = col[k], k) by member
// v: least significant digit first, digits of up to kRsBits bits, all of about
// the same width.  A pass counts the digits of each tile of keys (k_rs_hist),
// scans the counts bin by bin across tiles, and moves every key to its bin's
// place (k_rs_scatter).  Inside a tile a wave takes 64 consecutive keys at a
// time: ballots of the digit's bits give every lane the lanes with its digit,
// so its place among them, and one of them advances the wave's own counter of
// the digit; equal digits keep their order in the wave, and the scan over
// (digit, wave) keeps it in the tile.
//
// What bounds it: memory, 20 B per key and pass, the last pass's scattered maps
// and the ballots; so few passes of wide digits.  10^7 keys of 21 bits, counts,
// scans and moves: 3 passes of 7 bits 0.43 ms, 6 of 4 bits (counters per
// thread) 0.68 ms.  22,000 keys of 13 bits: 2 passes 25 us, 4 passes 100 us.
// A primal build's lists are sorted without the items that the filter drops, and
// carry the item along: 8 B more per key and pass, but no gather of it at the end, no
// flags, scan and compaction of the lists after.  3.7*10^7 incidences, three
// quarters kept, 24-bit members: 1.19 ms of scatters where those and the
// filter's passes took 2.03.
// 9 bits, as keys of 17 and 18 bits then take two passes and not three: 4.5*10^7
// of 18 bits with two values 1.14 ms (three passes with one value 1.44).
constexpr int kRsBits = 9;
constexpr int kRsBins = 1 << kRsBits;
constexpr int kRsThreads = 256;
static_assert(kRsBins == 2 * kRsThreads, "two digits per thread");
constexpr int kRsWaves = kRsThreads / kWave;
// Keys per thread: with fewer keys than kRsFewKeys, smaller tiles fill more CUs.
constexpr int kRsItems = 16, kRsItemsFew = 4;
constexpr int64_t kRsFewKeys = 1 << 19;
// What a scatter moves with each key.
constexpr int kRsOne = 0, kRsTwo = 1, kRsLists = 2;

// Digit counts of each tile, bin-major: hist[bin * ntiles + tile].  w2: keys with
// a negative value there are left out.  n_dev: at most *n_dev keys.
template <int ITEMS>
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const int32_t *keys, const int32_t *w2,
                                                        int64_t n, const int32_t *n_dev, int shift,
                                                        int bits, int32_t *hist, int32_t ntiles) {
    __shared__ int32_t h[kRsWaves][kRsBins];
    const int t = threadIdx.x, w = t / kWave;
    if (n_dev) n = min(n, (int64_t)*n_dev);
    for (int i = 0; i < kRsWaves; ++i) h[i][t] = h[i][t + kRsThreads] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRsThreads * ITEMS;
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t p = base + i * kRsThreads + t;
        if (p < n && (!w2 || w2[p] >= 0)) atomicAdd(&h[w][((uint32_t)keys[p] >> shift) & mask], 1);
    }
    __syncthreads();
    for (int d = t; d <= (int)mask; d += kRsThreads) {
        int32_t c = 0;
        for (int i = 0; i < kRsWaves; ++i) c += h[i][d];
        hist[(int64_t)d * ntiles + blockIdx.x] = c;
    }
}

// Move the keys of each tile to their place: off[bin * ntiles + tile] is the
// first output slot of the tile's keys with that digit.  vin null: the value
// of key p is p.  With `last`, the values become the final maps instead: kT[q] =
// value (the incidence), colT[q] = rowid[value] (its item), posT[value] = q (kT,
// posT may be null).  kRsTwo: a second value moves along (win to wout); with `last`
// nothing else is done.  kRsLists: as kRsTwo, but keys with a negative second value are left
// out; the number of the others goes to *n_dev in the first pass, and is read
// from there in later ones; in the last, the second value goes to colT[q], and posT[value] = q + 1.
template <int ITEMS, int MODE>
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(
    const int32_t *kin, const int32_t *vin, const int32_t *win, int64_t n, int32_t *n_dev,
    int32_t first, int shift, int bits, const int32_t *off, int32_t ntiles, int32_t *kout,
    int32_t *vout, int32_t *wout, int32_t last, const int32_t *rowid, int32_t *colT, int32_t *kT,
    int32_t *posT) {
    constexpr int TILE = kRsThreads * ITEMS;
    constexpr bool TWO = MODE != kRsOne, LISTS = MODE == kRsLists;
    __shared__ int32_t cnt[kRsWaves][kRsBins];  // keys of a digit so far; then their place
    __shared__ int32_t sk[TILE], sv[TILE];      // the tile in sorted order
    __shared__ int32_t sw[TWO ? TILE : 1];
    __shared__ int32_t sh[kScanThreads / kWave + 1];
    __shared__ int32_t dst[kRsBins];            // output slot less tile position, per digit
    const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t base = (int64_t)blockIdx.x * TILE;
    if (LISTS) {
        if (first) {
            if (blockIdx.x == 0 && t == 0) *n_dev = off[(int64_t)ntiles << bits];
        } else {
            n = min(n, (int64_t)*n_dev);
            if (base >= n) return;
        }
    }
    for (int i = 0; i < kRsWaves; ++i) cnt[i][t] = cnt[i][t + kRsThreads] = 0;
    __syncthreads();
    const int64_t mine = base + (int64_t)w * ITEMS * kWave + lane;
    int32_t key[ITEMS], val[ITEMS], two[TWO ? ITEMS : 1], rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t p = mine + i * kWave;
        key[i] = 0;
        val[i] = (int32_t)p;
        if (LISTS) two[i] = -1;
        if (p < n) {
            key[i] = kin[p];
            if (vin) val[i] = vin[p];
            if (TWO) two[i] = win[p];
        }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool ok = mine + i * kWave < n && (!LISTS || two[i] >= 0);
        const uint32_t d = ((uint32_t)key[i] >> shift) & mask;
        uint64_t same = __ballot(ok);
        for (int b = 0; b < bits; ++b) {
            const bool set = (d >> b) & 1u;
            const uint64_t m = __ballot(set);
            same &= set ? m : ~m;
        }
        const int32_t below = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        const int32_t before = ok ? cnt[w][d] : 0;
        rank[i] = before + below;
        __builtin_amdgcn_wave_barrier();  // every lane has read its counter
        if (ok && below == 0) cnt[w][d] = before + __popcll(same);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread t: digits 2 t and 2 t + 1
    int32_t sum = 0;
    for (int d = 2 * t; d < 2 * t + 2; ++d)
        for (int i = 0; i < kRsWaves; ++i) sum += cnt[i][d];
    int32_t total;
    int32_t run = block_excl_scan<int32_t>(sum, sh, total);
    for (int d = 2 * t; d < 2 * t + 2; ++d) {
        dst[d] = (d <= (int)mask ? off[(int64_t)d * ntiles + blockIdx.x] : 0) - run;
        for (int i = 0; i < kRsWaves; ++i) {
            const int32_t c = cnt[i][d];
            cnt[i][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (mine + i * kWave >= n || (LISTS && two[i] < 0)) continue;
        const int32_t r = cnt[w][((uint32_t)key[i] >> shift) & mask] + rank[i];
        sk[r] = key[i];
        sv[r] = val[i];
        if (TWO) sw[r] = two[i];
    }
    __syncthreads();
    // each bin's run with consecutive lanes
    const int32_t tn = LISTS ? total : (int32_t)(n - base < TILE ? n - base : TILE);
#pragma unroll 4
    for (int32_t j = t; j < tn; j += kRsThreads) {
        const int32_t k = sk[j], v = sv[j];
        const int32_t q = dst[((uint32_t)k >> shift) & mask] + j;
        kout[q] = k;
        if (!last || MODE == kRsTwo) {
            vout[q] = v;
            if (TWO) wout[q] = sw[j];
        } else if (LISTS) {
            if (posT) posT[v] = q + 1;
            colT[q] = sw[j];
        } else {
            if (kT) kT[q] = v;
            if (posT) posT[v] = q;
            colT[q] = rowid[v];
        }
    }
}

// Row pointers of the transpose from the sorted members: ptr[v] = first slot
// with member >= v, for v = 0..n (members outside [0, n) are clamped; they
// only occur in input that the row checks reject).  A thread per slot writes the
// pointers between its member and the one before, and of a long run of members in
// no list (those of all the items that the filter drops) only the ends: the
// blocks of kWave members within it a wave writes at once, after a search
// (left to one thread, such runs took 0.24 ms in a batch of 10 graphs).
__global__ __launch_bounds__(256) void k_rs_bounds(const int32_t *sk, int64_t nnz, int32_t n,
                                                   int32_t *ptr, const int32_t *n_dev) {
    if (n_dev) nnz = min(nnz, (int64_t)*n_dev);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = t; p <= nnz; p += nt) {
        int32_t hi = p < nnz ? sk[p] : n;
        int32_t lo = p > 0 ? sk[p - 1] : -1;
        hi = hi < 0 ? 0 : (hi > n ? n : hi);
        lo = lo < -1 ? -1 : (lo > n ? n : lo);
        if (hi - lo > 2 * kWave) {
            const int32_t c0 = (lo + kWave) & ~(kWave - 1);  // first block after lo
            const int32_t c1 = (int32_t)(((int64_t)hi + 1) & ~(int64_t)(kWave - 1));
            for (int32_t v = lo + 1; v < c0; ++v) ptr[v] = (int32_t)p;
            lo = c1 - 1;
        }
        for (int32_t v = lo + 1; v <= hi; ++v) ptr[v] = (int32_t)p;
    }
    const int64_t blocks = ((int64_t)n + 1) / kWave;
    const int lane = lane_id();
    for (int64_t c0 = t - lane; c0 < blocks; c0 += nt) {
        const int64_t first = (c0 + lane) * kWave;
        int32_t lo = 0;
        bool gap = false;
        if (c0 + lane < blocks) {
            int32_t end = (int32_t)nnz;  // first slot with member >= first
            while (lo < end) {
                const int32_t mid = lo + ((end - lo) >> 1);
                if (sk[mid] < first) lo = mid + 1;
                else end = mid;
            }
            gap = lo >= nnz || sk[lo] >= first + kWave - 1;
        }
        for (uint64_t m = __ballot(gap); m; m &= m - 1) {
            const int src = __builtin_ctzll(m);
            ptr[(c0 + src) * kWave + lane] = __shfl(lo, src, kWave);
        }
    }
}

// -------------------------------------------------------- s filtering

// Member-list entries below which the filter compares sizes entry by entry.
constexpr int64_t kFilterFew = 1 << 20;

// The s filter of a dual build, whose item sizes are known once the lists are
// transposed, as a stream compaction: the filtered lists N_s(v), one after
// the other, are the kept entries of the member lists in their order, so the
// position of a kept entry is the number of kept entries before it.
// kept[it] = 1 if item it has |S| >= s; then keep[p] = kept[itmM[p]] for entry p
// of the member lists (one gather per entry instead of the item's two bounds).
__global__ void k_item_kept(const int32_t *ptrI, int32_t N, int32_t s, int32_t *kept) {
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < N;
         it += (int64_t)gridDim.x * blockDim.x)
        kept[it] = ptrI[it + 1] - ptrI[it] >= s ? 1 : 0;
}

// kept null: the sizes are compared here (short inputs, whose list bounds stay
// in cache: one launch less).
__global__ void k_filter_flags(const int32_t *itmM, int64_t nnz, const int32_t *kept,
                               const int32_t *ptrI, int32_t s, int32_t *keep,
                               const int32_t *err) {
    if (err && (*err & kErrColRange)) return;  // items that index nothing
    if (!kept) {
        for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz;
             p += (int64_t)gridDim.x * blockDim.x) {
            const int32_t it = itmM[p];
            keep[p] = ptrI[it + 1] - ptrI[it] >= s ? 1 : 0;
        }
        return;
    }
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz;
         p += (int64_t)gridDim.x * blockDim.x)
        keep[p] = kept[itmM[p]];
}

// After the exclusive scan of the flags (pos[p], pos[nnz] = kept total): kept
// entry p goes to itmS[pos[p]], and the item's own entry sets its
// back-pointer start[inv[p]] to the position after it; ptrS[v] = pos[ptrM[v]].
// Where ranks pay, itmS receives the items' ranks among the kept ones, and orig
// the item of every rank.
__global__ void k_filter_scatter(const int32_t *itmM, int64_t nnz, const int32_t *pos,
                                 const int32_t *ptrM, int32_t M, int32_t *ptrS, int32_t *itmS,
                                 const int32_t *inv, int32_t *start, int32_t N,
                                 const int32_t *crank, int32_t *orig, const int32_t *err) {
    if (err && (*err & kErrColRange)) return;
    int64_t n = nnz > (int64_t)M + 1 ? nnz : (int64_t)M + 1;
    if (crank && !ranks_pay(crank[N], N)) crank = nullptr;
    if (crank && N > n) n = N;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        if (p < nnz) {
            const int32_t q = pos[p];
            if (pos[p + 1] != q) {
                const int32_t it = itmM[p];
                itmS[q] = crank ? crank[it] : it;
                if (start) start[inv[p]] = q + 1;
            }
        }
        if (p <= M) ptrS[p] = pos[ptrM[p]];
        if (crank && p < N) {
            const int32_t r = crank[p];
            if (crank[p + 1] != r) orig[r] = (int32_t)p;
        }
    }
}

// orig[r] = the kept item with rank r, where ranks pay.
__global__ void k_rank_items(const int32_t *crank, int32_t N, int32_t *orig) {
    if (!ranks_or_null(crank, N)) return;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < N;
         it += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = crank[it];
        if (crank[it + 1] != r) orig[r] = (int32_t)it;
    }
}

// W_a = sum over members v of the number of kept items b > a in N_s(v); 0 for
// items with |S_a| < s.  For every member incidence k of a kept item,
// start[k] = index in itmS of the first item > a in N_s(v) (the back-pointer
// where a's walk over v begins).  totals (in rows): kept items, their
// incidences, W.
__global__ __launch_bounds__(256) void k_cost(const int32_t *ptrI, const int32_t *memI,
                                              int32_t N, int32_t s, const int32_t *s_item,
                                              const int32_t *ptrS, const int32_t *itmS,
                                              int64_t *cost, int32_t *start, int64_t *totals,
                                              int32_t full, int32_t have_start,
                                              const int32_t *err) {
    if (err && *err) return;  // lists or members that index nothing
    int64_t kept = 0, kept_nnz = 0, wedges = 0;  // counted by each row's first lane
    for_all_rows<32, true>(ptrI, N, [&](int64_t a, int gl, int W) {
        const int32_t b = ptrI[a], e = ptrI[a + 1];
        if (e - b < (s_item ? s_item[a] : s)) {
            if (gl == 0) cost[a] = 0;
            return;
        }
        int64_t c = 0;
        if (have_start) {
            for (int32_t k0 = b + gl; k0 < e; k0 += kRowLoads * W) {
                int32_t hi[kRowLoads], st[kRowLoads];
#pragma unroll
                for (int q = 0; q < kRowLoads; ++q) {
                    const int32_t k = min(k0 + q * W, e - 1);
                    st[q] = start[k];
                    hi[q] = memI[k];
                }
#pragma unroll
                for (int q = 0; q < kRowLoads; ++q) hi[q] = ptrS[hi[q] + 1];
#pragma unroll
                for (int q = 0; q < kRowLoads; ++q)
                    if (k0 + q * W < e) c += hi[q] - st[q];
            }
        } else {
            for (int32_t k = b + gl; k < e; k += W) {
                const int32_t v = memI[k];
                const int32_t lo = ptrS[v], hi = ptrS[v + 1];
                const int32_t st = full ? lo : upper_bound(itmS, lo, hi, (int32_t)a);
                start[k] = st;
                c += hi - st;
            }
        }
        if (W != 1) c = W == kWave ? wave_sum(c) : group_sum<kGroup>(c);
        if (gl == 0) {
            cost[a] = c;
            kept += 1;
            kept_nnz += e - b;
            wedges += c;
        }
    });
    // one atomic per counter and block (same-address atomics serialize)
    kept = wave_sum(kept);
    kept_nnz = wave_sum(kept_nnz);
    wedges = wave_sum(wedges);
    __shared__ int64_t red[3][256 / kWave];
    const int wid = threadIdx.x / kWave;
    if (lane_id() == 0) {
        red[0][wid] = kept;
        red[1][wid] = kept_nnz;
        red[2][wid] = wedges;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        int64_t t = 0;
        for (int w = 0; w < 256 / kWave; ++w) t += red[threadIdx.x][w];
        if (t)
            atomicAdd((unsigned long long *)&totals[(blockIdx.x % kSumRows) * kTotalCols + threadIdx.x],
                      (unsigned long long)t);
    }
}

// Per kept item: flag as lookup-only the min(s - 1, kMaxLookup) members with
// the most candidates after a (ties to the lower incidence), by setting the
// sign bit of start[k].  At least one member stays unflagged, as |S_a| >= s
// for a kept item.  The item's planning cost becomes the wedges of its
// inserting members (they fill the table), but at least a third of W_a
// (every wedge is still read).  A lane looks at each item, and the wave then takes
// those that the task kernel counts, one after the other: they are few (a
// group of lanes for every item took 0.31 ms for 5*10^6 of them, this 0.09).  Rows of up to
// 256 and up to 2048 members keep their keys in registers, so the rounds only
// exchange maxima; longer rows read their members again in
// every round (as all above 256 did: one of 2000 members kept the kernel up 0.25 ms).
// The lane that owns incidence k is the one that flags it.
constexpr int kKeysFew = 4, kKeysMany = 32;

__global__ __launch_bounds__(256) void k_mark_lookup(PlanItems I, const int32_t *memI,
                                                     const int32_t *ptrS, int32_t *start,
                                                     int64_t *cost, const int32_t *err) {
    if (err && *err) return;
    I.crank = ranks_or_null(I.crank, I.N);
    constexpr int W = kWave;
    const int gl = lane_id();
    auto best_of = [&](uint64_t v) { return group_max<kWave>(v); };
    // only items that the task kernel counts: the others count every wedge
    auto counted = [&](int64_t a) {
        if (a >= I.N) return false;
        const int64_t w = cost[a];
        if (w <= I.small_max) return false;
        if (I.ptrI[a + 1] - I.ptrI[a] < (I.s_item ? I.s_item[a] : I.s)) return false;
        int32_t kind, ranges;
        return direct_tasks(I, (int32_t)a, w, kind, ranges) == 0;
    };
    auto mark = [&](int64_t a) {
        const int32_t b = I.ptrI[a], e = I.ptrI[a + 1];
        const int32_t s = I.s_item ? I.s_item[a] : I.s;
        const int32_t rounds = min(min(s - 1, kMaxLookup), e - b - 1);
        int64_t flagged = 0;
        // the row's keys in K registers of each lane
        auto keyed = [&](auto per_lane) {
            constexpr int K = decltype(per_lane)::value;
            uint64_t key[K];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const int32_t k = b + gl + i * W;
                key[i] = 0;
                if (k < e) {
                    const int32_t st = start[k];
                    const int32_t c = ptrS[memI[k] + 1] - st;
                    if (st >= 0)
                        key[i] = ((uint64_t)(uint32_t)c << 32) | (uint32_t)(INT32_MAX - k);
                }
            }
            for (int32_t r = 0; r < rounds; ++r) {
                uint64_t best = 0;
#pragma unroll
                for (int i = 0; i < K; ++i) best = key[i] > best ? key[i] : best;
                best = best_of(best);
                if ((best >> 32) == 0) break;  // no member with candidates left
                const int32_t k = INT32_MAX - (int32_t)(uint32_t)best;
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    if (key[i] == best) {  // keys are distinct: one owner
                        key[i] = 0;
                        start[k] |= (int32_t)0x80000000u;
                    }
                }
                flagged += (int64_t)(best >> 32);
            }
        };
        if (e - b <= W * kKeysFew) {
            keyed(std::integral_constant<int, kKeysFew>{});
        } else if (e - b <= W * kKeysMany) {
            keyed(std::integral_constant<int, kKeysMany>{});
        } else for (int32_t r = 0; r < rounds; ++r) {
            // best unflagged member: most candidates, then lowest k
            uint64_t best = 0;
            for (int32_t k = b + gl; k < e; k += W) {
                const int32_t st = start[k];
                if (st < 0) continue;
                const int32_t c = ptrS[memI[k] + 1] - st;
                const uint64_t key = ((uint64_t)(uint32_t)c << 32) | (uint32_t)(INT32_MAX - k);
                best = key > best ? key : best;
            }
            best = best_of(best);
            if ((best >> 32) == 0) break;  // no member with candidates left
            const int32_t k = INT32_MAX - (int32_t)(uint32_t)best;
            if ((k - b) % W == gl) start[k] |= (int32_t)0x80000000u;
            flagged += (int64_t)(best >> 32);
        }
        if (gl == 0 && flagged) {
            const int64_t w = cost[a];
            // an item with too many wedges for the sieve keeps a cost that is
            // too many as well, and one with too many for a lane (which counts
            // all W_a of a tiny item) likewise
            constexpr int64_t sieve = (int64_t)kSieveWedges * kSieveLarge, lane = 3 * kTinyMaxCost;
            cost[a] = max(max(w - flagged, (w + 2) / 3), min(w, (w > sieve ? sieve : lane) + 1));
        }
    };
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    for (int64_t base = wave * kWave; base < I.N; base += nwaves * kWave)
        for (uint64_t m = __ballot(counted(base + gl)); m; m &= m - 1) mark(base + __builtin_ctzll(m));
}

// Product filter, one block per tile of kFilterTile entries (256 threads x
// 16): pass 1 counts the kept entries of the tile, pass 2 writes them at
// off[tile] in their original order.
__global__ __launch_bounds__(256) void k_product_filter(const int32_t *a, const int32_t *b,
                                                        const int32_t *w, int64_t n, int32_t s,
                                                        int32_t *cnt, const int64_t *off,
                                                        int32_t *oa, int32_t *ob, int32_t *ow) {
    __shared__ int32_t sh[kScanThreads / kWave + 1];
    constexpr int PER = kFilterTile / 256;
    const int64_t t0 = (int64_t)blockIdx.x * kFilterTile;
    int32_t keep[PER];
    int32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int64_t k = t0 + (int64_t)threadIdx.x * PER + i;
        keep[i] = k < n && b[k] > a[k] && w[k] >= s;
        mine += keep[i];
    }
    int32_t total;
    const int32_t ex = block_excl_scan<int32_t>(mine, sh, total);
    if (!oa) {
        if (threadIdx.x == 0) cnt[blockIdx.x] = total;
        return;
    }
    int64_t o = off[blockIdx.x] + ex;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (keep[i]) {
            const int64_t k = t0 + (int64_t)threadIdx.x * PER + i;
            oa[o] = a[k];
            ob[o] = b[k];
            if (ow) ow[o] = w[k];
            ++o;
        }
    }
}

}  // namespace

// ------------------------------------------------------------ launchers

hipError_t launch_product_filter(hipStream_t st, const int32_t *a, const int32_t *b, const int32_t *w,
                                 int64_t n, int32_t s, int32_t *cnt, const int64_t *off,
                                 int32_t *out_a, int32_t *out_b, int32_t *out_w) {
    if (n <= 0) return hipSuccess;
    const int64_t tiles = (n + kFilterTile - 1) / kFilterTile;
    k_product_filter<<<(unsigned)tiles, 256, 0, st>>>(a, b, w, n, s, cnt, off, out_a, out_b, out_w);
    return hipGetLastError();
}

hipError_t launch_check_rowptr(hipStream_t st, const int32_t *rp, int32_t m, int32_t *seen) {
    k_check_rowptr<<<grid_for((int64_t)m + 1, 256), 256, 0, st>>>(rp, m, seen);
    return hipGetLastError();
}

hipError_t launch_report(hipStream_t st, const Report &R) {
    k_report<<<1, kWave, 0, st>>>(R);
    return hipGetLastError();
}

hipError_t launch_rows(hipStream_t st, const int32_t *rp, const int32_t *col, int32_t m,
                       int32_t n, int64_t nnz, int check_order, int32_t *rowid, int32_t *err,
                       int32_t s, const int32_t *s_item, const int32_t *crank) {
    if (m <= 0) return hipSuccess;
    k_rows<<<rows_grid(m, 16384), 256, 0, st>>>(rp, col, m, n, nnz, check_order, s, s_item, crank,
                                                rowid, err);
    return hipGetLastError();
}

hipError_t launch_ranks(hipStream_t st, const int32_t *ptrI, int32_t N, int32_t s, int32_t *kept,
                        int32_t *crank, int32_t *part32) {
    k_item_kept<<<grid_for(N, 256, 65536), 256, 0, st>>>(ptrI, N, s, kept);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_scan_i32(st, kept, N, crank, part32);
}

hipError_t launch_rank_items(hipStream_t st, const int32_t *crank, int32_t N, int32_t *orig) {
    k_rank_items<<<grid_for(N, 256, 65536), 256, 0, st>>>(crank, N, orig);
    return hipGetLastError();
}

hipError_t launch_fill_i32(hipStream_t st, int32_t *p, int64_t n, int32_t v) {
    if (n <= 0) return hipSuccess;
    k_fill<int32_t><<<grid_for(n, 256, 65536), 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_i64(hipStream_t st, int64_t *p, int64_t n, int64_t v) {
    if (n <= 0) return hipSuccess;
    k_fill<int64_t><<<grid_for(n, 256, 65536), 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_copy_i32(hipStream_t st, int32_t *dst, const int32_t *src, int64_t n) {
    if (n <= 0) return hipSuccess;
    k_copy<<<grid_for(n, 256, 65536), 256, 0, st>>>(dst, src, n);
    return hipGetLastError();
}

int64_t scan_partials(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

template <typename TI, typename TO>
static hipError_t scan_impl(hipStream_t st, const TI *in, int64_t n, TO *out, TO *partial) {
    if (n <= 0) {
        k_zero_total<TO><<<1, 1, 0, st>>>(out);
        return hipGetLastError();
    }
    if (n <= kScanOneMax) {
        k_scan_one<TI, TO><<<1, kScanOneThreads, 0, st>>>(in, n, out);
        return hipGetLastError();
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    k_scan_reduce<TI, TO><<<(unsigned)nb, kScanThreads, 0, st>>>(in, n, partial);
    if (nb <= kScanSumTiles) {
        k_scan_down<TI, TO, true><<<(unsigned)nb, kScanThreads, 0, st>>>(in, n, partial, out);
    } else {
        k_scan_partials<TO><<<1, kScanThreads, 0, st>>>(partial, nb);
        k_scan_down<TI, TO, false><<<(unsigned)nb, kScanThreads, 0, st>>>(in, n, partial, out);
    }
    return hipGetLastError();
}

hipError_t launch_scan_i32(hipStream_t st, const int32_t *in, int64_t n, int32_t *out,
                           int32_t *partial) {
    return scan_impl<int32_t, int32_t>(st, in, n, out, partial);
}

hipError_t launch_scan_i32_to_i64(hipStream_t st, const int32_t *in, int64_t n, int64_t *out,
                                  int64_t *partial) {
    return scan_impl<int32_t, int64_t>(st, in, n, out, partial);
}



hipError_t launch_start_from_map(hipStream_t st, int64_t nnz, const int32_t *map, int32_t *start) {
    if (nnz <= 0) return hipSuccess;
    k_start_from_map<<<grid_for(nnz, 256, 65536), 256, 0, st>>>(nnz, map, start);
    return hipGetLastError();
}







static int64_t rs_tiles(int64_t nnz) {
    const int64_t tile = (int64_t)kRsThreads * (nnz < kRsFewKeys ? kRsItemsFew : kRsItems);
    return (nnz + tile - 1) / tile;
}

int64_t transpose_hist(int64_t nnz) { return (int64_t)kRsBins * rs_tiles(nnz) + 1; }

static int key_bits(int32_t n) {
    int bits = 0;
    while (bits < 31 && ((int64_t)1 << bits) < (int64_t)n) ++bits;
    return std::max(1, bits);
}

int transpose_passes(int32_t n) { return (key_bits(n) + kRsBits - 1) / kRsBits; }

// The passes of a sort of `keys` in [0, n), each counted, scanned and moved:
// move(p, last, few, keys in, ntiles, shift, bits) launches the scatter of pass p.
// w, n_dev: see k_rs_hist (w in the first pass, n_dev in later ones).
template <typename Move>
static hipError_t rs_passes(hipStream_t st, const int32_t *keys, int64_t nnz, int32_t n,
                            int32_t *const rsK[2], int32_t *hist, int32_t *part32,
                            const int32_t *w, const int32_t *n_dev, Move move) {
    const int passes = transpose_passes(n);
    const int32_t ntiles = (int32_t)rs_tiles(nnz);
    const bool few = nnz < kRsFewKeys;
    const int total = key_bits(n), width = (total + passes - 1) / passes;
    hipError_t e = hipSuccess;
    for (int p = 0; p < passes && e == hipSuccess; ++p) {
        const int32_t *kin = p == 0 ? keys : rsK[(p - 1) & 1];
        const int shift = p * width, bits = std::min(width, total - shift);
        auto *const count = few ? k_rs_hist<kRsItemsFew> : k_rs_hist<kRsItems>;
        count<<<ntiles, kRsThreads, 0, st>>>(kin, p == 0 ? w : nullptr, nnz, p == 0 ? nullptr : n_dev,
                                             shift, bits, hist, ntiles);
        e = hipGetLastError();
        if (e == hipSuccess) e = launch_scan_i32(st, hist, (int64_t)ntiles << bits, hist, part32);
        if (e != hipSuccess) break;
        move(p, p == passes - 1 ? 1 : 0, few, kin, ntiles, shift, bits);
        e = hipGetLastError();
    }
    return e;
}

// Scatter of a launch's tile size.
template <int MODE>
static auto rs_move(bool few) {
    return few ? k_rs_scatter<kRsItemsFew, MODE> : k_rs_scatter<kRsItems, MODE>;
}

static hipError_t rs_bounds(hipStream_t st, const int32_t *sorted, int64_t nnz, int32_t n,
                            int32_t *ptr, const int32_t *n_dev) {
    k_rs_bounds<<<grid_for(std::max<int64_t>(nnz, n / kWave) + 1, 256, 65536), 256, 0, st>>>(sorted, nnz, n, ptr, n_dev);
    return hipGetLastError();
}

hipError_t launch_transpose(hipStream_t st, const int32_t *col, int64_t nnz, int32_t n,
                            const int32_t *rowid, int32_t *const rsK[2], int32_t *const rsV[2],
                            int32_t *hist, int32_t *part32, int32_t *ptrT, int32_t *colT,
                            int32_t *kT, int32_t *posT) {
    if (nnz <= 0) return launch_fill_i32(st, ptrT, (int64_t)n + 1, 0);
    const hipError_t e = rs_passes(
        st, col, nnz, n, rsK, hist, part32, nullptr, nullptr,
        [&](int p, int last, bool few, const int32_t *kin, int32_t ntiles, int shift, int bits) {
            rs_move<kRsOne>(few)<<<ntiles, kRsThreads, 0, st>>>(
                kin, p == 0 ? nullptr : rsV[(p - 1) & 1], nullptr, nnz, nullptr, p == 0, shift, bits,
                hist, ntiles, rsK[p & 1], rsV[p & 1], nullptr, last, rowid, colT, kT, posT);
        });
    return e != hipSuccess ? e
                           : rs_bounds(st, rsK[(transpose_passes(n) - 1) & 1], nnz, n, ptrT, nullptr);
}

hipError_t launch_member_lists(hipStream_t st, const int32_t *col, int32_t *item, int64_t nnz,
                               int32_t n, int32_t *const rsK[2], int32_t *const rsV[2],
                               int32_t *rsW, int32_t *hist, int32_t *part32, int32_t *n_dev,
                               int32_t *ptr, int32_t *itm, int32_t *start) {
    if (nnz <= 0) return launch_fill_i32(st, ptr, (int64_t)n + 1, 0);
    int32_t *const w[2] = {rsW, item};  // the first pass leaves `item` free
    const hipError_t e = rs_passes(
        st, col, nnz, n, rsK, hist, part32, item, n_dev,
        [&](int p, int last, bool few, const int32_t *kin, int32_t ntiles, int shift, int bits) {
            rs_move<kRsLists>(few)<<<ntiles, kRsThreads, 0, st>>>(
                kin, p == 0 ? nullptr : rsV[(p - 1) & 1], p == 0 ? item : w[(p - 1) & 1], nnz, n_dev,
                p == 0, shift, bits, hist, ntiles, rsK[p & 1], rsV[p & 1], w[p & 1], last, nullptr,
                itm, nullptr, start);
        });
    return e != hipSuccess ? e
                           : rs_bounds(st, rsK[(transpose_passes(n) - 1) & 1], nnz, n, ptr, n_dev);
}

hipError_t launch_sort_values(hipStream_t st, const int32_t *key, const int32_t *v,
                              const int32_t *w, int64_t nnz, int32_t n, int32_t *const rsK[2],
                              int32_t *const rsV[2], int32_t *const rsW[2], int32_t *hist,
                              int32_t *part32, int32_t *ptr) {
    if (nnz <= 0) return launch_fill_i32(st, ptr, (int64_t)n + 1, 0);
    const hipError_t e = rs_passes(
        st, key, nnz, n, rsK, hist, part32, nullptr, nullptr,
        [&](int p, int, bool few, const int32_t *kin, int32_t ntiles, int shift, int bits) {
            const int32_t *vin = p == 0 ? v : rsV[(p - 1) & 1];
            const int32_t *win = p == 0 || !w ? w : rsW[(p - 1) & 1];
            (w ? rs_move<kRsTwo>(few) : rs_move<kRsOne>(few))<<<ntiles, kRsThreads, 0, st>>>(
                kin, vin, win, nnz, nullptr, p == 0, shift, bits, hist, ntiles, rsK[p & 1],
                rsV[p & 1], rsW[p & 1], 0, nullptr, nullptr, nullptr, nullptr);
        });
    return e != hipSuccess ? e
                           : rs_bounds(st, rsK[(transpose_passes(n) - 1) & 1], nnz, n, ptr, nullptr);
}

hipError_t launch_filter(hipStream_t st, const int32_t *ptrM, const int32_t *itmM, int32_t M,
                         int64_t nnz, const int32_t *ptrI, int32_t N, int32_t s,
                         int32_t *kept, int32_t *pos, int32_t *part32, int32_t *ptrS,
                         int32_t *itmS, const int32_t *inv, int32_t *start, int32_t *crank,
                         int32_t *orig, const int32_t *err) {
    if (M <= 0) return hipSuccess;
    if (nnz > 0) {
        const bool few = !crank && nnz < kFilterFew;
        if (!few) k_item_kept<<<grid_for(N, 256, 65536), 256, 0, st>>>(ptrI, N, s, kept);
        k_filter_flags<<<grid_for(nnz, 256, 65536), 256, 0, st>>>(itmM, nnz, few ? nullptr : kept,
                                                                 ptrI, s, pos, err);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && crank) e = launch_scan_i32(st, kept, N, crank, part32);
        if (e != hipSuccess) return e;
    } else {
        crank = nullptr;  // no member lists to number
    }
    // in place: every scan thread reads its inputs before writing them
    hipError_t e = launch_scan_i32(st, pos, nnz, pos, part32);
    if (e != hipSuccess) return e;
    const int64_t most = std::max<int64_t>({nnz, (int64_t)M + 1, crank ? (int64_t)N : 0});
    k_filter_scatter<<<grid_for(most, 256, 65536), 256, 0, st>>>(
        itmM, nnz, pos, ptrM, M, ptrS, itmS, inv, start, N, crank, orig, err);
    return hipGetLastError();
}

hipError_t launch_cost(hipStream_t st, const int32_t *ptrI, const int32_t *memI, int32_t N,
                       int32_t s, const int32_t *s_item, const int32_t *ptrS, const int32_t *itmS,
                       int64_t *cost, int32_t *start, int64_t *totals, int32_t full,
                       int32_t have_start, const int32_t *err) {
    if (N <= 0) return hipSuccess;
    k_cost<<<rows_grid(N, 4096), 256, 0, st>>>(
        ptrI, memI, N, s, s_item, ptrS, itmS, cost, start, totals, full, have_start, err);
    return hipGetLastError();
}

hipError_t launch_mark_lookup(hipStream_t st, const PlanItems &I, const int32_t *memI,
                              const int32_t *ptrS, int32_t *start, int64_t *cost,
                              const int32_t *err) {
    if (I.N <= 0) return hipSuccess;
    k_mark_lookup<<<grid_for(I.N, 256, 16384), 256, 0, st>>>(I, memI, ptrS, start, cost, err);
    return hipGetLastError();
}

}  // namespace sl
