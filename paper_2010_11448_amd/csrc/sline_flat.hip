// Direct counting of libsline for gfx950: items with enough wedges for the
// width of their candidate range are counted in LDS counters indexed by the
// candidate, with no keys and no probing.
//
// A workgroup takes one task, an item and a run of its ranges of candidates,
// and works a range at a time:
//   1. every thread takes one member of the item and finds the part of its
//      list N_s(v) that lies in the range.  Ranges start at multiples of
//      kFlatBlock candidates, and long lists have the position of every such
//      multiple in a table (k_flat_bounds), so this is two reads and no
//      search; short lists are taken whole and filtered by candidate;
//   2. an exclusive scan of the parts' lengths numbers the range's wedges, and
//      a bit per wedge marks where a part begins: a wave reads the bits of 64
//      wedges, and the count of the bits up to a lane's own is that lane's
//      member.  Every lane of every load then has a wedge, whatever the lists'
//      lengths are;
//   3. a wedge adds one to its candidate's counter, and the add that makes a
//      counter reach s sets the candidate's bit in a bit map;
//   4. the map is read in order: the bits before a pair's own are its place.
//      Counters are read for pairs only, and cleared with wide stores.
// A counter has 4, 8 or 16 bits, enough for the item's size, which bounds
// every overlap; a range is as wide as the counters fit in kFlatWords words.
//
// What bounds it: vector instructions (about 20 per 64 wedges and 250 per wave
// and range; 56% of a SIMD's cycles by the counters), and the waits of a range that is
// too short to hide them (54% of a wave's cycles): LDS reads one after the other,
// three barriers, lists that are read for the first time.  Two workgroups of 512
// threads share a CU, so one counts while the other waits or clears.  A wave's chunks are counted eight at a time,
// the last ones in groups of eight, four or two: 10^6 hyperedges, s = 2 (8.7*10^9
// wedges, most of them here): 20.6 ms, 22.0 with eight for all, 24.0 before the
// kernel was compiled apart for the fill mode and for s = 1 (21.4 since it takes the
// items of one or two ranges too, of which it relieves the sieves).
#include <algorithm>

#include "sline_count.h"

namespace sl {

namespace {

constexpr int kFlatChunks = kFlatKeep / kWave;  // 64-wedge chunks marked at a time

// Position of every multiple of kFlatBlock candidates in each list that is at
// least as long as the table row it needs: bnd[ptrS[v] + r] = the first entry
// of N_s(v) that is >= r * kFlatBlock, r = 0..blocks.  A row lies over its
// list's own entries, so rows need no index of their own.  The row of the list
// [b, e), by one wave:
__device__ __forceinline__ void flat_bounds_row(const int32_t *itmS, int32_t b, int32_t e,
                                                int32_t blocks, int32_t *bnd) {
    int32_t last = -1;  // block of the entry before this step's first
    for (int32_t q = b; q <= e; q += kWave) {
        const int32_t p = q + lane_id();
        const int32_t cur = p < e ? itmS[p] / kFlatBlock : blocks;
        int32_t prev = __shfl_up(cur, 1, kWave);
        if (lane_id() == 0) prev = last;
        if (p <= e)
            for (int32_t x = prev + 1; x <= cur; ++x) bnd[b + x] = p;
        last = lane63(cur);
    }
}

// A wave looks at 64 lists, or at fewer if that leaves waves idle, and takes those of
// up to kMidList entries that need a row; longer ones go to a list of their own, of
// which every wave of a second kernel takes one.  (64 long lists in turn, as of the
// only members there are or of hubs with neighbouring ids, would keep the build
// waiting: 16 lists of 6,250 items, 0.47 ms of a build of 1.34, now 0.92.)
constexpr int32_t kMidList = 512;

__global__ __launch_bounds__(256) void k_flat_bounds(const int32_t *ptrS, const int32_t *itmS,
                                                     int32_t M, const int32_t *crank, int32_t N,
                                                     int32_t per, int32_t *bnd,
                                                     int32_t *long_lists, int32_t *n_long,
                                                     const int32_t *n_flat,
                                                     const int32_t *err) {
    if ((err && *err) || *n_flat == 0) return;
    crank = ranks_or_null(crank, N);
    const int32_t blocks = flat_blocks(cand_of(crank, N));
    if (blocks < 2) return;  // every item's candidates fit one range of any width
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    for (int64_t base = wave * per; base < M; base += nwaves * per) {
        const int64_t r = base + lane_id();
        const bool mine = lane_id() < per && r < M;
        const int32_t b0 = mine ? ptrS[r] : 0, e0 = mine ? ptrS[r + 1] : 0;
        const bool row = e0 - b0 > blocks, far = row && e0 - b0 > kMidList;
        if (const uint64_t m = __ballot(far)) {
            int32_t at = 0;
            if (lane_id() == 0) at = atomicAdd(n_long, (int32_t)__popcll(m));
            at = uniform(at) + (int32_t)lanes_below(m);
            if (far) long_lists[at] = (int32_t)r;
        }
        for (uint64_t m = __ballot(row && !far); m; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            flat_bounds_row(itmS, __builtin_amdgcn_readlane(b0, l), __builtin_amdgcn_readlane(e0, l),
                            blocks, bnd);
        }
    }
}

__global__ __launch_bounds__(256) void k_flat_long(const int32_t *ptrS, const int32_t *itmS,
                                                   const int32_t *crank, int32_t N, int32_t *bnd,
                                                   const int32_t *long_lists, const int32_t *n_long) {
    crank = ranks_or_null(crank, N);
    const int32_t blocks = flat_blocks(cand_of(crank, N)), n = *n_long;
    const int32_t nwaves = gridDim.x * (256 / kWave);
    for (int32_t i = blockIdx.x * (256 / kWave) + wave_id(); i < n; i += nwaves) {
        const int32_t v = long_lists[i];
        flat_bounds_row(itmS, uniform(ptrS[v]), uniform(ptrS[v + 1]), blocks, bnd);
    }
}

// v << n for the low five bits of n: the instruction itself, as the compiler
// masks n before it where it knows some bit of it.
__device__ __forceinline__ uint32_t shift_left(uint32_t v, uint32_t n) {
    uint32_t r;
    asm("v_lshlrev_b32 %0, %1, %2" : "=v"(r) : "v"(n), "v"(v));
    return r;
}

// One member of an item: its walk [st, en) of N_s(v), and the list's row of the
// bounds table (-1: none, the list is taken whole).
struct FlatMember {
    int32_t st, en, row;
};

// A task, and what the counting needs of its item.
struct FlatTask {
    int32_t t, a, part, k0, size, first, nend, s;
    int64_t cost;
};

template <bool FILL, bool ONES>
__global__ __launch_bounds__(kFlatThreads, 4) void k_count_flat(CountArgs A) {
    constexpr int NT = kFlatThreads, NW = NT / kWave;
    constexpr int kKeep = kFlatKeep / NT;  // wedges a lane holds (s = 1)
    constexpr int kLoad = 8;               // chunks a wave loads at a time
    __shared__ __align__(16) uint32_t ctr[kFlatWords + kWave];  // + a spare word per lane
    __shared__ __align__(16) uint4 bmp[kFlatWords / 16];        // a bit per candidate
    __shared__ int32_t adj[NT];  // the wedge map's positions; hits while pairs are written
    __shared__ __align__(8) uint32_t marks[2 * kFlatChunks];
    __shared__ int32_t msh[3 * NW], wtot[NW];
    // the task after the next one, in two words by turns: a skipped task has no other
    // barrier, and a late wave may still be reading the word of the task before it
    __shared__ int32_t sh_task[2];
    __shared__ int32_t sh_hits, sh_ok;
    __shared__ uint64_t sh_off, pool_cur[3];
    __shared__ int32_t log_cur[3];
    if (count_idle(A)) return;  // uniform: every thread reads the same words
    const int32_t n_flat = A.task_counts[kKindFlat * kCountStride];
    if (n_flat == 0) return;
    use_ranks(A);
    const int tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    const int32_t blocks = flat_blocks(cand_of(A.crank, A.N));
    uint4 *const c4 = reinterpret_cast<uint4 *>(ctr);
    for (int i = tid; i < kFlatWords / 4; i += NT) c4[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = tid; i < kFlatWords / 16; i += NT) bmp[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = tid; i < 2 * kFlatChunks; i += NT) marks[i] = 0;
    if (tid == 0) {
        stage_begin(A, kKindFlat, pool_cur, log_cur);
        sh_hits = 0;
        sh_task[0] = atomicAdd(A.queue + 1, 2);
    }
    int64_t passes = 0, my_wedges = 0, my_nnz = 0, my_pairs = 0;  // thread 0's are used
    __syncthreads();
    int32_t r = sh_task[0], r1 = r + 1;  // this task and the next in the list
    int turn = 0;

    WedgeMap<NT, kFlatChunks> map;
    map.adj_all = adj;
    map.marks_all = marks;
    map.sh = msh;
    auto load_task = [&](int32_t q) {
        FlatTask d{};
        if (q < n_flat) {
            d.t = A.big_tasks[A.n_tasks - 1 - q];
            d.a = A.task_item[d.t];
            d.part = A.task_part[d.t];
        }
        return d;
    };
    auto load_item = [&](FlatTask &d) {
        d.k0 = A.ptrI[d.a];
        d.size = A.ptrI[d.a + 1] - d.k0;
        d.first = cand_first(A.crank, 0, d.a);
        d.nend = cand_end(A.crank, A.item_end, A.N, d.a);
        d.cost = A.cost[d.a];
        d.s = A.s_item ? A.s_item[d.a] : A.s;
    };
    // member of incidence k of the current batch: st, and v in en
    auto load_member = [&](int32_t k, int32_t k1) {
        FlatMember m{0, -1, -1};
        if (k < k1) {
            m.en = A.memI[k];
            m.st = A.start[k] & kStartMask;
        }
        return m;
    };
    auto load_list = [&](FlatMember &m, bool table) {
        const int32_t v = m.en;
        m.en = 0;
        if (v >= 0) {
            const int32_t b = A.ptrS[v];
            m.en = A.ptrS[v + 1];
            if (table && m.en - b > blocks) m.row = b;
        }
    };
    // The next task is looked up while this one is counted.
    FlatTask cur = load_task(r);
    load_item(cur);
    while (r < n_flat) {
        int32_t r2 = 0;
        if (tid == 0) r2 = atomicAdd(A.queue + 1, 1);
        map.narrow = uniform(cur.size) <= kWave;
        FlatMember mem = load_member(cur.k0 + map.member(), cur.k0 + cur.size);
        FlatTask nxt = load_task(r1);
        const int32_t t = uniform(cur.t), a = uniform(cur.a), s = uniform(cur.s);
        const int32_t k0 = uniform(cur.k0), k1 = k0 + uniform(cur.size);
        const int32_t first = uniform(cur.first), nend = uniform(cur.nend);
        const FlatShape F = flat_shape(first, nend, k1 - k0);
        const int64_t cost = ((int64_t)uniform((int32_t)(cur.cost >> 32)) << 32) |
                             (uint32_t)uniform((int32_t)cur.cost);
        const int32_t per = flat_ranges_per_task(F, cost);
        const int32_t part = uniform(cur.part);
        const int32_t p0 = part * per, p1 = min(F.ranges, p0 + per);
        const bool skip = FILL && A.need && !A.need[t];
        // bits per counter as a shift, counters per word as a shift
        const uint32_t lb = F.lbits, psh = 5u - lb;
        const bool keep = ONES && flat_keeps(s, cost, k1 - k0);
        if (part == 0 && !FILL) {
            my_wedges += cost;
            my_nnz += k1 - k0;
        }
        load_list(mem, F.ranges > 1 && !keep);
        int32_t produced = 0;
        int32_t hits = 0;  // pairs found by this wave
        // What a counter holds before the add that makes a pair: s - 1, which is less
        // than the all-ones of a lane without a count as long as s is no more than
        // the item's size.  An item of fewer members (kept with SLINE_NO_PRUNE)
        // is in no pair: a value that no counter has.
        const uint32_t s_1 = s <= k1 - k0 ? (uint32_t)s - 1u : ~0u;

        // Count wedges, x = candidate - first of the range (>= span: none).
        auto count = [&](const auto &j, int32_t lo, uint32_t span) {
            constexpr int K = sizeof(j) / sizeof(j[0]);
            uint32_t x[K], at[K], old[K];
#pragma unroll
            for (int u = 0; u < K; ++u) {
                x[u] = (uint32_t)(j[u] - lo);
                at[u] = x[u] << lb;  // the counter's bit
                old[u] = ~0u;        // no count: all ones, not s_1
                if (x[u] < span) old[u] = atomicAdd(&ctr[at[u] >> 5], shift_left(1u, at[u]));
            }
#pragma unroll
            for (int u = 0; u < K; ++u) {
                const bool hit = __builtin_amdgcn_ubfe(old[u], at[u], 1u << lb) == s_1;
                const uint64_t m = __ballot(hit);
                if (m) {
                    if (hit)
                        atomicOr(reinterpret_cast<uint32_t *>(bmp) + (x[u] >> 5),
                                 1u << (x[u] & 31u));
                    hits += __popcll(m);
                }
            }
        };
        // Thread 0: room for `total` pairs of the task.
        auto reserve = [&](int32_t total) {
            bool ok = true;
            if (!FILL && A.mode == kModeStage) {
                uint64_t off;
                int32_t rec;
                ok = stage_reserve(A, pool_cur, log_cur, total, 1, off, rec);
                if (ok) {
                    StageRec sr;
                    sr.off = (int64_t)off;
                    sr.t = t;
                    sr.rel = produced;
                    sr.n = total;
                    sr.pad = 0;
                    A.log[rec] = sr;
                } else if (atomicExch(&A.need[t], 1) == 0) {
                    atomicAdd(A.need_count, 1);
                }
                sh_off = off;
            }
            sh_ok = ok && (FILL || A.mode != kModeCount) ? 1 : 0;
        };
        // Where reserved pairs go.
        struct Dest {
            int32_t *a, *b, *w;
            int64_t at;
            int32_t shift;
        };
        auto dest = [&]() {
            if (!FILL) return Dest{nullptr, A.pool_b, A.pool_w, (int64_t)sh_off, 0};
            const OutDst od = out_dst(A, a, A.task_off[t] + produced);
            return Dest{od.a, od.b, od.w, od.base, od.shift};
        };
        auto put = [&](const Dest &d, int64_t o, int32_t cand, int32_t w) {
            if (FILL) {
                d.a[o] = a - d.shift;
                d.b[o] = item_of(A, cand) - d.shift;
            } else {
                d.b[o] = cand;
            }
            if (d.w) d.w[o] = w;
        };
        // The pairs of the range, in order.  Wave w owns a run of quads (128
        // candidates) of the map.
        auto emit = [&](int32_t lo, int32_t total, int32_t q0, int32_t q1) {
            constexpr int IT = (kFlatWords / 16 / NW + kWave - 1) / kWave;
            uint4 w[IT];
            int32_t np[IT], mine = 0;
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int32_t q = q0 + i * kWave + lane;
                w[i] = make_uint4(0u, 0u, 0u, 0u);
                if (q < q1) {
                    w[i] = bmp[q];
                    bmp[q] = make_uint4(0u, 0u, 0u, 0u);
                }
                np[i] = __popc(w[i].x) + __popc(w[i].y) + __popc(w[i].z) + __popc(w[i].w);
                mine += np[i];
            }
            mine = lane63(wave_incl(mine));
            if (lane == 0) wtot[wid] = mine;
            if (tid == 0) reserve(total);
            __syncthreads();
            if (tid == 0) sh_hits = 0;
            if (!sh_ok || !mine) return;
            Dest d = dest();
#pragma unroll
            for (int v = 0; v < NW; ++v) d.at += v < wid ? wtot[v] : 0;
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int32_t incl = wave_incl(np[i]);
                const int32_t all = lane63(incl);
                int32_t o = incl - np[i];
                const uint32_t x0 = (uint32_t)(q0 + i * kWave + lane) << 7;
                uint32_t word = w[i].x, rest = 0;
                auto next = [&]() {  // the lane's next pair
                    while (word == 0u) {
                        ++rest;
                        word = rest == 1u ? w[i].y : rest == 2u ? w[i].z : w[i].w;
                    }
                    const uint32_t x = x0 + rest * 32u + (uint32_t)__builtin_ctz(word);
                    word &= word - 1u;
                    return x;
                };
                auto value = [&](uint32_t x) {
                    return (int32_t)__builtin_amdgcn_ubfe(ctr[x >> psh], x << lb, 1u << lb);
                };
                if (all <= kWave) {
                    // few: line them up, a pair per lane
                    int32_t *const line = adj + wid * kWave;
                    for (int32_t n = np[i]; n > 0; --n) line[o++] = (int32_t)next();
                    __builtin_amdgcn_wave_barrier();
                    if (lane < all) {
                        const uint32_t x = (uint32_t)line[lane];
                        put(d, d.at + lane, lo + (int32_t)x, value(x));
                    }
                    __builtin_amdgcn_wave_barrier();
                } else {
                    for (int32_t n = np[i]; n > 0; --n) {
                        const uint32_t x = next();
                        put(d, d.at + o++, lo + (int32_t)x, value(x));
                    }
                }
                d.at += all;
            }
        };

        load_item(nxt);
        if (skip) {
            // nothing to count again
        } else if (keep) {
            // s = 1: every candidate is a pair.  Every wedge goes into a register
            // once; a range has a bit per candidate, the bits before a
            // candidate's own are its rank, and wedges are counted by rank.
            uint32_t *const cand = ctr, *const set = ctr + kFlatWords / 2;  // cand: by rank
            uint16_t *const pre = reinterpret_cast<uint16_t *>(bmp);  // bits before each 64
            uint16_t *const cnt = pre + kFlatWords / 4;
            const uint64_t *const set64 = reinterpret_cast<const uint64_t *>(set);
            map.number(mem.st, max(mem.en - mem.st, 0));
            const auto run = map.window(0);
            const int32_t n = run.nc;
            int32_t j[kKeep];
#pragma unroll
            for (int u = 0; u < kKeep; u += kLoad) {
                int32_t part[kLoad];
#pragma unroll
                for (int v = 0; v < kLoad; ++v) part[v] = -1;
                if (u < n) map.load(A.itmS, run, u, part);
#pragma unroll
                for (int v = 0; v < kLoad; ++v) j[u + v] = part[v];
            }
            const int32_t np = keep_ranges(first, nend);
            for (int32_t p = 0; p < np; ++p) {
                const int32_t lo = first + p * kKeepWidth;
                const uint32_t span = (uint32_t)min((int64_t)nend - lo, (int64_t)kKeepWidth);
                uint32_t mine = 0;  // bit u: wedge u is the first of its candidate
                ++passes;
#pragma unroll
                for (int u = 0; u < kKeep; ++u) {
                    if (u >= n) break;
                    const uint32_t x = (uint32_t)(j[u] - lo), bit = 1u << (x & 31u);
                    bool made = false;
                    if (x < span) {
                        made = (atomicOr(&set[x >> 5], bit) & bit) == 0u;
                        if (made) mine |= 1u << u;
                    }
                    hits += __popcll(__ballot(made));
                }
                if (lane == 0 && hits) atomicAdd(&sh_hits, hits);
                hits = 0;
                __syncthreads();
                const int32_t ranks = sh_hits;
                if (ranks > 0) {
                    // bits before each 64 candidates: eight of those per thread
                    const bool used = tid * 512u < span;
                    uint4 q[4];
                    int32_t sum = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        q[i] = make_uint4(0u, 0u, 0u, 0u);
                        if (used) q[i] = reinterpret_cast<const uint4 *>(set)[tid * 4 + i];
                        sum += __popc(q[i].x) + __popc(q[i].y) + __popc(q[i].z) + __popc(q[i].w);
                    }
                    const int32_t incl = wave_incl(sum);
                    if (lane == 63) wtot[wid] = incl;
                    if (tid == 0) reserve(min(ranks, kKeepRanks));
                    __syncthreads();
                    if (tid == 0) sh_hits = 0;
                    int32_t run = incl - sum;
#pragma unroll
                    for (int v = 0; v < NW; ++v) run += v < wid ? wtot[v] : 0;
                    uint32_t pk[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        pk[i] = (uint32_t)run;
                        run += __popc(q[i].x) + __popc(q[i].y);
                        pk[i] |= (uint32_t)run << 16;
                        run += __popc(q[i].z) + __popc(q[i].w);
                    }
                    uint4 *const pre8 = reinterpret_cast<uint4 *>(pre) + tid;
                    if (used) *pre8 = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                    __syncthreads();
                    for (int32_t r0 = 0; r0 < ranks; r0 += kKeepRanks) {
                        const int32_t nr = min(ranks - r0, kKeepRanks);
#pragma unroll
                        for (int u = 0; u < kKeep; ++u) {
                            if (u >= n) break;
                            const uint32_t x = (uint32_t)(j[u] - lo);
                            if (x < span) {
                                const uint64_t below = set64[x >> 6] & ~(~0ull << (x & 63u));
                                const uint32_t k = pre[x >> 6] + __popcll(below) - (uint32_t)r0;
                                if (k < (uint32_t)nr) {
                                    atomicAdd(reinterpret_cast<uint32_t *>(cnt) + (k >> 1),
                                              1u << ((k & 1u) << 4));
                                    if ((mine >> u) & 1u) cand[k] = (uint32_t)j[u];
                                }
                            }
                        }
                        if (r0 > 0 && tid == 0) reserve(nr);
                        __syncthreads();
                        // a run of ranks for each wave
                        const int32_t rpw = (nr + NW * kWave - 1) / (NW * kWave) * kWave;
                        const int32_t k0w = min(nr, wid * rpw), k1w = min(nr, k0w + rpw);
                        if (k0w < k1w) {
                            const bool out = sh_ok;
                            const Dest d = dest();
                            for (int32_t k = k0w + lane; k < k1w; k += kWave) {
                                if (out) put(d, d.at + k, (int32_t)cand[k], (int32_t)cnt[k]);
                                cnt[k] = 0;
                            }
                        }
                        produced += nr;
                        if (r0 + kKeepRanks < ranks) __syncthreads();  // the ranks are counted again
                    }
                    if (used) *pre8 = make_uint4(0u, 0u, 0u, 0u);  // other items' map
#pragma unroll
                    for (int u = 0; u < kKeep; ++u) {
                        if (u >= n) break;
                        const uint32_t x = (uint32_t)(j[u] - lo);
                        if (x < span) set[x >> 5] = 0u;
                    }
                }
                __syncthreads();
            }
            // the counters of other items take the place of `cand`
            for (int i = tid; i < kKeepRanks / 4; i += NT) c4[i] = make_uint4(0u, 0u, 0u, 0u);
        } else {
            const bool one = k1 - k0 <= NT;  // every member has a thread
            const bool table = F.ranges > 1;
            // position of the next range's first candidate in this thread's list
            int32_t ahead = 0;
            if (mem.row >= 0) ahead = A.bnd[mem.row + (F.base + p0 * F.width) / kFlatBlock];
            for (int32_t p = p0; p < p1; ++p) {
                const int32_t lo = F.base + p * F.width;
                const int32_t hi = (int32_t)min((int64_t)nend, (int64_t)lo + F.width);
                const uint32_t span = (uint32_t)(hi - lo);
                const int32_t blk0 = lo / kFlatBlock;
                const int32_t blk1 =
                    min(blocks, (int32_t)(((int64_t)hi + kFlatBlock - 1) / kFlatBlock));
                ++passes;
                for (int32_t kb = k0; kb < k1; kb += NT) {
                    // the part of each member's list in the range
                    if (!one) {
                        mem = load_member(kb + tid, k1);
                        load_list(mem, table);
                        if (mem.row >= 0) ahead = A.bnd[mem.row + blk0];
                    }
                    int32_t b = mem.st, e = mem.en;
                    if (mem.row >= 0) {
                        b = max(b, ahead);
                        ahead = A.bnd[mem.row + blk1];
                        // the table of a list out of order (SLINE_SKIP_VALIDATE) has
                        // entries that were never written
                        e = min(e, ahead);
                    }
                    map.number(b, max(e - b, 0));
                    for (int32_t w0 = 0; w0 < map.total; w0 += kFlatChunks * kWave) {
                        const auto run = map.window(w0);
                        if (run.nc > 0) {
                            // the next chunks are loaded while these are counted;
                            // the last ones in as many as there are
                            int32_t u = 0;
                            if (run.nc >= kLoad) {
                                int32_t ja[kLoad], jb[kLoad];
                                map.load(A.itmS, run, 0, ja);
                                for (;;) {
                                    u += kLoad;
                                    if (u + kLoad > run.nc) {
                                        count(ja, lo, span);
                                        break;
                                    }
                                    map.load(A.itmS, run, u, jb);
                                    count(ja, lo, span);
                                    u += kLoad;
                                    if (u + kLoad > run.nc) {
                                        count(jb, lo, span);
                                        break;
                                    }
                                    map.load(A.itmS, run, u, ja);
                                    count(jb, lo, span);
                                }
                            }
                            const int32_t last = run.nc - u;
                            if (last > 4) {
                                int32_t j[8];
                                map.load(A.itmS, run, u, j);
                                count(j, lo, span);
                            } else if (last > 2) {
                                int32_t j[4];
                                map.load(A.itmS, run, u, j);
                                count(j, lo, span);
                            } else if (last > 0) {
                                int32_t j[2];
                                map.load(A.itmS, run, u, j);
                                count(j, lo, span);
                            }
                        }
                        if (!map.narrow) __syncthreads();  // the map is used again
                    }
                    if (!map.narrow && map.total == 0) __syncthreads();
                }
                if (lane == 0 && hits) atomicAdd(&sh_hits, hits);
                hits = 0;
                __syncthreads();
                const int32_t nq = (int32_t)((span + 127u) >> 7), qpw = (nq + NW - 1) / NW;
                const int32_t q0 = min(nq, wid * qpw), q1 = min(nq, q0 + qpw);
                const int32_t found = sh_hits;  // written before the last barrier
                if (found > 0) {
                    emit(lo, found, q0, q1);
                    produced += found;
                }
                // a quad's counters are 1 << lb times four words
                for (int32_t i = (q0 << lb) + lane; i < (q1 << lb); i += kWave)
                    c4[i] = make_uint4(0u, 0u, 0u, 0u);
                __syncthreads();
            }
        }
        if (!skip && !FILL && tid == 0) {
            A.task_cnt[t] = produced;
            my_pairs += produced;
        }
        turn ^= 1;
        if (tid == 0) sh_task[turn] = r2;
        __syncthreads();
        r = r1;
        r1 = sh_task[turn];
        cur = nxt;
    }
    if (tid == 0 && A.passes && !FILL) {
        unsigned long long *wk = stat_row(A);
        if (passes) atomicAdd(&wk[0], (unsigned long long)passes);
        if (my_nnz) atomicAdd(&wk[1], (unsigned long long)my_nnz);
        if (my_wedges) atomicAdd(&wk[2], (unsigned long long)my_wedges);
        if (my_pairs) atomicAdd(&wk[3], (unsigned long long)my_pairs);
    }
}

}  // namespace

hipError_t launch_flat_bounds(hipStream_t st, const int32_t *ptrS, const int32_t *itmS, int32_t M,
                              const int32_t *crank, int32_t N, int64_t nnz, int32_t *bnd,
                              int32_t *long_lists, int32_t *n_long, const int32_t *n_flat,
                              const int32_t *err) {
    if (M <= 0 || N <= kFlatBlock) return hipSuccess;
    const int32_t per = lanes_per_wave(M);
    const int64_t g = std::min<int64_t>(((int64_t)M + 4 * per - 1) / (4 * per), 4096);
    k_flat_bounds<<<(unsigned)g, 256, 0, st>>>(ptrS, itmS, M, crank, N, per, bnd, long_lists, n_long,
                                               n_flat, err);
    const hipError_t e = hipGetLastError();
    const int64_t most = nnz / kMidList;  // lists of more than kMidList entries
    if (e != hipSuccess || most == 0) return e;
    k_flat_long<<<(unsigned)std::min<int64_t>((most + 3) / 4, 1024), 256, 0, st>>>(
        ptrS, itmS, crank, N, bnd, long_lists, n_long);
    return hipGetLastError();
}

hipError_t launch_count_flat(hipStream_t st, const CountArgs &A) {
    // A.s is the least s of a batch; only items with s = 1 keep their wedges
    const bool fill = A.mode == kModeFill, ones = A.s <= 1;
    auto *const count = fill ? (ones ? k_count_flat<true, true> : k_count_flat<true, false>)
                             : (ones ? k_count_flat<false, true> : k_count_flat<false, false>);
    count<<<A.grid[kKindFlat], kFlatThreads, 0, st>>>(A);
    return hipGetLastError();
}

}  // namespace sl
