// Batched builds: many hypergraphs, each with its own s and role (primal or
// dual), counted in one pass of the plain pipeline.
//
// The graphs are independent, so their items can share one id space: graph
// g's items take the ids [ibase_g, ibase_g + N_g) and its members the ids
// [mbase_g, mbase_g + M_g).  Two items of different graphs share no member,
// so the combined L_s (each item compared with its own graph's s) is the
// disjoint union of the graphs' L_s, and sorting by (a, b) keeps every
// graph's pairs contiguous.  The kernels here build the combined item CSR
// (checking every caller CSR on the way), give every item its graph's s,
// and hand the combined result back per graph: directly, when the library
// allocates the results (the fill writes each pair into its graph's arrays),
// or by splitting a combined result into caller buffers.
//
// A dual graph's items are its vertices: their member lists are the rows of
// H_g^T, built by transposing XD, the row concatenation of all dual graphs'
// H_g (columns shifted by vdbase_g so the graphs' vertices do not collide).
#include <algorithm>

#include "sline_internal.h"

namespace sl {

namespace {

inline int grid_for(int64_t work, int per_block, int cap = 1 << 20) {
    const int64_t g = (work + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// last g with base[g] <= x, for base ascending with base[0] = 0 <= x
template <typename T>
__device__ __forceinline__ int32_t find_graph(const T *base, int32_t G, int64_t x) {
    int32_t lo = 0, hi = G;  // base[lo] <= x < base[hi] (base[G] = total)
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (base[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The graph of x, where `first` is the same in every lane of the wave and not
// above x: one search for the wave, by scalar loads, and only lanes with an x
// in a later graph search by themselves.  G: base[G] = total.
template <typename T>
__device__ __forceinline__ int32_t wave_graph(const T *base, int32_t G, int64_t first, int64_t x) {
    const int32_t g = __builtin_amdgcn_readfirstlane(find_graph(base, G, first));
    return x < base[g + 1] ? g : find_graph(base, G, x);
}

// A value of 64 bits that is the same in every lane of the wave, in scalar registers.
__device__ __forceinline__ int64_t wave_first(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Per graph: nnz (row_ptr[m]) and the row_ptr[0] == 0 check.
__global__ void k_batch_nnz(const BatchGraph *gr, int32_t G, int64_t *nnz, int32_t *err) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    const BatchGraph d = gr[g];
    int64_t z = 0;
    if (d.m > 0) {
        if (d.rp[0] != 0) atomicOr(err, kErrRowPtr0);
        z = d.rp[d.m];
    }
    nnz[g] = z;
}

// Entries k, k + step, .. of row r of XD, [rb, re) in its graph d.
__device__ __forceinline__ void concat_row(const BatchGraph *gr, int64_t r, int32_t k, int32_t step,
                                           int32_t rb, int32_t re, int32_t *xcol, int32_t *xrow,
                                           int32_t &bad) {
    const BatchGraph d = *gr;
    for (; k < re; k += step) {
        const int32_t v = d.col[k], before = d.col[k > rb ? k - 1 : k];
        const bool in = v >= 0 && v < d.n;
        if (!in) bad |= kErrColRange;
        if (k > rb && before >= v) bad |= kErrColOrder;
        const int64_t o = d.dzbase + k;
        xcol[o] = in ? (int32_t)(d.vdbase + v) : 0;
        xrow[o] = (int32_t)r;
    }
}

// Rows of XD (the dual graphs' rows, in graph order): columns shifted by
// vdbase and the row id of every entry (what the transpose reads); range and
// order checks.  A wave takes 64 rows, or fewer if that leaves waves idle: those of up
// to kShortRow entries a lane each, then those of up to kMidRow in turn; longer
// ones go to a list, of which
// every wave of a second kernel takes one (64 such rows in turn would keep the
// whole batch waiting: 100 rows of 20,000 entries took 5.6 ms, and take 0.11 so).
// Bounds on latency (a row's graph, its bounds, its entries); a wave per row, which
// searched the graph for each, took 0.72 ms for 64 graphs of 40,000 rows in the
// mean, this takes 0.18.
constexpr int kShortRow = 16;
constexpr int kMidRow = 256;

__global__ __launch_bounds__(256) void k_batch_concat(const BatchGraph *gr, const int32_t *dual_ids,
                                                      const int64_t *dbase, int32_t GD, int64_t E,
                                                      int32_t per, int32_t *xcol, int32_t *xrow,
                                                      int32_t *long_rows, int32_t room,
                                                      int32_t *n_long, int32_t *err) {
    if (*err & kErrPlanShape) return;  // a replayed plan keeps its last lists
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    int32_t bad = 0;
    for (int64_t e0 = wave_first(wave * per); e0 < E; e0 += nwaves * per) {
        const int64_t e = e0 + lane;
        int32_t b = 0, en = 0, q = 0;
        if (lane < per && e < E) {
            q = wave_graph(dbase, GD, e0, e);
            const BatchGraph *d = gr + dual_ids[q];
            const int32_t *rp = d->rp + (e - dbase[q]);
            b = rp[0];
            en = rp[1];
            // a row outside [0, nnz) is reported and never read (its entries of
            // XD stay zero, so later kernels index safely until the error returns)
            if (b < 0 || en < b || en > d->nnz) {
                bad |= kErrRowPtrOrder;
                b = en = 0;
            }
        }
        const bool far = en - b > kMidRow;
        if (const uint64_t m = __ballot(far)) {
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(n_long, (int32_t)__popcll(m));
            at = __builtin_amdgcn_readfirstlane(at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            // rows that overlap, which another row's bounds give away, may be
            // more than there is room for
            if (far && at < room) long_rows[at] = (int32_t)e;
            if (far) b = en;
        }
        const bool longer = en - b > kShortRow;
        if (en > b && !longer) concat_row(gr + dual_ids[q], e, b, 1, b, en, xcol, xrow, bad);
        for (uint64_t m = __ballot(longer); m; m &= m - 1) {
            const int src = __builtin_ctzll(m);
            const int32_t rb = __shfl(b, src), re = __shfl(en, src);
            concat_row(gr + dual_ids[__shfl(q, src)], e0 + src, rb + lane, kWave, rb, re, xcol, xrow,
                       bad);
        }
    }
    if (bad) atomicOr(err, bad);
}

__global__ __launch_bounds__(256) void k_batch_long(const BatchGraph *gr, const int32_t *dual_ids,
                                                    const int64_t *dbase, int32_t GD,
                                                    const int32_t *long_rows, int32_t room,
                                                    const int32_t *n_long, int32_t *xcol,
                                                    int32_t *xrow, int32_t *err) {
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    const int32_t n = min(*n_long, room);
    int32_t bad = 0;
    for (int64_t i = wave_first(wave); i < n; i += nwaves) {
        const int32_t e = long_rows[i], q = find_graph(dbase, GD, e);
        const BatchGraph *d = gr + dual_ids[q];
        const int32_t *rp = d->rp + (e - dbase[q]);
        const int32_t b = rp[0], en = rp[1];
        concat_row(d, e, b + lane_id(), kWave, b, en, xcol, xrow, bad);
    }
    if (bad) atomicOr(err, bad);
}

// One thread per combined item: its row length, its graph's s and the end of
// its graph's items (candidates of an item never lie beyond it).
__global__ void k_batch_len(const BatchGraph *gr, const int64_t *ibase, int32_t G, int64_t NI,
                            const int32_t *ptrT, int32_t *len, int32_t *s_item, int32_t *item_end,
                            int32_t *err) {
    if (*err & kErrPlanShape) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < NI;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = wave_graph(ibase, G, wave_first(i - lane_id()), i);
        const BatchGraph d = gr[g];
        const int32_t loc = (int32_t)(i - ibase[g]);
        int32_t l;
        if (d.dual) {
            const int64_t r = d.vdbase + loc;
            l = ptrT[r + 1] - ptrT[r];
        } else {
            const int32_t b = d.rp[loc], en = d.rp[loc + 1];
            l = en - b;
            if (b < 0 || en < b || en > d.nnz) {
                atomicOr(err, kErrRowPtrOrder);
                l = 0;
            }
            // members: the range is checked per incidence by k_batch_rows,
            // the order within each row on the combined lists (the combined
            // member ids of a primal graph keep its members' order)
        }
        len[i] = l;
        s_item[i] = d.s;
        item_end[i] = (int32_t)ibase[g + 1];
    }
}

// First combined incidence of every graph: zb[g] = ptrC[ibase[g]], g = 0..G.
__global__ void k_batch_zbase(const int64_t *ibase, int32_t G, const int32_t *ptrC, int32_t *zb) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g <= G) zb[g] = ptrC[ibase[g]];
}

// Combined incidences z.  Graph g's incidences are the contiguous range
// [zb[g], zb[g + 1]) in graph order: a primal graph's are its col array (rows
// checked by k_batch_len), shifted to the combined member ids; a dual graph's
// are its block of XD^T (rows of its vertices), whose entries are combined row
// ids of XD turned into member ids.  A wave takes kWaveEntries of them, as its search
// for the first one's graph is a chain of loads (3.7*10^7 incidences of 128
// graphs took 0.33 ms with a search for each 64, and take 0.10 so).
constexpr int kWaveEntries = 1024;

__global__ __launch_bounds__(256) void k_batch_rows(const BatchGraph *gr, const int32_t *zb,
                                                    int32_t G, int64_t ZT, const int32_t *ptrT,
                                                    const int32_t *colT, int32_t *memC,
                                                    int32_t *err) {
    if (*err & kErrPlanShape) return;
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    bool bad = false;
    for (int64_t z0 = wave_first(wave * kWaveEntries); z0 < ZT; z0 += nwaves * kWaveEntries) {
        const int64_t z1 = min(z0 + kWaveEntries, ZT);
        int32_t g = __builtin_amdgcn_readfirstlane(find_graph(zb, G, z0));
        for (int64_t at = z0; at < z1; ++g) {
            if (g >= G) {
                // rows with bad bounds (reported by k_batch_len) have no
                // entries, so the graphs may end before ZT: the rest gets a
                // member that later kernels can index by
                for (int64_t z = at + lane; z < z1; z += kWave) memC[z] = 0;
                break;
            }
            const BatchGraph d = gr[g];
            const int64_t first = zb[g], end = min((int64_t)zb[g + 1], z1);
            const int32_t *from = d.dual ? colT + ptrT[d.vdbase] : d.col;
            const int32_t shift = d.dual ? (int32_t)(d.mbase - d.dbase) : (int32_t)d.mbase;
#pragma unroll 4
            for (int64_t z = at + lane; z < end; z += kWave) {
                const int64_t k = z - first;
                // a primal graph with bad row bounds (reported by k_batch_len)
                // may map past its col
                int32_t v = d.dual || k < d.nnz ? from[k] : 0;
                if (!d.dual && (v < 0 || v >= d.n)) {
                    bad = true;
                    v = 0;
                }
                memC[z] = v + shift;
            }
            at = end > at ? end : at;
        }
    }
    if (bad) atomicOr(err, kErrColRange);
}

// One thread per graph: first pair of the graph in the combined result
// (items of graph g are [ibase_g, ibase_{g+1}); `a` is sorted).
__global__ void k_batch_bounds(const int64_t *ibase, int32_t G, const int32_t *a, int64_t P,
                               int64_t *off) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g > G) return;
    if (g == G) {
        off[G] = P;
        return;
    }
    const int64_t key = ibase[g];
    int64_t lo = 0, hi = P;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    off[g] = lo;
}

// Grid-stride over the combined pairs: each goes to its graph's output with
// the graph's item base taken off both ids.
__global__ void k_batch_split(const int64_t *ibase, const int64_t *off, int32_t G,
                              const int32_t *a, const int32_t *b, const int32_t *w, int64_t P,
                              int32_t *const *oa, int32_t *const *ob, int32_t *const *ow) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = wave_graph(off, G, wave_first(k - lane_id()), k);
        const int64_t r = k - off[g];
        const int32_t base = (int32_t)ibase[g];
        oa[g][r] = a[k] - base;
        ob[g][r] = b[k] - base;
        if (w && ow[g]) ow[g][r] = w[k];
    }
}

// One thread per graph boundary g = 0..G: the first pair of graph g.
__global__ void k_batch_graph_off(const int32_t *task_item, int32_t T, const int64_t *task_off,
                                  const int64_t *g_ibase, int32_t G, int64_t *g_off,
                                  const int64_t *T_dev) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g > G) return;
    if (T_dev) T = (int32_t)min(*T_dev, (int64_t)T);
    const int64_t first = g_ibase[g];
    int32_t lo = 0, hi = T;  // first task with task_item >= first
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((int64_t)task_item[mid] < first) lo = mid + 1;
        else hi = mid;
    }
    g_off[g] = task_off[lo];
}

// Replayed plans: the caller's row_ptr must still start at 0 and end at the
// nnz the plan was sized for (every later kernel bounds its reads by it).
__global__ void k_plan_check_shape(const BatchGraph *gr, int32_t G, int32_t *err) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    const BatchGraph d = gr[g];
    if (d.m > 0 && (d.rp[0] != 0 || (int64_t)d.rp[d.m] != d.nnz)) atomicOr(err, kErrPlanShape);
}

__global__ void k_plan_guard(const int64_t *value, int64_t cap, int32_t bit, int32_t *err) {
    if (threadIdx.x == 0 && *value > cap) atomicOr(err, bit);
}

}  // namespace

hipError_t launch_batch_graph_off(hipStream_t st, const int32_t *task_item, int32_t n_tasks,
                                  const int64_t *task_off, const int64_t *g_ibase, int32_t G,
                                  int64_t *g_off, const int64_t *n_tasks_dev) {
    if (G <= 0) return hipSuccess;
    k_batch_graph_off<<<grid_for((int64_t)G + 1, 256), 256, 0, st>>>(task_item, n_tasks, task_off,
                                                                     g_ibase, G, g_off, n_tasks_dev);
    return hipGetLastError();
}

hipError_t launch_plan_check_shape(hipStream_t st, const BatchGraph *gr, int32_t G, int32_t *err) {
    if (G <= 0) return hipSuccess;
    k_plan_check_shape<<<grid_for(G, 256), 256, 0, st>>>(gr, G, err);
    return hipGetLastError();
}

hipError_t launch_plan_guard(hipStream_t st, const int64_t *value, int64_t cap, int32_t bit,
                             int32_t *err) {
    k_plan_guard<<<1, kWave, 0, st>>>(value, cap, bit, err);
    return hipGetLastError();
}

hipError_t launch_batch_nnz(hipStream_t st, const BatchGraph *gr, int32_t G, int64_t *nnz,
                            int32_t *err) {
    if (G <= 0) return hipSuccess;
    k_batch_nnz<<<grid_for(G, 256), 256, 0, st>>>(gr, G, nnz, err);
    return hipGetLastError();
}

hipError_t launch_batch_concat(hipStream_t st, const BatchGraph *gr, const int32_t *dual_ids,
                               const int64_t *dbase, int32_t GD, int64_t E, int64_t ZD,
                               int32_t *xcol, int32_t *xrow, int32_t *long_rows, int32_t *n_long,
                               int32_t *err) {
    if (E <= 0) return hipSuccess;
    const int32_t room = (int32_t)(ZD / kMidRow);  // rows of more than kMidRow entries
    const int32_t per = lanes_per_wave(E);
    k_batch_concat<<<grid_for(E, 4 * per, 65536), 256, 0, st>>>(gr, dual_ids, dbase, GD, E, per, xcol,
                                                                xrow, long_rows, room, n_long, err);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || room == 0) return e;
    k_batch_long<<<grid_for(room, 4, 2048), 256, 0, st>>>(gr, dual_ids, dbase, GD, long_rows, room,
                                                          n_long, xcol, xrow, err);
    return hipGetLastError();
}

hipError_t launch_batch_len(hipStream_t st, const BatchGraph *gr, const int64_t *ibase, int32_t G,
                            int64_t NI, const int32_t *ptrT, int32_t *len, int32_t *s_item,
                            int32_t *item_end, int32_t *err) {
    if (NI <= 0) return hipSuccess;
    k_batch_len<<<grid_for(NI, 256, 65536), 256, 0, st>>>(gr, ibase, G, NI, ptrT, len, s_item,
                                                          item_end, err);
    return hipGetLastError();
}

hipError_t launch_batch_rows(hipStream_t st, const BatchGraph *gr, const int64_t *ibase, int32_t G,
                             int64_t ZT, const int32_t *ptrT, const int32_t *colT,
                             const int32_t *ptrC, int32_t *zb, int32_t *memC, int32_t *err) {
    if (G <= 0) return hipSuccess;
    k_batch_zbase<<<grid_for((int64_t)G + 1, 256), 256, 0, st>>>(ibase, G, ptrC, zb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ZT <= 0) return e;
    k_batch_rows<<<grid_for(ZT, 4 * kWaveEntries, 65536), 256, 0, st>>>(gr, zb, G, ZT, ptrT, colT, memC, err);
    return hipGetLastError();
}

hipError_t launch_batch_bounds(hipStream_t st, const int64_t *ibase, int32_t G, const int32_t *a,
                               int64_t P, int64_t *off) {
    k_batch_bounds<<<grid_for((int64_t)G + 1, 256), 256, 0, st>>>(ibase, G, a, P, off);
    return hipGetLastError();
}

hipError_t launch_batch_split(hipStream_t st, const int64_t *ibase, const int64_t *off, int32_t G,
                              const int32_t *a, const int32_t *b, const int32_t *w, int64_t P,
                              int32_t *const *oa, int32_t *const *ob, int32_t *const *ow) {
    if (P <= 0) return hipSuccess;
    k_batch_split<<<grid_for(P, 256, 65536), 256, 0, st>>>(ibase, off, G, a, b, w, P, oa, ob, ow);
    return hipGetLastError();
}

}  // namespace sl
