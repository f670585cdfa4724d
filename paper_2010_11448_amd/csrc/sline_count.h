// Device helpers shared by the counting kernels (sline_count.hip,
// sline_flat.hip).
#pragma once

#include "sline_internal.h"

namespace sl {

namespace {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
// Wave index inside the workgroup, as a wave-uniform (scalar) value.
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
}

template <typename T>
__device__ __forceinline__ T wave_total(T v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ void use_ranks(CountArgs &A) {
    A.crank = ranks_or_null(A.crank, A.N);
    if (!A.crank) A.orig = nullptr;
}

// The item a candidate stands for.  (A row that lists a member twice, let in by
// SLINE_SKIP_VALIDATE, can leave candidates that are none.)
__device__ __forceinline__ int32_t item_of(const CountArgs &A, int32_t cand) {
    return A.orig ? A.orig[min((uint32_t)cand, (uint32_t)A.N - 1u)] : cand;
}

// Where the pairs of item `item` at combined output position `pos` go: the
// single output, or (batches written per graph) the arrays of the item's
// graph at the position inside it, ids to be written less `shift`.
struct OutDst {
    int32_t *a, *b, *w;
    int64_t base;
    int32_t shift;
};

__device__ __forceinline__ OutDst out_dst(const CountArgs &A, int32_t item, int64_t pos) {
    OutDst d{A.out_a, A.out_b, A.out_w, pos, 0};
    const int32_t G = A.n_graphs;
    if (G > 0) {
        int32_t lo = 0, hi = G;  // g_ibase[lo] <= item < g_ibase[hi]
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (A.g_ibase[mid] <= item) lo = mid;
            else hi = mid;
        }
        d.shift = (int32_t)A.g_ibase[lo];
        if (A.g_out) {
            d.a = A.g_out[lo];
            d.b = A.g_out[G + lo];
            d.w = A.g_out[2 * G + lo];
            d.base = pos - A.g_off[lo];
        }
    }
    return d;
}

// Sum over the wave of n (0 <= n < 32) and the sum over the lanes below this
// one, from the ballots of its bits (nb = bits of n that can be set).
__device__ __forceinline__ void wave_bits_prefix(int32_t n, int nb, int32_t &before, int32_t &step) {
    before = 0;
    step = 0;
    for (int b = 0; b < nb; ++b) {
        const uint64_t m = __ballot((n >> b) & 1);
        before += (int32_t)lanes_below(m) << b;
        step += (int32_t)__popcll(m) << b;
    }
}

// Thread 0 of a workgroup of a kind's kernel, at its start: its own first chunks
// of the pool and the log, if it has some (a small build needs no others, and
// so no atomics on the heads).
__device__ __forceinline__ void stage_begin(const CountArgs &A, int kind, uint64_t *pool_cur,
                                            int32_t *log_cur) {
    const bool own = A.mode == kModeStage && A.pool_own > 0;
    pool_cur[0] = pool_cur[1] = 0;
    log_cur[0] = log_cur[1] = 0;
    pool_cur[2] = (uint64_t)A.pool_chunk[kind];
    log_cur[2] = A.log_chunk[kind];
    if (own) {
        pool_cur[0] = (uint64_t)A.pool_first[kind] + (uint64_t)blockIdx.x * pool_cur[2];
        pool_cur[1] = pool_cur[0] + pool_cur[2];
        log_cur[0] = A.log_first[kind] + (int32_t)blockIdx.x * log_cur[2];
        log_cur[1] = log_cur[0] + log_cur[2];
    }
}

// The row of A.passes a workgroup adds to.
__device__ __forceinline__ unsigned long long *stat_row(const CountArgs &A) {
    return (unsigned long long *)A.passes + (blockIdx.x % kSumRows) * kStatCols;
}

// Stage mode, thread 0 of a workgroup: room for `total` pairs in the pool and
// `nrec` consecutive log records, taken from this workgroup's chunks (pool_cur and
// log_cur: next, end and size of a chunk, see stage_begin; one
// global atomic per new chunk; records of a chunk left unused stay zero, i.e.
// empty).  Returns false if the pool or the log has no room left.
__device__ __forceinline__ bool stage_reserve(const CountArgs &A, uint64_t *pool_cur,
                                              int32_t *log_cur, int32_t total, int32_t nrec,
                                              uint64_t &off, int32_t &rec) {
    off = pool_cur[0];
    rec = 0;
    if (off + (uint64_t)total > pool_cur[1]) {
        const uint64_t size = max((uint64_t)total, pool_cur[2]);
        off = (uint64_t)A.pool_own + atomicAdd(A.pool_head, (unsigned long long)size);
        if (off + size <= (uint64_t)A.pool_cap) {
            pool_cur[1] = off + size;
        } else if (off + (uint64_t)total <= (uint64_t)A.pool_cap) {
            pool_cur[1] = (uint64_t)A.pool_cap;
        } else {
            pool_cur[1] = 0;
            return false;
        }
    }
    pool_cur[0] = off + (uint64_t)total;
    if (log_cur[0] + nrec > log_cur[1]) {
        const int32_t size = max(nrec, log_cur[2]);
        const int32_t r = A.log_own + atomicAdd(A.log_head, size);
        log_cur[0] = r;
        log_cur[1] = (int32_t)min((int64_t)r + size, (int64_t)A.log_cap);
    }
    rec = log_cur[0];
    if (rec + nrec > log_cur[1]) return false;
    log_cur[0] = rec + nrec;
    return true;
}

// A counting launch with nothing to do: the plan's bounds were exceeded (or
// its input is malformed), or a fill pass that only recounts tasks flagged in
// `need` while none is flagged.
__device__ __forceinline__ bool count_idle(const CountArgs &A) {
    if (A.abort && *A.abort != 0) return true;
    return A.mode == kModeFill && A.need && A.need_count && *A.need_count == 0;
}

// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ int32_t wave_incl(int32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// The least of the lanes' values, in every lane.
__device__ __forceinline__ int32_t wave_least(int32_t v) {
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int32_t lane63(int32_t v) { return __builtin_amdgcn_readlane(v, 63); }

__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// The wedges of an item (or of one range of it), numbered 0, 1, ... over its
// members' list parts one after the other.  A bit per wedge marks where a part
// begins: the count of the bits up to a wedge's own is its part.  Every lane of
// every load then has a wedge, whatever the parts' lengths are.
//
// A window of CHUNKS * 64 wedges is shared out to the waves, a run of 64-wedge
// chunks each; a lane holds the bits of one chunk of its wave's run, so taking
// a chunk reads no memory but the part's position.  With up to 64 parts
// (narrow) every wave numbers all of them by itself, in its own area: no
// barrier.  With more, each thread has one part and two barriers order them.
template <int NT, int CHUNKS>
struct WedgeMap {
    static constexpr int NW = NT / kWave, PER = CHUNKS / NW;
    static_assert(PER <= kWave && PER * NW == CHUNKS, "a lane per chunk of a run");

    int32_t *adj_all;     // NT: 4 * (list position less wedge number), per part that has wedges
    uint32_t *marks_all;  // 2 * CHUNKS words, all zero between windows
    int32_t *sh;          // 3 * NW
    bool narrow;
    int32_t *adj;
    int32_t off, len, rank, total;  // this thread's part, and all wedges

    // a run: the bits of chunk c0 + lane but the first (bit i: a part begins at
    // wedge i + 1), the part of its first wedge and the byte offset of that one's
    // list entry; the chunks that lie in one part (bit per chunk), chunks and
    // wedges of the run
    struct Run {
        uint32_t lo, hi;
        int32_t base, pos;
        uint64_t whole;
        int32_t nc, t0, n;
    };

    // Which member this thread looks after: narrow maps have one per lane.
    __device__ __forceinline__ int member() const { return narrow ? lane_id() : (int)threadIdx.x; }

    // Number the parts: this thread's is [b, b + n).
    __device__ __forceinline__ void number(int32_t b, int32_t n) {
        len = n;
        const int32_t incl = wave_incl(n);
        const uint64_t has = __ballot(n > 0);
        off = incl - n;
        rank = (int32_t)lanes_below(has);
        total = lane63(incl);
        adj = adj_all;
        if (narrow) {
            adj += wave_id() * kWave;
        } else if (NW > 1) {
            const int wid = wave_id();
            if (lane_id() == 0) {
                sh[wid] = total;
                sh[NW + wid] = __popcll(has);
            }
            __syncthreads();
            total = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int32_t l = uniform(sh[w]), c = uniform(sh[NW + w]);
                off += w < wid ? l : 0;
                rank += w < wid ? c : 0;
                total += l;
            }
        }
        if (n > 0) adj[rank] = (int32_t)((uint32_t)(b - off) << 2);
    }

    // The wave's run of the window that starts at wedge w0 < total.
    __device__ __forceinline__ Run window(int32_t w0) {
        const int lane = lane_id(), wid = wave_id();
        const int32_t n = min(total - w0, CHUNKS * kWave);
        const int32_t nch = (n + kWave - 1) / kWave, cpw = (nch + NW - 1) / NW;
        const int32_t c0 = min(nch, wid * cpw);
        Run r;
        r.nc = min(nch, c0 + cpw) - c0;
        r.t0 = w0 + c0 * kWave;
        r.n = min(n - c0 * kWave, r.nc * kWave);
        uint32_t *marks = marks_all;
        int32_t before;
        if (narrow) {
            marks += wid * 2 * PER;
            const int32_t in = off - r.t0;
            if (len > 0 && in >= 0 && in < r.n) atomicOr(marks + (in >> 5), 1u << (in & 31));
            before = (int32_t)__popcll(__ballot(len > 0 && in < 0)) - 1;
        } else {
            const int32_t in = off - w0;
            if (len > 0 && in >= 0 && in < n) atomicOr(marks + (in >> 5), 1u << (in & 31));
            // parts up to the wedge before each run
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int32_t d = in - w * cpw * kWave;
                if (len > 0 && d <= 0 && d + len > 0) sh[2 * NW + w] = d < 0 ? rank : rank - 1;
            }
            __syncthreads();
            marks += 2 * c0;
            before = uniform(sh[2 * NW + wid]);
        }
        __builtin_amdgcn_wave_barrier();
        r.lo = r.hi = 0u;
        if (lane < r.nc) {
            uint2 *const m = reinterpret_cast<uint2 *>(marks) + lane;
            const uint2 v = *m;
            *m = make_uint2(0u, 0u);
            r.lo = v.x;
            r.hi = v.y;
        }
        const int32_t pop = __popc(r.lo) + __popc(r.hi);
        r.base = before + wave_incl(pop) - pop + (int32_t)(r.lo & 1u);
        r.lo = (r.lo >> 1) | (r.hi << 31);
        r.hi >>= 1;
        r.pos = 0;
        if (lane < r.nc) r.pos = adj[r.base] + ((r.t0 + lane * kWave) << 2);
        r.whole = __ballot((r.lo | r.hi) == 0u);
        return r;
    }

    // Byte offsets of the list entries of chunk u < nc of the run (a lane past
    // the run's end gets its last wedge's).
    __device__ __forceinline__ uint32_t position(const Run &r, int32_t u, bool full) const {
        if (full && ((r.whole >> u) & 1u))
            return (uint32_t)__builtin_amdgcn_readlane(r.pos, u) + ((uint32_t)lane_id() << 2);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)r.lo, u);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)r.hi, u);
        const uint32_t q = __builtin_amdgcn_mbcnt_hi(
            hi, __builtin_amdgcn_mbcnt_lo(lo, (uint32_t)__builtin_amdgcn_readlane(r.base, u)));
        const int32_t in = full ? u * kWave + lane_id() : min(u * kWave + lane_id(), r.n - 1);
        return (uint32_t)adj[q] + ((uint32_t)(r.t0 + in) << 2);
    }

    // A list entry; positions lie below 2^30, so a 32-bit offset reaches it.
    static __device__ __forceinline__ int32_t entry(const int32_t *itmS, uint32_t at) {
        return *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(itmS) + at);
    }

    // Candidates of chunks u0 .. u0 + K - 1 of the run, -1 past its end.
    template <int K>
    __device__ __forceinline__ void load(const int32_t *itmS, const Run &r, int32_t u0,
                                         int32_t (&j)[K]) const {
        uint32_t p[K];
        if ((u0 + K) * kWave <= r.n) {
#pragma unroll
            for (int v = 0; v < K; ++v) p[v] = position(r, u0 + v, true);
#pragma unroll
            for (int v = 0; v < K; ++v) j[v] = entry(itmS, p[v]);
        } else {
#pragma unroll
            for (int v = 0; v < K; ++v) p[v] = position(r, min(u0 + v, r.nc - 1), false);
#pragma unroll
            for (int v = 0; v < K; ++v) {
                j[v] = entry(itmS, p[v]);
                if ((u0 + v) * kWave + lane_id() >= r.n) j[v] = -1;
            }
        }
    }
};

}  // namespace

}  // namespace sl
