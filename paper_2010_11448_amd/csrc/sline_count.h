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

__device__ __forceinline__ int32_t wave_total(int32_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Candidate numbers (see ranks_pay): a kernel drops crank and orig at its start
// when the build does not use ranks; a candidate's number is then its item's id.
__device__ __forceinline__ const int32_t *ranks_or_null(const int32_t *crank, int32_t N) {
    return crank && ranks_pay(crank[N], N) ? crank : nullptr;
}

__device__ __forceinline__ void use_ranks(CountArgs &A) {
    A.crank = ranks_or_null(A.crank, A.N);
    if (!A.crank) A.orig = nullptr;
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

// The item a candidate stands for.
__device__ __forceinline__ int32_t item_of(const int32_t *orig, int32_t cand) {
    return orig ? orig[cand] : cand;
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

// Stage mode, thread 0 of a workgroup: room for `total` pairs in the pool and
// `nrec` consecutive log records, taken from this workgroup's chunks (one
// global atomic per new chunk; records of a chunk left unused stay zero, i.e.
// empty).  Returns false if the pool or the log has no room left.
__device__ __forceinline__ bool stage_reserve(const CountArgs &A, uint64_t *pool_cur,
                                              int32_t *log_cur, int32_t total, int32_t nrec,
                                              uint64_t &off, int32_t &rec) {
    off = pool_cur[0];
    rec = 0;
    if (off + (uint64_t)total > pool_cur[1]) {
        const uint64_t size = max((uint64_t)total, (uint64_t)A.pool_chunk);
        off = atomicAdd(A.pool_head, (unsigned long long)size);
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
        const int32_t size = max(nrec, A.log_chunk);
        const int32_t r = atomicAdd(A.log_head, size);
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

}  // namespace

}  // namespace sl
