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

__device__ __forceinline__ void use_ranks(CountArgs &A) {
    A.crank = ranks_or_null(A.crank, A.N);
    if (!A.crank) A.orig = nullptr;
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

__device__ __forceinline__ int32_t lane63(int32_t v) { return __builtin_amdgcn_readlane(v, 63); }

__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// The wedges of an item (or of one range of it), numbered 0, 1, ... over its
// members' list parts one after the other, one part per thread at most.  A bit
// per wedge marks where a part begins: a wave reads the bits of 64 wedges, and
// the count of the bits up to a lane's own is that lane's part.  Every lane of
// every load then has a wedge, whatever the parts' lengths are.
template <int NT, int CHUNKS>
struct WedgeMap {
    static constexpr int NW = NT / kWave;
    int32_t *adj;     // NT: list position less wedge number, per part that has wedges
    uint64_t *marks;  // CHUNKS, all zero when a window is marked
    int32_t *wlen, *wpart;  // NW each
    int32_t *before0;

    // Number the parts: this thread's is [b, b + len).  One barrier inside.
    __device__ __forceinline__ void number(int32_t b, int32_t len, int32_t &off, int32_t &rank,
                                           int32_t &total) const {
        const int32_t incl = wave_incl(len);
        const uint64_t has = __ballot(len > 0);
        off = incl - len;
        rank = (int32_t)lanes_below(has);
        total = lane63(incl);
        if (NW > 1) {
            const int wid = wave_id();
            if (lane_id() == 0) {
                wlen[wid] = total;
                wpart[wid] = __popcll(has);
            }
            __syncthreads();
            total = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (w < wid) {
                    off += wlen[w];
                    rank += wpart[w];
                }
                total += wlen[w];
            }
        }
        if (len > 0) adj[rank] = b - off;
    }
    // Mark the parts of the window that starts at wedge w0.
    __device__ __forceinline__ void mark(int32_t w0, int32_t off, int32_t len, int32_t rank) const {
        const int32_t in = off - w0;
        if (len > 0 && in >= 0 && in < CHUNKS * kWave)
            atomicOr(reinterpret_cast<uint32_t *>(marks) + (in >> 5), 1u << (in & 31));
        // parts that begin before the window
        if (len > 0 && in <= 0 && in + len > 0) *before0 = in < 0 ? rank : rank - 1;
    }
    // Parts that begin before chunk c0 of the window.
    __device__ __forceinline__ int32_t parts_before(int32_t c0) const {
        int32_t n = 0;
        if (c0 > 0) {
#pragma unroll
            for (int i = 0; i < (CHUNKS + kWave - 1) / kWave; ++i) {
                const int c = i * kWave + lane_id();
                if (c < c0) n += __popcll(marks[c]);
            }
            n = lane63(wave_incl(n));
        }
        return uniform(*before0) + n;
    }
    // The candidate of this lane's wedge of chunk c (ok: it has one), and the
    // parts so far.
    __device__ __forceinline__ int32_t wedge(const int32_t *itmS, int32_t w0, int32_t c, bool ok,
                                             int32_t &before) const {
        const uint64_t raw = marks[c];
        const uint64_t m = ((uint64_t)(uint32_t)uniform((int32_t)(raw >> 32)) << 32) |
                           (uint32_t)uniform((int32_t)raw);
        const int32_t q = before + (int32_t)(m & 1u) + (int32_t)lanes_below(m >> 1);
        before += __popcll(m);
        return ok ? itmS[adj[q] + w0 + c * kWave + lane_id()] : -1;
    }
};

}  // namespace

}  // namespace sl
