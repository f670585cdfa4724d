// Counting kernels of libsline for gfx950: for each kept item a, count the
// members it shares with every kept item b > a and emit the pairs with count
// >= s, sorted by b.
//
// Method (Sec. IV-B/IV-C): item a reaches candidate b only through a shared
// member v, by walking the kept items of N_s(v) that follow a (strictly upper
// triangle).  The paper's per-thread `visited` array becomes a counter table
// in LDS, so every candidate is counted once per shared member and its final
// count is the overlap w_ab itself.  Items smaller than s never appear
// (degree-based pruning: they are dropped from the member lists and from the
// task list).
//
// Work units: item a with W_a wedges is cut into P_a tasks covering equal
// sub-ranges of its candidate range (a, N); P_a = ceil(W_a / target), so every
// task carries about the same number of wedges.  A workgroup takes a group of
// up to `group_parts` consecutive tasks of one item and walks them in order,
// keeping for each member v the cursor into N_s(v) in a register: the walk of
// the first range starts at the back-pointer of (a, v) computed with W_a, and
// each range ends where the list reaches the range's upper bound, found by
// reading the list forward (no search).  Tasks are listed in (a, sub-range)
// order, and an exclusive scan of the per-task pair counts places each task's
// output directly in canonical (a, b) order.
//
// Table: one 32-bit LDS word per slot, 0 = empty, for a range [lo, hi):
//   * dense  (hi - lo <= slots): slot = j - lo, the word is the count;
//   * hashed (hi - lo  > slots): the word packs (j - lo + 1) above the low
//     `cb` bits, which hold the count (cb = bit length of |S_a|, so a count
//     never reaches the key field; ranges too wide for the key field are
//     split).  Slots form buckets of four words read with one 16-byte LDS
//     load.  Home bucket = (j - lo) * buckets / (hi - lo), one v_mul_hi_u32;
//     a candidate takes its home bucket or, when that is full, the next
//     bucket with room (no wrap-around; `pad` extra slots at the end).  The
//     map is monotone, so a bucket with a free slot separates smaller from
//     larger candidates: candidates can only be out of order inside a run of
//     full buckets ended by a non-full one (a cluster), and extraction ranks
//     each candidate against its cluster to write it to its final position.
//     A probe that runs off the table marks the range, which is then cleared
//     and split in halves (depth-first, left half first).
//
// Insertion cutoff (s > 1): the members flagged lookup-only (the s - 1
// longest lists of the item, at most kMaxLookup) walk after the others,
// behind a barrier, and only add to keys already in the table: a candidate
// whose overlap reaches s lies in at least one list that inserts it.
//
// Kernels: k_count_small (one wave per item with W_a <= small_max), k_count_tasks
// (one workgroup per task group), k_count_tiny (one lane per item), k_count_item
// (whole items of up to a few thousand wedges) and k_count_flat (sline_flat.hip: wedges
// dense in their candidate range).  Normally one counting pass
// stages every extracted range's (b, w) in a pool and logs where it goes;
// after the exclusive scan of the pairs per task, k_stage_copy moves each
// range to its task's offset, writing (a, b, w).  Tasks that found no room in
// the pool, or every task when no pool could be had, are counted again in a
// fill pass that writes at the task's offset directly.  In product mode
// (`full`, the SpGEMM companion) every b in [0, N) counts, a itself included.
#include <algorithm>
#include <type_traits>

#include "sline_count.h"

namespace sl {

namespace {

constexpr int kR = 8;        // member cursors per thread held in registers
constexpr int kPiece = 256;  // planned entries per piece of a long member run

// first index p in [lo, hi) with arr[p] >= key (arr ascending), hi if none
__device__ __forceinline__ int32_t lower_bound(const int32_t *arr, int32_t lo, int32_t hi,
                                               int32_t key) {
    while (lo < hi) {
        int32_t mid = lo + ((hi - lo) >> 1);
        if (arr[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

struct Range {
    int32_t lo;      // first candidate id
    int32_t hi;      // one past the last candidate id
    uint32_t span;   // hi - lo
    uint32_t mul;    // hashed: home bucket = mulhi(j - lo, mul); 0 = dense
    int32_t limit;   // words in use (home slots + pad when hashed; a multiple of 4)
    int32_t cb;      // hashed: count bits of a slot word
    uint32_t cmask;  // (1 << cb) - 1
    uint32_t psh;    // dense: 2^psh counters per word (4 x 8, 2 x 16 or 1 x 32 bits)
};

// Counters per table word, as a shift, for overlaps of up to 2^cb - 1: four
// 8-bit counters when the item has at most 255 members, two 16-bit ones up
// to 65535, else one.
__device__ __forceinline__ uint32_t pack_shift(int32_t cb) { return cb <= 8 ? 2u : cb <= 16 ? 1u : 0u; }

// Dense ranges (span <= slots << pack_shift(cb)) count candidate j in
// counter j - lo directly: candidate order is counter order, no hashing and
// no overflow (an overlap never exceeds the item's size).  Wider ranges hash.
__device__ __forceinline__ Range make_range(int32_t lo, int32_t hi, int32_t slots, int32_t pad,
                                            int32_t cb) {
    Range r;
    r.lo = lo;
    r.hi = hi;
    const int64_t span = (int64_t)hi - lo;
    r.span = (uint32_t)span;
    r.cb = cb;
    r.cmask = (1u << cb) - 1u;
    r.psh = pack_shift(cb);
    if (span <= ((int64_t)slots << r.psh)) {
        r.mul = 0;
        r.limit = (int32_t)((span + (1 << r.psh) - 1) >> r.psh);
    } else {
        r.psh = 0;
        r.mul = (uint32_t)(((uint64_t)(slots >> 2) << 32) / (uint64_t)span);
        r.limit = slots + pad;
    }
    return r;
}

// A hashed range whose ids do not fit the key field of a slot word.
__device__ __forceinline__ bool too_wide(const Range &R) {
    return R.mul != 0 && (uint64_t)R.span >= (1ull << (32 - R.cb));
}

// The free word a new key takes in a bucket read as (w0..w3): the first free
// one going round from word ws; 4 if the bucket is full.
__device__ __forceinline__ uint32_t free_word(uint32_t ws, uint32_t w0, uint32_t w1, uint32_t w2,
                                              uint32_t w3) {
    const uint32_t f = (w0 == 0u ? 1u : 0u) | (w1 == 0u ? 2u : 0u) | (w2 == 0u ? 4u : 0u) |
                       (w3 == 0u ? 8u : 0u);
    const uint32_t r = ((f | (f << 4)) >> ws) & 15u;
    return r ? ((ws + (uint32_t)__builtin_ctz(r)) & 3u) : 4u;
}

// Hashed insertion of a wedge with key field `tag`, starting at bucket b whose
// contents were read as q.  Returns false if the probe came to bucket nb.
__device__ __forceinline__ bool tab_probe(uint32_t *tab, const Range &R, uint32_t tag,
                                          uint32_t ws, int32_t b, int32_t nb, uint4 q) {
    const uint32_t hmask = ~R.cmask;
    const uint4 *t4 = reinterpret_cast<const uint4 *>(tab);
    for (;;) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        int32_t hit = -1;
#pragma unroll
        for (int i = 3; i >= 0; --i)
            if ((w[i] & hmask) == tag) hit = i;
        const uint32_t fw = free_word(ws, q.x, q.y, q.z, q.w);
        const int32_t empty = fw < 4u ? (int32_t)fw : -1;
        if (hit >= 0) {
            atomicAdd(&tab[4 * b + hit], 1u);
            return true;
        }
        if (empty >= 0) {
            const uint32_t old = atomicCAS(&tab[4 * b + empty], 0u, tag | 1u);
            if (old == 0u) return true;  // inserted with count 1
            if ((old & hmask) == tag) {
                atomicAdd(&tab[4 * b + empty], 1u);
                return true;
            }
            // another candidate took the slot: look at this bucket again
        } else if (++b >= nb) {
            return false;  // full bucket without the key: next bucket
        }
        q = t4[b];
    }
}

// Pick word i of a bucket (i in 0..3) without indexing registers dynamically.
__device__ __forceinline__ uint32_t pick4(int32_t i, uint32_t a0, uint32_t a1, uint32_t a2,
                                          uint32_t a3) {
    return i == 0 ? a0 : i == 1 ? a1 : i == 2 ? a2 : a3;
}

constexpr int32_t kAllProbes = 1 << 20;  // no limit: every bucket of a table

// Count up to four wedges (a candidate >= R.hi means none).  The four home
// buckets are read together; every wedge that finds its key there is counted
// with one atomic add and every new key is claimed with one compare-and-swap,
// all four swaps in flight before any result is looked at.  A new key takes
// the first free word going round from its start word, the quarter of its
// bucket's share of the range it falls in: neighbouring entries of a sorted
// list, inserted by neighbouring lanes at once, share a home bucket but
// mostly not a start word, so their swaps do not collide.  Words never become
// free again during a pass, so a key is found in its home bucket or, if that
// bucket was full when it came, in a later one, and a bucket with a free word
// ends any search.  Wedges whose home bucket is full, or whose free word was
// taken by another key meanwhile, finish in the probe loop, which gives up after
// `probes` buckets (the range is then split, as where the table ends).
__device__ __forceinline__ bool tab_add4(uint32_t *tab, uint32_t *spare, const Range &R,
                                         int32_t j0, int32_t j1, int32_t j2, int32_t j3,
                                         int32_t probes = kAllProbes) {
    // this lane's spare word: atomics with nothing to count go there, so the
    // atomics need no branches
    uint32_t *const dummy = spare + lane_id();
    const int32_t j[4] = {j0, j1, j2, j3};
    uint32_t x[4];
    bool in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = (uint32_t)(j[i] - R.lo);
        in[i] = j[i] < R.hi && x[i] < R.span;
    }
    if (R.mul == 0) {
        const uint32_t pm = (1u << R.psh) - 1u, bsh = 5u - R.psh;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            atomicAdd(in[i] ? &tab[x[i] >> R.psh] : dummy, 1u << ((x[i] & pm) << bsh));
        return true;
    }
    const uint32_t hmask = ~R.cmask;
    const uint4 *t4 = reinterpret_cast<const uint4 *>(tab);
    int32_t b[4];
    uint32_t tag[4], ws[4];
    uint4 q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // a wedge outside the range reads bucket 0 and is ignored below
        b[i] = in[i] ? (int32_t)__umulhi(x[i], R.mul) : 0;
        // where the key lies inside its bucket's share of the range
        ws[i] = (x[i] * R.mul) >> 30;
        tag[i] = (x[i] + 1u) << R.cb;
        q[i] = t4[b[i]];
    }
    // first pass: add to a found key, or claim a free word
    uint32_t addr[4], old[4];
    uint32_t pend = 0;  // bit i: wedge i issued a compare-and-swap
    uint32_t slow = 0;  // bit i: wedge i continues in the probe loop
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w0 = q[i].x, w1 = q[i].y, w2 = q[i].z, w3 = q[i].w;
        const uint32_t fw = free_word(ws[i], w0, w1, w2, w3);
        // same key <=> the words differ only in the count bits (an empty
        // word never matches: the tag is above the count bits)
        int32_t hit = -1;
        if ((w3 ^ tag[i]) <= R.cmask) hit = 3;
        if ((w2 ^ tag[i]) <= R.cmask) hit = 2;
        if ((w1 ^ tag[i]) <= R.cmask) hit = 1;
        if ((w0 ^ tag[i]) <= R.cmask) hit = 0;
        addr[i] = 4u * (uint32_t)b[i] + (hit >= 0 ? (uint32_t)hit : (fw & 3u));
        const bool add = in[i] && hit >= 0;
        const bool cas = in[i] && hit < 0 && fw < 4u;
        const bool full = in[i] && hit < 0 && fw >= 4u;
        atomicAdd(add ? &tab[addr[i]] : dummy, 1u);
        old[i] = atomicCAS(cas ? &tab[addr[i]] : dummy, 0u, tag[i] | 1u);
        pend |= cas ? 1u << i : 0u;
        slow |= full ? 1u << i : 0u;
        b[i] += full ? 1 : 0;  // home bucket full without the key: continue after it
    }
    // second pass: the swaps' results
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool taken = ((pend >> i) & 1u) && old[i] != 0u;
        const bool same = taken && (old[i] & hmask) == tag[i];
        atomicAdd(same ? &tab[addr[i]] : dummy, 1u);
        slow |= (taken && !same) ? 1u << i : 0u;  // another key took the word: look again
    }
    bool ok = true;
    const int32_t nb = R.limit >> 2;
    while (slow) {
        const int32_t i = __builtin_ctz(slow);
        slow &= slow - 1u;
        const int32_t bi = i == 0 ? b[0] : i == 1 ? b[1] : i == 2 ? b[2] : b[3];
        const uint32_t ti = pick4(i, tag[0], tag[1], tag[2], tag[3]);
        const uint32_t wi = pick4(i, ws[0], ws[1], ws[2], ws[3]);
        if (bi >= nb) {
            ok = false;
        } else {
            ok &= tab_probe(tab, R, ti, wi, bi, min(nb, bi + probes), t4[bi]);
        }
    }
    return ok;
}

// Count up to four wedges whose keys, if present, were inserted before (the
// candidate cannot reach s without them, so an absent key is skipped).  Dense
// ranges add unconditionally: a candidate counted only here stays below s.
__device__ __forceinline__ void tab_look4(uint32_t *tab, const Range &R, int32_t j0, int32_t j1,
                                          int32_t j2, int32_t j3) {
    const int32_t j[4] = {j0, j1, j2, j3};
    uint32_t x[4];
    bool in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = (uint32_t)(j[i] - R.lo);
        in[i] = j[i] < R.hi && x[i] < R.span;
    }
    if (R.mul == 0) {
        const uint32_t pm = (1u << R.psh) - 1u, bsh = 5u - R.psh;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (in[i]) atomicAdd(&tab[x[i] >> R.psh], 1u << ((x[i] & pm) << bsh));
        return;
    }
    const uint4 *t4 = reinterpret_cast<const uint4 *>(tab);
    const int32_t nb = R.limit >> 2;
    uint32_t tag[4];
    int32_t b[4];
    uint4 q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        tag[i] = (x[i] + 1u) << R.cb;
        b[i] = in[i] ? (int32_t)__umulhi(x[i], R.mul) : 0;
        q[i] = in[i] ? t4[b[i]] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (!in[i]) continue;
        for (;;) {
            const uint32_t w0 = q[i].x, w1 = q[i].y, w2 = q[i].z, w3 = q[i].w;
            const bool h0 = (w0 ^ tag[i]) <= R.cmask, h1 = (w1 ^ tag[i]) <= R.cmask;
            const bool h2 = (w2 ^ tag[i]) <= R.cmask, h3 = (w3 ^ tag[i]) <= R.cmask;
            if (h0 || h1 || h2 || h3) {
                atomicAdd(&tab[4 * b[i] + (h0 ? 0 : h1 ? 1 : h2 ? 2 : 3)], 1u);
                break;
            }
            // a bucket with a free word ends the search: the key is absent
            if (w0 == 0u || w1 == 0u || w2 == 0u || w3 == 0u || ++b[i] >= nb) break;
            q[i] = t4[b[i]];
        }
    }
}

struct Smem {
    uint32_t *tab;       // table words
    int2 *runs;          // long member runs of the current range
    int32_t *taken;      // per run: entries of the run inside the current range
    int32_t *misc;       // see kMisc*
    int2 *stack;         // ranges still to process
    uint32_t *spare;     // one word per lane, past the table (targets of idle atomics)
    uint64_t *pool_cur;  // this workgroup's pool chunk (see stage_begin)
    int32_t *log_cur;    // and log chunk
};

// misc words: run pieces, overflow flag, stack depth, staging reservation
// (ok, offset low, offset high), then one word per wave.
constexpr int kMiscRuns = 0, kMiscOverflow = 1, kMiscDepth = 2, kMiscStageOk = 3,
              kMiscStageLo = 4, kMiscStageHi = 5, kMiscWave = 6;

// One member's walk over [cur, end) of N_s(v) for the range R, one lane:
// reads four entries at a time and stops at the first id >= R.hi.  Returns
// the new cursor.
__device__ __forceinline__ int32_t walk_lane(const int32_t *itmS, int32_t cur, int32_t end,
                                             const Range &R, const Smem &S, bool look, bool &ok) {
    int32_t p = cur;
    while (p < end) {
        const int32_t j0 = itmS[p];
        const int32_t j1 = (p + 1 < end) ? itmS[p + 1] : INT32_MAX;
        const int32_t j2 = (p + 2 < end) ? itmS[p + 2] : INT32_MAX;
        const int32_t j3 = (p + 3 < end) ? itmS[p + 3] : INT32_MAX;
        if (look) tab_look4(S.tab, R, j0, j1, j2, j3);
        else ok &= tab_add4(S.tab, S.spare, R, j0, j1, j2, j3);
        const int32_t taken = (j0 < R.hi) + (j1 < R.hi) + (j2 < R.hi) + (j3 < R.hi);
        p += taken;
        if (taken < 4) break;
    }
    return p;
}

// Insert every wedge of item a whose candidate lies in R.  Members with few
// expected candidates in R are walked by their owning lane; the others are
// queued and walked by whole waves, up to 256 entries per step (sized by the
// expected run length).  On return nc[] holds the advanced cursors of the
// thread's members (not yet committed) and misc[1] is set if a probe ran off
// the table.
template <int NT, int RUNCAP>
__device__ __forceinline__ void insert_range(const CountArgs &A, const Smem &S, const Range &R,
                                             int32_t k0, int32_t k1, const int32_t (&cur)[kR],
                                             const int32_t (&end)[kR], uint32_t lookm, bool look,
                                             int32_t nend, int32_t (&nc)[kR]) {
    constexpr int W = NT / kWave;
    const int lane = lane_id(), wid = wave_id();
    const float frac = (float)R.span / (float)((int64_t)nend - R.lo);
    const float light_len = (float)A.tune.light_len;
    bool ok = true;
    uint32_t light = 0;  // bit i: member i is walked by this lane
    int32_t slot[kR];
#pragma unroll
    for (int i = 0; i < kR; ++i) {
        slot[i] = -1;
        if (!look) nc[i] = cur[i];
    }
#pragma unroll
    for (int i = 0; i < kR; ++i) {
        const int32_t k = k0 + (int32_t)threadIdx.x + i * NT;
        if (k < k1 && cur[i] < end[i] && (((lookm >> i) & 1u) != 0u) == look) {
            const float est = (float)(end[i] - cur[i]) * frac;
            int32_t sl = -1;
            if (est > light_len) {
                // K pieces of 256 planned entries (the last one open-ended)
                const int32_t K = min(16, (int32_t)((est * 1.25f + 16.0f) * (1.0f / kPiece)) + 1);
                const int32_t s0 = atomicAdd(&S.misc[kMiscRuns], K);
                if (s0 + K <= RUNCAP) {
                    for (int32_t k = 0; k < K; ++k) {
                        const int32_t b = cur[i] + k * kPiece;
                        S.runs[s0 + k] = make_int2(b, k == K - 1 ? end[i] : min(end[i], b + kPiece));
                        S.taken[s0 + k] = 0;
                    }
                    sl = s0 | (K << 16);
                } else {
                    // no room: blank the slots this reservation holds, walk by
                    // lane.  A blank piece is empty and its clamped index
                    // (end - 1) lies in the member's own run.
                    for (int32_t k = s0; k < min(s0 + K, RUNCAP); ++k)
                        S.runs[k] = make_int2(end[i], end[i]);
                }
            }
            if (sl < 0) light |= 1u << i;
            slot[i] = sl;
        }
    }
    // members walked by their own lane, one at a time (one copy of the walk)
    while (light) {
        const uint32_t bit = light & (0u - light);  // lowest member still to walk
        light ^= bit;
        int32_t c = 0, e = 0;
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            c = (bit & (1u << r)) ? cur[r] : c;
            e = (bit & (1u << r)) ? end[r] : e;
        }
        const int32_t n = walk_lane(A.itmS, c, e, R, S, look, ok);
#pragma unroll
        for (int r = 0; r < kR; ++r) nc[r] = (bit & (1u << r)) ? n : nc[r];
    }
    // members past the register window: locate the range by binary search
    for (int32_t k = k0 + (int32_t)threadIdx.x + kR * NT; k < k1; k += NT) {
        const int32_t st = A.start[k];
        // dense ranges count every member in one pass (lookup-only ones too)
        if (R.mul != 0 && (st < 0) != look) continue;
        const int32_t v = A.memI[k];
        const int32_t e0 = A.ptrS[v + 1];
        const int32_t b = lower_bound(A.itmS, st & kStartMask, e0, R.lo);
        walk_lane(A.itmS, b, e0, R, S, look, ok);
    }
    __syncthreads();
    // Pieces: each wave keeps four in flight (one 64-entry load each per
    // step), taking pieces h = wid, wid + W, ... in turn.  The entries below
    // R.hi form a prefix of a member's run, so the pieces' counts add up to it.
    const int32_t npiece = __builtin_amdgcn_readfirstlane(min(S.misc[kMiscRuns], RUNCAP));
    int32_t next = wid;
    int32_t pr[4], pp[4], pe[4], pg[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) pr[k] = -1;
    for (;;) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (pr[k] < 0 && next < npiece) {
                const int2 rr = S.runs[next];
                pr[k] = next;
                pp[k] = __builtin_amdgcn_readfirstlane(rr.x);
                pe[k] = __builtin_amdgcn_readfirstlane(rr.y);
                pg[k] = 0;
                next += W;
            }
            any |= pr[k] >= 0;
        }
        if (!any) break;
        int32_t j[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            j[k] = INT32_MAX;
            if (pr[k] >= 0) {
                // the clamped index lies in the piece's member run: pe - 1 is
                // its last entry, also for empty pieces (blank, or planned
                // past the run's end), which read it and count nothing
                const int32_t v = A.itmS[min(pp[k] + lane, pe[k] - 1)];
                if (pp[k] + lane < pe[k]) j[k] = v;
            }
        }
        if (look) tab_look4(S.tab, R, j[0], j[1], j[2], j[3]);
        else ok &= tab_add4(S.tab, S.spare, R, j[0], j[1], j[2], j[3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (pr[k] < 0) continue;
            const int32_t n = __popcll(__ballot(j[k] < R.hi));
            pg[k] += n;
            pp[k] += kWave;
            if (n < kWave || pp[k] >= pe[k]) {
                if (lane == 0 && pg[k]) S.taken[pr[k]] = pg[k];
                pr[k] = -1;
            }
        }
    }
    if (!ok) S.misc[kMiscOverflow] = 1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kR; ++i) {
        if (slot[i] >= 0) {
            const int32_t s0 = slot[i] & 0xffff, K = slot[i] >> 16;
            int32_t t = S.runs[s0].x;
            for (int32_t k = 0; k < K; ++k) t += S.taken[s0 + k];
            nc[i] = t;
        }
    }
}

// Zero table words [0, limit); `tab` is 16-byte aligned.
template <int NT>
__device__ __forceinline__ void tab_clear(uint32_t *tab, int32_t limit) {
    uint4 *t4 = reinterpret_cast<uint4 *>(tab);
    const int32_t n4 = limit >> 2;
    for (int32_t i = threadIdx.x; i < n4; i += NT) t4[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int32_t i = (n4 << 2) + threadIdx.x; i < limit; i += NT) tab[i] = 0u;
}

__device__ __forceinline__ uint32_t slot_count(uint32_t w, const Range &R) {
    return R.mul ? (w & R.cmask) : w;
}

// Counters >= s of one word of a packed dense range (2^psh counters of
// 32 >> psh bits each).
__device__ __forceinline__ int32_t packed_hits(uint32_t w, uint32_t psh, uint32_t s) {
    if (psh == 2u)
        return ((w & 0xffu) >= s) + (((w >> 8) & 0xffu) >= s) + (((w >> 16) & 0xffu) >= s) +
               ((w >> 24) >= s);
    return ((w & 0xffffu) >= s) + ((w >> 16) >= s);
}

// Pairs (counters >= s) in the bucket of four words q.
__device__ __forceinline__ int32_t bucket_pairs(const uint4 &q, const Range &R, uint32_t s) {
    if (R.psh == 0u)
        return (slot_count(q.x, R) >= s) + (slot_count(q.y, R) >= s) + (slot_count(q.z, R) >= s) +
               (slot_count(q.w, R) >= s);
    return packed_hits(q.x, R.psh, s) + packed_hits(q.y, R.psh, s) + packed_hits(q.z, R.psh, s) +
           packed_hits(q.w, R.psh, s);
}

__device__ __forceinline__ void cswap(uint32_t &x, uint32_t &y) {
    const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
    x = lo;
    y = hi;
}

__device__ __forceinline__ bool bucket_full(const uint4 &q) {
    return q.x != 0u && q.y != 0u && q.z != 0u && q.w != 0u;
}

// Extract the candidates with count >= s and return their number
// (block-uniform).  Each lane holds one bucket (four slots, one 16-byte LDS
// read), so the order inside a bucket is settled in registers; only buckets
// in a run of full buckets (or right after one) rank their entries against
// the neighbouring buckets of the run.  Fill mode writes (a, b, w) in b order
// at task_off[t] + rel; stage mode reserves room in the pool, writes (b, w)
// there and logs the range (or flags task t when the pool or the log is
// full).  Leaves the table cleared.  FILL: whether the mode is fill, if
// compiled for one of them (else -1); LISTED: the lists hold every bucket.
template <int NT, int RUNCAP, int FILL = -1, bool LISTED = false>
__device__ __forceinline__ int32_t tab_extract(const CountArgs &A, const Smem &S, const Range &R,
                                               int32_t a, int32_t sa, int32_t t, int64_t rel) {
    constexpr int W = NT / kWave;
    // each wave lists the buckets of its block that hold pairs, in order, in
    // the run arrays (idle during extraction): LCAP 16-bit entries per wave
    constexpr int LCAP = (int)(RUNCAP * sizeof(int2) / sizeof(uint16_t)) / W;
    const int lane = lane_id(), wid = wave_id();
    const int32_t L = R.limit;
    const int32_t nbk = (L + 3) >> 2;  // words past L are zero
    const int32_t per_wave = ((nbk + W * kWave - 1) / (W * kWave)) * kWave;
    const int32_t b0 = wid * per_wave;
    const int32_t b1 = min(nbk, b0 + per_wave);
    const uint32_t s = (uint32_t)sa;
    const uint4 *t4 = reinterpret_cast<const uint4 *>(S.tab);
    uint16_t *const lst = reinterpret_cast<uint16_t *>(S.runs) + wid * LCAP;
    __syncthreads();  // the insertion has finished reading the run arrays
    // bits of a bucket's pair count: up to 4 pairs, or 16 with packed counters
    const int nbits = R.psh ? 5 : 3;
    int32_t mine = 0, nact = 0;
    for (int32_t i = b0; i < b1; i += kWave) {
        const int32_t bk = i + lane;
        const uint4 q = bk < b1 ? t4[bk] : make_uint4(0u, 0u, 0u, 0u);
        const int32_t n = bucket_pairs(q, R, s);
        int32_t nb_before, nb_step;
        wave_bits_prefix(n, nbits, nb_before, nb_step);
        mine += nb_step;
        const uint64_t am = __ballot(n > 0);
        const int32_t slot = nact + (int32_t)lanes_below(am);
        if (n > 0 && slot < LCAP) lst[slot] = (uint16_t)bk;
        nact += (int32_t)__popcll(am);
    }
    if (lane == 0) S.misc[kMiscWave + wid] = mine;
    __syncthreads();
    int32_t run = 0, total = 0;
    for (int w = 0; w < W; ++w) {
        const int32_t tw = S.misc[kMiscWave + w];
        if (w < wid) run += tw;
        total += tw;
    }
    bool write = false;
    int64_t base = 0;
    int32_t shift = 0;  // fill mode, batches written per graph: the graph's item base
    int32_t *dst_a = nullptr, *dst_b = nullptr, *dst_w = nullptr;
    const bool fill = FILL < 0 ? A.mode == kModeFill : FILL != 0;
    if (total && fill) {
        write = true;
        const OutDst od = out_dst(A, a, A.task_off[t] + rel);
        base = od.base;
        shift = od.shift;
        dst_a = od.a;
        dst_b = od.b;
        dst_w = od.w;
    } else if (total && A.mode == kModeStage) {
        if (threadIdx.x == 0) {
            uint64_t off;
            int32_t rec;
            const bool ok = stage_reserve(A, S.pool_cur, S.log_cur, total, 1, off, rec);
            if (ok) {
                StageRec r;
                r.off = (int64_t)off;
                r.t = t;
                r.rel = (int32_t)rel;
                r.n = total;
                r.pad = 0;
                A.log[rec] = r;
            } else if (atomicExch(&A.need[t], 1) == 0) {
                atomicAdd(A.need_count, 1);
            }
            S.misc[kMiscStageOk] = ok ? 1 : 0;
            S.misc[kMiscStageLo] = (int32_t)(uint32_t)(off & 0xffffffffull);
            S.misc[kMiscStageHi] = (int32_t)(uint32_t)(off >> 32);
        }
        __syncthreads();
        if (S.misc[kMiscStageOk]) {
            write = true;
            base = (int64_t)(((uint64_t)(uint32_t)S.misc[kMiscStageHi] << 32) |
                             (uint64_t)(uint32_t)S.misc[kMiscStageLo]);
            dst_b = A.pool_b;
            dst_w = A.pool_w;
        }
    }
    if (write) {
        // One bucket per lane (bk, valid when vb): its pairs go to
        // run + (pairs of this wave's buckets before it).  `listed`: the
        // lanes hold the listed buckets, not consecutive ones.
        bool prev_full = R.mul && b0 > 0 && b0 < b1 && bucket_full(t4[b0 - 1]);
        const bool outs = FILL < 0 ? dst_a != nullptr : FILL != 0;  // ids of items, and a
        auto emit = [&](auto listed, int32_t bk, bool vb) {
            const uint4 q = vb ? t4[bk] : make_uint4(0u, 0u, 0u, 0u);
            const uint32_t wv[4] = {q.x, q.y, q.z, q.w};
            uint32_t c[4];
            bool ok[4];
            int32_t n = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                c[k] = slot_count(wv[k], R);
                ok[k] = c[k] >= s;
                n += ok[k];
            }
            if (R.psh) n = bucket_pairs(q, R, s);
            // exclusive prefix of n over the lanes
            int32_t before, step;
            wave_bits_prefix(n, nbits, before, step);
            if (R.mul == 0 && R.psh) {
                // packed dense: counter order is candidate order
                const uint32_t per = 1u << R.psh, cbits = 32u >> R.psh;
                const uint32_t cm = (cbits == 32u) ? 0xffffffffu : ((1u << cbits) - 1u);
                int32_t pos = run + before;
                for (int k = 0; k < 4 && n; ++k) {
                    for (uint32_t j = 0; j < per; ++j) {
                        const uint32_t cnt = (wv[k] >> (j * cbits)) & cm;
                        if (cnt >= s) {
                            const int32_t b = R.lo + (int32_t)(((uint32_t)(4 * bk + k) << R.psh) + j);
                            if (outs) dst_a[base + pos] = a - shift;
                            dst_b[base + pos] = outs ? item_of(A, b) - shift : b;
                            if (dst_w) dst_w[base + pos] = (int32_t)cnt;
                            ++pos;
                        }
                    }
                }
            } else if (R.mul == 0) {
                // dense: slot order is candidate order
                int32_t pos = run + before;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (ok[k]) {
                        if (outs) dst_a[base + pos] = a - shift;
                        const int32_t b = R.lo + 4 * bk + k;
                        dst_b[base + pos] = outs ? item_of(A, b) - shift : b;
                        if (dst_w) dst_w[base + pos] = (int32_t)c[k];
                        ++pos;
                    }
                }
            } else {
                // the bucket's kept words in candidate order (a word orders
                // like its key, which sits above the count bits; words not
                // kept sort last): five compare-exchanges
                uint32_t key[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) key[k] = ok[k] ? wv[k] : 0xFFFFFFFFu;
                cswap(key[0], key[1]);
                cswap(key[2], key[3]);
                cswap(key[0], key[2]);
                cswap(key[1], key[3]);
                cswap(key[1], key[2]);
                uint32_t tag[4];
                int32_t rank[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    tag[k] = key[k] >> R.cb;
                    rank[k] = k;
                }
                // runs of full buckets: a bucket ends a run unless it is full
                const bool full = bucket_full(q) && vb;
                bool pf;  // the bucket before this one is full
                if (decltype(listed)::value) {
                    pf = vb && bk > 0 && bucket_full(t4[bk - 1]);
                } else {
                    const uint64_t fm = __ballot(full);
                    pf = lane ? ((fm >> (lane - 1)) & 1ull) != 0 : prev_full;
                    prev_full = ((fm >> 63) & 1ull) != 0;
                }
                int32_t left = 0;
                if (n && (full || pf)) {
                    // full buckets before this one in the same run
                    for (int32_t b2 = bk - 1; b2 >= 0; --b2) {
                        const uint4 lv = t4[b2];
                        if (!bucket_full(lv)) break;
                        const uint32_t l[4] = {lv.x, lv.y, lv.z, lv.w};
#pragma unroll
                        for (int k2 = 0; k2 < 4; ++k2) {
                            if ((l[k2] & R.cmask) >= s) {
                                ++left;
                                const uint32_t tg = l[k2] >> R.cb;
#pragma unroll
                                for (int k = 0; k < 4; ++k) rank[k] += tg < tag[k];
                            }
                        }
                    }
                    // buckets after this one up to the first that is not full
                    bool more = full;
                    for (int32_t b2 = bk + 1; more && b2 < nbk; ++b2) {
                        const uint4 rv = t4[b2];
                        more = bucket_full(rv);
                        const uint32_t r[4] = {rv.x, rv.y, rv.z, rv.w};
#pragma unroll
                        for (int k2 = 0; k2 < 4; ++k2) {
                            if ((r[k2] & R.cmask) >= s) {
                                const uint32_t tg = r[k2] >> R.cb;
#pragma unroll
                                for (int k = 0; k < 4; ++k) rank[k] += tg < tag[k];
                            }
                        }
                    }
                }
                const int32_t pos = run + before - left;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (k < n) {
                        const int32_t p = pos + rank[k];
                        if (outs) dst_a[base + p] = a - shift;
                        const int32_t b = R.lo + (int32_t)tag[k] - 1;
                        dst_b[base + p] = outs ? item_of(A, b) - shift : b;
                        if (dst_w) dst_w[base + p] = (int32_t)(key[k] & R.cmask);
                    }
                }
            }
            run += step;
        };
        if (LISTED || nact <= LCAP) {
            // only the buckets that hold pairs, 64 at a time
            for (int32_t i = 0; i < nact; i += kWave) {
                const bool vb = i + lane < nact;
                emit(std::true_type{}, vb ? (int32_t)lst[i + lane] : 0, vb);
            }
        } else {
            for (int32_t i = b0; i < b1; i += kWave)
                emit(std::false_type{}, i + lane, i + lane < b1);
        }
    }
    __syncthreads();
    tab_clear<NT>(S.tab, L);
    __syncthreads();
    return total;
}

// Candidates [lo, hi) of item a with a table of `slots` home slots: insert,
// split on overflow, extract; the member cursors advance to hi.  Returns the
// pairs produced (block-uniform).
template <int NT, int PAD, int RUNCAP>
__device__ __forceinline__ int64_t run_range(const CountArgs &A, const Smem &S, int32_t a,
                                             int32_t sa, int32_t nend, int32_t t, int32_t lo,
                                             int32_t hi, int32_t slots,
                                             int32_t cb, int32_t k0, int32_t k1, int32_t (&cur)[kR],
                                             const int32_t (&end)[kR], uint32_t lookm,
                                             int64_t &passes) {
    if (threadIdx.x == 0) {
        S.stack[0] = make_int2(lo, hi);
        S.misc[kMiscDepth] = 1;
    }
    __syncthreads();
    int64_t produced = 0;
    for (;;) {
        // every thread reads the stack before anyone may change it (the next
        // call's thread 0 rewrites it as soon as it leaves this loop)
        const int32_t depth = S.misc[kMiscDepth];
        const int2 top = depth ? S.stack[depth - 1] : make_int2(0, 0);
        __syncthreads();
        if (depth == 0) break;
        if (threadIdx.x == 0) {
            S.misc[kMiscDepth] = depth - 1;
            S.misc[kMiscRuns] = 0;
            S.misc[kMiscOverflow] = 0;
        }
        __syncthreads();
        const Range R = make_range(top.x, top.y, slots, PAD, cb);
        bool split = too_wide(R);
        if (!split) {
            int32_t nc[kR];
            // a dense range has room for every candidate: all members count in
            // one pass, lookup-only ones included
            const uint32_t lm = R.mul ? lookm : 0u;
            insert_range<NT, RUNCAP>(A, S, R, k0, k1, cur, end, lm, false, nend, nc);
            ++passes;
            split = S.misc[kMiscOverflow] != 0;
            if (!split && sa > 1 && R.mul != 0) {
                // members marked lookup-only count candidates the others inserted
                __syncthreads();
                if (threadIdx.x == 0) S.misc[kMiscRuns] = 0;
                __syncthreads();
                insert_range<NT, RUNCAP>(A, S, R, k0, k1, cur, end, lm, true, nend, nc);
            }
            if (!split) {
                produced += tab_extract<NT, RUNCAP>(A, S, R, a, sa, t, produced);
#pragma unroll
                for (int i = 0; i < kR; ++i) cur[i] = nc[i];
                continue;
            }
            // a probe ran off the table: clear it
            __syncthreads();
            tab_clear<NT>(S.tab, R.limit);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const int32_t mid = (int32_t)(((int64_t)top.x + top.y) / 2);
            const int32_t d = S.misc[kMiscDepth];
            S.stack[d] = make_int2(mid, top.y);
            S.stack[d + 1] = make_int2(top.x, mid);
            S.misc[kMiscDepth] = d + 2;
        }
        __syncthreads();
    }
    return produced;
}

// Cursors of the thread's members for a walk starting at candidate lo (first:
// the item's first candidate, where the back-pointers point).
template <int NT>
__device__ __forceinline__ void init_cursors(const CountArgs &A, int32_t first, int32_t lo,
                                             int32_t k0, int32_t k1, int32_t (&cur)[kR], int32_t (&end)[kR],
                                             uint32_t &lookm) {
    lookm = 0;
#pragma unroll
    for (int i = 0; i < kR; ++i) {
        const int32_t k = k0 + (int32_t)threadIdx.x + i * NT;
        cur[i] = 0;
        end[i] = 0;
        if (k < k1) {
            const int32_t v = A.memI[k];
            const int32_t e = A.ptrS[v + 1];
            const int32_t st = A.start[k];
            lookm |= (uint32_t)(st < 0) << i;
            int32_t c = st & kStartMask;
            if (lo > first) c = lower_bound(A.itmS, c, e, lo);
            cur[i] = c;
            end[i] = e;
        }
    }
}

// Count bits for item a: its size bounds every overlap.
__device__ __forceinline__ int32_t count_bits(int32_t size) {
    return 32 - __clz((uint32_t)max(size, 1));
}

// Number of tasks of an item: P = ceil(cost / target) equal sub-ranges of
// its candidate range of `span` ids, each about `target` wedges.  When the
// item's candidates are dense enough -- at least dense_min wedges (by the
// planning cost) on average in each sub-range narrow enough for its packed
// dense counters (slots << pack_shift(size)) -- the item is cut into that many
// sub-ranges instead (if more): counting one of them costs an add per wedge
// and an in-order scan, with no hashing.  dense_min = 0 keeps P as is.
__device__ __forceinline__ int32_t task_parts(int64_t cost, int32_t small_max, int32_t target,
                                              int64_t span, int32_t size, int32_t dense_min,
                                              int32_t slots) {
    if (cost <= 0) return 0;
    if (cost <= small_max) return 1;
    int64_t P = (cost + target - 1) / target;
    if (dense_min > 0 && span > 0) {
        const int64_t cap = (int64_t)slots << pack_shift(32 - __clz((uint32_t)max(size, 1)));
        const int64_t Pd = (span + cap - 1) / cap;
        if (Pd > P && cost >= (int64_t)dense_min * Pd) P = Pd;
    }
    return (int32_t)min(P, (int64_t)INT32_MAX);
}

// Number of candidates of item a.
__device__ __forceinline__ int64_t item_span(const int32_t *crank, const int32_t *item_end,
                                             int32_t N, int32_t full, int32_t a) {
    return (int64_t)cand_end(crank, item_end, N, a) - cand_first(crank, full, a);
}

// Sub-range p of P of the candidate range [first, N) of an item.
__device__ __forceinline__ void task_range(int32_t first_id, int32_t N, int32_t p, int32_t P,
                                           int32_t &lo, int32_t &hi) {
    const int64_t first = first_id, span = (int64_t)N - first;
    lo = (int32_t)(first + span * p / P);
    hi = (int32_t)(first + span * (p + 1) / P);
}

constexpr int kSmallPad = 64;
constexpr int kSmallRunCap = 128;
constexpr int kTaskPad = 64;
constexpr int kTaskRunCap = 256;
constexpr int kStack = 64;

// --------------------------------------------------------------- small

// SLOTS: home slots of the wave's table (Tuning::small_slots).
template <int SLOTS>
__global__ __launch_bounds__(kWave) void k_count_small(CountArgs A) {
    constexpr int LIM = SLOTS + kSmallPad;
    __shared__ __align__(16) uint32_t tab[LIM + kWave];
    __shared__ int2 runs[kSmallRunCap];
    __shared__ int32_t taken[kSmallRunCap];
    __shared__ int2 stack[kStack];
    __shared__ int32_t misc[kMiscWave + 1];
    __shared__ uint64_t pool_cur[3];
    __shared__ int32_t log_cur[3];
    const Smem S{tab, runs, taken, misc, stack, tab + LIM, pool_cur, log_cur};
    if (count_idle(A)) return;  // uniform: every thread reads the same words
    use_ranks(A);
    if (threadIdx.x == 0) {
        stage_begin(A, kKindSmall, pool_cur, log_cur);
    }
    tab_clear<kWave>(tab, LIM);
    const int32_t n_small = A.task_counts[kKindSmall * kCountStride];
    int64_t passes = 0;
    __syncthreads();
    for (int32_t r = blockIdx.x; r < n_small; r += gridDim.x) {
        const int32_t t = A.small_tasks[r];
        if (A.mode == kModeFill && A.need && !A.need[t]) continue;
        const int32_t a = A.small_items[r];
        const int64_t c = A.cost[a];
        // 2 W_a home slots (load <= 1/2), rounded up to whole waves
        int32_t want = (int32_t)std::min<int64_t>(2 * c, SLOTS);
        want = std::min(SLOTS, std::max(kWave, ((want + kWave - 1) / kWave) * kWave));
        const int32_t k0 = A.ptrI[a], k1 = A.ptrI[a + 1];
        int32_t cur[kR], end[kR];
        uint32_t lookm;
        const int32_t first = cand_first(A.crank, A.full, a);
        const int32_t nend = cand_end(A.crank, A.item_end, A.N, a);
        init_cursors<kWave>(A, first, first, k0, k1, cur, end, lookm);
        const int64_t produced = run_range<kWave, kSmallPad, kSmallRunCap>(
            A, S, a, A.s_item ? A.s_item[a] : A.s, nend, t, first, nend, want,
            count_bits(k1 - k0), k0, k1, cur, end, lookm, passes);
        if (A.mode != kModeFill && threadIdx.x == 0) A.task_cnt[t] = (int32_t)produced;
        __syncthreads();
    }
    if (threadIdx.x == 0 && passes && A.passes)
        atomicAdd(stat_row(A), (unsigned long long)passes);
}

// ---------------------------------------------------------- whole items

// An item counted at once by one workgroup, all its wedges through a wedge map.
//
// With up to kMiniWedges wedges (KIND kKindMini) every wedge goes into the hash
// table in one step of a wave.  With more and s > 1 most candidates are met
// once and are no pair, so they are sieved: a first walk sets, for every
// wedge, a bit chosen by the candidate (its low bits) in `seen`, and where that
// was set already, in `twice`; a second walk inserts only the wedges whose
// `twice` bit is set, which counts them exactly, every wedge of a pair among
// them.  (Two candidates that share a bit only bring wedges that stay below
// s.)  The wedges let through are collected first, so that a table step has a
// wedge in every lane.
//
// What bounds it: the chain of reads from an item to its wedges (item, list
// bounds, members, their lists, candidates), then instructions, about 25 per
// 64 wedges and walk and 30 per 64 wedges let through.  So the next item's
// part of the chain is read while this one is counted, and small items get a
// single wave, whose barriers cost nothing and whose per-item steps are not
// repeated by other waves.  FILL: compiled for the fill mode, or for the two
// others; one kernel for all modes kept twice the arguments, half of them
// spilled (109 scalar registers, 342 reads of them), and a third more
// instructions.  4 KB of LDS for up to 256 wedges, 10.8 KB (15 waves
// per CU) for up to 2048, 40 KB and four waves for up to 8192.
constexpr int kSieveList = 5 * kWave;  // wedges a wave collects
// A hash table holds candidates in their order, and where they crowd in a small part
// of the range, as with neighbours whose ids are close, probes get long.  So a key
// that finds no room within kItemProbes buckets of its own ends the pass, and another
// pass measures the range's candidates: if direct counters fit what they span, these
// count it, else it is split at their mean, which sets few distant candidates apart
// from the others at once.
// s = 2, with probes to the end of the table and splits at the middle of the range, and
// so: 300,000 items of 5 to 30 members within 400 of 60,000 vertices 14.1 and 4.0 ms,
// one member in 20 anywhere 11.8 and 6.2; 783,766 vertices in cliques of some 500
// neighbours, s = 8, 8.1 and 4.9 (hashed tasks, with wider counters, took 5.3).  128
// graphs with members anywhere, replayed, lose 2 % by the code for it (10.12, 10.34); with
// 4 buckets 10.38, with 2 10.8.
constexpr int32_t kItemProbes = 8;

// What the counting needs of an item.
struct ItemDesc {
    int32_t a, t, k0, size, first, nend, s;
};

__device__ __forceinline__ ItemDesc item_desc(const CountArgs &A, int32_t a) {
    ItemDesc d{};
    d.a = a;
    if (a >= 0) {
        d.t = (int32_t)A.tbase[a];
        d.k0 = A.ptrI[a];
        d.size = A.ptrI[a + 1] - d.k0;
        d.first = cand_first(A.crank, 0, a);
        d.nend = cand_end(A.crank, A.item_end, A.N, a);
        d.s = A.s_item ? A.s_item[a] : A.s;
    }
    return d;
}

template <int KIND, int NT, int LIM, int CHUNKS, int MINB, bool FILL>
__global__ __launch_bounds__(NT, MINB) void k_count_item(CountArgs A) {
    constexpr int NW = NT / kWave;
    constexpr bool SIEVE = KIND != kKindMini;
    constexpr int SLOTS = LIM - kTaskPad;  // home slots of the LIM table words
    constexpr int kLoad = SIEVE ? 8 : 4;   // chunks a wave loads at a time
    constexpr int RUNCAP = ((LIM / 4 / NW + kWave - 1) / kWave * kWave) * NW * 2 / 8;
    constexpr int LISTS = SIEVE ? NW * kSieveList : RUNCAP * 2;
    static_assert(LISTS * sizeof(int32_t) >= RUNCAP * sizeof(int2), "list area");
    static_assert(RUNCAP * sizeof(int2) / sizeof(uint16_t) >= LIM / 4, "every bucket listed");
    static_assert(!SIEVE || (LIM & (LIM - 1)) == 0, "bits are chosen by a mask");
    __shared__ __align__(16) uint32_t tab[LIM + kWave];  // first walk: `seen`; then the table
    __shared__ __align__(16) uint32_t twice[SIEVE ? LIM : 4];
    __shared__ __align__(16) int32_t list[LISTS];
    __shared__ int32_t adj[NT];
    __shared__ __align__(8) uint32_t marks[2 * CHUNKS];
    __shared__ int32_t msh[3 * NW];
    __shared__ int2 stack[kStack];
    __shared__ int32_t misc[kMiscWave + NW];
    __shared__ int2 span;    // of a measured range: its least and its largest candidate,
    __shared__ float2 sums;  // their sum less the range's start, and their number
    __shared__ uint64_t pool_cur[3];
    __shared__ int32_t log_cur[3];
    if (count_idle(A)) return;  // uniform: every thread reads the same words
    const int32_t n_items = A.task_counts[KIND * kCountStride];
    if ((int32_t)blockIdx.x >= n_items) return;
    use_ranks(A);
    const int32_t *const items =
        (KIND == kKindMini ? A.small_items : KIND == kKindSieve1 ? A.small_tasks : A.tiny_tasks) +
        (A.n_tasks - 1);
    const int tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    const Smem S{tab, reinterpret_cast<int2 *>(list), nullptr, misc, stack, tab + LIM, pool_cur,
                 log_cur};
    WedgeMap<NT, CHUNKS> map;
    map.adj_all = adj;
    map.marks_all = marks;
    map.sh = msh;
    if (tid == 0) {
        stage_begin(A, KIND, pool_cur, log_cur);
    }
    tab_clear<NT>(tab, LIM);
    if (SIEVE) tab_clear<NT>(twice, LIM);
    for (int i = tid; i < 2 * CHUNKS; i += NT) marks[i] = 0;
    int64_t my_wedges = 0, my_nnz = 0, my_pairs = 0, passes = 0;  // thread 0's are used
    const int32_t stride = (int32_t)gridDim.x;
    auto item_at = [&](int64_t q) { return q < n_items ? items[-q] : -1; };
    // a member's list (v, -1: none) and the first entry of the walk
    auto load_member = [&](const ItemDesc &d, int32_t &v, int32_t &b) {
        map.narrow = NT == kWave || uniform(d.size) <= kWave;
        const int32_t k = map.member();
        v = -1;
        b = 0;
        if (k < d.size) {
            v = A.memI[d.k0 + k];
            b = A.start[d.k0 + k] & kStartMask;
        }
    };
    auto load_end = [&](int32_t v) { return v >= 0 ? A.ptrS[v + 1] : 0; };
    int64_t r = blockIdx.x;
    ItemDesc cur = item_desc(A, item_at(r));
    int32_t ahead = item_at(r + stride);  // the next item
    int32_t v, b;
    load_member(cur, v, b);
    int32_t e = load_end(v);
    __syncthreads();
    for (; r < n_items; r += stride) {
        const ItemDesc nxt = item_desc(A, ahead);
        ahead = item_at(r + 2 * (int64_t)stride);
        const int32_t t = uniform(cur.t), a = uniform(cur.a), s = uniform(cur.s);
        const int32_t size = uniform(cur.size);
        const int32_t first = uniform(cur.first), nend = uniform(cur.nend);
        const bool skip = FILL && A.need && !A.need[t];
        map.narrow = NT == kWave || size <= kWave;
        int32_t nv = -1, nb = 0, ne = 0;
        if (!skip) {
            map.number(b, max(e - b, 0));
            const int32_t total = map.total;
            const auto run = map.window(0);
            int32_t j[kLoad];
            if (run.nc > 0) map.load(A.itmS, run, 0, j);
            const bool narrow = map.narrow;
            load_member(nxt, nv, nb);
            map.narrow = narrow;
            // call body(j) with kLoad candidates per lane (-1: none), over the
            // wave's chunks; the first ones are loaded
            // as long as it returns true
            auto walk = [&](bool again, auto body) {
                for (int32_t u = 0; u < run.nc; u += kLoad) {
                    if (u > 0 || again) map.load(A.itmS, run, u, j);
                    if (!body()) break;
                }
            };
            // home slots: two per candidate, and a pair takes two wedges at least
            const int32_t slots = SIEVE && s > 1 ? total / 2 : 2 * total;
            const int32_t want =
                min(SLOTS, max(kWave, (slots + kWave - 1) / kWave * kWave));
            const int32_t cb = count_bits(size);
            // a range that direct counters fit needs no sieve
            const bool sieve =
                SIEVE && s > 1 && make_range(first, nend, want, kTaskPad, cb).mul != 0;
            // bits: 16 per wedge, a power of two
            const int32_t words =
                min(LIM, max(kWave, 1 << (32 - __clz(max(total, 2) / 2 - 1))));
            const uint32_t bmask = (uint32_t)words * 32u - 1u;
            if (sieve) {
                walk(false, [&]() {
                    uint32_t old[kLoad];
#pragma unroll
                    for (int u = 0; u < kLoad; ++u) {
                        const uint32_t h = (uint32_t)j[u] & bmask;
                        if (j[u] >= 0) old[u] = atomicOr(&tab[h >> 5], 1u << (h & 31u));
                    }
#pragma unroll
                    for (int u = 0; u < kLoad; ++u) {
                        const uint32_t h = (uint32_t)j[u] & bmask;
                        if (j[u] >= 0 && __builtin_amdgcn_ubfe(old[u], h, 1u))
                            atomicOr(&twice[h >> 5], 1u << (h & 31u));
                    }
                    return true;
                });
                __syncthreads();
                tab_clear<NT>(tab, words);
            }
            ne = load_end(nv);
            if (tid == 0) {
                span = make_int2(INT32_MAX, -1);
                sums = make_float2(0.0f, 0.0f);
                stack[0] = make_int2(first, nend);
                misc[kMiscDepth] = 1;
                misc[kMiscOverflow] = 0;
            }
            __syncthreads();
            int32_t produced = 0;
            // the first walk left j at the run's last chunks
            bool again = sieve && run.nc > kLoad;
            bool measure = false;  // this pass looks at the candidates of the range alone
            if (SIEVE && NW == 1 && sieve) {
                // it starts with that where the last 128 of the first walk are close
                const int32_t x = wave_least(
                    (int32_t)min(min((uint32_t)j[0], (uint32_t)j[1]), (uint32_t)INT32_MAX));
                measure = ~wave_least(~max(j[0], j[1])) - x < want << pack_shift(cb);
            }
            // up to four candidates of the range per lane, to the table or measured;
            // whether the wave's all found room
            auto take4 = [&](const Range &R, int32_t x0, int32_t x1, int32_t x2, int32_t x3) {
                if (!measure)
                    return __ballot(!tab_add4(tab, S.spare, R, x0, x1, x2, x3, kItemProbes)) == 0;
                const int32_t x[4] = {x0, x1, x2, x3};
                int32_t least = INT32_MAX, last = -1, count = 0;
                float sum = 0.0f;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = x[u] >= R.lo && x[u] < R.hi;
                    if (in) least = min(least, x[u]);
                    if (in) last = max(last, x[u]);
                    if (in) sum += (float)(x[u] - R.lo);
                    count += (int32_t)__popcll(__ballot(in));
                }
                least = wave_least(least);
                last = ~wave_least(~last);
                sum = wave_total(sum);
                if (lane == 0) {
                    atomicMin(&span.x, least);
                    atomicMax(&span.y, last);
                    atomicAdd(&sums.x, sum);
                    atomicAdd(&sums.y, (float)count);
                }
                return true;
            };
            for (;;) {
                const int32_t depth = misc[kMiscDepth];
                const int2 top = depth ? stack[depth - 1] : make_int2(0, 0);
                if (depth == 0) break;
                const Range R = make_range(top.x, top.y, want, kTaskPad, cb);
                bool split = too_wide(R) && !measure;
                if (!split) {
                    if (!measure) ++passes;
                    bool ok = true;  // of the wave
                    if (SIEVE) {
                        int32_t *const mine = list + wid * kSieveList;
                        int32_t n = 0;  // wedges collected
                        walk(again, [&]() {
                            uint32_t w[kLoad];
                            if (sieve) {
#pragma unroll
                                for (int u = 0; u < kLoad; ++u)
                                    w[u] = twice[((uint32_t)j[u] & bmask) >> 5];
                            }
#pragma unroll
                            for (int u = 0; u < kLoad; ++u) {
                                bool in = j[u] >= R.lo && j[u] < R.hi;
                                if (sieve) in = in && __builtin_amdgcn_ubfe(w[u], (uint32_t)j[u], 1u);
                                const uint64_t m = __ballot(in);
                                if (m == 0) continue;
                                if (in) mine[n + (int32_t)lanes_below(m)] = j[u];
                                n += __popcll(m);
                                if (n >= 4 * kWave) {
                                    __builtin_amdgcn_wave_barrier();
                                    ok = ok && take4(R, mine[lane], mine[kWave + lane],
                                                     mine[2 * kWave + lane], mine[3 * kWave + lane]);
                                    n -= 4 * kWave;
                                    if (lane < n) mine[lane] = mine[4 * kWave + lane];
                                    __builtin_amdgcn_wave_barrier();
                                }
                            }
                            return ok;
                        });
                        again = run.nc > kLoad;
                        __builtin_amdgcn_wave_barrier();
                        if (ok && n > 0) {
                            int32_t x[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                x[u] = u * kWave + lane < n ? mine[u * kWave + lane] : -1;
                            ok = take4(R, x[0], x[1], x[2], x[3]);
                        }
                    } else {
                        if (run.nc > 0) ok = take4(R, j[0], j[1], j[2], j[3]);
                    }
                    if (!ok) misc[kMiscOverflow] = 1;
                    __syncthreads();
                    split = misc[kMiscOverflow] != 0;
                    if (measure) {
                        // nothing went to the table
                    } else if (!split) {
                        produced += tab_extract<NT, RUNCAP, FILL ? 1 : 0, true>(A, S, R, a, s, t, produced);
                    } else {
                        tab_clear<NT>(tab, R.limit);
                    }
                }
                __syncthreads();
                if (tid == 0) {
                    int32_t d = depth - 1;
                    if (measure) {
                        // what the candidates span, if direct counters fit it; else
                        // its parts below and above their mean
                        const int2 r = make_int2(span.x, span.y + 1);
                        if (r.x >= r.y) {
                            // none at all
                        } else if ((uint32_t)(r.y - r.x) <= (uint32_t)want << pack_shift(cb)) {
                            stack[d++] = r;
                        } else {
                            int32_t mid = d < kStack / 2 ? R.lo + (int32_t)(sums.x / sums.y)
                                                         : (int32_t)(((int64_t)r.x + r.y) / 2);
                            mid = min(max(mid, r.x + 1), r.y - 1);
                            stack[d] = make_int2(mid, r.y);
                            stack[d + 1] = make_int2(r.x, mid);
                            d += 2;
                        }
                    } else if (split) {
                        ++d;  // the range stays, to be measured
                        misc[kMiscOverflow] = 0;
                        span = make_int2(INT32_MAX, -1);
                        sums = make_float2(0.0f, 0.0f);
                    }
                    misc[kMiscDepth] = d;
                }
                __syncthreads();
                measure = split && !measure;
            }
            if (sieve) tab_clear<NT>(twice, words);
            if (!FILL) {
                if (tid == 0) A.task_cnt[t] = produced;
                my_wedges += total;
                my_nnz += size;
                my_pairs += produced;
            }
            __syncthreads();
        } else {
            load_member(nxt, nv, nb);
            ne = load_end(nv);
        }
        cur = nxt;
        b = nb;
        e = ne;
    }
    if (tid == 0 && A.passes && !FILL) {
        unsigned long long *wk = stat_row(A);
        if (passes) atomicAdd(&wk[0], (unsigned long long)passes);
        if (KIND != kKindMini) {  // work figures: the kernels of heavier items
            if (my_nnz) atomicAdd(&wk[1], (unsigned long long)my_nnz);
            if (my_wedges) atomicAdd(&wk[2], (unsigned long long)my_wedges);
            if (my_pairs) atomicAdd(&wk[3], (unsigned long long)my_pairs);
        }
    }
}

// --------------------------------------------------------------- tiny

// One lane per tiny item: an item with at most Tuning::tiny_max_wedges wedges
// (three times as many with s > 2, see is_tiny) and at most kTinyCap members, outside
// product mode.  The lane copies the candidates of all its members' walks
// into its own column of an LDS buffer, sorts them, and counts each run of
// equal ids: that count is the overlap.  The candidates come out ascending,
// in output order.  A workgroup stages the pairs of its 256 items with one
// reservation.
__global__ __launch_bounds__(kTinyThreads) void k_count_tiny(CountArgs A) {
    constexpr int NT = kTinyThreads;
    __shared__ int32_t buf[kTinyCap * NT];  // column of lane i: buf[q * NT + i]
    __shared__ int32_t red[2][NT / kWave];
    __shared__ uint64_t pool_cur[3];
    __shared__ int32_t log_cur[3];
    __shared__ int32_t res[4];  // ok, offset low, offset high, first record
    if (count_idle(A)) return;
    use_ranks(A);
    if (threadIdx.x == 0) {
        stage_begin(A, kKindTiny, pool_cur, log_cur);
    }
    const int tid = threadIdx.x, lane = lane_id(), wid = tid / kWave;
    int32_t *col = buf + tid;
    const int32_t n_tiny = A.task_counts[kKindTiny * kCountStride];
    __syncthreads();
    for (int32_t base = blockIdx.x * NT; base < n_tiny; base += gridDim.x * NT) {
        const int32_t r = base + tid;
        bool act = r < n_tiny;
        int32_t t = 0, a = 0, nc = 0, np = 0, sa = 1;
        if (act) {
            t = A.tiny_tasks[r];
            a = A.tiny_items[r];
            if (A.mode == kModeFill && A.need && !A.need[t]) act = false;
        }
        if (act) {
            sa = A.s_item ? A.s_item[a] : A.s;
            const int32_t k0 = A.ptrI[a], k1 = A.ptrI[a + 1];
            for (int32_t k = k0; k < k1; ++k) {
                const int32_t v = A.memI[k];
                const int32_t e = A.ptrS[v + 1];
                for (int32_t p = A.start[k] & kStartMask; p < e; ++p) {
                    if (nc == kTinyCap) {
                        atomicOr(A.err, kErrInternal);  // the planning bound was wrong
                        break;
                    }
                    col[nc * NT] = A.itmS[p];
                    ++nc;
                }
            }
            // insertion sort of the lane's column
            for (int32_t i = 1; i < nc; ++i) {
                const int32_t x = col[i * NT];
                int32_t j = i - 1;
                while (j >= 0 && col[j * NT] > x) {
                    col[(j + 1) * NT] = col[j * NT];
                    --j;
                }
                col[(j + 1) * NT] = x;
            }
            for (int32_t i = 0; i < nc;) {
                int32_t j = i + 1;
                while (j < nc && col[j * NT] == col[i * NT]) ++j;
                np += (j - i) >= sa;
                i = j;
            }
        }
        if (act && A.mode != kModeFill) A.task_cnt[t] = np;
        // where this lane's pairs go
        int32_t *dst_a = nullptr, *dst_b = nullptr, *dst_w = nullptr;
        int64_t at = 0;
        int32_t shift = 0;
        if (A.mode == kModeFill) {
            if (act && np) {
                const OutDst od = out_dst(A, a, A.task_off[t]);
                dst_a = od.a;
                dst_b = od.b;
                dst_w = od.w;
                at = od.base;
                shift = od.shift;
            }
        } else if (A.mode == kModeStage) {
            // pairs and records before this lane in the workgroup
            int32_t pb, pstep;
            wave_bits_prefix(np, 6, pb, pstep);
            const uint64_t hm = __ballot(np > 0);
            if (lane == 0) {
                red[0][wid] = pstep;
                red[1][wid] = (int32_t)__popcll(hm);
            }
            __syncthreads();
            int32_t pbefore = pb, rbefore = (int32_t)lanes_below(hm), total = 0, nrec = 0;
            for (int w = 0; w < NT / kWave; ++w) {
                if (w < wid) {
                    pbefore += red[0][w];
                    rbefore += red[1][w];
                }
                total += red[0][w];
                nrec += red[1][w];
            }
            if (tid == 0) {
                uint64_t off = 0;
                int32_t rec = 0;
                const bool ok = total > 0 && stage_reserve(A, pool_cur, log_cur, total, nrec, off, rec);
                res[0] = ok ? 1 : 0;
                res[1] = (int32_t)(uint32_t)(off & 0xffffffffull);
                res[2] = (int32_t)(uint32_t)(off >> 32);
                res[3] = rec;
            }
            __syncthreads();
            if (act && np) {
                if (res[0]) {
                    const int64_t off = (int64_t)(((uint64_t)(uint32_t)res[2] << 32) |
                                                  (uint64_t)(uint32_t)res[1]);
                    at = off + pbefore;
                    dst_b = A.pool_b;
                    dst_w = A.pool_w;
                    StageRec rec;
                    rec.off = at;
                    rec.t = t;
                    rec.rel = 0;
                    rec.n = np;
                    rec.pad = 0;
                    A.log[res[3] + rbefore] = rec;
                } else if (atomicExch(&A.need[t], 1) == 0) {
                    atomicAdd(A.need_count, 1);  // counted again by the fill pass
                }
            }
            __syncthreads();  // res and red are rewritten by the next round
        }
        if (dst_b) {
            int32_t q = 0;
            for (int32_t i = 0; i < nc;) {
                int32_t j = i + 1;
                const int32_t b = col[i * NT];
                while (j < nc && col[j * NT] == b) ++j;
                if (j - i >= sa) {
                    if (dst_a) dst_a[at + q] = a - shift;
                    dst_b[at + q] = dst_a ? item_of(A, b) - shift : b;
                    if (dst_w) dst_w[at + q] = j - i;
                    ++q;
                }
                i = j;
            }
        }
    }
}

// --------------------------------------------------------------- tasks

// SLOTS: home slots of the workgroup's table (Tuning::task_slots); MINB:
// waves per SIMD the register budget is planned for (the table's LDS allows
// no more); NT: threads per workgroup.
template <int SLOTS, int MINB, int NT>
__global__ __launch_bounds__(NT, MINB) void k_count_tasks(CountArgs A) {
    constexpr int LIM = SLOTS + kTaskPad;
    __shared__ __align__(16) uint32_t tab[LIM + kWave];
    __shared__ int2 runs[kTaskRunCap];
    __shared__ int32_t taken[kTaskRunCap];
    __shared__ int2 stack[kStack];
    __shared__ int32_t misc[kMiscWave + NT / kWave];
    __shared__ int32_t sh_task;
    __shared__ uint64_t pool_cur[3];
    __shared__ int32_t log_cur[3];
    const Smem S{tab, runs, taken, misc, stack, tab + LIM, pool_cur, log_cur};
    if (count_idle(A)) return;  // uniform: every thread reads the same words
    use_ranks(A);
    if (threadIdx.x == 0) {
        stage_begin(A, kKindGroups, pool_cur, log_cur);
    }
    tab_clear<NT>(tab, LIM);
    const int32_t n_groups = A.task_counts[kKindGroups * kCountStride];
    int64_t passes = 0;
    int64_t my_wedges = 0, my_nnz = 0, my_pairs = 0;
    __syncthreads();
    for (;;) {
        if (threadIdx.x == 0) sh_task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int32_t r = sh_task;
        __syncthreads();
        if (r >= n_groups) break;
        const int32_t t0 = A.big_tasks[r];
        const int32_t a = A.task_item[t0];
        const int32_t p0 = A.task_part[t0];
        const int32_t P = task_parts(A.cost[a], A.tune.small_max_wedges, A.tune.task_wedges,
                                     item_span(A.crank, A.item_end, A.N, A.full, a),
                                     A.ptrI[a + 1] - A.ptrI[a], A.tune.dense_min_wedges,
                                     SLOTS);
        const int32_t p1 = min(P, p0 + A.tune.group_parts);
        const int32_t k0 = A.ptrI[a], k1 = A.ptrI[a + 1];
        const int32_t cb = count_bits(k1 - k0);
        const int32_t sa = A.s_item ? A.s_item[a] : A.s;
        const int32_t first = cand_first(A.crank, A.full, a);
        const int32_t nend = cand_end(A.crank, A.item_end, A.N, a);
        int32_t cur[kR], end[kR];
        uint32_t lookm = 0;
        bool fresh = true;  // cursors must be placed at the range start
        for (int32_t q = p0; q < p1; ++q) {
            int32_t lo, hi;
            task_range(first, nend, q, P, lo, hi);
            const int32_t t = t0 + (q - p0);
            if (A.mode == kModeFill && A.need && !A.need[t]) {
                fresh = true;
                continue;
            }
            if (fresh) {
                init_cursors<NT>(A, first, lo, k0, k1, cur, end, lookm);
                if (q == 0 && A.mode != kModeFill) {
                    // work figures of this kernel: the item's incidences and wedges
#pragma unroll
                    for (int i = 0; i < kR; ++i) my_wedges += end[i] - cur[i];
                    for (int32_t k = k0 + (int32_t)threadIdx.x + kR * NT; k < k1; k += NT)
                        my_wedges += A.ptrS[A.memI[k] + 1] - (A.start[k] & kStartMask);
                    my_nnz += k1 - k0;
                }
            }
            fresh = false;
            const int64_t produced = run_range<NT, kTaskPad, kTaskRunCap>(
                A, S, a, sa, nend, t, lo, hi, SLOTS, cb, k0, k1, cur, end, lookm, passes);
            if (A.mode != kModeFill && threadIdx.x == 0) {
                A.task_cnt[t] = (int32_t)produced;
                my_pairs += produced;
            }
        }
        __syncthreads();
    }
    if (A.passes && A.mode != kModeFill) {
        // one atomic per counter and workgroup (same-address atomics serialize)
        unsigned long long *wk = stat_row(A);
        int64_t w = my_wedges;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) w += __shfl_xor(w, d, kWave);
        __shared__ int64_t red[NT / kWave];
        if (lane_id() == 0) red[threadIdx.x / kWave] = w;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t t = 0;
            for (int i = 0; i < NT / kWave; ++i) t += red[i];
            if (t) atomicAdd(&wk[2], (unsigned long long)t);
            if (my_nnz) atomicAdd(&wk[1], (unsigned long long)my_nnz);
            if (my_pairs) atomicAdd(&wk[3], (unsigned long long)my_pairs);
        }
    }
    if (threadIdx.x == 0 && passes && A.passes)
        atomicAdd(stat_row(A), (unsigned long long)passes);
}

// ----------------------------------------------------------- task lists

__device__ __forceinline__ int32_t plan_parts(const PlanItems &I, int64_t cost, int32_t a) {
    return task_parts(cost, I.small_max, I.target,
                      item_span(I.crank, I.item_end, I.N, I.full, a), I.ptrI[a + 1] - I.ptrI[a],
                      I.dense_min, I.slots);
}

// A tiny item: one task, at most kTinyCap members and tiny_max wedges, or with
// s > 2, where few pairs are left to write, three times as many, outside
// product mode (see k_count_tiny).
__device__ __forceinline__ bool is_tiny(const PlanItems &I, int32_t a, int64_t c,
                                        int32_t tiny_max) {
    if (I.full || c > 3 * tiny_max || I.ptrI[a + 1] - I.ptrI[a] > kTinyCap) return false;
    return c <= tiny_max || (I.s_item ? I.s_item[a] : I.s) > 2;
}

// Tasks of item a and the kind of kernel that counts them.
__device__ __forceinline__ int32_t item_tasks(const PlanItems &I, int32_t a, int64_t c,
                                              int32_t tiny_max, int32_t &kind, int32_t &ranges) {
    ranges = 0;
    kind = kKindTiny;
    if (c > 0 && c <= I.small_max && is_tiny(I, a, c, tiny_max)) return 1;
    const int32_t direct = direct_tasks(I, a, c, kind, ranges);
    if (direct > 0) return direct;
    kind = c > I.small_max ? kKindGroups : kKindSmall;
    return plan_parts(I, c, a);
}

__global__ __launch_bounds__(256) void k_task_count(const int64_t *cost, PlanItems I,
                                                    int32_t tiny_max, int32_t bound,
                                                    int32_t *ntask, int64_t *sums) {
    I.crank = ranks_or_null(I.crank, I.N);
    __shared__ int32_t sh[1 + kKinds];
    if (threadIdx.x < 1 + kKinds) sh[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < I.N;
         base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = base + threadIdx.x;
        int32_t kind = -1, r = 0;
        if (i < I.N) {
            const int32_t a = (int32_t)i;
            const int64_t c = cost[a];
            int32_t n = item_tasks(I, a, c, tiny_max, kind, r);
            if (n == 0) kind = -1;
            // at a larger s the item's cost is no higher, but its ranges may
            // come to have too few wedges to be counted directly, and the
            // other way round; either way it has at most one task per
            // `target` wedges
            if (bound && c > 0)
                n = max(n, (int32_t)min((c + I.target - 1) / I.target, (int64_t)INT32_MAX));
            ntask[a] = n;
        }
        r = wave_total(r);
        if (lane_id() == 0 && r) atomicAdd(&sh[0], r);
#pragma unroll
        for (int k = 0; k < kKinds; ++k) {
            const int32_t n = (int32_t)__popcll(__ballot(kind == k));
            if (lane_id() == 0 && n) atomicAdd(&sh[1 + k], n);
        }
    }
    __syncthreads();
    // one atomic per sum and block (same-address atomics serialize)
    if (threadIdx.x < 1 + kKinds && sh[threadIdx.x])
        atomicAdd((unsigned long long *)&sums[(blockIdx.x % kSumRows) * kTotalCols + threadIdx.x],
                  (unsigned long long)sh[threadIdx.x]);
}

// counts[kind * kCountStride] receives the length of each kind's list.
//
// Each workgroup fills the tasks of a contiguous chunk of items.  The slots
// of the two lists are claimed with one global atomic per list and workgroup
// (same-address atomics serialize), then handed out inside the workgroup
// with LDS atomics, one per wave and step.
__global__ __launch_bounds__(256) void k_task_fill(
    const int64_t *cost, PlanItems I, int32_t tiny_max, int32_t group, const int64_t *tbase,
    int32_t *task_item, int32_t *task_part, int32_t *small_tasks, int32_t *small_items,
    int32_t *tiny_tasks, int32_t *tiny_items, int32_t *groups, int32_t cap, int32_t *counts,
    int32_t chunk, const int32_t *abort) {
    if (abort && *abort != 0) return;
    I.crank = ranks_or_null(I.crank, I.N);
    const int32_t N = I.N;
    __shared__ int32_t sh[kKinds];
    const int lane = lane_id();
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < N ? lo + chunk : N;
    if (threadIdx.x < kKinds) sh[threadIdx.x] = 0;
    __syncthreads();
    // list entries of n tasks of a kind: task groups hold several
    auto entries = [&](int32_t kind, int32_t n) {
        return kind == kKindGroups ? (n + group - 1) / group : n;
    };
    // pass 1: list entries of the chunk
    int32_t ne[kKinds] = {};
    for (int64_t a = lo + threadIdx.x; a < hi; a += blockDim.x) {
        int32_t kind, ranges;
        const int32_t n = item_tasks(I, (int32_t)a, cost[a], tiny_max, kind, ranges);
        const int32_t e = entries(kind, n);
#pragma unroll
        for (int k = 0; k < kKinds; ++k) ne[k] += k == kind ? e : 0;
    }
#pragma unroll
    for (int k = 0; k < kKinds; ++k) {
        const int32_t n = wave_total(ne[k]);
        if (lane == 0 && n) atomicAdd(&sh[k], n);
    }
    __syncthreads();
    if (threadIdx.x < kKinds && sh[threadIdx.x])
        sh[threadIdx.x] = atomicAdd(&counts[threadIdx.x * kCountStride], sh[threadIdx.x]);
    __syncthreads();
    // pass 2: tasks, and the list entries at the claimed slots
    for (int64_t base = lo + (threadIdx.x & ~(kWave - 1)); base < hi; base += blockDim.x) {
        const int64_t a = base + lane;
        int32_t n = 0, kind = -1, ranges;
        int64_t t0 = 0;
        if (a < hi) {
            n = item_tasks(I, (int32_t)a, cost[a], tiny_max, kind, ranges);
            if (n > 0) t0 = tbase[a];
        }
        for (int32_t p = 0; p < n; ++p) {
            task_item[t0 + p] = (int32_t)a;
            task_part[t0 + p] = p;
        }
        // this lane's first entry in the list of its kind
        int32_t at = 0;
#pragma unroll
        for (int k = 0; k < kKinds; ++k) {
            const bool is = n > 0 && kind == k;
            const uint64_t m = __ballot(is);
            if (m == 0) continue;
            const bool several = k == kKindGroups || k == kKindFlat;
            const int32_t e = is ? entries(k, n) : 0;
            const int32_t incl = several ? wave_incl(e) : (int32_t)lanes_below(m) + e;
            const int32_t tot = several ? lane63(incl) : (int32_t)__popcll(m);
            int32_t first = 0;
            if (lane == 0) first = atomicAdd(&sh[k], tot);
            first = uniform(first);
            if (is) at = first + incl - e;
        }
        if (n == 0) continue;
        if (kind == kKindSmall) {
            small_tasks[at] = (int32_t)t0;
            small_items[at] = (int32_t)a;
        } else if (kind == kKindTiny) {
            tiny_tasks[at] = (int32_t)t0;
            tiny_items[at] = (int32_t)a;
        } else if (kind == kKindSieve1) {
            small_tasks[cap - 1 - at] = (int32_t)a;
        } else if (kind == kKindSieve4) {
            tiny_tasks[cap - 1 - at] = (int32_t)a;
        } else if (kind == kKindMini) {
            small_items[cap - 1 - at] = (int32_t)a;
        } else if (kind == kKindFlat) {
            for (int32_t p = 0; p < n; ++p) groups[cap - 1 - (at + p)] = (int32_t)(t0 + p);
        } else {
            for (int32_t g = 0; g * group < n; ++g)
                groups[at + g] = (int32_t)(t0 + (int64_t)g * group);
        }
    }
}

__global__ void k_reset_queue(int32_t *q) { q[0] = q[1] = 0; }

// One wave per staged range (grid-stride): pool -> final (a, b, w).
// A record as the stage pass wrote it, checked all the same: it guards the
// indices the copy uses.
__device__ __forceinline__ bool stage_rec_ok(const CountArgs &A, const StageRec &rec) {
    return rec.t >= 0 && rec.t < A.n_tasks && rec.n >= 0 && rec.off >= 0 &&
           rec.off + rec.n <= A.pool_cap;
}

// Records of at most this many pairs are copied by one lane each (a task of a
// tiny or small item stages a handful of pairs); longer ones by a whole wave.
constexpr int32_t kLaneRec = 32;

__global__ __launch_bounds__(256) void k_stage_copy(CountArgs A, int32_t n_rec) {
    if (A.abort && *A.abort != 0) return;
    use_ranks(A);
    if (n_rec < 0) n_rec = min(A.log_own + *A.log_head, A.log_cap);
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / kWave;
    // short records: one lane each
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n_rec;
         r += (int64_t)gridDim.x * blockDim.x) {
        const StageRec rec = A.log[r];
        if (rec.n > kLaneRec) continue;  // a wave's, below
        if (!stage_rec_ok(A, rec)) {
            atomicOr(A.err, kErrInternal);
            continue;
        }
        if (rec.n == 0 || A.need[rec.t]) continue;
        const int32_t a = A.task_item[rec.t];
        const int64_t dst = A.task_off[rec.t] + rec.rel;
        if (rec.rel < 0 || dst + rec.n > A.task_off[rec.t + 1]) {
            atomicOr(A.err, kErrInternal);
            continue;
        }
        const OutDst od = out_dst(A, a, dst);
        for (int32_t i = 0; i < rec.n; ++i) {
            od.a[od.base + i] = a - od.shift;
            od.b[od.base + i] = item_of(A, A.pool_b[rec.off + i]) - od.shift;
            if (od.w) od.w[od.base + i] = A.pool_w[rec.off + i];
        }
    }
    // long records: one wave each
    for (int64_t r = wave; r < n_rec; r += nwaves) {
        const StageRec rec = A.log[r];
        if (rec.n <= kLaneRec) continue;  // copied above
        if (!stage_rec_ok(A, rec)) {
            if (lane == 0) atomicOr(A.err, kErrInternal);
            continue;
        }
        if (A.need[rec.t]) continue;
        const int32_t a = A.task_item[rec.t];
        const int64_t dst = A.task_off[rec.t] + rec.rel;
        if (rec.rel < 0 || dst + rec.n > A.task_off[rec.t + 1]) {
            if (lane == 0) atomicOr(A.err, kErrInternal);
            continue;
        }
        const OutDst od = out_dst(A, a, dst);
        // four loads per lane in flight before the stores
        for (int32_t i0 = 0; i0 < rec.n; i0 += 4 * kWave) {
            int32_t bv[4], wv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t i = i0 + u * kWave + lane;
                bv[u] = 0;
                wv[u] = 0;
                if (i < rec.n) {
                    bv[u] = item_of(A, A.pool_b[rec.off + i]);
                    if (od.w) wv[u] = A.pool_w[rec.off + i];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t i = i0 + u * kWave + lane;
                if (i < rec.n) {
                    od.a[od.base + i] = a - od.shift;
                    od.b[od.base + i] = bv[u] - od.shift;
                    if (od.w) od.w[od.base + i] = wv[u];
                }
            }
        }
    }
}

inline int grid_for(int64_t work, int per_block, int cap) {
    int64_t g = (work + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

}  // namespace

hipError_t launch_task_count(hipStream_t st, const int64_t *cost, const PlanItems &I,
                             int32_t tiny_max, int32_t *ntask, int64_t *sums, int32_t bound) {
    if (I.N <= 0) return hipSuccess;
    k_task_count<<<grid_for(I.N, 256, 2048), 256, 0, st>>>(cost, I, tiny_max, bound, ntask, sums);
    return hipGetLastError();
}

hipError_t launch_task_fill(hipStream_t st, const int64_t *cost, const PlanItems &I,
                            int32_t tiny_max, int32_t group, const int64_t *tbase,
                            int32_t *task_item, int32_t *task_part, int32_t *small_tasks,
                            int32_t *small_items, int32_t *tiny_tasks, int32_t *tiny_items,
                            int32_t *big_tasks, int32_t cap, int32_t *counts,
                            const int32_t *abort) {
    if (I.N <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>(1024, ((int64_t)I.N + 255) / 256);
    const int32_t chunk = (int32_t)((((int64_t)I.N + blocks - 1) / blocks + 255) / 256 * 256);
    const int64_t grid = ((int64_t)I.N + chunk - 1) / chunk;
    k_task_fill<<<(unsigned)grid, 256, 0, st>>>(cost, I, tiny_max, std::max(1, group), tbase,
                                                task_item, task_part, small_tasks, small_items,
                                                tiny_tasks, tiny_items, big_tasks, cap, counts,
                                                chunk, abort);
    return hipGetLastError();
}

hipError_t launch_count(hipStream_t st, const CountArgs &A, hipEvent_t mid) {
    if (A.N <= 0) return hipSuccess;
    const int32_t *g = A.grid;
    if (g[kKindTiny] > 0 && A.tune.tiny_max_wedges > 0 && !A.full)
        k_count_tiny<<<g[kKindTiny], kTinyThreads, 0, st>>>(A);
    if (g[kKindSmall] > 0) {
        switch (A.tune.small_slots) {
        case 512: k_count_small<512><<<g[kKindSmall], kWave, 0, st>>>(A); break;
        case 2048: k_count_small<2048><<<g[kKindSmall], kWave, 0, st>>>(A); break;
        default: k_count_small<1024><<<g[kKindSmall], kWave, 0, st>>>(A); break;
        }
    }
    const bool fill = A.mode == kModeFill;
    if (g[kKindMini] > 0) {
        constexpr int LIM = 2 * kMiniWedges + kTaskPad, CHUNKS = kMiniWedges / kWave;
        auto *const count = fill ? k_count_item<kKindMini, kWave, LIM, CHUNKS, 7, true>
                                 : k_count_item<kKindMini, kWave, LIM, CHUNKS, 7, false>;
        count<<<g[kKindMini], kWave, 0, st>>>(A);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g[kKindGroups] > 0 || g[kKindFlat] > 0) k_reset_queue<<<1, 1, 0, st>>>(A.queue);
    if (mid) {
        e = hipEventRecord(mid, st);
        if (e != hipSuccess) return e;
    }
    if (g[kKindFlat] > 0) {
        e = launch_count_flat(st, A);
        if (e != hipSuccess) return e;
    }
    if (g[kKindSieve4] > 0) {
        constexpr int LIM = kSieveLarge * 16, CHUNKS = kSieveLarge * kSieveWedges / kWave;
        auto *const count = fill ? k_count_item<kKindSieve4, kSieveLarge, LIM, CHUNKS, 4, true>
                                 : k_count_item<kKindSieve4, kSieveLarge, LIM, CHUNKS, 4, false>;
        count<<<g[kKindSieve4], kSieveLarge, 0, st>>>(A);
    }
    if (g[kKindSieve1] > 0) {
        constexpr int LIM = kSieveSmall * 16, CHUNKS = kSieveSmall * kSieveWedges / kWave;
        auto *const count = fill ? k_count_item<kKindSieve1, kSieveSmall, LIM, CHUNKS, 4, true>
                                 : k_count_item<kKindSieve1, kSieveSmall, LIM, CHUNKS, 4, false>;
        count<<<g[kKindSieve1], kSieveSmall, 0, st>>>(A);
    }
    if (g[kKindGroups] > 0) {
        const int gh = g[kKindGroups];
        switch (A.tune.task_slots) {
        case 4480: k_count_tasks<4480, 4, 256><<<gh, 256, 0, st>>>(A); break;
        case 13440: k_count_tasks<13440, 2, 256><<<gh, 256, 0, st>>>(A); break;
        // twice the table and twice the threads: two workgroups per CU keep
        // four waves per SIMD, as four of 256 threads do
        case 17920: k_count_tasks<17920, 4, 512><<<gh, 512, 0, st>>>(A); break;
        default: k_count_tasks<8960, 4, 256><<<gh, 256, 0, st>>>(A); break;
        }
    }
    return hipGetLastError();
}

int32_t set_grids(CountArgs &A, const int64_t *items) {
    // workgroups a CU holds: tiny four (32 KB of LDS each), item kernels 28 of one
    // wave (registers; 20 where items are few, as each costs room in the pool), 15
    // and four (LDS), direct counters two; the hashed kernels as tuned
    const int per_cu[kKinds] = {A.tune.small_grid_per_cu, A.tune.task_grid_per_cu, 4, 2, 15, 4, 20};
    // Item kernels share their items out evenly, but not their time: with just the
    // workgroups that fit, few were left at work in the end (2.1 of 3.75 waves per
    // SIMD in the mean).  So several rounds of them, as long as each has
    // kRoundItems items to take; 128 graphs: sieve of one wave 3.4 ms in one
    // round, 2.3 in four; up to 256 wedges 1.8 and 1.6; 10^6 hyperedges, sieve of
    // four waves 6.5 and 6.0.  More rounds gained little and cost room
    // in pool and log.
    constexpr int kRounds[kKinds] = {1, 1, 2, 1, 6, 4, 5};
    constexpr int64_t kRoundItems = 8;
    int32_t total = 0;
    for (int k = 0; k < kKinds; ++k) {
        int64_t g = std::max(1, A.n_cu * per_cu[k]);
        const int64_t n = k == kKindTiny ? (items[k] + kTinyThreads - 1) / kTinyThreads : items[k];
        g = std::max(g, std::min(g * kRounds[k], n / kRoundItems));
        // items in groups or ranges take several workgroups each
        if (n == 0 || (k != kKindGroups && k != kKindFlat)) g = std::min(g, n);
        A.grid[k] = (int32_t)g;
        total += (int32_t)g;
    }
    return total;
}

void set_chunks(CountArgs &A) {
    // Chunks so small that a kind's workgroups hold a share of pool and log: 1/16
    // for the kernels whose ranges bring many pairs (so that what is left of a
    // chunk when the next range does not fit it is little), 1/64 for the others.
    int64_t pool = 0, log = 0;
    for (int k = 0; k < kKinds; ++k) {
        const bool big = k == kKindGroups || k == kKindFlat || k == kKindSieve4;
        const int64_t parts = (big ? 16 : 64) * std::max<int64_t>(A.grid[k], 1);
        A.pool_chunk[k] =
            std::max<int64_t>(kPoolChunkMin, std::min<int64_t>(1 << 16, A.pool_cap / parts));
        A.log_chunk[k] =
            (int32_t)std::max<int64_t>(8, std::min<int64_t>(256, (int64_t)A.log_cap / parts));
        A.pool_first[k] = pool;
        A.log_first[k] = (int32_t)log;
        pool += A.pool_chunk[k] * A.grid[k];
        log += (int64_t)A.log_chunk[k] * A.grid[k];
    }
    // first chunks without atomics, where that leaves room for others
    const bool fits = A.mode == kModeStage && pool * 2 <= A.pool_cap && log * 2 <= A.log_cap;
    A.pool_own = fits ? pool : 0;
    A.log_own = fits ? (int32_t)log : 0;
}

hipError_t launch_stage_copy(hipStream_t st, const CountArgs &A, int32_t n_rec) {
    if (n_rec == 0 || (n_rec < 0 && A.log_cap <= 0)) return hipSuccess;
    const int64_t most = n_rec < 0 ? A.log_cap : n_rec;
    k_stage_copy<<<grid_for(most * kWave, 256, 16384), 256, 0, st>>>(A, n_rec);
    return hipGetLastError();
}

}  // namespace sl
