// The claim-word push: the masked product x_{k+1} = A^T[V_{k+1}, V_k] x_k of
// Theorem 1 with the visited mask and the parent select folded into one
// 64-bit word per vertex.
//
// Word w(v) = (level << 32) | parent; while v is unreached its top bit is set
// (above every offer).  At level k, frontier column u offers the key
// ((k + 1) << 32) | u to every row v it holds, by atomicMin on w(v):
//   - a row visited at level <= k has a smaller word: the offer changes nothing
//     (the mask V_{k+1} of the product);
//   - an unreached row keeps the smallest key offered during the level, i.e.
//     the smallest frontier in-neighbour (the min-parent reading of the
//     paper's Algorithm 3 parent array);
//   - the one atomic that finds the top bit set lists v for the next level, so every
//     reached vertex is listed once (Theorem 2's single claim per row).
// Nothing else needs a barrier inside a level, and the level and parent of a
// vertex are never written before its final value is known: a pass at the
// end splits the words into the callers' level and parent arrays.
//
// Three forms:
//   - deep (thin graphs: every out-degree at most 8 - grids, road-like graphs,
//     thousands of thin levels): waves go on from their share of the list by
//     themselves for up to 128 levels, the rows they improve queued in LDS, with
//     no barrier and no launch between levels;
//   - narrow: one workgroup of 1024 threads runs level after level with the
//     frontier in LDS (up to 8192 columns and 2^16 entries per level), so a
//     level costs a few dependent memory round trips and a workgroup barrier
//     instead of a grid-wide launch (the first and last levels of the others);
//   - wide: a launch per level over the frontier lists in global memory
//     (short columns a lane each, long ones in chunks of 1024 entries a wave
//     each, as the paper's work-splitting of long columns suggests).
// Several queries on different graphs share the launches: query q owns the
// virtual ids [base_q, base_q + n_q), its words, and its graph's arrays.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bfs_device.h"
#include "bfs_internal.h"

namespace bfsi {

namespace {

// Unreached words have the top bit set (no offer has it: levels stay below
// 2^31); bit 62 is clear for the rows of kCwLong entries or more, so the offer
// that reaches a row learns its class without reading its column pointers.
constexpr unsigned long long kUnreached = ~0ull;
constexpr unsigned long long kUnreachedLong = ~0ull ^ (1ull << 62);
__device__ __forceinline__ bool unreached(unsigned long long w) { return (w >> 63) != 0ull; }
__device__ __forceinline__ bool long_row(unsigned long long w) { return ((w >> 62) & 1ull) == 0ull; }
constexpr uint32_t kCwGroup = 4;               // narrow: columns a thread expands at once
constexpr uint32_t kCwUnroll = 4;              // wide: entries a lane offers at once
constexpr uint32_t kCwStage = 512;             // wide: a wave's staged appends (LDS entries)

__device__ __forceinline__ unsigned long long offer_key(uint32_t level, uint32_t u) {
    return ((unsigned long long)level << 32) | u;
}

// The query owning virtual id x: the last q with bases[q] <= x.
__device__ __forceinline__ uint32_t query_of(const CwParams &P, uint32_t x) {
    if (P.nq == 1) return 0;
    uint32_t lo = 0, hi = P.nq;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (P.bases[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

struct Col {                                   // a frontier column
    const int32_t *ptr, *idx;                  // its graph
    uint32_t base;                             // its query's first virtual id
    uint32_t u;                                // its vertex (graph-local)
    int32_t r0;                                // its first entry
    uint32_t deg;                              // its entries
};

__device__ __forceinline__ Col column(const CwParams &P, uint32_t x) {
    const CwQuery &Q = P.q[query_of(P, x)];
    Col c;
    c.ptr = Q.out_ptr;
    c.idx = Q.out_idx;
    c.base = Q.base;
    c.u = x - Q.base;
    c.r0 = c.ptr[c.u];
    c.deg = (uint32_t)(c.ptr[c.u + 1] - c.r0);
    return c;
}

// Append x (with deg out-entries) to the level list of count slot t, called
// by every lane of the wave (own = lane has a vertex); short columns through
// one atomic per wave, long ones (with their chunk map) per lane.
__device__ __forceinline__ void append_wide(const CwParams &P, const CwLists &L, uint32_t t, bool own,
                                            uint32_t x, uint32_t deg) {
    CwState *st = P.st;
    const bool sh = own && deg < kCwLong;
    const unsigned long long bm = __ballot(sh);
    if (bm) {
        const uint32_t leader = (uint32_t)__ffsll((long long)bm) - 1u;
        uint32_t base = 0;
        if (lane_id() == leader) base = atomicAdd(&st->cnt[t][0], (uint32_t)__popcll(bm));
        base = __shfl(base, (int)leader, 64);
        if (sh) L.s[base + lanes_below(bm)] = x;
    }
    if (own && deg >= kCwLong) {
        const uint32_t nch = (deg + kCwChunk - 1) / kCwChunk;
        const uint32_t li = atomicAdd(&st->cnt[t][1], 1u);
        const uint32_t cb = atomicAdd(&st->cnt[t][2], nch);
        L.l[li] = x;
        L.lbase[li] = cb;
        for (uint32_t c = 0; c < nch; ++c) L.cmap[cb + c] = li;
    }
}

struct Ref {                                   // a column's graph and query
    const int32_t *ptr, *idx;
    uint32_t base;
};

struct RowRef {                                // a thin graph's fixed-width rows and the query
    const int4 *rows;
    uint32_t base, quads;
};

template <bool kSingle>
__device__ __forceinline__ Ref ref_of(const CwParams &P, const Ref &one, uint32_t x) {
    if (kSingle) return one;
    const CwQuery &Q = P.q[query_of(P, x)];
    return Ref{Q.out_ptr, Q.out_idx, Q.base};
}

// An empty statement that takes x as read and rewritten: the results of a
// batch of atomics issued under each lane's own condition are first examined
// after every atomic of the batch is in flight (the compiler would otherwise
// examine each result inside its condition, right after its atomic, waiting
// for it there).  It emits no instruction.
__device__ __forceinline__ void settle_after_issue(unsigned long long &x) {
    asm volatile("" : "+v"(x));
}
__device__ __forceinline__ void settle_after_issue32(uint32_t &x) {
    asm volatile("" : "+v"(x));
}

// A wave's staging of the next level's short columns in LDS: appends are
// gathered here (a ballot and an LDS write per batch) and go to the global
// list kCwStage - 64 at a time, one counter atomic each (a per-append
// counter atomic would serialise every append of the level on one word).
struct Stage {
    uint32_t *buf;                             // the wave's kCwStage LDS entries
    uint32_t n;                                // entries held (uniform in the wave)
};

__device__ __forceinline__ void stage_flush(const CwParams &P, const CwLists &N, uint32_t t, Stage &S) {
    if (S.n == 0) return;
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&P.st->cnt[t][0], S.n);
    base = __shfl(base, 0, 64);
    for (uint32_t i = lane_id(); i < S.n; i += 64) N.s[base + i] = S.buf[i];
    S.n = 0;
}

// After an offer to row v (of column c's graph) that found word `old`: if
// the offer reached v first, list it for the next level (its class from the
// word; the entry count read only for the long ones).  Every lane calls it.
__device__ __forceinline__ void reach(const CwParams &P, const CwLists &N, uint32_t t, const Col &c, int32_t v,
                                      unsigned long long old, Stage &S) {
    const bool own = unreached(old);
    const bool lg = own && long_row(old);
    uint32_t deg = 0;
    if (lg) deg = (uint32_t)(c.ptr[v + 1] - c.ptr[v]);
    append_wide(P, N, t, lg, c.base + (uint32_t)v, deg);           // long rows (with their chunks)
    const bool sh = own && !lg;
    const unsigned long long bm = __ballot(sh);
    if (bm) {
        if (sh) S.buf[S.n + lanes_below(bm)] = c.base + (uint32_t)v;
        S.n += (uint32_t)__popcll(bm);
        if (S.n > kCwStage - 64) stage_flush(P, N, t, S);
    }
}

// kCwUnroll offers of one lane's column c at once: entries e0 + q * stride
// (those with ok[q]); their entry loads, word tests and atomics are each
// issued for the whole batch before the first result is used.  Every lane
// calls it.
__device__ __forceinline__ void offer_batch(const CwParams &P, const CwLists &N, uint32_t t, const Col &c,
                                            unsigned long long key, bool pre, const bool *ok, int32_t e0,
                                            int32_t stride, Stage &S) {
    int32_t v[kCwUnroll];
    unsigned long long old[kCwUnroll];
#pragma unroll
    for (uint32_t q = 0; q < kCwUnroll; ++q) {
        v[q] = 0;
        if (ok[q]) v[q] = c.idx[e0 + (int32_t)q * stride];
    }
    bool go[kCwUnroll];
#pragma unroll
    for (uint32_t q = 0; q < kCwUnroll; ++q) go[q] = ok[q];
    if (pre) {
        unsigned long long w[kCwUnroll];
#pragma unroll
        for (uint32_t q = 0; q < kCwUnroll; ++q) {
            w[q] = 0ull;
            if (ok[q]) w[q] = P.cw[c.base + (uint32_t)v[q]];
        }
#pragma unroll
        for (uint32_t q = 0; q < kCwUnroll; ++q) settle_after_issue(w[q]);
        // the words only decrease, so a stale copy is never below the true value
#pragma unroll
        for (uint32_t q = 0; q < kCwUnroll; ++q) go[q] = ok[q] && w[q] > key;
    }
#pragma unroll
    for (uint32_t q = 0; q < kCwUnroll; ++q) {
        old[q] = 0ull;
        if (go[q]) old[q] = atomicMin(&P.cw[c.base + (uint32_t)v[q]], key);
    }
#pragma unroll
    for (uint32_t q = 0; q < kCwUnroll; ++q) settle_after_issue(old[q]);
#pragma unroll
    for (uint32_t q = 0; q < kCwUnroll; ++q) reach(P, N, t, c, v[q], old[q], S);
}

// Exclusive prefix sum over the 1024 threads of the narrow workgroup; *total
// receives the sum.  Every thread calls it.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t *s_w, uint32_t *total) {
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(x);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        const uint32_t v = lane < kCwNarrowThreads / 64 ? s_w[lane] : 0u;
        const uint32_t vi = wave_incl_scan(v);
        if (lane < kCwNarrowThreads / 64) s_w[lane] = vi - v;
        if (lane == kCwNarrowThreads / 64 - 1) s_w[kCwNarrowThreads / 64] = vi;
    }
    __syncthreads();
    const uint32_t r = s_w[wave] + inc - x;
    *total = s_w[kCwNarrowThreads / 64];
    __syncthreads();
    return r;
}

}  // namespace

// Words to unreached (with the row class), every count zero, then the
// sources: word (0, s) and the level-0 lists.  A block row per query.
__global__ __launch_bounds__(kCwBlock) void k_cw_fill(CwParams P) {
    const CwQuery &Q = P.q[blockIdx.y];
    for (uint32_t v = blockIdx.x * kCwBlock + threadIdx.x; v < Q.n; v += gridDim.x * kCwBlock) {
        const uint32_t deg = (uint32_t)(Q.out_ptr[v + 1] - Q.out_ptr[v]);
        P.cw[Q.base + v] = deg >= kCwLong ? kUnreachedLong : kUnreached;
        if (P.stamp) P.stamp[Q.base + v] = 0u;
    }
    const uint32_t gid = (blockIdx.y == 0) ? blockIdx.x * kCwBlock + threadIdx.x : 0xFFFFFFFFu;
    if (gid < 12) P.st->cnt[gid / 4][gid % 4] = 0u;
    if (gid == 0) {
        P.st->level = 0u;
        P.st->done = 0u;
        P.st->last = 0u;
    }
}

__global__ __launch_bounds__(kCwBlock) void k_cw_roots(CwParams P) {
    const uint32_t q = blockIdx.x * kCwBlock + threadIdx.x;
    bool own = false;
    uint32_t x = 0, deg = 0;
    if (q < P.nq) {
        const CwQuery &Q = P.q[q];
        x = Q.base + (uint32_t)Q.source;
        P.cw[x] = offer_key(0u, (uint32_t)Q.source);
        deg = (uint32_t)(Q.out_ptr[Q.source + 1] - Q.out_ptr[Q.source]);
        own = true;
    }
    append_wide(P, P.lists[0], 0u, own, x, deg);
}

// Level k, wide form.  Items: the short columns, 64 to a wave (a lane each,
// entries taken in lockstep rounds so that the next level's appends gather
// per wave), then the chunks of the long columns (a wave each).  The atomic
// is skipped where the row's word is already at or below the offer.
__global__ __launch_bounds__(kCwBlock) void k_cw_wide(CwParams P, uint32_t k) {
    __shared__ uint32_t s_stage[kCwBlock / 64][kCwStage];
    CwState *st = P.st;
    const uint32_t t0 = k % 3, t1 = (k + 1) % 3, t2 = (k + 2) % 3;
    const CwLists C = P.lists[k & 1], N = P.lists[(k + 1) & 1];
    const uint32_t lane = lane_id();
    const uint32_t gw = blockIdx.x * (kCwBlock / 64) + (threadIdx.x >> 6);
    const uint32_t nw = gridDim.x * (kCwBlock / 64);
    // the lane's entry of the wave's first step, read together with the
    // counts (before it is known to exist: the list has room for V entries)
    // instead of one round trip after them
    const uint32_t i_first = gw * 64u + lane;
    uint32_t x_first = C.s[i_first < P.V ? i_first : 0u];
    const uint32_t ns = st->cnt[t0][0], nc = st->cnt[t0][2];
    settle_after_issue32(x_first);
    if (blockIdx.x == 0 && threadIdx.x < 4) st->cnt[t2][threadIdx.x] = 0u;   // level k+2's lists
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->level = k + 1;
        if (ns + nc != 0) st->last = k;                          // the deepest level with a frontier
    }
    const uint32_t sw = (ns + 63) / 64;
    // test the row's word before the atomic on wide levels (most rows are
    // settled there; the test saves their atomics), not on thin ones (where a
    // level's cost is its chain of dependent round trips)
    const bool pre = ns + 64u * nc >= kCwPrecheck;
    Stage S{s_stage[threadIdx.x >> 6], 0u};
    for (uint32_t it = gw; it < sw + nc; it += nw) {             // uniform per wave
        if (it < sw) {
            const uint32_t i = it * 64 + lane;
            Col c{};
            if (i < ns) c = column(P, it == gw ? x_first : C.s[i]);
            const unsigned long long key = offer_key(k + 1, c.u);
            const uint32_t rounds = (uint32_t)wave_max((int32_t)c.deg);
            for (uint32_t r = 0; r < rounds; r += kCwUnroll) {
                bool ok[kCwUnroll];
#pragma unroll
                for (uint32_t q = 0; q < kCwUnroll; ++q) ok[q] = r + q < c.deg;
                offer_batch(P, N, t1, c, key, pre, ok, c.r0 + (int32_t)r, 1, S);
            }
        } else {
            const uint32_t ch = it - sw;
            const uint32_t li = C.cmap[ch];
            const Col c = column(P, C.l[li]);
            const int32_t e0 = c.r0 + (int32_t)((ch - C.lbase[li]) * kCwChunk);
            const int32_t end = c.r0 + (int32_t)c.deg;
            const int32_t e1 = (e0 + (int32_t)kCwChunk < end) ? e0 + (int32_t)kCwChunk : end;
            const unsigned long long key = offer_key(k + 1, c.u);
            for (int32_t eb = e0; eb < e1; eb += 64 * (int32_t)kCwUnroll) {
                bool ok[kCwUnroll];
#pragma unroll
                for (uint32_t q = 0; q < kCwUnroll; ++q) ok[q] = eb + (int32_t)(q * 64u + lane) < e1;
                offer_batch(P, N, t1, c, key, pre, ok, eb + (int32_t)lane, 64, S);
            }
        }
    }
    stage_flush(P, N, t1, S);
}

// Levels in one workgroup, the frontier in LDS, from level k0 (listed in the
// global lists) until the search ends, a level is too wide (more than
// kCwCap columns, kCwLongCap columns of more than four entries or
// kCwNarrowEdges entries: its frontier goes back to the global lists
// unexpanded), or max_levels levels are done.  Per level: each thread takes
// up to kCwPer columns, kCwGroup at a time, reading their first four entries
// and making their offers with every load and atomic of the group in flight;
// the rest of the longer columns follow in 256-entry pieces, a wave each.
template <bool kSingle>
__global__ __launch_bounds__(kCwNarrowThreads) void k_cw_narrow(CwParams P, uint32_t k0, uint32_t max_levels,
                                                                uint32_t max_next, uint32_t max_edges) {
    __shared__ uint32_t s_f[2][kCwCap];        // frontier, next frontier (virtual ids)
    __shared__ uint32_t s_lx[kCwLongCap];      // columns of more than four entries
    __shared__ int32_t s_lr0[kCwLongCap];      //   their entries after the first four
    __shared__ uint32_t s_ldeg[kCwLongCap];
    __shared__ uint32_t s_lpre[kCwLongCap + 1];   // 256-entry pieces before each
    __shared__ uint32_t s_scan[kCwNarrowThreads / 64 + 1];
    __shared__ uint32_t s_n[2], s_nl, s_edges;
    __shared__ uint32_t s_cs, s_cl, s_cc;
    CwState *st = P.st;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const Ref one = Ref{P.q[0].out_ptr, P.q[0].out_idx, P.q[0].base};   // the query, when there is one
    uint32_t k = k0;
    {
        const uint32_t t0 = k % 3, ns = st->cnt[t0][0], nl = st->cnt[t0][1];
        if (ns + nl > kCwCap) return;                             // the host checks this first
        const CwLists C = P.lists[k & 1];
        for (uint32_t i = tid; i < ns + nl; i += kCwNarrowThreads) s_f[0][i] = i < ns ? C.s[i] : C.l[i - ns];
        if (tid == 0) s_n[0] = ns + nl;
    }
    __syncthreads();
    uint32_t cur = 0;
    // Hand frontier f (n columns: the first min(n, kCwCap) in LDS array
    // `lds`, the rest in P.spill) to the global lists of level `lv`.
    auto to_global = [&](const uint32_t *lds, uint32_t n, uint32_t lv) {
        const uint32_t t = lv % 3;
        const CwLists L = P.lists[lv & 1];
        if (tid == 0) {
            s_cs = 0;
            s_cl = 0;
            s_cc = 0;
        }
        __syncthreads();
        for (uint32_t i = tid; i < n; i += kCwNarrowThreads) {
            const uint32_t x = i < kCwCap ? lds[i] : P.spill[i - kCwCap];
            const Col c = column(P, x);
            if (c.deg < kCwLong) {
                L.s[atomicAdd(&s_cs, 1u)] = x;
            } else {
                const uint32_t nch = (c.deg + kCwChunk - 1) / kCwChunk;
                const uint32_t li = atomicAdd(&s_cl, 1u);
                const uint32_t cb = atomicAdd(&s_cc, nch);
                L.l[li] = x;
                L.lbase[li] = cb;
                for (uint32_t j = 0; j < nch; ++j) L.cmap[cb + j] = li;
            }
        }
        __syncthreads();
        if (tid == 0) {
            st->cnt[t][0] = s_cs;
            st->cnt[t][1] = s_cl;
            st->cnt[t][2] = s_cc;
            for (int j = 0; j < 3; ++j) {
                st->cnt[(lv + 1) % 3][j] = 0u;
                st->cnt[(lv + 2) % 3][j] = 0u;
            }
            st->level = lv;
        }
    };
    for (uint32_t done = 0;; ++done, ++k) {
        const uint32_t nf = s_n[cur];
        if (nf == 0) {
            if (tid == 0) {
                for (int t = 0; t < 3; ++t)
                    for (int j = 0; j < 3; ++j) st->cnt[t][j] = 0u;
                st->level = k;
                st->done = 1u;
            }
            return;
        }
        if (done == max_levels) {
            to_global(s_f[cur], nf, k);
            return;
        }
        if (tid == 0) {
            s_nl = 0;
            s_edges = 0;
            s_n[cur ^ 1] = 0;
        }
        __syncthreads();
        // The level's columns: extents, width.  Loads are issued under a
        // lane's own condition with the result left in place otherwise, and
        // nothing reads a result before every load of the batch is issued, so
        // the batch's loads are in flight together.
        uint32_t xs[kCwPer];
        int32_t r0s[kCwPer];
        uint32_t degs[kCwPer];
        Ref refs[kCwPer];
        uint32_t my_edges = 0;
#pragma unroll
        for (uint32_t j = 0; j < kCwPer; ++j) {
            const uint32_t i = tid + j * kCwNarrowThreads;
            xs[j] = s_f[cur][i < nf ? i : 0u];
            refs[j] = ref_of<kSingle>(P, one, xs[j]);
        }
        int32_t pa[kCwPer], pb[kCwPer];
#pragma unroll
        for (uint32_t j = 0; j < kCwPer; ++j) {
            pa[j] = 0;
            pb[j] = 0;
            if (tid + j * kCwNarrowThreads < nf) {
                const uint32_t u = xs[j] - refs[j].base;
                pa[j] = refs[j].ptr[u];
                pb[j] = refs[j].ptr[u + 1];
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kCwPer; ++j) {
            r0s[j] = pa[j];
            degs[j] = (uint32_t)(pb[j] - pa[j]);
            my_edges += degs[j];
            if (my_edges > kCwNarrowEdges) my_edges = kCwNarrowEdges + 1u;   // saturate
            if (degs[j] > 4u) {
                const uint32_t li = atomicAdd(&s_nl, 1u);
                if (li < kCwLongCap) {
                    s_lx[li] = xs[j];
                    s_lr0[li] = r0s[j] + 4;
                    s_ldeg[li] = degs[j] - 4u;
                }
            }
        }
        if (my_edges) atomicAdd(&s_edges, my_edges);
        __syncthreads();
        if (s_edges > max_edges || s_nl > kCwLongCap) {            // too wide: back to the lists
            to_global(s_f[cur], nf, k);
            return;
        }
        const uint32_t nl = s_nl;
        uint32_t *nxt = s_f[cur ^ 1];
        // the first four entries of every column, kCwGroup columns at a time
#pragma unroll
        for (uint32_t g0 = 0; g0 < kCwPer; g0 += kCwGroup) {
            int32_t v[kCwGroup][4];
            unsigned long long old[kCwGroup][4];
#pragma unroll
            for (uint32_t j = 0; j < kCwGroup; ++j)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    v[j][e] = -1;
                    if (e < degs[g0 + j]) v[j][e] = refs[g0 + j].idx[r0s[g0 + j] + (int32_t)e];
                }
#pragma unroll
            for (uint32_t j = 0; j < kCwGroup; ++j) {
                const unsigned long long key = offer_key(k + 1, xs[g0 + j] - refs[g0 + j].base);
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    old[j][e] = 0ull;
                    if (e < degs[g0 + j])
                        old[j][e] = atomicMin(&P.cw[refs[g0 + j].base + (uint32_t)v[j][e]], key);
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < kCwGroup; ++j)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) settle_after_issue(old[j][e]);
#pragma unroll
            for (uint32_t j = 0; j < kCwGroup; ++j)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (unreached(old[j][e])) {
                        const uint32_t pos = atomicAdd(&s_n[cur ^ 1], 1u);
                        const uint32_t x = refs[g0 + j].base + (uint32_t)v[j][e];
                        if (pos < kCwCap) nxt[pos] = x;
                        else P.spill[pos - kCwCap] = x;
                    }
        }
        // the rest of the longer columns: 256-entry pieces, a wave each
        if (nl) {
            uint32_t total = 0;
            // nl <= 2048: two columns per thread
            const uint32_t i0 = 2 * tid, i1 = 2 * tid + 1;
            const uint32_t p0 = i0 < nl ? (s_ldeg[i0] + 255u) / 256u : 0u;
            const uint32_t p1 = i1 < nl ? (s_ldeg[i1] + 255u) / 256u : 0u;
            const uint32_t ex = block_excl_scan(p0 + p1, s_scan, &total);
            if (i0 < nl) s_lpre[i0] = ex;
            if (i1 < nl) s_lpre[i1] = ex + p0;
            if (tid == 0) s_lpre[nl] = total;
            __syncthreads();
            for (uint32_t it = wave; it < total; it += kCwNarrowThreads / 64) {
                uint32_t lo = 0, hi = nl;                  // s_lpre[lo] <= it < s_lpre[hi]
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_lpre[mid] <= it) lo = mid;
                    else hi = mid;
                }
                const uint32_t x = s_lx[lo];
                const Ref r = ref_of<kSingle>(P, one, x);
                const int32_t e0 = s_lr0[lo] + (int32_t)((it - s_lpre[lo]) * 256u);
                const int32_t end = s_lr0[lo] + (int32_t)s_ldeg[lo];
                const unsigned long long key = offer_key(k + 1, x - r.base);
                int32_t vv[4];
                unsigned long long oo[4];
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    const int32_t ei = e0 + (int32_t)(e * 64u + lane);
                    vv[e] = -1;
                    if (ei < end) vv[e] = r.idx[ei];
                }
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) {
                    oo[e] = 0ull;
                    if (e0 + (int32_t)(e * 64u + lane) < end) oo[e] = atomicMin(&P.cw[r.base + (uint32_t)vv[e]], key);
                }
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) settle_after_issue(oo[e]);
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (unreached(oo[e])) {
                        const uint32_t pos = atomicAdd(&s_n[cur ^ 1], 1u);
                        const uint32_t y = r.base + (uint32_t)vv[e];
                        if (pos < kCwCap) nxt[pos] = y;
                        else P.spill[pos - kCwCap] = y;
                    }
            }
        }
        __syncthreads();
        if (s_n[cur ^ 1] > max_next) {                     // the next frontier is too wide
            to_global(nxt, s_n[cur ^ 1], k + 1);
            return;
        }
        cur ^= 1;
    }
}

// ---------------------------------------------------------------------------
// the deep form: many levels per launch, a wave at a time
// ---------------------------------------------------------------------------

// Orders a wave's LDS writes before the same wave's later LDS reads by other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A thin graph's out-lists in rows of `width` entries (4 or 8), -1 past a
// list's end.
__global__ __launch_bounds__(kCwBlock) void k_cw_rows(const int32_t *ptr, const int32_t *idx, int32_t n, int32_t width,
                                                      int32_t *rows) {
    const size_t stride = (size_t)gridDim.x * kCwBlock, cells = (size_t)n * (size_t)width;
    for (size_t i = (size_t)blockIdx.x * kCwBlock + threadIdx.x; i < cells; i += stride) {
        const size_t v = i / (size_t)width;
        const int32_t e = ptr[v] + (int32_t)(i % (size_t)width);
        rows[i] = e < ptr[v + 1] ? idx[e] : -1;
    }
}

// The rows of virtual id x's query: one query (mode 0), queries on one graph
// (mode 1: the bases are multiples of its size), queries on any (mode 2).
template <int kMode>
__device__ __forceinline__ RowRef deep_ref(const CwParams &P, const RowRef &one, uint32_t x) {
    if (kMode == 0) return one;
    if (kMode == 1) return RowRef{one.rows, x - x % P.same_n, one.quads};
    const CwQuery &Q = P.q[query_of(P, x)];
    return RowRef{Q.rows, Q.base, Q.quads};
}

// A wave's queue of improved vertices: virtual ids and the levels they were
// improved to.
struct DeepQueue {
    uint32_t x[kDeepQueue], l[kDeepQueue];
};
constexpr uint32_t kDeepFirst = 0u;            // no improved row has level 0

// The lanes' vertices x (those with ok) onto the next launch's list, each
// vertex once per launch: the first to raise its stamp lists it.  Every lane
// calls it.
__device__ __forceinline__ void deep_list(const CwParams &P, const CwLists &N, uint32_t t, uint32_t tag, bool ok,
                                          uint32_t x) {
    const bool fresh = ok && atomicMax(&P.stamp[x], tag) < tag;
    const unsigned long long bm = __ballot(fresh);
    if (!bm) return;
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&P.st->cnt[t][0], (uint32_t)__popcll(bm));
    base = __shfl(base, 0, 64);
    if (fresh) N.s[base + lanes_below(bm)] = x;
}

// The queue's n entries onto the next launch's list: the stamps of 256 at a
// time in flight together, the fresh ones gathered at the queue's front, then
// one counter atomic for all of them.  Entries of level kDeepFirst (flat
// launches: rows reached for the first time, which one offer each finds) need
// no stamp; a row improved once more in the same launch may then be listed
// twice, so a list holds up to 2 V entries (its array and the long columns'
// behind it, which a thin graph has none of).
__device__ __forceinline__ void deep_spill(const CwParams &P, const CwLists &N, uint32_t t, uint32_t tag,
                                           DeepQueue &q, uint32_t n) {
    const uint32_t lane = lane_id();
    uint32_t kept = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 256u) {                          // uniform
        uint32_t x[4], old[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            const uint32_t i = i0 + 64u * j + lane;
            x[j] = q.x[i < n ? i : n - 1u];
            old[j] = i < n ? 0u : tag;
            if (i < n && q.l[i] != kDeepFirst) old[j] = atomicMax(&P.stamp[x[j]], tag);
        }
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) settle_after_issue32(old[j]);
        wave_lds_sync();
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            const bool fresh = old[j] < tag;
            const unsigned long long bm = __ballot(fresh);
            if (fresh) q.x[kept + lanes_below(bm)] = x[j];              // kept <= i0 + 64 j: read already
            kept += (uint32_t)__popcll(bm);
        }
        wave_lds_sync();
    }
    if (!kept) return;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&P.st->cnt[t][0], kept);
    base = __shfl(base, 0, 64);
    for (uint32_t i = lane; i < kept; i += 64u) N.s[base + i] = q.x[i];
}

// U columns per lane (x at level l, those with ok): offers to all their rows
// (a thin graph keeps its lists in fixed-width rows of kE entries, -1 past a
// list's end, so one load gives a column with no look at its bounds), every load and then every atomic of the lane in flight
// together; the rows improved go to queue q (its size m, the same in every
// lane), or to the next launch's list once it is full.
template <int kMode, int kE, int U>
__device__ __forceinline__ void deep_expand(const CwParams &P, const CwLists &N, const RowRef &one, uint32_t t,
                                            uint32_t tag, bool pre, bool flat, const uint32_t (&x)[U],
                                            const uint32_t (&l)[U], const bool (&ok)[U], DeepQueue &q, uint32_t &m) {
    constexpr int kQuads = kE / 4;
    uint32_t base[U];
    int4 d[U][kQuads];
#pragma unroll
    for (int c = 0; c < U; ++c) {
        const RowRef r = deep_ref<kMode>(P, one, x[c]);
        base[c] = r.base;
#pragma unroll
        for (int h = 0; h < kQuads; ++h) {
            d[c][h] = make_int4(-1, -1, -1, -1);
            // (graphs of either width may share a launch of the wider kind)
            const uint32_t quads = kMode == 2 ? r.quads : (uint32_t)kQuads;
            if (ok[c] && (uint32_t)h < quads) d[c][h] = r.rows[(size_t)(x[c] - r.base) * quads + h];
        }
    }
    uint32_t v[U][kE];
    bool on[U][kE];
#pragma unroll
    for (int c = 0; c < U; ++c)
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const int4 &w = d[c][e / 4];
            const int32_t i = (e & 3) == 0 ? w.x : ((e & 3) == 1 ? w.y : ((e & 3) == 2 ? w.z : w.w));
            on[c][e] = i >= 0;
            v[c][e] = base[c] + (uint32_t)(i >= 0 ? i : 0);
        }
    unsigned long long old[U][kE];
    if (pre) {
#pragma unroll
        for (int c = 0; c < U; ++c)
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                old[c][e] = 0ull;
                if (on[c][e]) old[c][e] = P.cw[v[c][e]];
            }
#pragma unroll
        for (int c = 0; c < U; ++c)
#pragma unroll
            for (int e = 0; e < kE; ++e) settle_after_issue(old[c][e]);
    }
#pragma unroll
    for (int c = 0; c < U; ++c) {
        const unsigned long long key = offer_key(l[c] + 1u, x[c] - base[c]);
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            // the words only decrease, so a stale copy is never below the true value
            const bool go = on[c][e] && (!pre || old[c][e] > key);
            old[c][e] = 0ull;
            if (go) old[c][e] = atomicMin(&P.cw[v[c][e]], key);
        }
    }
#pragma unroll
    for (int c = 0; c < U; ++c)
#pragma unroll
        for (int e = 0; e < kE; ++e) settle_after_issue(old[c][e]);
#pragma unroll
    for (int c = 0; c < U; ++c)
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            // a lower level than the row had (or its first): the row's own
            // offers follow; the same level: only its parent changed
            const bool imp = (uint32_t)(old[c][e] >> 32) > l[c] + 1u;
            const unsigned long long bm = __ballot(imp);
            if (!bm) continue;
            const uint32_t pos = m + lanes_below(bm);
            if (imp && pos < kDeepQueue) {
                q.x[pos] = v[c][e];
                q.l[pos] = (flat && unreached(old[c][e])) ? kDeepFirst : l[c] + 1u;
            }
            const uint32_t end = m + (uint32_t)__popcll(bm);
            if (end > kDeepQueue) deep_list(P, N, t, tag, imp && pos >= kDeepQueue, v[c][e]);
            m = end < kDeepQueue ? end : kDeepQueue;
        }
}

// A wave per block takes a share of the list and goes on from it by itself:
// the rows its offers improve are its next columns, level after level, in LDS,
// with no word to the other waves.  Nothing waits at a level's end, so a level
// costs the chain row - atomics - LDS instead of a launch with its counts and lists around that chain.  Waves drift apart, so a
// row may first be offered a level above its own; the word's minimum sets it
// right whenever the smaller offer comes, and whoever lowers a row's level
// makes that row's own offers again.  When no improved row is left every word
// holds its smallest offer from columns that made theirs at their final
// level: the level, and the smallest in-neighbour one level up.
//
// After `iters` levels (or with kDeepStop rows in the queue: the frontier
// grows, other waves should share it) the queue goes to the next launch's
// list, whose entries carry no level: the next launch reads it from the
// word.  A list longer than one step of the whole grid is expanded one level
// only, as the wide form does: it keeps every wave busy by itself, and a wave
// going on alone would run ahead of columns still waiting in the list.
template <int kMode, int kE>
__global__ __launch_bounds__(64) void k_cw_deep(CwParams P, uint32_t seq, uint32_t iters) {
    __shared__ DeepQueue s_q[2];
    CwState *st = P.st;
    const uint32_t t0 = seq % 3, t1 = (seq + 1) % 3, t2 = (seq + 2) % 3;
    const CwLists C = P.lists[seq & 1], N = P.lists[(seq + 1) & 1];
    const uint32_t lane = lane_id(), tag = seq + 1u;
    const uint32_t ns = st->cnt[t0][0];
    if (blockIdx.x == 0 && lane < 4) st->cnt[t2][lane] = 0u;
    const bool flat = ns > kDeepWaves * 64u;
    const uint32_t nw = flat ? gridDim.x : kDeepWaves;
    if (blockIdx.x >= nw) return;
    const RowRef one = RowRef{P.q[0].rows, P.q[0].base, P.q[0].quads};
    const uint32_t want = (ns + nw - 1u) / nw;
    const uint32_t per = flat ? 64u : (want < kDeepShare ? kDeepShare : want);
    const bool pre = ns >= kDeepCheck;
    uint32_t m = 0;                                                     // entries of s_q[0], flat only
    for (uint32_t b = blockIdx.x * per; b < ns; b += nw * per) {        // uniform; once unless flat
        uint32_t x1[1] = {0u}, l1[1] = {0u};
        bool ok1[1] = {lane < per && b + lane < ns};
        if (ok1[0]) {
            x1[0] = C.s[b + lane];
            l1[0] = (uint32_t)(ld_agent64(&P.cw[x1[0]]) >> 32);
        }
        if (flat) {
            deep_expand<kMode, kE, 1>(P, N, one, t1, tag, pre, true, x1, l1, ok1, s_q[0], m);
            if (m > kDeepQueue / 2) {
                wave_lds_sync();
                deep_spill(P, N, t1, tag, s_q[0], m);
                m = 0;
            }
            continue;
        }
        uint32_t cur = 0, n = 0;
        deep_expand<kMode, kE, 1>(P, N, one, t1, tag, pre, false, x1, l1, ok1, s_q[0], n);
        wave_lds_sync();
        for (uint32_t i = 1; i < iters && n != 0u && n <= kDeepStop; ++i) {     // uniform
            DeepQueue &q = s_q[cur], &o = s_q[cur ^ 1u];
            uint32_t no = 0;
            if (n <= 64u) {
                uint32_t x[1] = {q.x[lane < n ? lane : 0u]}, l[1] = {q.l[lane < n ? lane : 0u]};
                const bool ok[1] = {lane < n};
                deep_expand<kMode, kE, 1>(P, N, one, t1, tag, pre, false, x, l, ok, o, no);
            } else {
                for (uint32_t j = 0; j < n; j += 128u) {                // uniform
                    const uint32_t i0 = j + lane, i1 = j + 64u + lane;
                    uint32_t x[2] = {q.x[i0 < n ? i0 : 0u], q.x[i1 < n ? i1 : 0u]};
                    uint32_t l[2] = {q.l[i0 < n ? i0 : 0u], q.l[i1 < n ? i1 : 0u]};
                    const bool ok[2] = {i0 < n, i1 < n};
                    deep_expand<kMode, kE, 2>(P, N, one, t1, tag, pre, false, x, l, ok, o, no);
                }
            }
            wave_lds_sync();
            cur ^= 1u;
            n = no;
        }
        deep_spill(P, N, t1, tag, s_q[cur], n);
    }
    if (flat) {
        wave_lds_sync();
        deep_spill(P, N, t1, tag, s_q[0], m);
    }
}

// The words into the callers' arrays: a block row per query.  With deepest
// set, the largest level over all queries goes to st->last.
__global__ __launch_bounds__(kCwBlock) void k_cw_out(CwParams P, uint32_t deepest) {
    const CwQuery &Q = P.q[blockIdx.y];
    int32_t top = 0;
    for (uint32_t v = blockIdx.x * kCwBlock + threadIdx.x; v < Q.n; v += gridDim.x * kCwBlock) {
        const unsigned long long w = P.cw[Q.base + v];
        const bool r = !unreached(w);
        const int32_t l = r ? (int32_t)(w >> 32) : -1;
        Q.level[v] = l;
        Q.parent[v] = r ? (int32_t)(uint32_t)w : -1;
        top = l > top ? l : top;
    }
    if (deepest) {
        top = wave_max(top);
        if (lane_id() == 0 && (uint32_t)top > ld_agent(&P.st->last)) atomicMax(&P.st->last, (uint32_t)top);
    }
}

hipError_t launch_cw_init(const CwParams &p, hipStream_t s) {
    uint32_t g = (p.max_n + kCwBlock - 1) / kCwBlock;
    g = g < 2048u ? (g ? g : 1u) : 2048u;
    hipLaunchKernelGGL(k_cw_fill, dim3(g, p.nq), dim3(kCwBlock), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cw_roots, dim3((p.nq + kCwBlock - 1) / kCwBlock), dim3(kCwBlock), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_cw_wide(const CwParams &p, uint32_t k, uint32_t grid, hipStream_t s) {
    hipLaunchKernelGGL(k_cw_wide, dim3(grid), dim3(kCwBlock), 0, s, p, k);
    return hipGetLastError();
}

hipError_t launch_cw_rows(const int32_t *ptr, const int32_t *idx, int32_t n, int32_t width, int32_t *rows,
                          hipStream_t s) {
    const size_t want = ((size_t)n * (size_t)width + kCwBlock - 1) / kCwBlock;
    hipLaunchKernelGGL(k_cw_rows, dim3((uint32_t)(want < 8192 ? want : 8192)), dim3(kCwBlock), 0, s, ptr, idx, n,
                       width, rows);
    return hipGetLastError();
}

hipError_t launch_cw_deep(const CwParams &p, uint32_t seq, uint32_t iters, uint32_t grid, bool wide_rows,
                          hipStream_t s) {
    const dim3 g(grid), b(64);
    const int mode = p.nq == 1 ? 0 : (p.same_n ? 1 : 2);
    if (mode == 0) {
        if (wide_rows) hipLaunchKernelGGL((k_cw_deep<0, 8>), g, b, 0, s, p, seq, iters);
        else hipLaunchKernelGGL((k_cw_deep<0, 4>), g, b, 0, s, p, seq, iters);
    } else if (mode == 1) {
        if (wide_rows) hipLaunchKernelGGL((k_cw_deep<1, 8>), g, b, 0, s, p, seq, iters);
        else hipLaunchKernelGGL((k_cw_deep<1, 4>), g, b, 0, s, p, seq, iters);
    } else {
        if (wide_rows) hipLaunchKernelGGL((k_cw_deep<2, 8>), g, b, 0, s, p, seq, iters);
        else hipLaunchKernelGGL((k_cw_deep<2, 4>), g, b, 0, s, p, seq, iters);
    }
    return hipGetLastError();
}

hipError_t launch_cw_narrow(const CwParams &p, uint32_t k, uint32_t max_levels, uint32_t max_next,
                            uint32_t max_edges, hipStream_t s) {
    max_next = max_next < kCwCap ? max_next : kCwCap;
    max_edges = max_edges < kCwNarrowEdges ? max_edges : kCwNarrowEdges;
    if (p.nq == 1)
        hipLaunchKernelGGL(k_cw_narrow<true>, dim3(1), dim3(kCwNarrowThreads), 0, s, p, k, max_levels, max_next,
                           max_edges);
    else
        hipLaunchKernelGGL(k_cw_narrow<false>, dim3(1), dim3(kCwNarrowThreads), 0, s, p, k, max_levels, max_next,
                           max_edges);
    return hipGetLastError();
}

// The pack and its way back are streams: bound by HBM when every workgroup has
// the same share.  A block row of the grid per query, as many blocks as the
// largest one needed, left most of 65,536 workgroups empty and the largest
// query's with 32 rounds of one 4-byte load each (64 random graphs, 44.8 M
// entries: 138 us packed, 20 us unpacked).  So a workgroup takes a tile of the
// packed entries (or vertices), whichever queries lie in it.
constexpr uint32_t kPackEntries = 2048, kPackVerts = 1024, kPackBlocks = 2048;

// A 16-byte load from an address aligned to 4 bytes only (a tile starts anywhere
// in its query's list).
typedef int Int4Any __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint32_t pack_first(const PackQuery &Q, bool entries) { return entries ? Q.ebase : Q.base; }

// The query that holds packed entry (vertex) x: the last of [q, nq) that starts
// at or before it; q starts there too.  x is mostly q's or the next one's.
__device__ __forceinline__ uint32_t pack_query(const PackParams &P, uint32_t q, uint32_t x, bool entries) {
    for (uint32_t t = 0; t < 2; ++t) {
        if (q + 1 >= P.nq || x < pack_first(P.q[q + 1], entries)) return q;
        ++q;
    }
    uint32_t lo = q, hi = P.nq;                            // the answer is in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t m = lo + (hi - lo) / 2;
        if (pack_first(P.q[m], entries) <= x) lo = m;
        else hi = m;
    }
    return lo;
}

// The queries' out-lists into one block-diagonal CSR: row base_q + v holds
// query q's row v with every entry offset by base_q; and the packed sources.
// Workgroups below `entry_blocks` copy entries, consecutive tiles each (finding a
// tile's query by itself is a chain of reads as long as the copy: 116 us with a
// workgroup per tile), the others row offsets.
__global__ __launch_bounds__(kCwBlock) void k_pack(PackParams P, uint32_t entry_blocks) {
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x < entry_blocks) {
        const uint64_t tiles = ((uint64_t)P.pad_end + kPackEntries - 1) / kPackEntries;
        const uint64_t t0 = tiles * blockIdx.x / entry_blocks, t1 = tiles * (blockIdx.x + 1) / entry_blocks;
        uint32_t q = 0;
        for (uint64_t t = t0; t < t1; ++t) {
            const uint64_t e0 = t * kPackEntries;
            if (e0 < P.E) q = pack_query(P, q, (uint32_t)e0, true);
            const uint32_t end = q + 1 < P.nq ? P.q[q + 1].ebase : P.E;
            if (e0 + kPackEntries <= end) {                // one query's
                constexpr uint32_t quads = kPackEntries / (4 * kCwBlock);
                const int32_t *src = P.q[q].idx + (e0 - P.q[q].ebase);
                int32_t *dst = P.idx + e0;
                const int32_t add = (int32_t)P.q[q].base;
                Int4Any x[quads];
#pragma unroll
                for (uint32_t i = 0; i < quads; ++i) x[i] = *(const Int4Any *)(src + 4 * (i * kCwBlock + tid));
#pragma unroll
                for (uint32_t i = 0; i < quads; ++i)
                    *(int4 *)(dst + 4 * (i * kCwBlock + tid)) =
                        make_int4(x[i].x + add, x[i].y + add, x[i].z + add, x[i].w + add);
                continue;
            }
            uint32_t at = q;
            for (uint32_t i = tid; i < kPackEntries; i += kCwBlock) {
                const uint64_t e = e0 + i;
                if (e < P.E) {
                    at = pack_query(P, at, (uint32_t)e, true);
                    P.idx[e] = P.q[at].idx[e - P.q[at].ebase] + (int32_t)P.q[at].base;
                } else if (e < P.pad_end) {
                    P.idx[e] = 0;
                }
            }
        }
        return;
    }
    const uint64_t v0 = (uint64_t)(blockIdx.x - entry_blocks) * kPackVerts;
    uint32_t q = v0 < P.V ? pack_query(P, 0, (uint32_t)v0, false) : 0;
    for (uint32_t i = tid; i < kPackVerts; i += kCwBlock) {
        const uint64_t v = v0 + i;
        if (v < P.V) {
            q = pack_query(P, q, (uint32_t)v, false);
            const uint32_t at = (uint32_t)v - P.q[q].base;
            P.ptr[v] = P.q[q].ptr[at] + (int32_t)P.q[q].ebase;
            if (at == 0) P.roots[q] = (int32_t)P.q[q].base + P.q[q].source;
        } else if (v == P.V) {
            P.ptr[v] = (int32_t)P.E;
        }
    }
}

// The packed results into the callers' arrays (parents back to the query's ids).
__global__ __launch_bounds__(kCwBlock) void k_unpack(PackParams P) {
    const uint64_t v0 = (uint64_t)blockIdx.x * kPackVerts;
    uint32_t q = pack_query(P, 0, (uint32_t)v0, false);    // v0 < V
    constexpr uint32_t per = kPackVerts / kCwBlock;
    int32_t l[per], p[per];
#pragma unroll
    for (uint32_t i = 0; i < per; ++i) {
        const uint64_t v = v0 + i * kCwBlock + threadIdx.x;
        l[i] = v < P.V ? P.level[v] : 0;
        p[i] = v < P.V ? P.parent[v] : 0;
    }
#pragma unroll
    for (uint32_t i = 0; i < per; ++i) {
        const uint64_t v = v0 + i * kCwBlock + threadIdx.x;
        if (v >= P.V) break;
        q = pack_query(P, q, (uint32_t)v, false);
        const uint32_t base = P.q[q].base, at = (uint32_t)v - base;
        P.q[q].level[at] = l[i];
        P.q[q].parent[at] = p[i] >= 0 ? p[i] - (int32_t)base : -1;
    }
}

hipError_t launch_pack(const PackParams &p, hipStream_t s) {
    uint32_t et = (uint32_t)(((uint64_t)p.pad_end + kPackEntries - 1) / kPackEntries);
    et = et < kPackBlocks ? et : kPackBlocks;
    const uint32_t vt = (uint32_t)(((uint64_t)p.V + 1 + kPackVerts - 1) / kPackVerts);
    hipLaunchKernelGGL(k_pack, dim3(et + vt), dim3(kCwBlock), 0, s, p, et);
    return hipGetLastError();
}

hipError_t launch_unpack(const PackParams &p, hipStream_t s) {
    const uint32_t vt = (uint32_t)(((uint64_t)p.V + kPackVerts - 1) / kPackVerts);
    hipLaunchKernelGGL(k_unpack, dim3(vt), dim3(kCwBlock), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_cw_out(const CwParams &p, bool deepest, hipStream_t s) {
    uint32_t gx = (p.max_n + kCwBlock - 1) / kCwBlock;
    gx = gx < 1024u ? (gx ? gx : 1u) : 1024u;
    hipLaunchKernelGGL(k_cw_out, dim3(gx, p.nq), dim3(kCwBlock), 0, s, p, deepest ? 1u : 0u);
    return hipGetLastError();
}

}  // namespace bfsi
