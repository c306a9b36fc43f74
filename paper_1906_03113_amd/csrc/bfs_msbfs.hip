// Many searches on one graph at once: the masked product of Theorem 1 applied
// to Q sources side by side, 64 sources per 64-bit word per vertex.
//
// For source q, row v and level k the recurrence is the single-source one:
// v joins source q's frontier at level k+1 when some frontier vertex u of
// source q has an edge u -> v and v was not reached by q through level k.  So
// with cur[u] = the sources whose level-k frontier holds u and vis[v] = the
// sources that reached v through level k, one pass over the frontier's columns
// computes, for every entry (u, v),
//     new = cur[u] & ~vis[v]      and      nxt[v] |= new,
// i.e. one read of each column serves every source whose frontier holds it.
//
// The parent of v for source q is, as everywhere in this library, the
// smallest frontier in-neighbour.  The push form takes it with atomicMin over
// the entries it visits; the pull form scans v's in-neighbours in ascending
// order and gives each still-unassigned source bit to the first u whose
// cur[u] holds it (a wave scans 64 entries per step, and an OR prefix across
// its lanes gives each bit to the lowest lane that holds it).  Lists of
// kMsLong entries or more are split into chunks of kMsChunk entries handled
// by different waves, which combine with atomicMin (the same minimum).
// Results are staged vertex-major and written to the callers' per-source
// arrays at the end.  Level k's mask buffers rotate over three slots so the
// one that held F_{k-1} can be cleared while level k runs.  Results are
// bit-identical to single-source searches.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bfs_device.h"
#include "bfs_internal.h"

namespace bfsi {

namespace {

__device__ __forceinline__ const unsigned long long *row(const unsigned long long *m, int32_t v,
                                                         uint32_t W) {
    return m + (size_t)v * W;
}
__device__ __forceinline__ unsigned long long *row(unsigned long long *m, int32_t v, uint32_t W) {
    return m + (size_t)v * W;
}

// selects instead of indexing the parameter arrays with a runtime index
template <typename T>
__device__ __forceinline__ T pick3(T a, T b, T c, uint32_t s) {
    return s == 0 ? a : (s == 1 ? b : c);
}

__device__ __forceinline__ size_t stage(const MsLevel &p, int32_t v, uint32_t q) {
    return (size_t)v * (p.W * 64u) + q;
}

// Whether u may hold frontier bits at this level (always, without the bitmap).
__device__ __forceinline__ bool in_frontier(const MsLevel &p, int32_t u) {
    return !p.use_fbits || ((p.fbits[(uint32_t)u >> 6] >> ((uint32_t)u & 63u)) & 1ull) != 0ull;
}

// With the graph's degree-ordered copy the kernels walk search labels: the
// caller's id of label x and the label of the caller's vertex v (identities
// in the caller's order).
__device__ __forceinline__ int32_t caller_id(const MsLevel &p, int32_t x) {
    return p.orig ? p.orig[x] : x;
}
__device__ __forceinline__ int32_t label_of(const MsLevel &p, int32_t v) {
    return p.pos ? p.pos[v] : v;
}
// The staged row of label x: the label itself when the staged results are
// the library's own (k_ms_out maps them back), else the caller's id.
__device__ __forceinline__ int32_t srow(const MsLevel &p, int32_t x) {
    return p.stage_labels ? x : caller_id(p, x);
}

// One step of a scan by a group of G lanes (G = 16 or 64, aligned within the
// wave), a list entry per lane (its caller id uc) with its mask's bits
// restricted to the sources looked for (hit): each bit goes to the lowest lane
// that holds it, i.e. to the smallest in-neighbour of the step.  Returns the
// bits found (the same in every lane of the group).  vo is the row's staged
// results' row.
template <uint32_t G>
__device__ __forceinline__ unsigned long long scan_resolve(const MsLevel &p, int32_t vo, uint32_t w,
                                                           int32_t uc, unsigned long long hit,
                                                           bool owner_alone) {
    const uint32_t li = __lane_id() & (G - 1u);
    if (__ballot(hit != 0ull) == 0ull) return 0ull;        // (uniform) nothing found in the wave
    unsigned long long incl = hit;
#pragma unroll
    for (uint32_t d = 1; d < G; d <<= 1) {
        const unsigned long long t = __shfl_up(incl, d, (int)G);
        if (li >= d) incl |= t;
    }
    unsigned long long below = __shfl_up(incl, 1u, (int)G);
    if (li == 0) below = 0ull;
    unsigned long long own = hit & ~below;
    const unsigned long long found = __shfl(incl, (int)(G - 1u), (int)G);
    // each found bit's parent (the entry of the lane that owns it) through the
    // group's row of 64 LDS slots, then written by source: lane li takes
    // sources li, li + G, ..., so the staged row goes out in 64 / G stores
    // of consecutive entries instead of one store per bit
    __shared__ uint32_t s_par[kBlock / 64][(64 / G) * 64];   // a row per group of the wave
    uint32_t *slot = &s_par[threadIdx.x >> 6][(__lane_id() / G) * 64u];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    while (own) {
        const uint32_t b = (uint32_t)__ffsll((long long)own) - 1u;
        own &= own - 1ull;
        slot[b] = (uint32_t)uc;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t b = li; b < 64u; b += G) {
        if ((found >> b) & 1ull) {
            const size_t at = stage(p, vo, w * 64u + b);
            const uint32_t pu = slot[b];
            if (owner_alone) p.spar[at] = pu;
            else atomicMin(&p.spar[at], pu);
        }
    }
    return found;
}

}  // namespace

// Every mask and the first level planes to zero and every staged parent to
// 0xFFFFFFFF (parents are combined with atomicMin).
typedef int32_t v4i __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_ms_clear(MsLevel p) {
    const size_t gid = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * kBlock;
    const size_t nw = (size_t)p.n * p.W;
    for (size_t i = gid; i < nw; i += stride) {
        p.vis[i] = 0ull;
        p.m[0][i] = 0ull;
        p.m[1][i] = 0ull;
        p.m[2][i] = 0ull;
#pragma unroll
        for (uint32_t j = 0; j < kMsPlanesFirst; ++j) p.planes[nw * j + i] = 0ull;
    }
    for (size_t v = gid; v < (size_t)p.n; v += stride) p.flag[v] = 0u;
    // staged parents, 16 bytes at a time, streaming stores (not read by
    // this kernel, and far larger than the caches)
    const size_t ns = (size_t)p.n * p.W * 16u;
    const v4i ones = {-1, -1, -1, -1};
    for (size_t i = gid; i < ns; i += stride) __builtin_nontemporal_store(ones, reinterpret_cast<v4i *>(p.spar) + i);
    if (gid < 4) p.cnt[gid] = 0u;
    if (gid < 3) p.rcnt[gid] = 0u;
    if (gid < (size_t)kMsStatWords) p.mstat[gid] = 0ull;
}

// nw words to zero (a level plane before the first level that has its bit, a
// mask buffer that held other data).
__global__ __launch_bounds__(kBlock) void k_ms_zero(unsigned long long *a, size_t nw) {
    const size_t stride = (size_t)gridDim.x * kBlock;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < nw; i += stride) a[i] = 0ull;
}

// Lane t's word in every lane (t the same in all of them), and the lane's bit of
// such a word.
__device__ __forceinline__ unsigned long long word_of_lane(unsigned long long x, int t) {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, t) |
           ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), t) << 32);
}
__device__ __forceinline__ bool lane_bit(unsigned long long x, uint32_t lane) {
    return __builtin_amdgcn_inverse_ballot_w64(x);
}

// The planes into vertex-major levels in the same memory (plane j's words are
// [j n W, (j + 1) n W) of it, row v's levels the 32 words from 32 v W): row r0 =
// ceil(planes n / 32) and those after it lie behind every plane and are written
// first (part 0), while the planes' words that the rows before it need are
// copied to tmp (planes r0 W words, in one mask buffer: ms_levels_fit); part 1
// then writes those rows from tmp.  A wave takes 64 (row, word)s, fewer where
// there are not that many for each: a lane loads the words of one, then they go out
// one at a time with the 64 sources on the lanes, a 256-byte store each (their
// words are the same in every lane: each plane is one select by them).  With 64 for
// every wave a graph of 3,000 vertices took 13 us a part, all of it 47 waves' loops
// (kShare; where there are 64 for each the bound is a constant: directed 2^20, 256
// sources 135 us a part, 141 without).
template <bool kShare>
__global__ __launch_bounds__(kBlock) void k_ms_levels(MsLevel p, uint32_t planes, unsigned long long *tmp, uint32_t part) {
    const uint32_t W = p.W, lane = __lane_id();
    const size_t nw = (size_t)p.n * W;
    const size_t split = ms_levels_row(p.n, planes) * W;
    const size_t gid = (size_t)blockIdx.x * kBlock + threadIdx.x, stride = (size_t)gridDim.x * kBlock;
    // (staged row, word) i has its masks at the row's label
    const auto masks_of = [&](size_t i) -> size_t {
        const size_t r = W == 1 ? i : i / W;
        return p.stage_labels ? i : (size_t)label_of(p, (int32_t)r) * W + (i - r * W);
    };
    if (part == 0)
        for (size_t i = gid; i < split * planes; i += stride)
            tmp[i] = p.planes[nw * (i / split) + masks_of(i % split)];
    const size_t first = part == 0 ? split : 0, last = part == 0 ? nw : split;
    const size_t waves = stride / 64u, share = (last - first + waves - 1) / waves;
    const size_t per = kShare && share < 64 ? share : 64;
    for (size_t i0 = first + gid / 64u * per; i0 < last; i0 += waves * per) {    // uniform per wave
        const size_t i = lane < per && i0 + lane < last ? i0 + lane : last - 1;
        const size_t m = masks_of(i);
        const unsigned long long vis = p.vis[m];
        unsigned long long pl[kMsPlanes];
#pragma unroll
        for (uint32_t j = 0; j < kMsPlanes; ++j) {
            pl[j] = 0ull;
            if (j < planes) pl[j] = part != 0 ? tmp[split * j + i] : p.planes[nw * j + m];
        }
        const int items = (int)(last - i0 < per ? last - i0 : per);
        for (int t = 0; t < items; ++t) {                                       // uniform
            int32_t l = 0;
#pragma unroll
            for (uint32_t j = 0; j < kMsPlanes; ++j)
                if (j < planes) l |= lane_bit(word_of_lane(pl[j], t), lane) ? 1 << j : 0;
            __builtin_nontemporal_store(lane_bit(word_of_lane(vis, t), lane) ? l : -1, p.slev + (i0 + (size_t)t) * 64u + lane);
        }
    }
}

// Level k, push half.  Work items: the frontier list, up to 64 columns per
// wave step - the entries of those with at most kMsShort entries dealt out one per
// lane, each longer one below kMsLong entries taken by the whole wave - then
// the chunks of the graph's long columns, a wave each, skipped unless the
// column is in some frontier.  Per
// entry (u, v): new = cur[u] & ~vis[v] is ORed into nxt[v], each of its bits q
// takes atomicMin(parent_q(v), u) - over all the entries this is the smallest
// frontier in-neighbour of v for q - and v is listed for level k+1 once,
// through a per-wave LDS buffer flushed with one atomic per kMsFlush entries.
// Also clears the masks of F_{k-1} (slot (k+2) % 3).
constexpr uint32_t kMsWaveBuf = 256;
constexpr int kMsBits = 4;               // sources of an entry handled together
constexpr int32_t kMsShort = 16;         // longest column a group of lanes takes
constexpr uint32_t kMsFlush = kMsWaveBuf - 64;

__global__ __launch_bounds__(kBlock) void k_ms_push(MsLevel p, uint32_t k) {
    __shared__ int32_t s_buf[kBlock / 64][kMsWaveBuf];
    __shared__ int32_t s_pre[kBlock / 64][64];         // per wave: short columns' entry offsets
    __shared__ int32_t s_col[kBlock / 64][64];         // ... their column ids
    __shared__ int32_t s_e0[kBlock / 64][64];          // ... and first entries
    const uint32_t s0 = k % 3, s1 = (k + 1) % 3, s2 = (k + 2) % 3;
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s0);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], s1);
    unsigned long long *old = pick3(p.m[0], p.m[1], p.m[2], s2);
    const int32_t *fcur = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s0);
    int32_t *fnxt = pick3(p.fq[0], p.fq[1], p.fq[2], s1);
    const int32_t *fold = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s2);
    const uint32_t ncur = p.cnt[s0], nold = p.cnt[s2];
    const uint32_t W = p.W;
    const uint32_t gt = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    for (uint32_t t = gt; t < nold * W; t += gs) {
        const uint32_t u = (uint32_t)fold[t / W];
        old[(size_t)u * W + (t % W)] = 0ull;
    }
    const uint32_t lane = __lane_id();
    const uint32_t wid = threadIdx.x >> 6;
    int32_t *buf = s_buf[wid];
    uint32_t nbuf = 0;                    // the same in every lane
    const uint32_t tag = k + 2;           // "listed for level k+1"
    auto flush = [&]() {
        __builtin_amdgcn_wave_barrier();
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&p.cnt[s1], nbuf);
        base = __shfl(base, 0, 64);
        for (uint32_t i = lane; i < nbuf; i += 64) fnxt[base + i] = buf[i];
        __builtin_amdgcn_wave_barrier();
        nbuf = 0;
    };
    // one entry (u, v): the new bits of u's mask for v, their parents, the OR
    // into nxt[v]; true if this lane lists v for level k+1
    auto entry = [&](int32_t u, int32_t e, int32_t &v) -> bool {
        const unsigned long long *cu = row(cur, u, W);
        v = p.out_idx[e];
        const unsigned long long *vv = row(p.vis, v, W);
        unsigned long long *nv = row(nxt, v, W);
        bool listed = false, any = false;
        for (uint32_t w = 0; w < W; ++w) {
            const unsigned long long nb = cu[w] & ~vv[w];
            if (!nb) continue;
            // parents only decrease, so a stale pre-read can only let
            // an atomic through that was not needed (staged rows and parent
            // values in the caller's ids)
            const int32_t vo = p.stage_labels ? v : (p.out_ent ? p.out_ent[e] : v);
            const uint32_t uo = (uint32_t)caller_id(p, u);
            // kMsBits sources at a time: their pre-reads are all in flight before
            // the first atomic
            for (unsigned long long b = nb; b;) {
                uint32_t *at[kMsBits], cp[kMsBits];
#pragma unroll
                for (int x = 0; x < kMsBits; ++x) {
                    cp[x] = 0u;                             // no source: nothing to lower
                    at[x] = p.spar;
                    if (b) {
                        at[x] = &p.spar[stage(p, vo, w * 64u + (uint32_t)__ffsll((long long)b) - 1u)];
                        cp[x] = *at[x];
                    }
                    b &= b - 1ull;
                }
#pragma unroll
                for (int x = 0; x < kMsBits; ++x)
                    if (cp[x] > uo) atomicMin(at[x], uo);
            }
            if (W == 1) {
                // the lane whose OR turns nxt[v] nonzero lists v; a
                // pre-read (possibly stale: bits are only ever added)
                // skips ORs that would add nothing
                if (nb & ~nv[0]) listed = atomicOr(&nv[0], nb) == 0ull;
            } else {
                atomicOr(&nv[w], nb);
                any = true;
            }
        }
        if (W != 1) listed = any && atomicMax(&p.flag[v], tag) < tag;
        return listed;
    };
    // the wave's listed vertices into its LDS buffer (called by whole waves)
    auto emit = [&](bool listed, int32_t v) {
        const unsigned long long bm = __ballot(listed);
        if (bm) {
            if (listed) buf[nbuf + lanes_below(bm)] = v;
            nbuf += (uint32_t)__popcll(bm);
            if (nbuf > kMsFlush) flush();
        }
    };
    // the frontier list C columns per wave step, a lane per column: the
    // entries of the short columns (at most kMsShort) are dealt out over the
    // wave's lanes, one entry each, through an exclusive prefix sum of their
    // lengths in LDS; then each longer column below kMsLong, the whole wave
    // over its entries
    int32_t *pre = s_pre[wid];
    int32_t *cu_of = s_col[wid];
    int32_t *e0_of = s_e0[wid];
    // columns per wave step: 64 on graphs of low average degree (short
    // columns only: fewer, fuller steps), else a power of two up to 64 such
    // that the list spans about one step per wave (a short list of longer
    // columns then keeps every wave busy)
    const uint32_t nwaves = gs >> 6;
    const uint32_t want = (ncur + nwaves - 1) / nwaves;
    const uint32_t C = (p.wide_steps || want >= 64u) ? 64u
                     : (want <= 1u ? 1u : 1u << (32 - __clz((int)(want - 1u))));
    // waves per group of C columns: 2, 4 or 8 where the list leaves that many
    // (each takes every T-th 64 entries of a column longer than kMsShort, the
    // first also the short ones; a wave alone would scan a column of up to 511
    // entries in eight dependent steps)
    const uint32_t groups = (ncur + C - 1) / C;
    const uint32_t T = groups * 8u <= nwaves ? 8u : (groups * 4u <= nwaves ? 4u : (groups * 2u <= nwaves ? 2u : 1u));
    const uint32_t seg = (gt >> 6) % T;
    for (uint32_t b0 = (gt >> 6) / T * C; b0 < ncur; b0 += nwaves / T * C) {   // uniform per wave
        const uint32_t it = b0 + lane;
        int32_t u = -1, e0 = 0, d = 0;
        if (lane < C && it < ncur) {
            u = fcur[it];
            e0 = p.out_ptr[u];
            d = p.out_ptr[u + 1] - e0;
        }
        const int32_t ds = (d <= kMsShort && seg == 0u) ? d : 0;
        int32_t inc = ds;
#pragma unroll
        for (uint32_t o = 1; o < 64; o <<= 1) {
            const int32_t t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        const int32_t total = __shfl(inc, 63, 64);
        pre[lane] = inc - ds;
        cu_of[lane] = u;
        e0_of[lane] = e0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int32_t j0 = 0; j0 < total; j0 += 64) {                 // uniform
            const int32_t j = j0 + (int32_t)lane;
            int32_t v = -1;
            bool listed = false;
            if (j < total) {
                // the column holding entry j: the last one whose prefix is <= j
                uint32_t c = 0;
#pragma unroll
                for (uint32_t step = 32; step; step >>= 1)
                    if (c + step < 64u && pre[c + step] <= j) c += step;
                listed = entry(cu_of[c], e0_of[c] + (j - pre[c]), v);
            }
            emit(listed, v);
        }
        for (unsigned long long mm = __ballot(d > kMsShort && (uint32_t)d < kMsLong); mm; mm &= mm - 1ull) {
            const int src = (int)__ffsll((long long)mm) - 1;
            const int32_t mu = __shfl(u, src, 64), me0 = __shfl(e0, src, 64), md = __shfl(d, src, 64);
            for (int32_t eb = (int32_t)(64u * seg); eb < md; eb += (int32_t)(64u * T)) {    // uniform
                int32_t v = -1;
                const bool listed = (eb + (int32_t)lane < md) ? entry(mu, me0 + eb + (int32_t)lane, v) : false;
                emit(listed, v);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();                           // LDS reused by the next step
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // the chunks of the graph's long columns, a wave each, or a part of one where
    // there are fewer chunks than waves
    const uint32_t parts = p.nlo_chunks * 8u <= nwaves ? 8u : (p.nlo_chunks * 4u <= nwaves ? 4u
                         : (p.nlo_chunks * 2u <= nwaves ? 2u : 1u));
    for (uint32_t c8 = gt >> 6; c8 < p.nlo_chunks * parts; c8 += nwaves) {
        const uint32_t c = c8 / parts, part = c8 % parts;
        const MsLong L = p.lo[p.lomap[c]];
        const int32_t u = L.v;
        bool in_f = false;
        for (uint32_t w = 0; w < W; ++w) in_f = in_f || row(cur, u, W)[w] != 0ull;
        if (!in_f) continue;
        const int32_t r1 = p.out_ptr[u + 1], len = (int32_t)(kMsChunk / parts);
        const int32_t e0 = p.out_ptr[u] + (int32_t)((c - L.chunk_base) * kMsChunk) + (int32_t)part * len;
        const int32_t e1 = (e0 + len < r1) ? e0 + len : r1;
        for (int32_t eb = e0; eb < e1; eb += 64) {       // uniform: whole waves step together
            const int32_t e = eb + (int32_t)lane;
            int32_t v = -1;
            const bool listed = (e < e1) ? entry(u, e, v) : false;
            emit(listed, v);
        }
    }
    if (nbuf) flush();
}

// The calling block's share of list slot t's statistics (out-degree sum d,
// new pairs c) into the block's group lines of mstat, slot t and the running
// totals (one atomic per word per block).  Every thread calls it.
__device__ __forceinline__ void add_stats(const MsLevel &p, uint32_t t, unsigned long long d,
                                          unsigned long long c) {
    __shared__ unsigned long long s_d[kBlock / 64][2];
    d = wave_sum64(d);
    c = wave_sum64(c);
    if (__lane_id() == 0) {
        s_d[threadIdx.x >> 6][0] = d;
        s_d[threadIdx.x >> 6][1] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sd = 0, sc = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            sd += s_d[w][0];
            sc += s_d[w][1];
        }
        const int g = (int)(blockIdx.x % kMsDegGroups);
        if (sd) atomicAdd(&p.mstat[ms_line((int)t, g)], sd);
        if (sc) {
            atomicAdd(&p.mstat[ms_line((int)t, g) + 1], sc);
            atomicAdd(&p.mstat[ms_line(kMsCumSlot, g) + 1], sc);
        }
    }
}

// Whether the calling block is the launch's last to get here (every thread
// calls it): arrivals on a counter per group of blocks, the groups' last on
// one for the groups, in words 2 and 3 of mstat's lines; every counter is back
// at zero afterwards.  Each wave drains its memory operations first, so the
// last block finds every other block's atomics done.
constexpr int kWaitVmcnt0 = 0x0F70;           // s_waitcnt vmcnt(0) alone

__device__ __forceinline__ bool ms_last_to_arrive(const MsLevel &p) {
    __shared__ uint32_t s_last;
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    if (gridDim.x == 1) return true;                       // nobody else (the sources, small graphs)
    if (threadIdx.x == 0) {
        const uint32_t nb = gridDim.x;
        const uint32_t groups = nb < (uint32_t)kMsDegGroups ? nb : (uint32_t)kMsDegGroups;
        const uint32_t g = blockIdx.x % groups, in_group = (nb - g + groups - 1) / groups;
        unsigned long long *mine = &p.mstat[ms_line(0, (int)g) + 2], *top = &p.mstat[ms_line(0, 0) + 3];
        uint32_t last = 0;
        if (atomicAdd(mine, 1ull) == in_group - 1) {
            __hip_atomic_store(mine, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (atomicAdd(top, 1ull) == groups - 1) {
                __hip_atomic_store(top, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = 1;
            }
        }
        s_last = last;
    }
    __syncthreads();
    return s_last != 0;
}

// Sources nb of word w reach label x at level k >= 1.  Levels are kept as bit
// planes while the search is short: plane j, [n][W] like the masks, holds the
// (vertex, source) pairs whose level has bit j, so a level costs one or two
// mask-wide updates of consecutive words where staged levels cost a 4-byte store
// per pair into 256-byte rows (R-MAT s22, 64 sources: 1 GB of them, in lines
// written partly on each level and read again at the end).  With
// direct_levels (a search past 2^kMsPlanes levels has turned its planes into
// staged levels) they are stored one by one.
__device__ __forceinline__ void set_levels(const MsLevel &p, int32_t x, uint32_t w, uint32_t k,
                                           unsigned long long nb) {
    if (p.direct_levels) {
        const int32_t vo = srow(p, x);
        for (unsigned long long b = nb; b; b &= b - 1ull)
            p.slev[stage(p, vo, w * 64u + (uint32_t)__ffsll((long long)b) - 1u)] = (int32_t)k;
        return;
    }
    unsigned long long *at = p.planes + (size_t)x * p.W + w;
    const size_t step = (size_t)p.n * p.W;
    for (uint32_t bits = k; bits; bits &= bits - 1u) at[step * ((uint32_t)__ffs((int)bits) - 1u)] |= nb;
}

// The same, and they join vis, where the rows lie apart (a push's list): every word
// is loaded before the first is stored, one trip to memory instead of one for each
// word.  (Rows in order - the close of a pull - are bound by bandwidth: 59 us a
// level of directed 2^20, 256 sources, 64 this way.)
__device__ __forceinline__ void join_levels(const MsLevel &p, int32_t x, uint32_t w, uint32_t k,
                                            unsigned long long nb) {
    const size_t at = (size_t)x * p.W + w, step = (size_t)p.n * p.W;
    const unsigned long long seen = p.vis[at];
    if (p.direct_levels) {
        p.vis[at] = seen | nb;
        set_levels(p, x, w, k, nb);
        return;
    }
    unsigned long long pl[kMsPlanes];
#pragma unroll
    for (uint32_t j = 0; j < kMsPlanes; ++j) {
        pl[j] = 0ull;
        if (((k >> j) & 1u) != 0u) pl[j] = p.planes[step * j + at];
    }
    p.vis[at] = seen | nb;
#pragma unroll
    for (uint32_t j = 0; j < kMsPlanes; ++j)
        if (((k >> j) & 1u) != 0u) p.planes[step * j + at] = pl[j] | nb;
}

// The direction of level k: the network's argmin between push (0) and pull (1)
// over the level's twelve features, push when an output is not finite (or
// without a network).  Features, from f = |F_k| (the union frontier), d = its
// out-degree sum, c = the summed union frontier sizes of levels 0..k, u = the
// (vertex, source) pairs not reached through level k, q sources, k, n and nnz.
__device__ __forceinline__ float ms_feature(uint32_t i, float f, float d, float c, float u, float q,
                                            float k, float n, float nnz) {
    // a / b per lane, then one logarithm for all (a switch over the lanes runs
    // its cases one after another)
    const float a = i == 0 || i == 6                      ? f + 1.f
                  : i == 1 || i == 7 || i == 9 || i == 11 ? d + 1.f
                  : i == 2                                ? c + 1.f
                  : i == 3                                ? q + 1.f
                  : i == 4                                ? k + 1.f
                  : i == 5                                ? nnz
                  : i == 8                                ? u + 1.f
                  : i == 10                               ? (f + 1.f) * q
                                                          : 1.f;
    const float b = i == 5 || i == 6 || i == 10 ? n
                  : i == 7                      ? nnz + 1.f
                  : i == 8                      ? n * q
                  : i == 9                      ? f + 1.f
                  : i == 11                     ? nnz - d + 1.f
                                                : 1.f;
    const float x = a / b;
    return i == 5 ? x : logf(x);
}

// The next list (slot t) starts empty, its size and its statistics, and the summed
// sizes of the lists so far become `sum` (in lane 0): the first lanes of one wave.
__device__ __forceinline__ void ms_next_list(const MsLevel &p, uint32_t t, unsigned long long sum) {
    const uint32_t lane = __lane_id();
    p.mstat[ms_line((int)t, (int)lane)] = 0ull;
    p.mstat[ms_line((int)t, (int)lane) + 1] = 0ull;
    if (lane == 0) {
        p.mstat[ms_line(kMsCumSlot, 0)] = sum;
        p.cnt[t] = 0u;
    }
}

// Level k and its list's size, with the direction in the top bit, to the host.
__device__ __forceinline__ void ms_report(const MsLevel &p, uint32_t k, uint32_t size_dir) {
    // one word and relaxed: a release at system scope writes the L2 back first
    __hip_atomic_store((unsigned long long *)p.host_status, (unsigned long long)k | ((unsigned long long)size_dir << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The end of a level, by the last block of its last launch (a launch of its own
// for the direction cost 5 us a level): level k's list (slot k % 3) is
// complete, the next level's list starts empty (next_list), the direction of
// level k is decided, and the level, the list's size and the direction go to
// the host, which polls for them.  Every thread of the block calls it.
__device__ __forceinline__ void ms_close(const MsLevel &p, uint32_t k, bool next_list, bool report) {
    __shared__ float s_w[kMlpLds];
    const uint32_t lane = __lane_id(), t = k % 3, tn = (k + 1) % 3;
    uint32_t f = 0;
    unsigned long long d = 0, c = 0, r = 0;
    long long nnz = 0;
    if (threadIdx.x < 64) {
        f = ld_agent(&p.cnt[t]);
        if (p.mlp != nullptr) nnz = p.out_ptr[p.n];
    }
    if (threadIdx.x < (uint32_t)kMsDegGroups) {
        d = ld_agent64(&p.mstat[ms_line((int)t, (int)lane)]);
        c = ld_agent64(&p.mstat[ms_line(kMsCumSlot, (int)lane)]);
        r = ld_agent64(&p.mstat[ms_line(kMsCumSlot, (int)lane) + 1]);
    }
    if (p.mlp != nullptr) stage_mlp(p.mlp, s_w);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    if (next_list && lane < (uint32_t)kMsDegGroups) {
        if (lane == 0) c += f;                // this one with them
        ms_next_list(p, tn, c);
    }
    uint32_t dir = 0;
    if (p.mlp != nullptr && f != 0) {
        d = wave_sum64(d);
        c = wave_sum64(c);
        r = wave_sum64(r);
        const unsigned long long pairs = (unsigned long long)p.n * p.nq;
        const unsigned long long u = pairs > r ? pairs - r : 0ull;
        const float feat = ms_feature(lane, (float)f, (float)d, (float)c, (float)u, (float)p.nq, (float)k, (float)p.n,
                                      (float)nnz);
        const int b = mlp_argmin(s_w, feat, 2);
        dir = b < 0 ? 0u : (uint32_t)b;
    }
    if (lane == 0 && report) ms_report(p, k, f | (dir << 31));
}

// Sources: bit q set in cur and vis of its vertex, level 0, parent itself; each
// distinct source vertex enters the level-0 list once.
__global__ __launch_bounds__(kBlock) void k_ms_roots(MsLevel p) {
    const uint32_t gid = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    for (uint32_t q = gid; q < p.nq; q += gs) {
        const int32_t s = p.sources[q];                       // the caller's id
        const int32_t x = label_of(p, s);
        const unsigned long long bit = 1ull << (q & 63);
        atomicOr(&row(p.m[0], x, p.W)[q >> 6], bit);
        atomicOr(&row(p.vis, x, p.W)[q >> 6], bit);
        if (p.direct_levels) p.slev[stage(p, srow(p, x), q)] = 0;
        p.spar[stage(p, srow(p, x), q)] = (uint32_t)s;
        const int g = (int)(q % kMsDegGroups);
        atomicAdd(&p.mstat[ms_line(0, g) + 1], 1ull);              // one pair per source
        atomicAdd(&p.mstat[ms_line(kMsCumSlot, g) + 1], 1ull);
        if (atomicMax(&p.flag[x], 1u) < 1u) {
            p.fq[0][atomicAdd(&p.cnt[0], 1u)] = x;
            atomicAdd(&p.mstat[ms_line(0, g)], (unsigned long long)(p.out_ptr[x + 1] - p.out_ptr[x]));
            atomicAdd(&p.mstat[ms_line(kMsCumSlot, g)], 1ull);
        }
    }
    if (ms_last_to_arrive(p)) ms_close(p, 0u, false, true);
}

// Level k, settle half, one lane per newly listed vertex v: the new bits
// (nxt[v]) join vis and get level k+1 (their parents were set by the push).
// The level is reported only when it had a frontier, so levels launched past
// the end of the search (an empty frontier: push and settle then change
// nothing) leave the last level's report in place.  Where no direction is decided
// on it the level closes as this launch starts - its list is complete since the
// push - so that the next level's launches come meanwhile and no workgroup waits
// for the others (1.7 us of a thin level's 6.5).
__global__ __launch_bounds__(kBlock) void k_ms_settle(MsLevel p, uint32_t k) {
    const uint32_t s0 = k % 3, s1 = (k + 1) % 3;
    const unsigned long long *nxt = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s1);
    const int32_t *fnxt = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s1);
    const uint32_t nnext = p.cnt[s1], ncur = p.cnt[s0];
    const uint32_t W = p.W;
    const uint32_t gt = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    if (p.mlp == nullptr && gt < (uint32_t)kMsDegGroups) {
        ms_next_list(p, (k + 2) % 3, p.mstat[ms_line(kMsCumSlot, 0)] + nnext);
        if (gt == 0 && ncur != 0u) ms_report(p, k + 1, nnext);
    }
    unsigned long long deg = 0, pairs = 0;
    for (uint32_t i = gt; i < nnext; i += gs) {
        const int32_t v = fnxt[i];
        deg += (unsigned long long)(p.out_ptr[v + 1] - p.out_ptr[v]);
        for (uint32_t w = 0; w < W; ++w) {
            const unsigned long long nb = row(nxt, v, W)[w];
            if (!nb) continue;
            pairs += (unsigned long long)__popcll(nb);
            join_levels(p, v, w, k + 1, nb);
        }
    }
    add_stats(p, s1, deg, pairs);
    if (p.mlp != nullptr && ms_last_to_arrive(p)) ms_close(p, k + 1, true, ncur != 0u);
}

// The union-frontier bitmap of level k: bit v of fbits = some word of v's
// level-k mask is nonzero.  A wave per 64 consecutive vertices (one lane
// each), whose ballot is the word; every word is rewritten, so nothing needs
// clearing.
__global__ __launch_bounds__(kBlock) void k_ms_fbits(MsLevel p, uint32_t k) {
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], k % 3);
    const uint32_t W = p.W, lane = __lane_id();
    const uint32_t nw = (uint32_t)(((size_t)p.n + 63) / 64);
    const uint32_t wave = (blockIdx.x * kBlock + threadIdx.x) >> 6, nwaves = (gridDim.x * kBlock) >> 6;
    for (uint32_t i = wave; i < nw; i += nwaves) {           // uniform per wave
        const uint32_t v = i * 64u + lane;
        bool nz = false;
        if (v < (uint32_t)p.n)
            for (uint32_t w = 0; w < W; ++w) nz = nz || row(cur, (int32_t)v, W)[w] != 0ull;
        const unsigned long long bm = __ballot(nz);
        if (lane == 0) p.fbits[i] = bm;
    }
}

// Entries [e0, e1) of row v scanned by the whole wave for the sources in rem
// until every one is found; returns the bits found.  The first batch is one
// step of 64 entries (on a dense frontier most rows end there), every later
// one four steps: their index loads, then their bitmap tests, then their mask
// gathers, each four deep in flight.  With prune (a long row's
// chunk after its first), each batch first drops the sources that an earlier
// chunk of the row has settled at an in-neighbour below the batch's first
// entry: staged parents only decrease within the level, so a stale read only
// keeps a source longer.
__device__ __forceinline__ unsigned long long scan_wave4(const MsLevel &p, const unsigned long long *cur,
                                                         int32_t vo, uint32_t w, int32_t e0, int32_t e1,
                                                         unsigned long long rem, bool owner_alone,
                                                         bool prune) {
    const uint32_t W = p.W;
    const int32_t lane = (int32_t)__lane_id();
    unsigned long long found = 0ull;
    int32_t nst = 1;                                                    // steps in this batch
    for (int32_t eb = e0; eb < e1 && rem; eb += nst * 64, nst = 4) {
        int32_t uu[4], oo[4];                                           // labels, caller ids
        bool ok[4];
        unsigned long long mm[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int32_t e = eb + t * 64 + lane;
            const bool in = t < nst && e < e1;
            uu[t] = in ? p.in_idx[e] : -1;
        }
        if (prune) {
            const uint32_t first = (uint32_t)(p.ent ? p.ent[eb] : __shfl(uu[0], 0, 64));
            const uint32_t sp = p.spar[stage(p, vo, w * 64u + (uint32_t)lane)];
            rem &= ~__ballot(sp < first);
            if (!rem) break;                                            // uniform
        }
        if (p.use_fbits) {
            unsigned long long fb[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) fb[t] = uu[t] >= 0 ? p.fbits[(uint32_t)uu[t] >> 6] : 0ull;
#pragma unroll
            for (int t = 0; t < 4; ++t) ok[t] = ((fb[t] >> ((uint32_t)uu[t] & 63u)) & 1ull) != 0ull;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) ok[t] = uu[t] >= 0;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) mm[t] = ok[t] ? row(cur, uu[t], W)[w] : 0ull;
        // the caller's ids of the entries that may give a parent (with the
        // degree-ordered copy a lookup, mostly in the few megabytes of the
        // labels of largest degree; streaming every entry's id cost more)
#pragma unroll
        for (int t = 0; t < 4; ++t) oo[t] = (mm[t] & rem) ? caller_id(p, uu[t]) : -1;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (rem) {                                                  // uniform
                const unsigned long long f = scan_resolve<64>(p, vo, w, oo[t], mm[t] & rem, owner_alone);
                rem &= ~f;
                found |= f;
            }
        }
    }
    return found;
}

// Level k, pull form (for large frontiers): every vertex v whose sources are
// not all settled ORs, in ascending in-neighbour order, the frontier masks of
// its in-neighbours restricted to the sources that have not reached it; each
// source bit found first at u gets parent u (the smallest frontier
// in-neighbour for that source) and level k+1.  Rows of up to kMsSerial
// entries are scanned by one lane, longer ones by a wave (scan_step); the
// owner of such a row writes vis and the next mask without atomics, and rows
// with new bits are listed (one atomicAdd per block chunk).  The graph's long
// rows (kMsLong entries or more) are scanned in chunks by waves across the
// grid: each chunk gives its first hits (atomicMin on the staged parent) and
// ORs its bits into the next mask; k_ms_pull_close then folds those into vis and
// lists the rows.  Also clears F_{k-1}'s masks.
// Chunk j (kMsChunk entries) of long row v, scanned by one wave in ascending
// order until every unsettled source is found: first hits go to the staged
// parents by atomicMin, the bits found are ORed into the next mask and, for
// the row's first chunk (first = true), into vis as well.
__device__ __forceinline__ void long_chunk(const MsLevel &p, const unsigned long long *cur,
                                           unsigned long long *nxt, int32_t v, uint32_t j,
                                           uint32_t k, bool first) {
    const uint32_t W = p.W, tail = p.nq & 63u;
    const int32_t r1 = p.in_ptr[v + 1];
    const int32_t e0 = p.in_ptr[v] + (int32_t)(j * kMsChunk);
    const int32_t e1 = (e0 + (int32_t)kMsChunk < r1) ? e0 + (int32_t)kMsChunk : r1;
    unsigned long long *vis = row(p.vis, v, W);
    for (uint32_t w = 0; w < W; ++w) {
        const unsigned long long full = (w == W - 1 && tail) ? ((1ull << tail) - 1ull) : ~0ull;
        const unsigned long long found = scan_wave4(p, cur, srow(p, v), w, e0, e1, full & ~vis[w], false,
                                                    j != 0);
        if (found && __lane_id() == 0) {
            atomicOr(&row(nxt, v, W)[w], found);
            if (first) vis[w] |= found;
        }
    }
}

constexpr int kMsWriteRows = 8;          // rows whose staged results a wave writes together

__device__ __forceinline__ unsigned long long full_word(const MsLevel &p, uint32_t w) {
    const uint32_t tail = p.nq & 63u;
    return (w == p.W - 1u && tail) ? ((1ull << tail) - 1ull) : ~0ull;
}

// The rows of up to kMsSerial entries: a lane per (row, word), consecutive lanes
// on the words of one row.  A lane records, per found bit, the offset of the
// entry that gave it (LDS); then each wave writes its lanes' rows, one at a
// time with the 64 sources of the word on the 64 lanes, so that the staged
// results of a row go out as one 256-byte store.  Waves do not wait for each
// other anywhere.  Also clears F_{k-1}'s masks.
template <bool kOne>
__global__ __launch_bounds__(kBlock) void k_ms_pull_short(MsLevel p, uint32_t k) {
    __shared__ uint32_t s_off[kBlock][9];          // found bits: entry offset, 4 bits each
    __shared__ unsigned long long s_fnd[kBlock];   // found bits
    __shared__ int32_t s_e0[kBlock];
    const uint32_t s0 = k % 3, s1 = (k + 1) % 3, s2 = (k + 2) % 3;
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s0);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], s1);
    unsigned long long *old = pick3(p.m[0], p.m[1], p.m[2], s2);
    const int32_t *fold = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s2);
    const uint32_t nold = p.cnt[s2];
    const uint32_t W = kOne ? 1u : p.W;
    const uint32_t tid = threadIdx.x, lane = __lane_id();
    const uint32_t gt = blockIdx.x * kBlock + tid, gs = gridDim.x * kBlock;
    for (size_t t = gt; t < (size_t)nold * W; t += gs) {
        const uint32_t u = (uint32_t)fold[t / W];
        old[(size_t)u * W + (t % W)] = 0ull;
    }
    const size_t items = (size_t)p.n * W;
    for (size_t i0 = gt - lane; i0 < items; i0 += gs) {                          // uniform per wave
        const size_t item = i0 + lane;
        int32_t v = 0, e0 = 0, e1 = 0;
        uint32_t w = 0;
        unsigned long long rem = 0ull, found = 0ull, sv = 0ull;
        if (item < items) {
            v = (int32_t)(item / W);
            w = (uint32_t)(item - (size_t)v * W);
            e0 = p.in_ptr[v];
            e1 = p.in_ptr[v + 1];
            sv = p.vis[item];
            if (e1 - e0 <= kMsSerial) rem = full_word(p, w) & ~sv;
        }
        s_e0[tid] = e0;
#pragma unroll
        for (int i = 0; i < 8; ++i) s_off[tid][i] = 0u;
        // four entries at a time: their index and mask loads are all issued
        // before the first is used; positions past e1 repeat the last entry,
        // whose bits are then already taken
        for (int32_t e = e0; e < e1 && rem; e += 4) {
            int32_t uu[4];
            unsigned long long mm[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) uu[j] = p.in_idx[e + j < e1 ? e + j : e1 - 1];
#pragma unroll
            for (int j = 0; j < 4; ++j) mm[j] = in_frontier(p, uu[j]) ? row(cur, uu[j], W)[w] : 0ull;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned long long hit = mm[j] & rem;
                rem &= ~hit;
                found |= hit;
                const uint32_t off = (uint32_t)(e - e0 + j);
                while (hit) {
                    const uint32_t b = (uint32_t)__ffsll((long long)hit) - 1u;
                    hit &= hit - 1ull;
                    s_off[tid][b >> 3] |= off << ((b & 7u) * 4u);
                }
            }
        }
        if (found) nxt[item] = found;
        s_fnd[tid] = found;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // kMsWriteRows rows together: their parents (entries of the row's list)
        // are loaded for all of them before the first is stored
        const int32_t vo = found ? srow(p, v) : 0;
        for (unsigned long long rows = __ballot(found != 0ull); rows;) {         // uniform
            bool on[kMsWriteRows];
            size_t at[kMsWriteRows];
            int32_t u[kMsWriteRows];
#pragma unroll
            for (int x = 0; x < kMsWriteRows; ++x) {
                const int src = rows ? (int)__ffsll((long long)rows) - 1 : 0;
                const uint32_t rr = (tid & ~63u) + (uint32_t)src;
                on[x] = rows != 0ull && ((s_fnd[rr] >> lane) & 1ull) != 0ull;
                const int32_t rv = __shfl(vo, src, 64);
                const uint32_t rw = kOne ? 0u : (uint32_t)__shfl((int)w, src, 64);
                at[x] = stage(p, rv, rw * 64u + lane);
                const int32_t e = s_e0[rr] + (int32_t)((s_off[rr][lane >> 3] >> ((lane & 7u) * 4u)) & 15u);
                u[x] = 0;
                if (on[x]) u[x] = p.ent ? p.ent[e] : p.in_idx[e];
                rows &= rows - 1ull;
            }
#pragma unroll
            for (int x = 0; x < kMsWriteRows; ++x) {
                if (on[x]) p.spar[at[x]] = (uint32_t)u[x];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

constexpr uint32_t kMsAlone = 2;               // open rows from which each gets the whole wave
constexpr int kMsTogether = 4;                 // steps of 16 entries before each open row gets it in any case

// Row chunk c of the pull: rows [v0, v1), kMsWideRows at most.
__device__ __forceinline__ void row_chunk(const MsLevel &p, uint32_t c, int32_t &v0, int32_t &v1) {
    if (p.row_chunks) {
        v0 = p.row_chunks[c];
        v1 = p.row_chunks[c + 1];
        return;
    }
    v0 = (int32_t)c * kMsWideRows;
    v1 = p.n - v0 < kMsWideRows ? p.n : v0 + kMsWideRows;
}

// One mask word: the rows of more than kMsSerial entries below kMsLong, a wave
// per kMsWideRows consecutive rows, four rows to a step with 16 lanes each, four
// such steps (all sixteen rows) in flight together: a row's scan is a chain of
// dependent loads (entry, mask, caller's id), and with one row group after
// another a wave had one of them in flight at a time.  Once at most kMsAlone
// rows are open, or after kMsTogether steps, each is finished by the whole wave.  Before that the long
// rows, a wave per chunk: with long_split only each row's first chunk - it
// holds the row's smallest in-neighbours, so what it finds is final: those
// bits go into vis now and k_ms_pull_rest then scans the later chunks for the
// other sources only; without it every chunk here, all looking for the same
// unsettled sources.
__global__ __launch_bounds__(kBlock) void k_ms_pull_wide(MsLevel p, uint32_t k) {
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], k % 3);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], (k + 1) % 3);
    const uint32_t lane = __lane_id();
    const uint32_t gw = (blockIdx.x * kBlock + threadIdx.x) >> 6, nw = (gridDim.x * kBlock) >> 6;
    const uint32_t nitems = p.long_split ? p.nli : p.nli_chunks;
    for (uint32_t c = gw; c < nitems; c += nw) {                                 // uniform per wave
        int32_t v;
        uint32_t j = 0;
        if (p.long_split) {
            v = p.li[c].v;
        } else {
            const MsLong L = p.li[p.limap[c]];
            v = L.v;
            j = c - L.chunk_base;
        }
        long_chunk(p, cur, nxt, v, j, k, p.long_split != 0u);
    }
    const unsigned long long full = full_word(p, 0u);
    const int g = (int)(lane >> 4);
    const int32_t gl = (int32_t)(lane & 15u);
    for (uint32_t c = gw; c < p.nrow_chunks; c += nw) {                          // uniform per wave
        int32_t v0, v1, b = 0, e = 0;
        row_chunk(p, c, v0, v1);
        unsigned long long r0 = 0ull;
        if ((int32_t)lane < v1 - v0) {
            b = p.in_ptr[v0 + (int32_t)lane];
            e = p.in_ptr[v0 + (int32_t)lane + 1];
            r0 = full & ~p.vis[v0 + (int32_t)lane];
            if (e - b <= kMsSerial || (uint32_t)(e - b) >= kMsLong) r0 = 0ull;
        }
        unsigned long long open = __ballot(r0 != 0ull);
        if (!open) continue;
        int32_t at[4], end[4];
        unsigned long long rem[4], fnd[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int src = 4 * t + g;
            at[t] = __shfl(b, src, 64);
            end[t] = __shfl(e, src, 64);
            rem[t] = __shfl(r0, src, 64);
            fnd[t] = 0ull;
        }
        for (int step = 0; step < kMsTogether && (uint32_t)__popcll(open) > kMsAlone; ++step) {     // uniform
            int32_t uu[4], oo[4];
            bool ok[4];
            unsigned long long mm[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) uu[t] = (rem[t] && at[t] + gl < end[t]) ? p.in_idx[at[t] + gl] : -1;
            if (p.use_fbits) {
                unsigned long long fb[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) fb[t] = uu[t] >= 0 ? p.fbits[(uint32_t)uu[t] >> 6] : 0ull;
#pragma unroll
                for (int t = 0; t < 4; ++t) ok[t] = ((fb[t] >> ((uint32_t)uu[t] & 63u)) & 1ull) != 0ull;
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) ok[t] = uu[t] >= 0;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) mm[t] = ok[t] ? cur[uu[t]] : 0ull;
#pragma unroll
            for (int t = 0; t < 4; ++t) oo[t] = (mm[t] & rem[t]) ? caller_id(p, uu[t]) : -1;
            open = 0ull;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int32_t v = v0 + 4 * t + g;
                const unsigned long long f = scan_resolve<16>(p, srow(p, v < p.n ? v : 0), 0u, oo[t], mm[t] & rem[t],
                                                              true);
                rem[t] &= ~f;
                fnd[t] |= f;
                at[t] += 16;
                if (at[t] >= end[t]) rem[t] = 0ull;
                // row 4 t + g is open: one bit, from its group's first lane
                const unsigned long long o = __ballot(gl == 0 && rem[t] != 0ull);
                open |= ((o & 1ull) | ((o >> 15) & 2ull) | ((o >> 30) & 4ull) | ((o >> 45) & 8ull)) << (4 * t);
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            for (unsigned long long o = (open >> (4 * t)) & 15ull; o; o &= o - 1ull) {       // uniform
                const int og = (int)__ffsll((long long)o) - 1, src = 16 * og;
                const int32_t a = __shfl(at[t], src, 64), z = __shfl(end[t], src, 64);
                const unsigned long long rr = __shfl(rem[t], src, 64);
                const unsigned long long f = scan_wave4(p, cur, srow(p, v0 + 4 * t + og), 0u, a, z, rr, true, false);
                if (g == og) fnd[t] |= f;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (gl == 0 && fnd[t]) nxt[v0 + 4 * t + g] = fnd[t];
    }
}

// Level k, pull form, the later chunks of the long rows (after k_ms_pull):
// each looks only for the sources the row's first chunk left unsettled (vis
// holds those found there), gives its first hits to the staged parents by
// atomicMin (the smallest over the chunks) and ORs its bits into the next
// mask; k_ms_pull_close then folds those into vis and lists the rows.  The chunks
// are taken every row's second chunk first, then the third, ..., so that
// most chunks find their row's earlier chunks done and skip the sources
// those settled.
__global__ __launch_bounds__(kBlock) void k_ms_pull_rest(MsLevel p, uint32_t k) {
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], k % 3);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], (k + 1) % 3);
    const uint32_t gt = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    const uint32_t nrest = p.nli_chunks - p.nli;
    for (uint32_t i = gt >> 6; i < nrest; i += gs >> 6) {                // uniform per wave
        const uint32_t c = p.lirest[i];
        const MsLong L = p.li[p.limap[c]];
        long_chunk(p, cur, nxt, L.v, c - L.chunk_base, k, false);
    }
}

// ---------------------------------------------------------------------------
// several mask words per vertex (more than 64 sources)
// ---------------------------------------------------------------------------
//
// A lane of a scan step holds one word of one entry: lane l has word l % kWp
// and entry l / kWp of the step, so an entry's index is read once for kWp words
// and its mask words, which lie side by side, come in one access, where a scan
// per word reads the list and gathers a line per entry again for every word.
// Measured, directed R-MAT of 2^20 vertices, 256 sources (four words): the
// pulls of a call took 3.15 ms a word at a time.

// The bits of a step: each bit of a lane's hit goes to the lowest entry of the
// step that holds it.  Parents pass through the wave's LDS rows (one of 64
// slots per word) and go out by source, kWp * 64 consecutive entries of the
// staged row.  Returns the bits found of the lane's word.
template <uint32_t kWp>
__device__ __forceinline__ unsigned long long words_resolve(const MsLevel &p, int32_t vo, uint32_t w0, int32_t uc,
                                                            unsigned long long hit, bool owner_alone,
                                                            uint32_t *slots) {
    if (__ballot(hit != 0ull) == 0ull) return 0ull;        // uniform
    const uint32_t lane = __lane_id(), word = lane % kWp;
    unsigned long long incl = hit;
#pragma unroll
    for (uint32_t d = kWp; d < 64u; d <<= 1) {
        const unsigned long long t = __shfl_up(incl, d, 64);
        if (lane >= d) incl |= t;
    }
    unsigned long long below = __shfl_up(incl, kWp, 64);
    if (lane < kWp) below = 0ull;
    unsigned long long own = hit & ~below;
    const unsigned long long found = __shfl(incl, (int)(64u - kWp + word), 64);
    uint32_t *slot = slots + word * 64u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    while (own) {
        const uint32_t b = (uint32_t)__ffsll((long long)own) - 1u;
        own &= own - 1ull;
        slot[b] = (uint32_t)uc;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (uint32_t x = 0; x < kWp; ++x) {
        const unsigned long long fx = __shfl(found, (int)x, 64);
        if ((fx >> lane) & 1ull) {
            const size_t at = stage(p, vo, (w0 + x) * 64u + lane);
            const uint32_t pu = slots[x * 64u + lane];
            if (owner_alone) p.spar[at] = pu;
            else atomicMin(&p.spar[at], pu);
        }
    }
    return found;
}

// Entries [e0, e1) of row v scanned by the whole wave for words w0 .. w0 + kWp -
// 1 (rem: the sources looked for of the lane's word), four steps of 64 / kWp
// entries at a time; prune as scan_wave4.
template <uint32_t kWp>
__device__ __forceinline__ unsigned long long words_scan(const MsLevel &p, const unsigned long long *cur, int32_t vo,
                                                         uint32_t w0, int32_t e0, int32_t e1, unsigned long long rem,
                                                         bool owner_alone, bool prune, uint32_t *slots) {
    constexpr int32_t kStep = 64 / (int32_t)kWp;
    const uint32_t W = p.W, lane = __lane_id(), word = lane % kWp;
    const int32_t entry = (int32_t)(lane / kWp);
    const uint32_t w = w0 + word < W ? w0 + word : W - 1u;   // a word past the last looks for nothing
    unsigned long long found = 0ull;
    for (int32_t eb = e0; eb < e1 && __ballot(rem != 0ull); eb += 4 * kStep) {               // uniform
        int32_t uu[4], oo[4];
        unsigned long long mm[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int32_t e = eb + t * kStep + entry;
            uu[t] = e < e1 ? p.in_idx[e] : -1;
        }
        if (prune) {
            const uint32_t first = (uint32_t)(p.ent ? p.ent[eb] : __shfl(uu[0], 0, 64));
            uint32_t sp[kWp];
#pragma unroll
            for (uint32_t x = 0; x < kWp; ++x)
                sp[x] = w0 + x < W ? p.spar[stage(p, vo, (w0 + x) * 64u + lane)] : 0u;
#pragma unroll
            for (uint32_t x = 0; x < kWp; ++x) {
                const unsigned long long done = __ballot(sp[x] < first);
                if (word == x) rem &= ~done;
            }
            if (!__ballot(rem != 0ull)) break;                                              // uniform
        }
        bool ok[4];
        if (p.use_fbits) {
            unsigned long long fb[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) fb[t] = uu[t] >= 0 ? p.fbits[(uint32_t)uu[t] >> 6] : 0ull;
#pragma unroll
            for (int t = 0; t < 4; ++t) ok[t] = ((fb[t] >> ((uint32_t)uu[t] & 63u)) & 1ull) != 0ull;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) ok[t] = uu[t] >= 0;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) mm[t] = ok[t] ? row(cur, uu[t], W)[w] : 0ull;
#pragma unroll
        for (int t = 0; t < 4; ++t) oo[t] = (mm[t] & rem) ? caller_id(p, uu[t]) : -1;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const unsigned long long f = words_resolve<kWp>(p, vo, w0, oo[t], mm[t] & rem, owner_alone, slots);
            rem &= ~f;
            found |= f;
        }
    }
    return found;
}

// Chunk j of long row v by one wave, kWp words at a time (long_chunk's work).
template <uint32_t kWp>
__device__ __forceinline__ void words_chunk(const MsLevel &p, const unsigned long long *cur, unsigned long long *nxt,
                                            int32_t v, uint32_t j, uint32_t k, bool first, uint32_t *slots) {
    const uint32_t W = p.W, lane = __lane_id();
    const int32_t r1 = p.in_ptr[v + 1];
    const int32_t e0 = p.in_ptr[v] + (int32_t)(j * kMsChunk);
    const int32_t e1 = (e0 + (int32_t)kMsChunk < r1) ? e0 + (int32_t)kMsChunk : r1;
    for (uint32_t w0 = 0; w0 < W; w0 += kWp) {
        const uint32_t w = w0 + lane % kWp;
        const unsigned long long rem = w < W ? full_word(p, w) & ~row(p.vis, v, W)[w] : 0ull;
        const unsigned long long found =
            words_scan<kWp>(p, cur, srow(p, v), w0, e0, e1, rem, false, j != 0, slots);
        if (found && lane < kWp) {                          // lane x has word w0 + x
            atomicOr(&row(nxt, v, W)[w], found);
            if (first) row(p.vis, v, W)[w] |= found;
        }
    }
}

// k_ms_pull_wide for W >= 2 words: four rows of a wave's kMsWideRows in flight
// for their first step, kWp words each; a row with sources left goes on alone.
template <uint32_t kWp>
__global__ __launch_bounds__(kBlock) void k_ms_wide_words(MsLevel p, uint32_t k) {
    __shared__ uint32_t s_par[kBlock / 64][kWp * 64];
    constexpr int32_t kStep = 64 / (int32_t)kWp;
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], k % 3);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], (k + 1) % 3);
    const uint32_t W = p.W, lane = __lane_id(), word = lane % kWp;
    const int32_t entry = (int32_t)(lane / kWp);
    const uint32_t gw = (blockIdx.x * kBlock + threadIdx.x) >> 6, nw = (gridDim.x * kBlock) >> 6;
    uint32_t *slots = s_par[threadIdx.x >> 6];
    const uint32_t nitems = p.long_split ? p.nli : p.nli_chunks;
    for (uint32_t c = gw; c < nitems; c += nw) {                                 // uniform per wave
        int32_t v;
        uint32_t j = 0;
        if (p.long_split) {
            v = p.li[c].v;
        } else {
            const MsLong L = p.li[p.limap[c]];
            v = L.v;
            j = c - L.chunk_base;
        }
        words_chunk<kWp>(p, cur, nxt, v, j, k, p.long_split != 0u, slots);
    }
    for (uint32_t c = gw; c < p.nrow_chunks; c += nw) {                          // uniform per wave
        int32_t v0, v1, b = 0, e = 0;
        row_chunk(p, c, v0, v1);
        if ((int32_t)lane < v1 - v0) {
            b = p.in_ptr[v0 + (int32_t)lane];
            e = p.in_ptr[v0 + (int32_t)lane + 1];
        }
        unsigned long long wide = __ballot(e - b > kMsSerial && (uint32_t)(e - b) < kMsLong);
        while (wide) {                                                           // uniform
            int32_t v[4], at[4], end[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int src = wide ? (int)__ffsll((long long)wide) - 1 : 0;
                v[t] = wide ? v0 + src : -1;
                at[t] = wide ? __shfl(b, src, 64) : 0;
                end[t] = wide ? __shfl(e, src, 64) : 0;
                wide &= wide - 1ull;
            }
            for (uint32_t w0 = 0; w0 < W; w0 += kWp) {
                const uint32_t w = w0 + word;
                const bool has = w < W;
                unsigned long long rem[4], mm[4];
                int32_t uu[4], oo[4];
                bool ok[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    rem[t] = (has && v[t] >= 0) ? full_word(p, w) & ~row(p.vis, v[t], W)[w] : 0ull;
                    uu[t] = at[t] + entry < end[t] ? p.in_idx[at[t] + entry] : -1;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) ok[t] = uu[t] >= 0 && rem[t] != 0ull && in_frontier(p, uu[t]);
#pragma unroll
                for (int t = 0; t < 4; ++t) mm[t] = ok[t] ? row(cur, uu[t], W)[w] : 0ull;
#pragma unroll
                for (int t = 0; t < 4; ++t) oo[t] = (mm[t] & rem[t]) ? caller_id(p, uu[t]) : -1;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (v[t] < 0) continue;                                      // uniform
                    const int32_t vo = srow(p, v[t]);
                    unsigned long long f = words_resolve<kWp>(p, vo, w0, oo[t], mm[t] & rem[t], true, slots);
                    if (at[t] + kStep < end[t])
                        f |= words_scan<kWp>(p, cur, vo, w0, at[t] + kStep, end[t], rem[t] & ~f, true, false, slots);
                    if (f && lane < kWp) row(nxt, v[t], W)[w] = f;
                }
            }
        }
    }
}

// k_ms_pull_rest for W >= 2 words.
template <uint32_t kWp>
__global__ __launch_bounds__(kBlock) void k_ms_rest_words(MsLevel p, uint32_t k) {
    __shared__ uint32_t s_par[kBlock / 64][kWp * 64];
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], k % 3);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], (k + 1) % 3);
    const uint32_t gt = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    const uint32_t nrest = p.nli_chunks - p.nli;
    for (uint32_t i = gt >> 6; i < nrest; i += gs >> 6) {                       // uniform per wave
        const uint32_t c = p.lirest[i];
        const MsLong L = p.li[p.limap[c]];
        words_chunk<kWp>(p, cur, nxt, L.v, c - L.chunk_base, k, false, s_par[threadIdx.x >> 6]);
    }
}

// After a pull level, over all rows: the bits found join vis, the rows with any
// are listed (a block's kMsCloseRows rows through LDS, one counter atomic for
// them), the list's statistics are summed; the last block closes the level.
// Reading every row's mask once (W x 8 bytes in order) replaces a list kept by
// the pull's blocks, which tied their waves together with barriers.
constexpr uint32_t kMsCloseRows = 4 * kBlock;

__global__ __launch_bounds__(kBlock) void k_ms_pull_close(MsLevel p, uint32_t k) {
    __shared__ int32_t s_list[kMsCloseRows];
    __shared__ uint32_t s_n, s_base;
    const uint32_t s1 = (k + 1) % 3;
    const unsigned long long *nxt = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s1);
    int32_t *fnxt = pick3(p.fq[0], p.fq[1], p.fq[2], s1);
    const uint32_t W = p.W, tid = threadIdx.x;
    unsigned long long deg = 0, pairs = 0;
    for (uint32_t c0 = blockIdx.x * kMsCloseRows; c0 < (uint32_t)p.n; c0 += gridDim.x * kMsCloseRows) {
        if (tid == 0) s_n = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < kMsCloseRows / kBlock; ++j) {
            const uint32_t v = c0 + j * kBlock + tid;
            if (v >= (uint32_t)p.n) continue;
            bool any = false;
            for (uint32_t w = 0; w < W; ++w) {
                const unsigned long long nb = row(nxt, (int32_t)v, W)[w];
                if (!nb) continue;
                any = true;
                pairs += (unsigned long long)__popcll(nb);
                row(p.vis, (int32_t)v, W)[w] |= nb;
                set_levels(p, (int32_t)v, w, k + 1, nb);
            }
            if (any) {
                deg += (unsigned long long)(p.out_ptr[v + 1] - p.out_ptr[v]);
                s_list[atomicAdd(&s_n, 1u)] = (int32_t)v;
            }
        }
        __syncthreads();
        if (tid == 0 && s_n) s_base = atomicAdd(&p.cnt[s1], s_n);
        __syncthreads();
        for (uint32_t i = tid; i < s_n; i += kBlock) fnxt[s_base + i] = s_list[i];
        __syncthreads();
    }
    add_stats(p, s1, deg, pairs);
    if (ms_last_to_arrive(p)) ms_close(p, k + 1, true, true);
}

// The staged results into the callers' arrays: a block per 64 vertices and 64
// sources.  Parents go through an LDS tile, so that both the staged rows and the
// per-source output rows move in whole lines; each lane reads 4 sources of a
// staged row and writes 4 vertices of an output row (16 bytes, or 4 scalar
// stores where the caller's array is not 16-byte aligned or at the tail).
// Levels need no transpose while they are bit planes: source q's level of a
// vertex is bit q of the vertex's words, which the block keeps in LDS.  With
// kPlanes false (a search past the planes) they are staged and go as the parents
// do.  Pairs never reached become -1.
template <bool kPlanes>
__global__ __launch_bounds__(kBlock) void k_ms_out(MsLevel p, uint32_t planes) {
    // one 64 x 64 tile (+1 column against bank conflicts): 16.6 KB per block, so
    // that several blocks share a compute unit and keep more loads in flight
    __shared__ int32_t t_x[64][65];
    __shared__ __align__(16) unsigned long long s_word[1 + kMsPlanes][64];   // visited, planes
    __shared__ int32_t s_lab[64];
    const uint32_t W = p.W, S = W * 64u, tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const uint32_t ntiles = (uint32_t)(((size_t)p.n + 63) / 64);
    const uint32_t g4 = (tid & 15u) * 4u;          // first of this lane's 4 columns
    const size_t nw = (size_t)p.n * W;
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int32_t v0 = (int32_t)(tile * 64u);
        const bool in = v0 + (int32_t)lane < p.n;
        const int32_t xl = in ? label_of(p, v0 + (int32_t)lane) : 0;
        for (uint32_t w = 0; w < W; ++w) {
            if (wave == 0) {                       // a wave per kind of word, a lane per vertex
                s_word[0][lane] = in ? row(p.vis, xl, W)[w] : 0ull;
                s_lab[lane] = xl;
            }
            if (kPlanes)
                for (uint32_t j = (wave + 3u) & 3u; j < planes; j += 4u)
                    s_word[1 + j][lane] = in ? p.planes[nw * j + (size_t)xl * W + w] : 0ull;
            __syncthreads();
            int4 lv[4], pa[4];
            uint32_t bits[4];
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {            // this lane's 4 sources of 4 staged rows
                const uint32_t vi = (tid >> 4) + 16u * r;
                const int32_t v = v0 + (int32_t)vi;
                lv[r] = make_int4(-1, -1, -1, -1);
                pa[r] = lv[r];
                bits[r] = (uint32_t)(s_word[0][vi] >> g4) & 15u;
                if (bits[r]) {                          // read once: streaming loads
                    const size_t at = (size_t)(p.stage_labels ? s_lab[vi] : v) * S + w * 64u + g4;
                    const v4i b = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(p.spar + at));
                    pa[r] = make_int4(b.x, b.y, b.z, b.w);
                    if (!kPlanes) {
                        const v4i a = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(p.slev + at));
                        lv[r] = make_int4(a.x, a.y, a.z, a.w);
                    }
                }
            }
            int4 out_l[4], out_p[4];
            if (kPlanes) {
                // sources qi = (tid >> 4) + 16 r of vertices g4 .. g4 + 3 (r < 2: the
                // words' low halves)
                int32_t l[4][4];
#pragma unroll
                for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
                    for (uint32_t x = 0; x < 4; ++x) l[r][x] = 0;
#pragma unroll
                for (uint32_t j = 0; j <= kMsPlanes; ++j) {
                    if (j > planes) break;
                    const uint32_t sel = j < planes ? 1 + j : 0;         // the visited words last
                    unsigned long long m[4];
#pragma unroll
                    for (uint32_t x = 0; x < 4; ++x) m[x] = s_word[sel][g4 + x];
#pragma unroll
                    for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
                        for (uint32_t x = 0; x < 4; ++x) {
                            const uint32_t half = r < 2 ? (uint32_t)m[x] : (uint32_t)(m[x] >> 32);
                            const uint32_t bit = (half >> ((tid >> 4) + 16u * (r & 1u))) & 1u;
                            if (j < planes) l[r][x] |= (int32_t)(bit << j);
                            else l[r][x] = bit ? l[r][x] : -1;
                        }
                }
#pragma unroll
                for (uint32_t r = 0; r < 4; ++r) out_l[r] = make_int4(l[r][0], l[r][1], l[r][2], l[r][3]);
            }
            for (int half = kPlanes ? 1 : 0; half < 2; ++half) {         // levels, then parents
#pragma unroll
                for (uint32_t r = 0; r < 4; ++r) {        // staged rows -> tile[source][vertex]
                    const uint32_t vi = (tid >> 4) + 16u * r;
                    const int4 x = half ? pa[r] : lv[r];
                    t_x[g4 + 0][vi] = (bits[r] & 1u) ? x.x : -1;
                    t_x[g4 + 1][vi] = (bits[r] & 2u) ? x.y : -1;
                    t_x[g4 + 2][vi] = (bits[r] & 4u) ? x.z : -1;
                    t_x[g4 + 3][vi] = (bits[r] & 8u) ? x.w : -1;
                }
                __syncthreads();
#pragma unroll
                for (uint32_t r = 0; r < 4; ++r) {        // tile rows, 4 vertices per lane
                    const uint32_t qi = (tid >> 4) + 16u * r;
                    const int4 y = make_int4(t_x[qi][g4], t_x[qi][g4 + 1], t_x[qi][g4 + 2], t_x[qi][g4 + 3]);
                    if (half) out_p[r] = y;
                    else out_l[r] = y;
                }
                __syncthreads();
            }
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {            // output rows
                const uint32_t qi = (tid >> 4) + 16u * r;
                const uint32_t q = w * 64u + qi;
                if (q >= p.nq) continue;
                const bool full = v0 + (int32_t)g4 + 3 < p.n;
                const auto put = [&](int32_t *o, const int4 &a) {
                    if (full && (reinterpret_cast<uintptr_t>(o) & 15u) == 0) {
                        // written once and not read here again: streaming stores
                        const v4i av = {a.x, a.y, a.z, a.w};
                        __builtin_nontemporal_store(av, reinterpret_cast<v4i *>(o));
                        return;
                    }
                    const int32_t av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (v0 + (int32_t)g4 + j < p.n) o[j] = av[j];
                };
                put(p.level[q] + v0 + g4, out_l[r]);
                put(p.parent[q] + v0 + g4, out_p[r]);
            }
        }
    }
}

// Level k, pull form, pass r of the range order (dense levels, one mask
// word).  The in-neighbours are visited one vertex range at a time, in
// ascending order of ranges: pass r looks only at the in-list entries whose
// in-neighbour lies in [r n / R, (r + 1) n / R), so the frontier masks it
// gathers (2 MB) stay in the XCDs' L2.  A row's lists are sorted, so each
// pass continues where the row's previous pass stopped (rcur); a source found
// in an earlier range has its smallest frontier in-neighbour there, so what a
// pass finds is final - written at once, with no atomics between passes.
// Pass 0 looks at every row; a row still open after a pass (sources unfound,
// entries left) goes on the list of the next pass.  Rows of at most kRpShort
// entries are scanned by one lane (16 entries per step, then the wave writes
// the staged results of its lanes' rows one row at a time); longer rows by a
// whole wave, 64 entries per step.  Also clears F_{k-1}'s masks (pass 0).
constexpr int32_t kRpShort = 64;

// One wave, one row: its entries from e with in-neighbour below rend, 64 a
// step, until rem is empty.  Stages the first hits; returns the bits found and
// leaves e at the first entry not scanned.
__device__ __forceinline__ unsigned long long rp_wave_row(const MsLevel &p, const unsigned long long *cur,
                                                          int32_t v, int32_t &e, int32_t e1, uint32_t rend,
                                                          unsigned long long rem) {
    const uint32_t lane = __lane_id();
    unsigned long long found = 0ull;
    while (e < e1 && rem) {                                    // uniform
        const int32_t ei = e + (int32_t)lane;
        int32_t u = 0;
        bool in = false;
        if (ei < e1) {
            u = p.in_idx[ei];
            in = (uint32_t)u < rend;
        }
        unsigned long long hit = 0ull;
        if (in) hit = cur[u] & rem;
        // the step's entries in the range are a prefix of its lanes (sorted list)
        const uint32_t cnt = (uint32_t)__popcll(__ballot(in));
        if (__ballot(hit != 0ull)) {
            unsigned long long incl = hit;
#pragma unroll
            for (uint32_t d = 1; d < 64; d <<= 1) {
                const unsigned long long t = __shfl_up(incl, d, 64);
                if (lane >= d) incl |= t;
            }
            unsigned long long below = __shfl_up(incl, 1u, 64);
            if (lane == 0) below = 0ull;
            unsigned long long own = hit & ~below;
            while (own) {
                const uint32_t b = (uint32_t)__ffsll((long long)own) - 1u;
                own &= own - 1ull;
                const size_t at = stage(p, v, b);
                p.spar[at] = (uint32_t)u;
            }
            const unsigned long long f = __shfl(incl, 63, 64);
            rem &= ~f;
            found |= f;
        }
        e += (int32_t)cnt;
        if (cnt < 64u) break;                                 // the range or the row ended here
    }
    return found;
}

__global__ __launch_bounds__(kBlock) void k_ms_rpull(MsLevel p, uint32_t k, uint32_t r) {
    __shared__ int32_t s_list[kMsRows];                 // rows the level lists
    __shared__ int32_t s_wide[kMsRows];                 // rows for a whole wave
    __shared__ int32_t s_open[kMsRows];                 // rows open after this pass
    __shared__ int32_t s_ocur[kMsRows];                 //   and their next entries
    __shared__ uint32_t s_off[kBlock][9];               // a row's found bits: entry offset, 4 bits each
    __shared__ unsigned long long s_fnd[kBlock];
    __shared__ int32_t s_e0[kBlock];
    __shared__ uint32_t s_n, s_nw, s_no, s_base, s_obase;
    const uint32_t s0 = k % 3, s1 = (k + 1) % 3, s2 = (k + 2) % 3;
    const unsigned long long *cur = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s0);
    unsigned long long *nxt = pick3(p.m[0], p.m[1], p.m[2], s1);
    int32_t *fnxt = pick3(p.fq[0], p.fq[1], p.fq[2], s1);
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const uint32_t gt = blockIdx.x * kBlock + tid, gs = gridDim.x * kBlock;
    const uint32_t R = p.rp_ranges;
    const uint32_t rend = (r + 1 == R) ? (uint32_t)p.n : (uint32_t)(((uint64_t)(r + 1) * (uint64_t)p.n) / R);
    const unsigned long long full = (p.nq & 63u) ? ((1ull << (p.nq & 63u)) - 1ull) : ~0ull;
    if (r == 0) {
        unsigned long long *old = pick3(p.m[0], p.m[1], p.m[2], s2);
        const int32_t *fold = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s2);
        const uint32_t nold = p.cnt[s2];
        for (uint32_t t = gt; t < nold; t += gs) old[fold[t]] = 0ull;
    }
    if (gt == 0) p.rcnt[(r + 1) % 3] = 0u;                     // the next pass's open rows
    const bool all = (r == 0);
    const uint32_t nin = all ? (uint32_t)p.n : p.rcnt[(r + 2) % 3];   // pass r-1's open rows
    const int32_t *lin = p.rlist[(r + 1) & 1];
    int32_t *lout = p.rlist[r & 1];
    for (uint32_t c0 = blockIdx.x * kMsRows; c0 < nin; c0 += gridDim.x * kMsRows) {
        if (tid == 0) {
            s_n = 0;
            s_nw = 0;
            s_no = 0;
        }
        __syncthreads();
        const uint32_t c1 = (c0 + kMsRows < nin) ? c0 + kMsRows : nin;
        for (uint32_t r0 = c0; r0 < c1; r0 += kBlock) {
            const uint32_t i = r0 + tid;
            int32_t v = -1, e = 0, e1 = 0;
            unsigned long long sv = 0ull, rem = 0ull;
            bool act = false;
            if (i < c1) {
                v = all ? (int32_t)i : lin[i];
                const int32_t b0 = p.in_ptr[v];
                e1 = p.in_ptr[v + 1];
                e = all ? b0 : p.rcur[v];
                if (e < e1) {
                    sv = p.vis[v];
                    rem = full & ~sv;
                    if (rem) {
                        if (e1 - b0 > kRpShort) s_wide[atomicAdd(&s_nw, 1u)] = v;
                        else act = true;
                    }
                }
            }
            unsigned long long got = 0ull;
            const bool mine = act;
            // steps of up to 16 entries; after each, the wave writes its
            // lanes' staged results one row at a time
            while (__ballot(act)) {                               // uniform
                unsigned long long found = 0ull;
#pragma unroll
                for (int j = 0; j < 9; ++j) s_off[tid][j] = 0u;
                s_e0[tid] = e;
                if (act) {
                    const int32_t es = e;
                    bool more = true;
                    for (int bt = 0; bt < 4 && more && rem; ++bt) {
                        int32_t uu[4];
                        unsigned long long mm[4];
                        bool in[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) uu[j] = p.in_idx[e + j < e1 ? e + j : e1 - 1];
#pragma unroll
                        for (int j = 0; j < 4; ++j) in[j] = (e + j < e1) && (uint32_t)uu[j] < rend;
#pragma unroll
                        for (int j = 0; j < 4; ++j) mm[j] = in[j] ? cur[uu[j]] : 0ull;
                        int nin4 = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            nin4 += in[j] ? 1 : 0;
                            unsigned long long hit = mm[j] & rem;
                            rem &= ~hit;
                            found |= hit;
                            const uint32_t off = (uint32_t)(e - es + j);
                            while (hit) {
                                const uint32_t b = (uint32_t)__ffsll((long long)hit) - 1u;
                                hit &= hit - 1ull;
                                s_off[tid][b >> 3] |= off << ((b & 7u) * 4u);
                            }
                        }
                        e += nin4;
                        more = (nin4 == 4);
                    }
                    // open while sources are unfound and this range may hold more
                    act = more && rem && e < e1;
                }
                got |= found;
                s_fnd[tid] = found;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                for (unsigned long long rows = __ballot(found != 0ull); rows; rows &= rows - 1ull) {
                    const uint32_t rr = (tid & ~63u) + (uint32_t)__ffsll((long long)rows) - 1u;
                    const unsigned long long fm = s_fnd[rr];
                    if ((fm >> lane) & 1ull) {
                        const uint32_t j = (s_off[rr][lane >> 3] >> ((lane & 7u) * 4u)) & 15u;
                        const int32_t rv = all ? (int32_t)(r0 + rr) : lin[r0 + rr];
                        const size_t at = stage(p, rv, lane);
                        p.spar[at] = (uint32_t)p.in_idx[s_e0[rr] + (int32_t)j];
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (mine) {
                if (got) {
                    const unsigned long long before = nxt[v];
                    nxt[v] = before | got;
                    p.vis[v] = sv | got;
                    if (!before) s_list[atomicAdd(&s_n, 1u)] = v;
                }
                if (rem && e < e1) {                               // the next range continues here
                    const uint32_t o = atomicAdd(&s_no, 1u);
                    s_open[o] = v;
                    s_ocur[o] = e;
                }
            }
        }
        __syncthreads();
        // the longer rows: a wave each
        for (uint32_t wi = wave; wi < s_nw; wi += kBlock / 64) {
            const int32_t v = s_wide[wi];
            const int32_t b0 = p.in_ptr[v], e1 = p.in_ptr[v + 1];
            int32_t e = all ? b0 : p.rcur[v];
            const unsigned long long sv = p.vis[v];
            const unsigned long long rem = full & ~sv;
            const unsigned long long got = rp_wave_row(p, cur, v, e, e1, rend, rem);
            if (lane == 0) {
                if (got) {
                    const unsigned long long before = nxt[v];
                    nxt[v] = before | got;
                    p.vis[v] = sv | got;
                    if (!before) s_list[atomicAdd(&s_n, 1u)] = v;
                }
                if ((rem & ~got) && e < e1) {
                    const uint32_t o = atomicAdd(&s_no, 1u);
                    s_open[o] = v;
                    s_ocur[o] = e;
                }
            }
        }
        __syncthreads();
        if (tid == 0) {
            if (s_n) s_base = atomicAdd(&p.cnt[s1], s_n);
            if (s_no) s_obase = atomicAdd(&p.rcnt[r % 3], s_no);
        }
        __syncthreads();
        for (uint32_t i = tid; i < s_n; i += kBlock) fnxt[s_base + i] = s_list[i];
        for (uint32_t i = tid; i < s_no; i += kBlock) {
            lout[s_obase + i] = s_open[i];
            p.rcur[s_open[i]] = s_ocur[i];
        }
        __syncthreads();
    }
}

// After a range-ordered pull (whose passes list the rows themselves): the
// statistics of the level-(k+1) list, and the level's close.
__global__ __launch_bounds__(kBlock) void k_ms_report(MsLevel p, uint32_t k) {
    const uint32_t s1 = (k + 1) % 3;
    const uint32_t nnext = p.cnt[s1];
    const int32_t *fnxt = pick3<const int32_t *>(p.fq[0], p.fq[1], p.fq[2], s1);
    const unsigned long long *nxt = pick3<const unsigned long long *>(p.m[0], p.m[1], p.m[2], s1);
    const uint32_t W = p.W;
    const uint32_t gt = blockIdx.x * kBlock + threadIdx.x, gs = gridDim.x * kBlock;
    if (gt == 0)
        for (int t = 0; t < 3; ++t) p.rcnt[t] = 0u;           // the range passes' open rows
    unsigned long long deg = 0, pairs = 0;
    for (uint32_t i = gt; i < nnext; i += gs) {
        const int32_t v = fnxt[i];
        deg += (unsigned long long)(p.out_ptr[v + 1] - p.out_ptr[v]);
        for (uint32_t w = 0; w < W; ++w) {
            const unsigned long long nb = row(nxt, v, W)[w];
            pairs += (unsigned long long)__popcll(nb);
            if (nb) set_levels(p, v, w, k + 1, nb);
        }
    }
    add_stats(p, s1, deg, pairs);
    if (ms_last_to_arrive(p)) ms_close(p, k + 1, true, true);
}

hipError_t launch_ms_rpull(const MsLevel &p, uint32_t k, uint32_t r, uint32_t grid, hipStream_t s) {
    hipLaunchKernelGGL(k_ms_rpull, dim3(grid), dim3(kBlock), 0, s, p, k, r);
    return hipGetLastError();
}

hipError_t launch_ms(const MsLevel &p, MsPhase phase, uint32_t k, uint32_t grid, hipStream_t s) {
    // the walks over a level's list end in a few atomics per workgroup on the
    // same words: at most 2,048 workgroups for them (R-MAT s22: 25-31 us at
    // 8,192, 17-22 us at 1,024-2,048), and no more than the rows can fill
    const uint32_t rows = (uint32_t)(((size_t)p.n + kMsCloseRows - 1) / kMsCloseRows);
    const uint32_t small = grid < 2048u ? grid : 2048u;
    const uint32_t close = small < rows ? small : rows;
    const dim3 g(grid), b(kBlock);
    switch (phase) {
        case kMsClear: hipLaunchKernelGGL(k_ms_clear, g, b, 0, s, p); break;
        case kMsRoots: hipLaunchKernelGGL(k_ms_roots, dim3((p.nq + kBlock - 1) / kBlock), b, 0, s, p); break;
        case kMsPush: hipLaunchKernelGGL(k_ms_push, g, b, 0, s, p, k); break;
        case kMsSettle: hipLaunchKernelGGL(k_ms_settle, dim3(close), b, 0, s, p, k); break;
        case kMsFbits: hipLaunchKernelGGL(k_ms_fbits, g, b, 0, s, p, k); break;
        case kMsShortRows:
            if (p.W == 1) hipLaunchKernelGGL(k_ms_pull_short<true>, g, b, 0, s, p, k);
            else hipLaunchKernelGGL(k_ms_pull_short<false>, g, b, 0, s, p, k);
            break;
        case kMsWide:
            if (p.W == 1) hipLaunchKernelGGL(k_ms_pull_wide, g, b, 0, s, p, k);
            else if (p.W == 2) hipLaunchKernelGGL(k_ms_wide_words<2>, g, b, 0, s, p, k);
            else hipLaunchKernelGGL(k_ms_wide_words<4>, g, b, 0, s, p, k);
            break;
        case kMsRest:
            if (p.W == 1) hipLaunchKernelGGL(k_ms_pull_rest, g, b, 0, s, p, k);
            else if (p.W == 2) hipLaunchKernelGGL(k_ms_rest_words<2>, g, b, 0, s, p, k);
            else hipLaunchKernelGGL(k_ms_rest_words<4>, g, b, 0, s, p, k);
            break;
        case kMsClose: hipLaunchKernelGGL(k_ms_pull_close, dim3(close), b, 0, s, p, k); break;
        case kMsReport: hipLaunchKernelGGL(k_ms_report, dim3(small), b, 0, s, p, k); break;
    }
    return hipGetLastError();
}

hipError_t launch_ms_zero(unsigned long long *a, size_t words, hipStream_t s) {
    const size_t want = (words + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_ms_zero, dim3((uint32_t)(want < 8192 ? want : 8192)), dim3(kBlock), 0, s, a, words);
    return hipGetLastError();
}

hipError_t launch_ms_levels(const MsLevel &p, uint32_t planes, unsigned long long *tmp, uint32_t grid, hipStream_t s) {
    if (!ms_levels_fit(p.n, planes)) return hipErrorInvalidValue;
    const size_t behind = ms_levels_row(p.n, planes), waves = (size_t)grid * (kBlock / 64);     // (row, word)s of the parts
    const auto part = [&](uint32_t which, size_t rows) -> hipError_t {
        if (rows * p.W < 64 * waves) hipLaunchKernelGGL(k_ms_levels<true>, dim3(grid), dim3(kBlock), 0, s, p, planes, tmp, which);
        else hipLaunchKernelGGL(k_ms_levels<false>, dim3(grid), dim3(kBlock), 0, s, p, planes, tmp, which);
        return hipGetLastError();
    };
    const hipError_t e = part(0u, (size_t)p.n - behind);
    return e != hipSuccess || planes == 0 ? e : part(1u, behind);
}

hipError_t launch_ms_out(const MsLevel &p, uint32_t planes, uint32_t grid, hipStream_t s) {
    if (p.direct_levels) hipLaunchKernelGGL(k_ms_out<false>, dim3(grid), dim3(kBlock), 0, s, p, 0u);
    else hipLaunchKernelGGL(k_ms_out<true>, dim3(grid), dim3(kBlock), 0, s, p, planes);
    return hipGetLastError();
}

}  // namespace bfsi
