// One masked sparse-matrix x sparse-vector product y = A^T[R, C] x over a
// chosen semiring: the operation the method is built from (Definition 1's
// submatrix A^T[V_{k+1}, V_k] is a row mask over the unvisited rows), offered
// as a primitive the way masked-algebra libraries offer it.  The semirings are
// those the Notation section names - Boolean (OR, AND), arithmetic (+, x),
// tropical (min, +) - plus (min, select), which gives the smallest column.
// A is pattern-only (entries 1); values are unsigned 64-bit, arithmetic wraps
// modulo 2^64, and min-plus adds 1 with saturation at 2^64 - 1.
//
// Passes (one stream, the host waits at the end):
//   k_sp_check    every vector index in [0, n) (else no product runs)
//   k_sp_product  up to 64 columns a wave, their entries dealt evenly to the
//                 lanes; columns of kSpLong entries are listed for the chunk pass
//   k_sp_items    chunk offsets of the listed columns (one workgroup scan)
//   k_sp_long     chunks of kSpChunk entries, a wave each
//   k_sp_count / k_sp_scan / k_sp_write
//                 the support bitmap compacted in ascending order with the
//                 values, resetting the accumulator, the bitmap and the state as
//                 it goes; the outcome goes to a pinned host slot
// What bounds it: a product is a chain of dependent random reads (row, its mask
// word, its support word and accumulator) and then its atomics; a lane keeps
// kSpBatch of them in flight.  R-MAT of 2^20 vertices, the widest level of a
// search (min, select): product 161 + long columns 71 us with one entry after
// another, 140 + 57 with eight of a lane in flight (the call 395 -> 298 us); a
// random graph of 20,001 vertices 150 -> 50 us, most of it launches, copies and
// the lockstep over the longest column.
// Every product is an atomic on the row's accumulator (OR, add, or max of
// the complement for the min semirings, so that every identity is zero) and
// the row's support bit; products equal to the identity skip the value atomic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bfs_device.h"
#include "bfs_internal.h"

namespace bfsi {

namespace {

constexpr uint32_t kWaves = kBlock / 64;
constexpr int kScanBlock = 1024;

__device__ __forceinline__ bool allowed(const uint32_t *mask, uint32_t comp, int32_t v) {
    if (mask == nullptr) return true;
    return (((mask[(uint32_t)v >> 5] >> (v & 31)) & 1u) ^ comp) != 0u;
}

// 1 (x) v for the semiring (A's entries are 1)
__device__ __forceinline__ unsigned long long mul(uint32_t sr, unsigned long long v) {
    if (sr == kSrBoolean) return v != 0ull ? 1ull : 0ull;
    if (sr == kSrMinPlus) return v == ~0ull ? v : v + 1ull;
    return v;
}

// y(i) (+)= p for kSpBatch entries of a lane (those with on), and their rows join
// the support: the row-mask words of all of them are loaded together, then the
// support words and (min semirings) the accumulators, then the atomics that are
// still needed go out.  One entry after another a lane had one of these
// dependent loads in flight at a time.  The pre-reads may be stale: bits are only
// set and accumulators of the min semirings only raised, so a stale one lets an
// atomic through that changes nothing.
constexpr int kSpBatch = 8;

__device__ __forceinline__ void accumulate(const SpParams &P, const int32_t (&i)[kSpBatch],
                                           const unsigned long long (&p)[kSpBatch], bool (&on)[kSpBatch]) {
    uint32_t m[kSpBatch], w[kSpBatch];
    unsigned long long a[kSpBatch];
    if (P.row_mask != nullptr) {
#pragma unroll
        for (int x = 0; x < kSpBatch; ++x) m[x] = on[x] ? P.row_mask[(uint32_t)i[x] >> 5] : 0u;
#pragma unroll
        for (int x = 0; x < kSpBatch; ++x) on[x] = on[x] && (((m[x] >> (i[x] & 31)) & 1u) ^ P.row_comp) != 0u;
    }
    const bool lowest = P.semiring == kSrMinPlus || P.semiring == kSrMinSelect;
#pragma unroll
    for (int x = 0; x < kSpBatch; ++x) {
        w[x] = 0xFFFFFFFFu;
        a[x] = ~0ull;
        if (on[x]) {
            w[x] = P.touched[(uint32_t)i[x] >> 5];
            if (lowest) a[x] = P.acc[i[x]];
        }
    }
#pragma unroll
    for (int x = 0; x < kSpBatch; ++x) {
        if (!on[x]) continue;
        const uint32_t bit = 1u << (i[x] & 31);
        if ((w[x] & bit) == 0u) atomicOr(&P.touched[(uint32_t)i[x] >> 5], bit);
        if (lowest) {
            const unsigned long long c = ~p[x];              // min of p == max of ~p
            if (a[x] < c) atomicMax(&P.acc[i[x]], c);
        } else if (p[x]) {
            if (P.semiring == kSrBoolean) atomicOr(&P.acc[i[x]], 1ull);
            else atomicAdd(&P.acc[i[x]], p[x]);
        }
    }
}

// Exclusive prefix sum over a workgroup of kScanBlock threads, and the total:
// within the waves by shuffles, over their sums through LDS.
__device__ __forceinline__ unsigned long long block_scan(unsigned long long v, unsigned long long *s,
                                                         unsigned long long &total) {
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    unsigned long long inc = v;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const unsigned long long o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s[wave] = inc;
    __syncthreads();
    unsigned long long before = 0ull;
    total = 0ull;
    for (uint32_t k = 0; k < kScanBlock / 64; ++k) {
        const unsigned long long x = s[k];
        before += k < wave ? x : 0ull;
        total += x;
    }
    __syncthreads();
    return before + inc - v;
}

}  // namespace

__global__ __launch_bounds__(kBlock) void k_sp_check(SpParams P) {
    bool bad = false;
    for (uint32_t x = blockIdx.x * kBlock + threadIdx.x; x < (uint32_t)P.nx; x += gridDim.x * kBlock) {
        const int32_t j = P.x_idx[x];
        bad = bad || j < 0 || j >= P.n;
    }
    if (__ballot(bad) != 0ull && lane_id() == 0) atomicOr(&P.st->bad, 1u);
}

// The columns below kSpLong entries, C to a wave (64, or as few as spread the
// vector over all waves): their entries on one line (a prefix sum of their
// lengths), 64 kSpBatch of them a step whatever the columns' lengths.  Longer
// columns are listed for k_sp_long.
__global__ __launch_bounds__(kBlock) void k_sp_product(SpParams P) {
    __shared__ int32_t s_pre[kWaves][64];
    if (P.st->bad) return;
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t gw = blockIdx.x * kWaves + wave, nw = gridDim.x * kWaves;
    int32_t *pre = s_pre[wave];
    const uint32_t want = ((uint32_t)P.nx + nw - 1u) / nw;
    const uint32_t C = want >= 64u ? 64u : (want <= 1u ? 1u : 1u << (32 - __clz((int)(want - 1u))));
    for (uint32_t x0 = gw * C; x0 < (uint32_t)P.nx; x0 += nw * C) {              // uniform per wave
        const uint32_t x = x0 + lane;
        int32_t j = -1, r0 = 0, deg = 0;
        unsigned long long p = 0ull;
        if (lane < C && x < (uint32_t)P.nx) {
            j = P.x_idx[x];
            if (allowed(P.col_mask, P.col_comp, j)) {
                r0 = P.out_ptr[j];
                deg = P.out_ptr[j + 1] - r0;
                p = mul(P.semiring, P.x_val[x]);
            }
        }
        const int32_t dl = deg < (int32_t)kSpLong ? deg : 0;
        const int32_t inc = (int32_t)wave_incl_scan((uint32_t)dl);
        const int32_t total = __shfl(inc, 63, 64);
        pre[lane] = inc - dl;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int32_t t0 = 0; t0 < total; t0 += 64 * kSpBatch) {                  // uniform
            int32_t i[kSpBatch], at[kSpBatch];
            unsigned long long pp[kSpBatch];
            bool on[kSpBatch];
#pragma unroll
            for (int q = 0; q < kSpBatch; ++q) {
                const int32_t t = t0 + 64 * q + (int32_t)lane;
                on[q] = t < total;
                int c = 0;                                  // the last column with pre <= t
#pragma unroll
                for (int step = 32; step; step >>= 1)
                    if (pre[c + step] <= t) c += step;
                at[q] = __shfl(r0, c, 64) + (t - pre[c]);
                pp[q] = __shfl(p, c, 64);
            }
#pragma unroll
            for (int q = 0; q < kSpBatch; ++q) i[q] = on[q] ? P.out_idx[at[q]] : 0;
            accumulate(P, i, pp, on);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();                                        // pre is rewritten
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const bool lg = deg >= (int32_t)kSpLong;
        const unsigned long long bm = __ballot(lg);
        if (bm) {
            uint32_t slot = 0;
            if (lane == 0) slot = atomicAdd(&P.st->nitems, (uint32_t)__popcll(bm));
            slot = __shfl(slot, 0, 64) + lanes_below(bm);
            if (lg) {
                SpItem it2;
                it2.j = j;
                it2.nch = ((uint32_t)deg + kSpChunk - 1u) / kSpChunk;
                it2.v = p;
                it2.base = 0ull;
                P.items[slot] = it2;
            }
        }
    }
}

// Chunk offsets of the listed columns: one workgroup of kScanBlock threads.
__global__ __launch_bounds__(kScanBlock) void k_sp_items(SpParams P) {
    __shared__ unsigned long long s[kScanBlock / 64];
    if (P.st->bad) return;
    const uint32_t m = P.st->nitems;
    unsigned long long run = 0ull;
    for (uint32_t b = 0; b < m; b += kScanBlock) {
        const uint32_t t = b + threadIdx.x;
        const unsigned long long c = t < m ? (unsigned long long)P.items[t].nch : 0ull;
        unsigned long long total;
        const unsigned long long ex = block_scan(c, s, total);
        if (t < m) P.items[t].base = run + ex;
        run += total;
    }
    if (threadIdx.x == 0) P.st->nchunks = run;
}

__global__ __launch_bounds__(kBlock) void k_sp_long(SpParams P) {
    if (P.st->bad) return;
    const unsigned long long nch = P.st->nchunks;
    const uint32_t m = P.st->nitems;
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    for (unsigned long long c = (unsigned long long)blockIdx.x * kWaves + wave; c < nch;
         c += (unsigned long long)gridDim.x * kWaves) {
        uint32_t lo = 0, hi = m - 1;                      // last item with base <= c
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1u) >> 1;
            if (P.items[mid].base <= c) lo = mid; else hi = mid - 1u;
        }
        const SpItem it = P.items[lo];
        // positions within the chunk: 512 past an entry near 2^31 is no int32
        const int32_t e0 = P.out_ptr[it.j] + (int32_t)((c - it.base) * kSpChunk);
        const int32_t left = P.out_ptr[it.j + 1] - e0, len = left < (int32_t)kSpChunk ? left : (int32_t)kSpChunk;
        for (int32_t t0 = 0; t0 < len; t0 += 64 * kSpBatch) {              // uniform
            int32_t i[kSpBatch];
            unsigned long long pp[kSpBatch];
            bool on[kSpBatch];
#pragma unroll
            for (int q = 0; q < kSpBatch; ++q) {
                const int32_t t = t0 + 64 * q + (int32_t)lane;
                on[q] = t < len;
                i[q] = on[q] ? P.out_idx[e0 + t] : 0;
                pp[q] = it.v;
            }
            accumulate(P, i, pp, on);
        }
    }
}

// Output pass 1: set bits per workgroup of kSpOutWords words.
__global__ __launch_bounds__(kSpOutWords) void k_sp_count(SpParams P) {
    __shared__ uint32_t s[kSpOutWords / 64];
    const uint32_t w = blockIdx.x * kSpOutWords + threadIdx.x;
    uint32_t c = w < P.words ? (uint32_t)__popc(P.touched[w]) : 0u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if (lane_id() == 0) s[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (uint32_t k = 0; k < kSpOutWords / 64; ++k) t += s[k];
        P.block_off[blockIdx.x] = t;
    }
}

// Output pass 2 where there are more than kSpSelf workgroups: their exclusive
// offsets (one workgroup of kScanBlock threads).
__global__ __launch_bounds__(kScanBlock) void k_sp_scan(SpParams P, uint32_t nblocks) {
    __shared__ unsigned long long s[kScanBlock / 64];
    unsigned long long run = 0ull;
    for (uint32_t b = 0; b < nblocks; b += kScanBlock) {
        const uint32_t t = b + threadIdx.x;
        const unsigned long long c = t < nblocks ? (unsigned long long)P.block_off[t] : 0ull;
        unsigned long long total;
        const unsigned long long ex = block_scan(c, s, total);
        if (t < nblocks) P.block_off[t] = (uint32_t)(run + ex);
        run += total;
    }
}

// Output pass 3: each word's rows in ascending order with their values; the
// accumulator entries and the words go back to zero.  With summed set
// block_off holds the workgroups' offsets; otherwise their counts, which each
// workgroup sums up to its own (a launch less; kSpSelf counts at most).  After a
// bad vector no row is in the support and nothing is written.  The first
// workgroup reports that (host[0]) and resets the state for the next call, the
// last one reports the output's length (host[1]).
constexpr uint32_t kSpSelf = 4096;

__global__ __launch_bounds__(kSpOutWords) void k_sp_write(SpParams P, uint32_t summed) {
    __shared__ uint32_t s[kSpOutWords / 64], s_before[kSpOutWords / 64];
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t w = blockIdx.x * kSpOutWords + threadIdx.x;
    uint32_t bits = w < P.words ? P.touched[w] : 0u;
    const uint32_t c = (uint32_t)__popc(bits);
    const uint32_t incl = wave_incl_scan(c);
    uint32_t before = 0;
    if (summed) {
        if (threadIdx.x == 0) before = P.block_off[blockIdx.x];
    } else {
        for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kSpOutWords) before += P.block_off[b];
    }
    before = wave_sum(before);
    if (lane == 63) s[wave] = incl;
    if (lane == 0) s_before[wave] = before;
    __syncthreads();
    uint32_t pos = incl - c, total = 0;
#pragma unroll
    for (uint32_t k = 0; k < kSpOutWords / 64; ++k) {
        pos += (k < wave ? s[k] : 0u) + s_before[k];
        total += s[k] + s_before[k];
    }
    const bool min_sr = P.semiring == kSrMinPlus || P.semiring == kSrMinSelect;
    while (bits) {
        const int b = __ffs(bits) - 1;
        bits &= bits - 1u;
        const int32_t i = (int32_t)(w * 32u + (uint32_t)b);
        const unsigned long long a = P.acc[i];
        P.y_idx[pos] = i;
        P.y_val[pos] = min_sr ? ~a : a;
        P.acc[i] = 0ull;
        ++pos;
    }
    if (c) P.touched[w] = 0u;
    if (threadIdx.x != 0) return;
    if (blockIdx.x == gridDim.x - 1) P.host[1] = total;
    if (blockIdx.x == 0) {
        P.host[0] = P.st->bad;
        P.st->bad = 0;
        P.st->nitems = 0;
        P.st->nchunks = 0ull;
    }
}

SpLayout sp_layout(int32_t n, int32_t max_nx) {
    SpLayout L{};
    const size_t words = ((size_t)n + 31) / 32;
    const size_t nblocks = (words + kSpOutWords - 1) / kSpOutWords;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = (off + bytes + 255) & ~(size_t)255; return o; };
    L.state = take(sizeof(SpState));
    L.acc = take((size_t)n * 8);
    L.touched = take(words * 4);
    L.items = take((size_t)(max_nx > 0 ? max_nx : 1) * sizeof(SpItem));
    L.block_off = take(nblocks * 4);
    L.total = off;
    return L;
}

hipError_t launch_spmspv(const SpParams &p, uint32_t grid, hipStream_t s) {
    uint32_t cg = ((uint32_t)p.nx + kBlock - 1) / kBlock;
    if (cg > 1024) cg = 1024;
    if (cg == 0) cg = 1;
    hipLaunchKernelGGL(k_sp_check, dim3(cg), dim3(kBlock), 0, s, p);
    hipLaunchKernelGGL(k_sp_product, dim3(grid), dim3(kBlock), 0, s, p);
    hipLaunchKernelGGL(k_sp_items, dim3(1), dim3(kScanBlock), 0, s, p);
    hipLaunchKernelGGL(k_sp_long, dim3(grid), dim3(kBlock), 0, s, p);
    const uint32_t nb = (p.words + kSpOutWords - 1) / kSpOutWords;
    hipLaunchKernelGGL(k_sp_count, dim3(nb), dim3(kSpOutWords), 0, s, p);
    const bool summed = nb > kSpSelf;
    if (summed) hipLaunchKernelGGL(k_sp_scan, dim3(1), dim3(kScanBlock), 0, s, p, nb);
    hipLaunchKernelGGL(k_sp_write, dim3(nb), dim3(kSpOutWords), 0, s, p, summed ? 1u : 0u);
    return hipGetLastError();
}

}  // namespace bfsi
