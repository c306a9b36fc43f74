// Wave64 and memory-scope helpers shared by every gfx950 kernel file of the
// library.  Device code only; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bfs_internal.h"

namespace bfsi {

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Number of lanes below the calling lane whose bit is set in m.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    const uint32_t lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(x, d, 64);
        if (lane >= (uint32_t)d) x += t;
    }
    return x;
}

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(v, d, 64);
        v = o < v ? o : v;
    }
    return v;
}

__device__ __forceinline__ int32_t wave_max(int32_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int32_t o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Loads that see other compute units' atomics (coherent across the XCDs' L2s).
__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_agent64(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The selector network 12 -> 32 (ReLU) -> 32 (ReLU) -> 3: row-major weights
// [out][in] followed by the biases, then the feature mean and inverse std.
//
// A decision stands between two levels, so its latency counts in full.
// Evaluated from global memory it took 4 to 5 us, a dependent read for each
// layer; so a whole workgroup stages the weights in LDS first, one coalesced
// trip (which a caller's own reads share) by kBlock threads, the rows an odd number of words
// apart, so that 32 lanes reading one column hit 32 banks (rows of 32 words hit
// two).
constexpr int kMlpRow1 = kMlpIn + 1, kMlpRow2 = kMlpH + 1;
constexpr int kMlpAt2 = kMlpRow1 * kMlpH;                   // the second layer's rows
constexpr int kMlpAtRest = kMlpAt2 + kMlpRow2 * kMlpH;      // b1, b2, then W3 to the end as they are
constexpr int kMlpLds = kMlpAtRest + kMlpTotal - kMlpIn * kMlpH - kMlpH * kMlpH;

// (in two halves, so that reads of the caller's can be in flight as well)
struct MlpTrip {
    static constexpr int per = (kMlpTotal + kBlock - 1) / kBlock;
    float x[per];
};

__device__ __forceinline__ void load_mlp(const float *w, MlpTrip &m) {
#pragma unroll
    for (int t = 0; t < MlpTrip::per; ++t) {
        const int i = (int)threadIdx.x + t * kBlock;
        m.x[t] = w[i < kMlpTotal ? i : kMlpTotal - 1];
    }
}

__device__ __forceinline__ void store_mlp(const MlpTrip &m, float *s) {
    constexpr int B1 = kMlpIn * kMlpH, W2 = B1 + kMlpH, B2 = W2 + kMlpH * kMlpH;
#pragma unroll
    for (int t = 0; t < MlpTrip::per; ++t) {
        const int i = (int)threadIdx.x + t * kBlock;
        const int j = i < B1 ? i + i / kMlpIn
                    : i < W2 ? kMlpAtRest + (i - B1)
                    : i < B2 ? kMlpAt2 + (i - W2) + (i - W2) / kMlpH
                             : kMlpAtRest + kMlpH + (i - B2);
        if (i < kMlpTotal) s[j] = m.x[t];
    }
}

__device__ __forceinline__ void stage_mlp(const float *w, float *s) {
    MlpTrip m;
    load_mlp(w, m);
    store_mlp(m, s);
}

__device__ __forceinline__ float lane_value(float v, int i) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}

// Evaluated by one wave from staged weights: lane o < 32 holds hidden unit o,
// inputs pass between lanes (no arrays, so nothing spills).  Returns, in
// every lane, the argmin of the first `nout` predicted log-times, or -1 when
// one of them is not finite.
__device__ __forceinline__ int mlp_argmin(const float *s, float feat, int nout = kMlpOut) {
    const float *W2 = s + kMlpAt2, *b1 = s + kMlpAtRest, *b2 = b1 + kMlpH, *W3 = b2 + kMlpH,
                *b3 = W3 + kMlpH * kMlpOut, *mean = b3 + kMlpOut, *istd = mean + kMlpIn;
    const uint32_t lane = lane_id();
    const uint32_t li = lane < (uint32_t)kMlpIn ? lane : 0u;
    const float x = (lane < (uint32_t)kMlpIn) ? (feat - mean[li]) * istd[li] : 0.f;
    const uint32_t o = lane & (kMlpH - 1);
    float a = b1[o];
#pragma unroll
    for (int i = 0; i < kMlpIn; ++i) a = fmaf(s[o * kMlpRow1 + i], lane_value(x, i), a);
    const float h1 = a > 0.f ? a : 0.f;
    float c = b2[o];
#pragma unroll
    for (int i = 0; i < kMlpH; ++i) c = fmaf(W2[o * kMlpRow2 + i], lane_value(h1, i), c);
    const float h2 = (c > 0.f ? c : 0.f) * (lane < (uint32_t)kMlpH ? 1.f : 0.f);
    float y[kMlpOut];
#pragma unroll
    for (int u = 0; u < kMlpOut; ++u) y[u] = W3[u * kMlpH + o] * h2;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
        for (int u = 0; u < kMlpOut; ++u) y[u] += __shfl_xor(y[u], d, 64);
    int best = 0;
    float bestv = 0.f;
    bool ok = true;
#pragma unroll
    for (int u = 0; u < kMlpOut; ++u) {
        if (u >= nout) break;
        const float z = y[u] + b3[u];
        if (!(z == z) || z > 1e30f || z < -1e30f) ok = false;
        if (u == 0 || z < bestv) { bestv = z; best = u; }
    }
    return ok ? best : -1;
}

}  // namespace bfsi
