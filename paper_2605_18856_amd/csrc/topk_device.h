// Selection by threshold, device side (not installed): 64-bit keys in the order "greater value first,
// lower index among equal values", all of them different, and the threshold that a given number of them
// reach.  Shared by the top-k reduction and the selection of follower profiles.
#pragma once
#include <hip/hip_runtime.h>

namespace bsse {

constexpr int TK_T = 1024;               // threads of a select workgroup
constexpr int TK_BINS = 2 * TK_T;
constexpr int TK_LIST = 512;             // blocks that can be listed (>= 256, the greatest k, and some)
constexpr int TK_CAND = 4096;            // keys LDS holds
constexpr int TK_RANK = 512;             // keys that are ranked by counting (>= 256)

// index: below 2^32.  A value that is not a number counts as minus infinity, and -0 as 0.
__device__ __forceinline__ unsigned long long tk_key(float v, unsigned index)
{
    if (!(v == v)) v = -INFINITY;
    if (v == 0.0f) v = 0.0f;
    const unsigned b = __float_as_uint(v);
    const unsigned o = (b & 0x80000000u) ? ~b : b | 0x80000000u;
    return ((unsigned long long)o << 32) | (0xFFFFFFFFu - index);
}
__device__ __forceinline__ float tk_value(unsigned long long key)
{
    const unsigned o = (unsigned)(key >> 32);
    return __uint_as_float((o & 0x80000000u) ? o & 0x7FFFFFFFu : ~o);
}
__device__ __forceinline__ unsigned tk_index(unsigned long long key) { return 0xFFFFFFFFu - (unsigned)key; }

__device__ __forceinline__ unsigned long long tk_max(unsigned long long a, unsigned long long b) { return a > b ? a : b; }
__device__ __forceinline__ unsigned long long tk_min(unsigned long long a, unsigned long long b) { return a < b ? a : b; }

struct TkShared {
    unsigned hist[TK_BINS];
    unsigned long long cand[TK_CAND];
    unsigned list[TK_LIST];
    unsigned wsum[TK_T / 64];
    unsigned long long wmin[TK_T / 64], wmax[TK_T / 64];
    unsigned long long lo;
    unsigned total, above, n, nlist;
};

// Range of the keys that for_each(f) hands to f, over all threads (at least one key).
template <typename E> __device__ __forceinline__ void tk_range(TkShared &s, E for_each, unsigned long long &lo, unsigned long long &hi)
{
    unsigned long long mn = ~0ull, mx = 0;
    for_each([&](unsigned long long key) { mn = tk_min(mn, key); mx = tk_max(mx, key); });
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        mn = tk_min(mn, __shfl_xor(mn, d, 64));
        mx = tk_max(mx, __shfl_xor(mx, d, 64));
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { s.wmin[threadIdx.x >> 6] = mn; s.wmax[threadIdx.x >> 6] = mx; }
    __syncthreads();
    lo = s.wmin[0]; hi = s.wmax[0];
    for (int w = 1; w < TK_T / 64; ++w) { lo = tk_min(lo, s.wmin[w]); hi = tk_max(hi, s.wmax[w]); }
}

// A threshold that at least k and at most cap (>= k) of the keys in lo..hi reach.  Every key for_each
// hands over is at most hi, and at least k are in the range.
template <typename E>
__device__ __forceinline__ unsigned long long tk_threshold(TkShared &s, E for_each, unsigned k, unsigned cap, unsigned long long lo, unsigned long long hi)
{
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned above = 0;                                  // keys above hi
    for (;;) {
        const int bits = 64 - __clzll((long long)(hi - lo)), shift = bits > 11 ? bits - 11 : 0;
        s.hist[tid] = 0; s.hist[tid + TK_T] = 0;
        __syncthreads();
        for_each([&](unsigned long long key) { if (key >= lo && key <= hi) atomicAdd(&s.hist[(key - lo) >> shift], 1u); });
        __syncthreads();
        // from the top: thread t sums bins TK_BINS - 1 - 2t and the one below
        const unsigned b = TK_BINS - 1 - 2 * tid, c1 = s.hist[b], c0 = s.hist[b - 1];
        unsigned incl = c1 + c0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned o = __shfl_up(incl, d, 64);
            if (lane >= (unsigned)d) incl += o;
        }
        if (lane == 63) s.wsum[wave] = incl;
        __syncthreads();
        for (unsigned w = 0; w < wave; ++w) incl += s.wsum[w];
        const unsigned need = k - above, excl = incl - c1 - c0;
        if (excl < need && need <= incl) {               // one thread
            const bool first = excl + c1 >= need;
            s.lo = lo + ((unsigned long long)(first ? b : b - 1) << shift);
            s.above = above + excl + (first ? 0u : c1);
            s.total = above + excl + c1 + (first ? 0u : c0);
        }
        __syncthreads();
        lo = s.lo;
        if (s.total <= cap || shift == 0) return lo;
        above = s.above;
        hi = tk_min(hi, lo + (1ull << shift) - 1ull);
    }
}

}  // namespace bsse
