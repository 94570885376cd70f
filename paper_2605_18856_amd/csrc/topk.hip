// Top-k reduction over candidates: the k best (value, index) pairs in the order "greater value
// first, lower index among equal values" -- the order whose first element is the sweep's winner.
//
// That order is the order of 64-bit keys (value as an ordered integer, then the complement of the
// index), all of them different, so selection is by threshold: no tie needs a rule of its own and
// nothing depends on scheduling.  Two launches:
//   * heads: one wavefront per block of TK_BLOCK elements leaves the block's greatest key;
//   * select: one workgroup per set.  A threshold that at least k heads reach bounds the k-th key
//     from below, and every element that reaches it lies in one of the blocks whose head does: those
//     blocks (about k of them) are read again, what reaches the threshold is gathered in LDS and ranked
//     by counting.
// Thresholds come from a histogram of 2048 bins over the range of the keys, narrowed to the bin of
// the k-th key while too many keys reach it; the keys being different, the range runs out first.
// Values in sorted or clustered order only cost further passes.
//
// Bound by latency: the passes over memory are short, and each is followed by a few barriers.  k = 64
// of 2^20 values: heads 4 us, select 13 us; extracting k maxima one after the other in three
// levels of workgroups took 256 us.
#include "bsse_internal.h"
#include "topk_device.h"

namespace bsse {

namespace {

typedef unsigned long long u64;

constexpr int TK_BLOCK = 256;            // elements behind one head

// heads[set][nh] of the sets of `count` values at V + set * count
__global__ void __launch_bounds__(256)
topk_heads_kernel(const float *__restrict__ V, unsigned count, unsigned nh, u64 *__restrict__ heads)
{
    const unsigned lane = threadIdx.x & 63, b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= nh) return;                                 // whole wavefront
    const float *v = V + (size_t)blockIdx.y * count;
    u64 best = 0;
#pragma unroll
    for (unsigned q = 0; q < TK_BLOCK / 64; ++q) {
        const unsigned i = b * TK_BLOCK + q * 64 + lane;
        if (i < count) best = tk_max(best, tk_key(v[i], i));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) best = tk_max(best, __shfl_xor(best, d, 64));
    if (lane == 0) heads[(size_t)blockIdx.y * nh + b] = best;
}

__global__ void __launch_bounds__(TK_T) topk_select_kernel(TopkArgs a)
{
    __shared__ TkShared s;
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned count = a.count, set = blockIdx.x;
    const unsigned k = (unsigned)a.k;                    // <= count
    const unsigned nh = (count + TK_BLOCK - 1) / TK_BLOCK;
    const float *V = a.V + (size_t)set * count;

    // ---- the blocks to look into, and a bound from below
    u64 T = 0;
    unsigned nlist = nh;
    const bool listed = a.heads != nullptr && nh > k;
    if (tid == 0) { s.n = 0; s.nlist = 0; }
    if (listed) {
        const u64 *heads = a.heads + (size_t)set * nh;
        auto each_head = [&](auto f) __attribute__((always_inline)) {
#pragma unroll 4
            for (unsigned i = tid; i < nh; i += TK_T) f(heads[i]);
        };
        u64 lo, hi;
        tk_range(s, each_head, lo, hi);
        T = tk_threshold(s, each_head, k, k + k / 4 + 8, lo, hi);
        for (unsigned i = tid; i < nh; i += TK_T)
            if (heads[i] >= T) s.list[atomicAdd(&s.nlist, 1u)] = i;
        __syncthreads();
        nlist = s.nlist;
    } else {
        __syncthreads();
    }

    // ---- what reaches the bound, into LDS
    auto each_element = [&](auto f) __attribute__((always_inline)) {
        for (unsigned e = wave; e < nlist; e += TK_T / 64) {
            const unsigned first = (listed ? s.list[e] : e) * TK_BLOCK + lane;
            float v[TK_BLOCK / 64];
#pragma unroll
            for (unsigned q = 0; q < TK_BLOCK / 64; ++q) v[q] = V[first + q * 64 < count ? first + q * 64 : count - 1u];
#pragma unroll
            for (unsigned q = 0; q < TK_BLOCK / 64; ++q)
                if (first + q * 64 < count) f(tk_key(v[q], first + q * 64));
        }
    };
    auto gather = [&]() __attribute__((always_inline)) {
        each_element([&](u64 key) {
            if (key < T) return;
            const unsigned at = atomicAdd(&s.n, 1u);
            if (at < TK_CAND) s.cand[at] = key;
        });
    };
    gather();
    __syncthreads();
    unsigned n = s.n;
    if (n > TK_CAND) {                                   // workgroup-uniform, here and below
        u64 lo, hi;
        tk_range(s, each_element, lo, hi);
        T = tk_threshold(s, each_element, k, TK_RANK, tk_max(lo, T), hi);
        if (tid == 0) s.n = 0;
        __syncthreads();
        gather();
        __syncthreads();
        n = s.n;
    } else if (n > TK_RANK) {
        auto each_cand = [&](auto f) __attribute__((always_inline)) {
            for (unsigned i = tid; i < n; i += TK_T) f(s.cand[i]);
        };
        u64 lo, hi;
        tk_range(s, each_cand, lo, hi);
        T = tk_threshold(s, each_cand, k, TK_RANK, lo, hi);
        u64 mine[TK_CAND / TK_T];
#pragma unroll
        for (unsigned q = 0; q < TK_CAND / TK_T; ++q) mine[q] = tid + q * TK_T < n ? s.cand[tid + q * TK_T] : 0ull;
        __syncthreads();
        if (tid == 0) s.n = 0;
        __syncthreads();
#pragma unroll
        for (unsigned q = 0; q < TK_CAND / TK_T; ++q)
            if (tid + q * TK_T < n && mine[q] >= T) s.cand[atomicAdd(&s.n, 1u)] = mine[q];
        __syncthreads();
        n = s.n;
    }

    // ---- in order: n <= TK_RANK keys, ranked by how many are greater
    u64 my = 0;
    unsigned r = 0;
    if (tid < n) {
        my = s.cand[tid];
        for (unsigned i = 0; i < n; ++i) r += s.cand[i] > my ? 1u : 0u;
    }
    __syncthreads();
    if (tid < n && r < k) {
        s.list[r] = tk_index(my);
        a.val[(size_t)set * k + r] = tk_value(my);
        a.idx[(size_t)set * k + r] = a.index_base + (long long)tk_index(my);
    }
    __syncthreads();
    const unsigned m = (unsigned)a.m;
    const float *X = a.X + (size_t)set * count * m;
    for (unsigned e = tid; e < k * m; e += TK_T) {
        const unsigned row = e / m;
        const float x = X[(size_t)s.list[row] * m + (e - row * m)];
        a.rows[(size_t)set * k * m + e] = x;
        if (a.rows_host) a.rows_host[(size_t)set * k * m + e] = x;
    }
}

}  // namespace

// Up to here one workgroup reads all values itself sooner than a launch over the blocks ends.
constexpr long long TK_DIRECT = 16384;

size_t topk_heads_bytes(long long count, int sets)
{
    return count <= TK_DIRECT ? 0 : (size_t)((count + TK_BLOCK - 1) / TK_BLOCK) * sets * sizeof(u64);
}

hipError_t launch_topk(const TopkArgs &args, int sets, hipStream_t s)
{
    if (args.count == 0 || args.k <= 0 || sets <= 0) return hipSuccess;
    if (args.k > 256 || (unsigned)args.k > args.count) return hipErrorInvalidValue;
    TopkArgs a = args;
    if ((long long)a.count > TK_DIRECT) {
        if (!a.heads) return hipErrorInvalidValue;
        const unsigned nh = (a.count + TK_BLOCK - 1) / TK_BLOCK;
        hipLaunchKernelGGL(topk_heads_kernel, dim3((nh + 3) / 4, (unsigned)sets), dim3(256), 0, s, a.V, a.count, nh, a.heads);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else {
        a.heads = nullptr;
    }
    hipLaunchKernelGGL(topk_select_kernel, dim3((unsigned)sets), dim3(TK_T), 0, s, a);
    return hipGetLastError();
}

}  // namespace bsse
