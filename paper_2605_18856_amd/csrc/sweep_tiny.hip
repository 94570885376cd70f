// Fused sweep for short rows on the vector unit (steps 2-5, m <= 24, any n and K): one lane per
// candidate, the row in registers (M = m, padded with zeros beyond eight), payoffs [K][n][M] so that
// an action is M consecutive numbers.  Follower payoffs have the same address in every lane: they come
// through scalar loads, and a multiply-add takes one of them as its scalar operand.  An action costs M
// multiply-adds and four instructions of bookkeeping; the leader column at the best response is a gather.
//
// Few rows are cut over the types (blockIdx.y) like the matrix-core launches; a sweep whose types need no
// cutting is ONE launch: every workgroup leaves its best candidate with row, best responses and tie
// count in pinned memory and the host folds.  The best responses are found by evaluating that row
// again, one type per thread (same operations in the same order, hence the same decisions).
//
// Small calls are bound by latency, large ones by the vector unit: 5151 points of m = n = 3, K = 2: 6 us
// (sweep, fold and evaluation as three launches with the payoffs one scalar at a time: 20); 2^20 rows of
// m = 5, n = 7, K = 16: 96 us a call, 302 before.
#include "bsse_internal.h"
#include "done_device.h"
#include <limits.h>

namespace bsse {

namespace {

constexpr int TN_T = 256;
typedef const float __attribute__((address_space(4))) *scalar_ptr;      // loads through it are scalar

__device__ __forceinline__ float tn_round_bf16(float v)
{
    unsigned b = __float_as_uint(v);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return __uint_as_float(b & 0xFFFF0000u);
}

template <int M> __device__ __forceinline__ void tn_load_row(const float *row, int m, int x_bf16, float (&x)[M])
{
#pragma unroll
    for (int i = 0; i < M; ++i) {
        float v = M <= 8 || i < m ? row[i] : 0.0f;
        x[i] = x_bf16 ? tn_round_bf16(v) : v;
    }
}

// sum_i x[i] * p[i], i ascending
template <int M, typename P> __device__ __forceinline__ float tn_dot(const float (&x)[M], P p)
{
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < M; ++i) s = fmaf(x[i], p[i], s);
    return s;
}

// Exact tie-break of one type: of the actions whose follower payoff is `best`, the one with the greatest
// leader payoff, the lowest among those.  Returns how many there are.
template <int M, typename P>
__device__ __forceinline__ int tn_exact(const float (&x)[M], P Bt, const float *At, int n, float best, float &l, int &js)
{
    int hits = 0;
    for (int j = 0; j < n; ++j)
        if (tn_dot<M>(x, Bt + (size_t)j * M) == best) {
            const float lj = tn_dot<M>(x, At + (size_t)j * M);
            if (hits == 0 || lj > l) { l = lj; js = j; }
            ++hits;
        }
    return hits;
}

struct TnBest { float u; int j; bool tied; };
__device__ __forceinline__ void tn_take(TnBest &b, float u, int j)
{
    const bool gt = u > b.u, eq = u == b.u;
    b.u = gt ? u : b.u;
    b.j = gt ? j : b.j;
    b.tied = !gt && (b.tied || eq);
}

template <int M, bool EVAL>
__global__ void __launch_bounds__(TN_T) sweep_tiny_kernel(GameView g, SweepArgs a, TinyRecs r)
{
    __shared__ float sv[TN_T / 64];
    __shared__ unsigned sc[TN_T / 64], st[TN_T / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = g.m, n = g.n, K = g.K;
    const unsigned count = (unsigned)a.count;
    const int t0 = (int)blockIdx.y * a.slice_stages, t1 = t0 + a.slice_stages < K ? t0 + a.slice_stages : K;
    const scalar_ptr prior = (scalar_ptr)g.prior;
    float best_v = -INFINITY;
    unsigned best_c = 0xFFFFFFFFu, ties = 0;
    for (unsigned c0 = blockIdx.x * TN_T; c0 < count; c0 += gridDim.x * TN_T) {
        const unsigned c = c0 + tid;
        const bool valid = c < count;
        float x[M];
        tn_load_row<M>(a.X + (size_t)(valid ? c : count - 1u) * m, m, g.x_bf16, x);
        float V = 0.0f;
        for (int t = t0; t < t1; ++t) {
            const scalar_ptr Bt = (scalar_ptr)g.B + (size_t)t * n * M;
            const float *At = g.AT + (size_t)t * n * M;
            TnBest b = { -INFINITY, 0, false };
            int j = 0;
            for (; j + 4 <= n; j += 4) {
                float u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) u[q] = tn_dot<M>(x, Bt + (size_t)(j + q) * M);
#pragma unroll
                for (int q = 0; q < 4; ++q) tn_take(b, u[q], j + q);
            }
            for (; j < n; ++j) tn_take(b, tn_dot<M>(x, Bt + (size_t)j * M), j);
            int js = b.j;
            float l = tn_dot<M>(x, At + (size_t)js * M);
            if (__ballot(b.tied) != 0ull) {              // wavefront-uniform
                const bool real = b.u != -INFINITY;      // (an input that is not finite: unspecified, not counted)
                const int hits = tn_exact<M>(x, Bt, At, n, b.u, l, js);
                ties += valid && b.tied && real && hits >= 2 ? 1u : 0u;
            }
            V = fmaf(prior[t], l, V);
            if (EVAL && valid) {
                if (a.br_out) a.br_out[c * a.br_sc + t * a.br_st] = js;
                if (a.l_out) a.l_out[c * a.l_sc + t * a.l_st] = l;
            }
        }
        if (!(V == V)) V = -INFINITY;                    // not a number never wins
        if (EVAL) {
            if (valid && a.V_out) a.V_out[c] = V;
        } else if (valid && (V > best_v || best_c == 0xFFFFFFFFu)) {     // a lane's candidates ascend
            best_v = V; best_c = c;
        }
    }
    if (!EVAL) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const float ov = __shfl_xor(best_v, d, 64);
            const unsigned oc = __shfl_xor(best_c, d, 64);
            if (ov > best_v || (ov == best_v && oc < best_c)) { best_v = ov; best_c = oc; }
        }
    }
    if (a.tie_counter || r.rec) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) ties += __shfl_xor(ties, d, 64);
    }
    if (a.tie_counter && lane == 0 && ties) atomicAdd(a.tie_counter, (unsigned long long)ties);
    if (EVAL) {
        if (a.done.flag) signal_done(a.done, blockIdx.y * gridDim.x + blockIdx.x);
        return;
    }
    if (lane == 0) { sv[wave] = best_v; sc[wave] = best_c; st[wave] = ties; }
    __syncthreads();
    best_v = sv[0]; best_c = sc[0]; ties = st[0];
#pragma unroll
    for (int w = 1; w < TN_T / 64; ++w) {
        if (sv[w] > best_v || (sv[w] == best_v && sc[w] < best_c)) { best_v = sv[w]; best_c = sc[w]; }
        ties += st[w];
    }
    if (a.blk_v) {
        if (tid == 0) { a.blk_v[blockIdx.x] = best_v; a.blk_i[blockIdx.x] = a.index_base + (long long)best_c; }
        return;
    }
    // the record, in pinned memory: the workgroup's winner once more, a type per thread
    const float *row = a.X + (size_t)best_c * m;
    float x[M];
    tn_load_row<M>(row, m, g.x_bf16, x);
    for (int t = tid; t < K; t += TN_T) {
        const float *Bt = g.B + (size_t)t * n * M, *At = g.AT + (size_t)t * n * M;
        TnBest b = { -INFINITY, 0, false };
#pragma unroll 4
        for (int j = 0; j < n; ++j) tn_take(b, tn_dot<M>(x, Bt + (size_t)j * M), j);
        int js = b.j;
        if (b.tied) {
            float l = 0.0f;
            tn_exact<M>(x, Bt, At, n, b.u, l, js);
        }
        r.rec_br[(size_t)blockIdx.x * K + t] = js;
    }
    for (int i = tid; i < m; i += TN_T) r.rec_x[(size_t)blockIdx.x * m + i] = row[i];
    FinishRec &rec = r.rec[blockIdx.x];
    if (tid == 0) { rec.value = best_v; rec.index = a.index_base + (long long)best_c; rec.ties = ties; }
    const Done d = { &rec.seq, r.seq };
    signal_done(d, 0);
}

typedef void (*tiny_kernel_t)(GameView, SweepArgs, TinyRecs);
template <bool EVAL> tiny_kernel_t tiny_kernel_for(int mp)
{
    switch (mp) {
    case 1: return sweep_tiny_kernel<1, EVAL>;
    case 2: return sweep_tiny_kernel<2, EVAL>;
    case 3: return sweep_tiny_kernel<3, EVAL>;
    case 4: return sweep_tiny_kernel<4, EVAL>;
    case 5: return sweep_tiny_kernel<5, EVAL>;
    case 6: return sweep_tiny_kernel<6, EVAL>;
    case 7: return sweep_tiny_kernel<7, EVAL>;
    case 8: return sweep_tiny_kernel<8, EVAL>;
    case 10: return sweep_tiny_kernel<10, EVAL>;
    case 12: return sweep_tiny_kernel<12, EVAL>;
    case 16: return sweep_tiny_kernel<16, EVAL>;
    case 20: return sweep_tiny_kernel<20, EVAL>;
    case 24: return sweep_tiny_kernel<24, EVAL>;
    }
    return nullptr;
}

long long tiny_blocks(long long count) { return (count + TN_T - 1) / TN_T; }

}  // namespace

int tiny_pad(int m)
{
    static const int pads[] = { 1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 20, 24 };
    for (int p : pads)
        if (p >= m) return p;
    return 0;
}

// Unsliced: at most one resident set (eight wavefronts per SIMD), every workgroup then walking the same
// number of blocks up to one.
long long tiny_num_blocks(long long count)
{
    const long long blocks = tiny_blocks(count), cap = 2048, rounds = (blocks + cap - 1) / cap;
    return rounds > 0 ? (blocks + rounds - 1) / rounds : 1;
}

int tiny_slices(const GameView &g, long long count)
{
    // Fewer workgroups than compute units leave the types of a row one behind the other: cut them, but
    // not below 64 multiply-adds' worth of actions per slice (the second launch costs more than that
    // saves), until the grid is about twice the compute units.
    const long long blocks = tiny_blocks(count);
    const long long least = (64 * 16 + (long long)g.m * g.n - 1) / ((long long)g.m * g.n);      // types per slice
    if (blocks >= 256 || g.K < 2 * least) return 1;
    long long want = 512 / blocks;
    if (want > g.K / least) want = g.K / least;
    if (want < 2) return 1;
    const int per = (int)((g.K + want - 1) / want);
    return (g.K + per - 1) / per;
}
long long tiny_row_blocks(const GameView &g, long long count)
{
    const int slices = tiny_slices(g, count);
    return slices > 1 ? tiny_blocks(count) * slices : tiny_num_blocks(count);
}

hipError_t launch_sweep_tiny(const GameView &g, const SweepArgs &a, bool eval, int slices, const TinyRecs &r, hipStream_t s)
{
    if (a.count <= 0) return hipSuccess;
    const tiny_kernel_t k = eval ? tiny_kernel_for<true>(g.m_pad) : tiny_kernel_for<false>(g.m_pad);
    if (!k) return hipErrorNotSupported;
    SweepArgs b = a;
    b.slice_stages = (g.K + slices - 1) / slices;
    const int ny = (g.K + b.slice_stages - 1) / b.slice_stages;
    if (ny > 1 && (!eval || a.V_out)) return hipErrorInvalidValue;
    if (!eval && !a.blk_v && !r.rec) return hipErrorInvalidValue;
    const long long nx = ny > 1 ? tiny_blocks(a.count) : tiny_num_blocks(a.count);
    hipLaunchKernelGGL(k, dim3((unsigned)nx, (unsigned)ny), dim3(TN_T), 0, s, g, b, r);
    return hipGetLastError();
}

}  // namespace bsse
