// Follower profiles that a set of candidates realises, and the linear program of each on the device
// (see profile_lp.hip for the program, the simplex method on its dual and the starting basis).
//
// Profiles: an open-addressing table in device memory.  A slot names one candidate of its profile (rows
// of best responses are compared, so that no two profiles can be mistaken for one another) and collects
// the key -- value, then lowest index -- of the profile's best candidate.  A thread that finds its key
// beaten already leaves without an atomic: popular profiles would otherwise queue at one address.
//
// Programs: one workgroup each, the tableau in LDS; a thread owns columns, so that the update of a pivot
// needs no exchange.  The arithmetic, operation by operation (no contraction), and the choice of every
// pivot are those of solve_profile_lp: same vertex, same bits.  Bound by the chain entering column ->
// ratio test -> pivot row -> update, about a microsecond a pivot; 200 programs of 16 x 78 cells run at
// once in the time of the longest instead of one after the other on the host.
#include "bsse_internal.h"
#include "done_device.h"
#include "topk_device.h"

namespace bsse {

namespace {

typedef unsigned long long u64;

// A workgroup first brings its own candidates together by profile in a table in LDS, so that only one of
// them per profile goes to the table in memory: a popular profile's slot is otherwise an address that
// thousands of threads queue at (65536 candidates: 37 us, and 17 with the step in LDS).
constexpr int PI_T = 1024, PI_SLOTS = 2 * PI_T;
__global__ void __launch_bounds__(PI_T)
profile_insert_kernel(const float *__restrict__ V, const int32_t *__restrict__ br, unsigned count, int K,
                      unsigned *slots, u64 *best, unsigned mask)
{
    __shared__ unsigned own[PI_SLOTS];                   // candidate + 1
    __shared__ u64 own_best[PI_SLOTS];
    const unsigned tid = threadIdx.x, c = blockIdx.x * PI_T + tid;
#pragma unroll
    for (unsigned i = 0; i < PI_SLOTS / PI_T; ++i) { own[tid + i * PI_T] = 0u; own_best[tid + i * PI_T] = 0ull; }
    __syncthreads();
    // (both searches end: each table has twice as many slots as candidates)
    auto find = [&](unsigned cand, unsigned h, unsigned m, auto load, auto swap) {
        const int32_t *row = br + (size_t)cand * K;
        for (;; h = (h + 1u) & m) {
            unsigned o = load(h);
            if (o == 0u) o = swap(h);
            if (o == 0u) return h;
            const int32_t *other = br + (size_t)(o - 1u) * K;
            int t = 0;
            while (t < K && other[t] == row[t]) ++t;
            if (t == K) return h;
        }
    };
    auto hash = [&](unsigned cand) {
        const int32_t *row = br + (size_t)cand * K;
        unsigned h = 0x811C9DC5u;
        for (int t = 0; t < K; ++t) { h ^= (unsigned)row[t]; h *= 0x9E3779B1u; h ^= h >> 15; }
        return h;
    };
    if (c < count) {
        const unsigned h = find(c, hash(c) & (PI_SLOTS - 1u), PI_SLOTS - 1u, [&](unsigned i) { return __hip_atomic_load(&own[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); },
                                [&](unsigned i) { return atomicCAS(&own[i], 0u, c + 1u); });
        atomicMax(&own_best[h], tk_key(V[c], c));
    }
    __syncthreads();
#pragma unroll 1
    for (unsigned i = 0; i < PI_SLOTS / PI_T; ++i) {
        const u64 key = own_best[tid + i * PI_T];
        if (key == 0ull) continue;
        const unsigned cand = tk_index(key);
        const unsigned h = find(cand, hash(cand) & mask, mask, [&](unsigned q) { return __hip_atomic_load(&slots[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                                [&](unsigned q) { return atomicCAS(&slots[q], 0u, cand + 1u); });
        if (__hip_atomic_load(&best[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < key) atomicMax(&best[h], key);
    }
}

// The keys of the table's occupied slots, in any order: PL_PER slots a thread, one addition to the
// counter per workgroup.
constexpr unsigned PL_PER = 8;
__global__ void __launch_bounds__(1024)
profile_list_kernel(const u64 *__restrict__ best, unsigned nslots, u64 *__restrict__ list, unsigned *n)
{
    __shared__ unsigned wave_n[16], at;
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    u64 key[PL_PER];
    unsigned mine = 0;
#pragma unroll
    for (unsigned q = 0; q < PL_PER; ++q) {
        const unsigned i = (blockIdx.x * PL_PER + q) * 1024u + tid;
        key[q] = i < nslots ? best[i] : 0ull;
        mine += key[q] != 0ull;
    }
    unsigned upto = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned o = __shfl_up(upto, d, 64);
        if (lane >= (unsigned)d) upto += o;
    }
    if (lane == 63) wave_n[wave] = upto;
    __syncthreads();
    if (tid == 0) {
        unsigned total = 0;
        for (unsigned w = 0; w < 16; ++w) { const unsigned k = wave_n[w]; wave_n[w] = total; total += k; }
        at = total ? atomicAdd(n, total) : 0u;
    }
    __syncthreads();
    unsigned pos = at + wave_n[wave] + upto - mine;
#pragma unroll
    for (unsigned q = 0; q < PL_PER; ++q)
        if (key[q]) list[pos++] = key[q];
}

// The `most` best of the n profiles (all of them if there are no more), in any order.
__global__ void __launch_bounds__(TK_T)
profile_select_kernel(const u64 *__restrict__ list, const unsigned *__restrict__ n_ptr, unsigned most, u64 *__restrict__ sel)
{
    __shared__ TkShared s;
    const unsigned n = *n_ptr;
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll 4
        for (unsigned i = threadIdx.x; i < n; i += TK_T) f(list[i]);
    };
    u64 T = 0;
    if (threadIdx.x == 0) s.n = 0;
    if (n > most) {
        u64 lo, hi;
        tk_range(s, each, lo, hi);
        T = tk_threshold(s, each, most, most, lo, hi);
    }
    __syncthreads();
    each([&](u64 key) { if (key >= T) sel[atomicAdd(&s.n, 1u)] = key; });
}

// ------------------------------------------------------------------------------- programs
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    const u64 b = (u64)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((u64)(unsigned)hi << 32) | (unsigned)lo));
}
// Minimum over the wavefront, in every lane (a value that is not a number never is).
__device__ __forceinline__ double wave_min(double v)
{
    v = fmin(v, dpp_f64<0xB1>(v));       // lanes 1 apart, 2 apart, half row, row, 16 lanes, 32 lanes
    v = fmin(v, dpp_f64<0x4E>(v));
    v = fmin(v, dpp_f64<0x141>(v));
    v = fmin(v, dpp_f64<0x140>(v));
    v = fmin(v, dpp_f64<0x142>(v));
    v = fmin(v, dpp_f64<0x143>(v));
    const u64 b = (u64)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, 63), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double((long long)(((u64)hi << 32) | lo));
}
template <int T> __device__ __forceinline__ double block_min(double v, double *red)
{
    v = wave_min(v);
    if constexpr (T > 64) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        v = red[0];
        for (int w = 1; w < T / 64; ++w) v = fmin(v, red[w]);
    }
    return v;
}

// The tableau in registers: one wavefront, column c * 64 + lane in lane `lane`, rows 0..M-1 of it (zero
// from m on); right-hand side and basic variable of row i in lane i.  Per pivot the entering column goes
// to every lane through LDS and nothing else is exchanged but two minima.
// See solve_profile_lp for what every step is.
template <int M, int C>
__global__ void __launch_bounds__(64) profile_lp_small_kernel(LpArgs a)
{
#pragma clang fp contract(off)
    __shared__ __attribute__((aligned(16))) double fcol[M];
    __shared__ double near_ratio[M];
    __shared__ int near_basic[M];
    const int lane = threadIdx.x;
    const unsigned p = blockIdx.x;
    const unsigned n_sel = *a.n < a.most ? *a.n : a.most;
    if (p >= n_sel) return;
    const int m = a.m, n = a.n_act, K = a.K, R = K * (n - 1), ncol = 2 + R + m, col_s = 2 + R;
    const int32_t *profile = a.br + (size_t)tk_index(a.sel[p]) * K;

    double tab[C][M], d[C];
    double ci = 0.0;                                     // objective of row `lane`
    if (lane < m)
        for (int t = 0; t < K; ++t) ci += (double)a.prior[t] * (double)a.A[((size_t)t * m + lane) * n + profile[t]];
    double big = 0.0;                                    // minus the greatest difference
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = c * 64 + lane;
        const bool diff = j >= 2 && j < col_s;
        const int t = diff ? (j - 2) / (n - 1) : 0, r = diff ? (j - 2) % (n - 1) : 0, pt = profile[t], act = r < pt ? r : r + 1;
        const float *Bt = a.B + (size_t)t * m * n;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            double v = 0.0;
            if (i < m) {
                if (diff) {
                    const double g = (double)Bt[(size_t)i * n + pt] - (double)Bt[(size_t)i * n + act];
                    v = -g;
                    big = fmin(big, -fabs(g));
                } else {
                    v = j == 0 ? 1.0 : j == 1 ? -1.0 : j == col_s + i ? -1.0 : 0.0;
                }
            }
            tab[c][i] = v;
        }
    }
    const double scale = fmax(1.0, -wave_min(big));
    if (lane < M) fcol[lane] = ci;
    __syncthreads();
    double cmin = fcol[0], ck = fcol[0];
    int k = 0;
#pragma unroll
    for (int i = 1; i < M; ++i) {
        const double v = fcol[i];
        if (i < m && v < cmin) cmin = v;
        if (i < m && v > ck) { ck = v; k = i; }
    }
    __syncthreads();
    const double shift = 1.0 - cmin, rk = ck + shift;
    double rhs = lane == k ? rk : rk - (ci + shift);
    int basic = lane == k ? 0 : col_s + lane;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = c * 64 + lane;
        double pk = 0.0;
#pragma unroll
        for (int i = 0; i < M; ++i) pk = i == k ? tab[c][i] : pk;
#pragma unroll
        for (int i = 0; i < M; ++i) tab[c][i] = i == k || i >= m ? tab[c][i] : pk - tab[c][i];
        d[c] = j < ncol ? (j == 0 ? 1.0 : j == 1 ? -1.0 : 0.0) - pk : 0.0;
    }
    double z = rk;

    const double tol = 1e-11 * scale;
    const int max_iter = 200 * (m + R) + 1000;
    int stall = 0, rc = 2;
    for (int it = 0; it < max_iter; ++it) {
        // entering column
        double mn = d[0];
#pragma unroll
        for (int c = 1; c < C; ++c) mn = fmin(mn, d[c]);
        mn = wave_min(mn);
        if (!(mn < -tol)) {                              // optimal
            double x = 0.0, s = 0.0;
#pragma unroll 1
            for (int i = 0; i < m; ++i) {
                const int j = col_s + i;
                double v = d[0];
#pragma unroll
                for (int c = 1; c < C; ++c) v = j / 64 == c ? d[c] : v;
                v = __shfl(v, j & 63, 64);
                v = v > 0.0 ? v : 0.0;
                s += v;
                x = lane == i ? v : x;
            }
            if (s > 0.0) {
                if (lane < m) a.x[(size_t)p * m + lane] = x / s;
                rc = 0;
            }
            break;
        }
        int e = -1;
#pragma unroll
        for (int c = C - 1; c >= 0; --c) {
            const u64 hit = __ballot(stall < 40 ? d[c] == mn : d[c] < -tol);
            if (hit) e = c * 64 + __builtin_ctzll(hit);
        }
        e = __builtin_amdgcn_readfirstlane(e);
        const int ec = e >> 6, el = e & 63;
        if (lane == el) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (c == ec)
#pragma unroll
                    for (int i = 0; i < M; ++i) fcol[i] = tab[c][i];
        }
        __syncthreads();
        // leaving row: least ratio, lowest basic variable among near-equal ones
        const double fi = lane < m ? fcol[lane & (M - 1)] : 0.0;
        const double q = fi > tol ? rhs / fi : INFINITY;
        const double least = wave_min(q);
        if (least == INFINITY) { rc = 1; break; }        // dual unbounded
        // (a row apart from every other by ten times the tolerance below wins whatever the order)
        const u64 close = __ballot(q <= least + 1e-12 * (1.0 + fabs(least)));
        int l = __builtin_ctzll(close);
        double rl = least;
        if (close & (close - 1ull)) {
            if (lane < M) { near_ratio[lane] = q; near_basic[lane] = basic; }
            __syncthreads();
            l = -1;
            for (int i = 0; i < m; ++i) {
                if (!(fcol[i] > tol)) continue;
                const double r = near_ratio[i];
                if (l < 0 || r < rl - 1e-13 * (1.0 + fabs(rl)) ||
                    (r <= rl + 1e-13 * (1.0 + fabs(rl)) && near_basic[i] < near_basic[l])) {
                    l = i; rl = r;
                }
            }
            __syncthreads();
        }
        l = __builtin_amdgcn_readfirstlane(l);
        // pivot on (l, e)
        const double piv = fcol[l];
        double f[M];
#pragma unroll
        for (int i = 0; i < M; ++i) f[i] = fcol[i];
        double fd = d[0];
#pragma unroll
        for (int c = 1; c < C; ++c) fd = ec == c ? d[c] : fd;
        {
            const u64 b = (u64)__double_as_longlong(fd);
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, el), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), el);
            fd = __longlong_as_double((long long)(((u64)hi << 32) | lo));
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            double old = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) old = i == l ? tab[c][i] : old;
            const bool is_e = lane == el && c == ec;
            const double r = is_e ? 1.0 : old / piv;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const double v = f[i] * r, w = tab[c][i] - v;
                tab[c][i] = i == l ? r : is_e ? 0.0 : w;
            }
            const double v = fd * r;
            d[c] = is_e ? 0.0 : d[c] - v;
        }
        if (lane == l) {
            rhs = rl; basic = e;
        } else if (fi != 0.0) {
            const double v = fi * rl;
            double r = rhs - v;
            if (r < 0.0 && r > -1e-9 * (1.0 + fabs(rl))) r = 0.0;
            rhs = r;
        }
        const double zv = fd * rl, z_new = z + zv;
        stall = (z - z_new > 1e-14 * (1.0 + fabs(z))) ? 0 : stall + 1;
        z = z_new;
        __syncthreads();                                 // fcol is free
    }
    if (lane == 0) { a.v[p] = z - shift; a.rc[p] = rc; }
}

// Any tableau that LDS holds: T threads, each owning columns.
template <int T>
__global__ void __launch_bounds__(T) profile_lp_kernel(LpArgs a)
{
#pragma clang fp contract(off)
    extern __shared__ __attribute__((aligned(16))) double lp[];
    __shared__ double red[T / 64];
    const int tid = threadIdx.x;
    const unsigned p = blockIdx.x;
    const unsigned n_sel = *a.n < a.most ? *a.n : a.most;
    if (p >= n_sel) return;
    const int m = a.m, n = a.n_act, K = a.K, R = K * (n - 1), ncol = 2 + R + m, col_s = 2 + R;
    double *tab = lp, *d = tab + (size_t)m * ncol, *rhs = d + ncol, *c = rhs + m, *fcol = c + m, *ratio = fcol + m;
    int *basic = reinterpret_cast<int *>(ratio + m);
    const int32_t *profile = a.br + (size_t)tk_index(a.sel[p]) * K;

    // ---- objective and payoff differences
    for (int i = tid; i < m; i += T) {
        double v = 0.0;
        for (int t = 0; t < K; ++t) v += (double)a.prior[t] * (double)a.A[((size_t)t * m + i) * n + profile[t]];
        c[i] = v;
    }
    double big = 0.0;                                    // minus the greatest difference
    for (int j = tid; j < ncol; j += T) {
        if (j < 2 || j >= col_s) {
            for (int i = 0; i < m; ++i) tab[(size_t)i * ncol + j] = j == 0 ? 1.0 : j == 1 ? -1.0 : j == col_s + i ? -1.0 : 0.0;
            continue;
        }
        const int t = (j - 2) / (n - 1), r = (j - 2) % (n - 1), pt = profile[t], act = r < pt ? r : r + 1;
        const float *Bt = a.B + (size_t)t * m * n;
        for (int i = 0; i < m; ++i) {
            const double g = (double)Bt[(size_t)i * n + pt] - (double)Bt[(size_t)i * n + act];
            tab[(size_t)i * ncol + j] = -g;
            big = fmin(big, -fabs(g));
        }
    }
    const double scale = fmax(1.0, -block_min<T>(big, red));
    __syncthreads();
    double cmin = c[0];
    int k = 0;
    for (int i = 1; i < m; ++i) {
        cmin = c[i] < cmin ? c[i] : cmin;
        if (c[i] > c[k]) k = i;
    }
    const double shift = 1.0 - cmin;
    const double rk = c[k] + shift;
    for (int i = tid; i < m; i += T) {
        rhs[i] = i == k ? rk : rk - (c[i] + shift);
        basic[i] = i == k ? 0 : col_s + i;
    }
    for (int j = tid; j < ncol; j += T) {
        const double pk = tab[(size_t)k * ncol + j];
        for (int i = 0; i < m; ++i)
            if (i != k) tab[(size_t)i * ncol + j] = pk - tab[(size_t)i * ncol + j];
        d[j] = (j == 0 ? 1.0 : j == 1 ? -1.0 : 0.0) - pk;
    }
    double z = rk;

    const double tol = 1e-11 * scale;
    const int max_iter = 200 * (m + R) + 1000;
    int stall = 0, rc = 2;
    for (int it = 0; it < max_iter; ++it) {
        __syncthreads();                                 // the update of the pivot before
        // entering column
        double mn = INFINITY;
        for (int j = tid; j < ncol; j += T) mn = fmin(mn, d[j]);
        mn = block_min<T>(mn, red);
        if (!(mn < -tol)) {                              // optimal
            double s = 0.0;
            for (int i = 0; i < m; ++i) { const double v = d[col_s + i]; s += v > 0.0 ? v : 0.0; }
            if (s > 0.0) {
                for (int i = tid; i < m; i += T) {
                    const double v = d[col_s + i];
                    a.x[(size_t)p * m + i] = (v > 0.0 ? v : 0.0) / s;
                }
                rc = 0;
            }
            break;
        }
        double first = INFINITY;                         // lowest column that qualifies
        for (int j = tid; j < ncol; j += T)
            if (stall < 40 ? d[j] == mn : d[j] < -tol) { first = (double)j; break; }
        const int e = (int)block_min<T>(first, red);
        // leaving row: least ratio, lowest basic variable among near-equal ones
        double least = INFINITY;
        for (int i = tid; i < m; i += T) {
            const double v = tab[(size_t)i * ncol + e];
            fcol[i] = v;
            const double q = v > tol ? rhs[i] / v : INFINITY;
            ratio[i] = q;
            least = fmin(least, q);
        }
        least = block_min<T>(least, red);
        __syncthreads();
        if (least == INFINITY) { rc = 1; break; }        // dual unbounded
        int l = -1;
        {
            // (a row apart from every other by ten times the tolerance below wins whatever the order)
            const double near = least + 1e-12 * (1.0 + fabs(least));
            int hits = 0;
            for (int i = 0; i < m; ++i)
                if (ratio[i] <= near) { l = i; ++hits; }
            if (hits > 1) {
                l = -1;
                double best_ratio = 0.0;
                for (int i = 0; i < m; ++i) {
                    if (!(fcol[i] > tol)) continue;
                    const double q = ratio[i];
                    if (l < 0 || q < best_ratio - 1e-13 * (1.0 + fabs(best_ratio)) ||
                        (q <= best_ratio + 1e-13 * (1.0 + fabs(best_ratio)) && basic[i] < basic[l])) {
                        l = i; best_ratio = q;
                    }
                }
            }
        }
        // pivot on (l, e): every thread its columns
        const double piv = fcol[l], fd = d[e], rl = rhs[l] / piv;
        __syncthreads();
        for (int j = tid; j < ncol; j += T) {
            double q = tab[(size_t)l * ncol + j] / piv;
            if (j == e) q = 1.0;
            tab[(size_t)l * ncol + j] = q;
#pragma unroll 4
            for (int i = 0; i < m; ++i) {
                const double f = fcol[i];
                if (i == l || f == 0.0) continue;
                const double v = f * q;
                tab[(size_t)i * ncol + j] = j == e ? 0.0 : tab[(size_t)i * ncol + j] - v;
            }
            const double v = fd * q;
            d[j] = j == e ? 0.0 : d[j] - v;
        }
        for (int i = tid; i < m; i += T) {
            const double f = fcol[i];
            if (i == l) { rhs[i] = rl; basic[i] = e; continue; }
            if (f == 0.0) continue;
            const double v = f * rl;
            double r = rhs[i] - v;
            if (r < 0.0 && r > -1e-9 * (1.0 + fabs(rl))) r = 0.0;
            rhs[i] = r;
        }
        const double zv = fd * rl, z_new = z + zv;
        stall = (z - z_new > 1e-14 * (1.0 + fabs(z))) ? 0 : stall + 1;
        z = z_new;
    }
    if (tid == 0) { a.v[p] = z - shift; a.rc[p] = rc; }
}

// The best program (greatest optimum, then the most promising profile) to pinned host memory.
__global__ void __launch_bounds__(256) profile_pick_kernel(LpArgs a, LpBest *out, double *x_host, int32_t *profile_host, Done done)
{
    __shared__ double sv[4];
    __shared__ u64 sk[4];
    __shared__ int sp[4], sbad[4];
    const int tid = threadIdx.x;
    const unsigned n = *a.n < a.most ? *a.n : a.most;
    double bv = -INFINITY;
    u64 bk = 0;
    int bp = -1, bad = 0;
    auto take = [&](double v, u64 key, int p) {
        if (p >= 0 && (bp < 0 || v > bv || (v == bv && key > bk))) { bv = v; bk = key; bp = p; }
    };
    for (unsigned p = tid; p < n; p += 256) {
        const int rc = a.rc[p];
        bad |= rc == 2;
        if (rc == 0) take(a.v[p], a.sel[p], (int)p);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        take(__shfl_xor(bv, s, 64), __shfl_xor(bk, s, 64), __shfl_xor(bp, s, 64));
        bad |= __shfl_xor(bad, s, 64);
    }
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; sk[tid >> 6] = bk; sp[tid >> 6] = bp; sbad[tid >> 6] = bad; }
    __syncthreads();
    for (int w = 0; w < 4; ++w) { take(sv[w], sk[w], sp[w]); bad |= sbad[w]; }
    if (bp >= 0) {
        for (int i = tid; i < a.m; i += 256) x_host[i] = a.x[(size_t)bp * a.m + i];
        for (int t = tid; t < a.K; t += 256) profile_host[t] = a.br[(size_t)tk_index(bk) * a.K + t];
    }
    if (tid == 0) {
        LpBest r;
        r.value = bv; r.profiles = *a.n; r.solved = n; r.found = bp >= 0 ? 1 : 0; r.failed = bad;
        *out = r;
    }
    signal_done(done, 0);
}

}  // namespace

unsigned profile_table_slots(long long count)
{
    unsigned s = 256;
    while ((long long)s < 2 * count) s <<= 1;            // (count <= 2^27)
    return s;
}

// slots, best and n (which the caller has cleared) -> list (up to `count` keys) and n, then sel (up to
// `most` of them).
hipError_t launch_profiles(const float *V, const int32_t *br, long long count, int K, unsigned *slots,
                           unsigned long long *best, unsigned *n, unsigned long long *list, unsigned most,
                           unsigned long long *sel, hipStream_t s)
{
    const unsigned nslots = profile_table_slots(count);
    hipLaunchKernelGGL(profile_insert_kernel, dim3((unsigned)((count + PI_T - 1) / PI_T)), dim3(PI_T), 0, s, V, br, (unsigned)count, K,
                       slots, best, nslots - 1u);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(profile_list_kernel, dim3((nslots + 1024 * PL_PER - 1) / (1024 * PL_PER)), dim3(1024), 0, s, best, nslots, list, n);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(profile_select_kernel, dim3(1), dim3(TK_T), 0, s, list, n, most, sel);
    return hipGetLastError();
}

static size_t lp_lds(int m, int n, int K)
{
    const size_t ncol = 2 + (size_t)K * (n - 1) + m;
    return ((size_t)m * ncol + ncol + 4 * (size_t)m) * sizeof(double) + (size_t)m * sizeof(int);
}

// A tableau that LDS holds beside the kernel's own words.
constexpr int LP_LDS_MOST = 150 * 1024;
bool lp_on_device(int m, int n, int K) { return n > 1 && (double)m * (2.0 + (double)K * (n - 1) + m) < 20000.0 && lp_lds(m, n, K) <= LP_LDS_MOST; }

hipError_t launch_profile_lps(const LpArgs &a, LpBest *out, double *x_host, int32_t *profile_host, const Done &done, hipStream_t s)
{
    // Up to sixteen rows and two columns a lane the tableau fits the registers of a wavefront (200
    // programs of 16 x 78 cells: 97 us from LDS, 32 from registers); otherwise LDS, by four wavefronts
    // once the cells outnumber the barriers' cost.
    const int ncol = 2 + a.K * (a.n_act - 1) + a.m, cols = (ncol + 63) / 64;
    const size_t lds = lp_lds(a.m, a.n_act, a.K);
    const bool small = a.m <= 16 && cols <= 2, one = (size_t)a.m * ncol <= 4096;
    hipError_t e;
    if (small) {
        void (*k)(LpArgs) = a.m <= 8 ? (cols == 1 ? profile_lp_small_kernel<8, 1> : profile_lp_small_kernel<8, 2>)
                                     : (cols == 1 ? profile_lp_small_kernel<16, 1> : profile_lp_small_kernel<16, 2>);
        hipLaunchKernelGGL(k, dim3(a.most), dim3(64), 0, s, a);
    } else {
        const void *k = one ? (const void *)profile_lp_kernel<64> : (const void *)profile_lp_kernel<256>;
        if (lds > 48 * 1024 && (e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, LP_LDS_MOST)) != hipSuccess) return e;
        if (one) hipLaunchKernelGGL(profile_lp_kernel<64>, dim3(a.most), dim3(64), lds, s, a);
        else hipLaunchKernelGGL(profile_lp_kernel<256>, dim3(a.most), dim3(256), lds, s, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(profile_pick_kernel, dim3(1), dim3(256), 0, s, a, out, x_host, profile_host, done);
    return hipGetLastError();
}

}  // namespace bsse
