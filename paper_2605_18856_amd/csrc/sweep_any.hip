// Host side of the any-shape matrix-core kernel (sweep_any_impl.h), the kernel that packs payoffs for
// it, and the kernel that turns the per-type leader payoffs of a sliced launch into values.
#include "bsse_internal.h"
#include "sweep_any_impl.h"
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>
#include "done_device.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms1(int ks, int form, bool many);
any_impl::any_kernel_t any_kernel_terms3(int ks, int form, bool many);
any_impl::any_kernel_t any_kernel_terms6(int ks, int form, bool many);
any_impl::any_kernel_t any_kernel_half(int ks, int form, bool many);

namespace {

using any_impl::THREADS;

int roundup(int v, int to) { return (v + to - 1) / to * to; }
int payoff_parts(int terms) { return terms == 6 ? 3 : terms == 2 ? 2 : 1; }
int products(const AnyGeo &q) { return q.terms != 2 ? q.terms : q.ks == 3 ? 4 : 3; }

// Sums of half-precision parts decide only where nothing that they leave out or round can: the margin bounds, in
// |x|_2 |B_j|_2 of a row and a type as they are scaled, what a difference of two of them is off by, by Cauchy and Schwarz.
//   * What two parts leave of a number is 2^-23 of it at most, of a row's component and of a payoff; three products
//     also leave out low times low part, 2^-22.
//   * Matrix instructions lose at most 8 2^-24 of the sum of their absolute products, over all k-steps |x|_2 |B_j|_2
//     at most, and 6 2^-24 of the sum they go on with, each (test_gpu_matrix_terms.py); the products with a small part
//     stand at 2^-10 of the sum when they do, which the 2 % cover.
//   * Both sums of the difference move.  The sums in 64 bits are rounded to 32 and so may tie at a distance of
//     2 2^-24 of their size, and the threshold is rounded: three more.
//   * Where a part is subnormal, what is left is 2^-25 at most (of components and payoffs below 2^-16 of the greatest
//     of their row or type, which is scaled to 2^14 to 2^15): 2^-24 sqrt(m) (|x|_2 + |B_j|_2) in a difference, and
//     with both norms at least 2^14 no more than 2^-37 sqrt(m) |x|_2 |B_j|_2.
// 2 % for the roundings of the norms.
float half_margin(int ks)
{
    const double left_out = ks == 3 ? 4.0 : 8.0, instructions = 8.0 + 6.0 * ks;
    return (float)(1.02 * ((2.0 * (left_out + instructions) + 3.0) * 0x1p-24 + 0x1p-37 * std::sqrt(16.0 * ks)));
}
// Payoffs from here on: rows of ordinary size might have infinite sums, which scaled ones do not show.
constexpr float kHalfMost = 0x1p100f;

// (on the bits, which are ordered as the numbers are: whole numbers are compared several at a time)
float greatest_of(size_t elems, const float *B)
{
    int most = 0;
    for (size_t e = 0; e < elems; ++e) {
        int bits;
        memcpy(&bits, &B[e], 4);
        bits &= 0x7FFFFFFF;
        most = bits > most ? bits : most;
    }
    float v;
    memcpy(&v, &most, 4);
    return v;
}
// Where the payoffs behind the records begin (terms 2).
__host__ __device__ inline size_t exact_off(const AnyGeo &q) { return (size_t)q.units * q.rec_bytes; }

any_impl::any_kernel_t kernel_for(const AnyGeo &q, bool many)
{
    return q.terms == 1   ? any_kernel_terms1(q.ks, q.form, many)
           : q.terms == 2 ? any_kernel_half(q.ks, q.form, many)
           : q.terms == 3 ? any_kernel_terms3(q.ks, q.form, many)
                          : any_kernel_terms6(q.ks, q.form, many);
}

// bf16 part `p` of v: every part the nearest bf16 (ties to even) of what the parts before it leave
__device__ __forceinline__ unsigned bf16_part(float v, int p)
{
    for (int k = 0;; ++k) {
        unsigned b = __float_as_uint(v);
        b += 0x7FFFu + ((b >> 16) & 1u);
        b &= 0xFFFF0000u;
        if (k == p) return b >> 16;
        v -= __uint_as_float(b);
    }
}

// terms 2, one workgroup per type: the power of two that brings the greatest payoff to 2^14, and the margin of
// the sums' filter.
__global__ void __launch_bounds__(256)
any_margin_kernel(int m, int n, float relative, const float *__restrict__ B, float *__restrict__ scale, float *__restrict__ margin)
{
    __shared__ float part[2][4];
    const int t = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float *Bt = B + (size_t)t * m * n;
    auto greatest = [&](float v, int which) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
        if (lane == 0) part[which][wave] = v;
        __syncthreads();
        return fmaxf(fmaxf(part[which][0], part[which][1]), fmaxf(part[which][2], part[which][3]));
    };
    float most = 0.0f;
    for (int e = tid; e < m * n; e += 256) most = fmaxf(most, fabsf(Bt[e]));
    most = greatest(most, 0);
    const float s = most > 0.0f ? ldexpf(1.0f, 14 - ilogbf(most)) : 1.0f;
    float norm = 0.0f;
    for (int j = tid; j < n; j += 256) {
        float sum = 0.0f;
        for (int i = 0; i < m; ++i) {
            const float b = Bt[(size_t)i * n + j] * s;
            sum = fmaf(b, b, sum);
        }
        norm = fmaxf(norm, sum);
    }
    norm = greatest(norm, 1);
    if (tid == 0) {
        scale[t] = s;
        margin[t] = relative * sqrtf(norm);
    }
}

// One thread per 16-byte piece of the records: eight k-slots of a fragment, or four (fp32) or eight
// (bf16) entries of a leader row.  Runs once per game; the reads are strided by n but the payoffs fit
// the caches.
__device__ __forceinline__ unsigned half_part(float v, int p)
{
    const _Float16 first = (_Float16)v, part = p ? (_Float16)(v - (float)first) : first;
    return __builtin_bit_cast(unsigned short, part);
}
__global__ void __launch_bounds__(256)
any_pack_kernel(AnyGeo q, int m, int n, int K, const float *__restrict__ A, const float *__restrict__ B,
                const float *__restrict__ scale, uint4 *__restrict__ Bpack, size_t pieces)
{
    const int parts = q.terms == 6 ? 3 : q.terms == 2 ? 2 : 1, half = 8 * q.ks;
    const int rec16 = q.rec_bytes / 16, frag16 = q.form >= 8 ? 2 * parts * q.ks * 64 : q.tpg * parts * q.ks * 64;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < pieces; p += stride) {
        if (q.terms == 2 && p >= exact_off(q) / 16) {      // terms 2: the payoffs themselves behind the records
            const size_t o = p - exact_off(q) / 16, tj = o / (4 * q.ks), t = tj / n, j = tj % n;
            float v[4];
            for (int k = 0; k < 4; ++k) {
                const int i = (int)(o % (4 * q.ks)) * 4 + k;
                v[k] = i < m ? B[(t * m + i) * n + j] : 0.0f;
            }
            Bpack[p] = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
            continue;
        }
        const int u = (int)(p / rec16), o = (int)(p % rec16);
        unsigned e[8] = { 0, 0, 0, 0, 0, 0, 0, 0 };
        uint4 out = make_uint4(0u, 0u, 0u, 0u);
        if (o < frag16) {
            const int lane = o % 64, f = o / 64, part = f % parts, s = f / parts % q.ks, tile = f / (parts * q.ks);
            const int hh = lane / 32, row = lane % 32;
            int t, j;
            const float *P = B;
            if (q.form >= 8) {
                // the rows a lane half receives are whole types: register r of half h2 is row 8(r/4)+4*h2+r%4
                const int h2 = (row >> 2) & 1, r = (row >> 3) * 4 + (row & 3);
                t = (32 / q.form) * u + (q.form == 16 ? h2 : 2 * h2 + (r >> 3));
                j = q.form == 16 ? r : r & 7;
                t = t < K ? t : K - 1;               // a padded type behaves like the last one, at weight zero
                P = tile ? A : B;                    // the second tile of a record holds the leader's payoffs
            } else {
                t = u; j = tile * 32 + row;
            }
            if (j < n)
                for (int k = 0; k < 8; ++k) {
                    const int i = hh * half + 8 * s + k;
                    if (i >= m) continue;
                    const float v = P[((size_t)t * m + i) * n + j];
                    e[k] = q.terms == 2 ? half_part(v * scale[t], part) : bf16_part(v, part);
                }
            out = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
        } else if (q.lead_off >= 0 && o >= q.lead_off / 16) {
            const int byte = (o - q.lead_off / 16) * 16, j = byte / q.lead_stride, b0 = byte % q.lead_stride;
            if (j < n) {
                const int per = q.terms == 1 ? 8 : 4, i0 = b0 / (q.terms == 1 ? 2 : 4);
                for (int k = 0; k < per; ++k) {
                    const float v = i0 + k < m ? A[((size_t)u * m + i0 + k) * n + j] : 0.0f;
                    e[k] = q.terms == 1 ? bf16_part(v, 0) : __float_as_uint(v);
                }
                out = q.terms == 1 ? make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16)
                                   : make_uint4(e[0], e[1], e[2], e[3]);
            }
        }
        Bpack[p] = out;
    }
}

// Leader columns [K][n][16*ks], fp32 (bf16 for terms == 1), zero padded: the gather from global memory
// and the exact routine.
__global__ void __launch_bounds__(256)
any_pack_lead_kernel(AnyGeo q, int m, int n, int K, const float *__restrict__ A, void *__restrict__ ATpack)
{
    const int mp = 16 * q.ks;
    const size_t total = (size_t)K * n * mp, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += stride) {
        const int i = (int)(p % mp);
        const size_t tj = p / mp, t = tj / n, j = tj % n;
        const float v = i < m ? A[(t * m + i) * n + j] : 0.0f;
        if (q.terms == 1) reinterpret_cast<unsigned short *>(ATpack)[p] = (unsigned short)bf16_part(v, 0);
        else reinterpret_cast<float *>(ATpack)[p] = v;
    }
}

__global__ void __launch_bounds__(FINISH_ROWS) finish_rows_kernel(FinishRowsArgs f)
{
    __shared__ float sv[FINISH_ROWS / 64];
    __shared__ unsigned sc[FINISH_ROWS / 64];
    const int tid = threadIdx.x;
    const unsigned count = (unsigned)f.count, c = blockIdx.x * FINISH_ROWS + tid;
    const unsigned cc = c < count ? c : count - 1u;
    float v = 0.0f;
    int t0 = 0;
    for (; t0 + 8 <= f.K; t0 += 8) {                     // eight loads in flight: the loop is bound by their latency
        float l[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) l[k] = f.l[(size_t)(t0 + k) * count + cc];
#pragma unroll
        for (int k = 0; k < 8; ++k) v = fmaf(f.prior[t0 + k], l[k], v);
    }
    for (; t0 < f.K; ++t0) v = fmaf(f.prior[t0], f.l[(size_t)t0 * count + cc], v);
    if (!(v == v)) v = -INFINITY;
    if (f.V_out && c < count) f.V_out[c] = v;
    if (!f.blk_v && !f.rec) return;
    float bv = v;
    unsigned bc = cc;                                    // (a thread past the end repeats the last row)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const float ov = __shfl_xor(bv, d, 64);
        const unsigned oc = __shfl_xor(bc, d, 64);
        if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; }
    }
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; sc[tid >> 6] = bc; }
    __syncthreads();
    bv = sv[0]; bc = sc[0];
    for (int w = 1; w < FINISH_ROWS / 64; ++w)
        if (sv[w] > bv || (sv[w] == bv && sc[w] < bc)) { bv = sv[w]; bc = sc[w]; }
    if (f.blk_v) {
        if (tid == 0) { f.blk_v[blockIdx.x] = bv; f.blk_i[blockIdx.x] = f.index_base + bc; }
        return;
    }
    for (int t = tid; t < f.K; t += FINISH_ROWS) f.rec_br[(size_t)blockIdx.x * f.K + t] = f.br[(size_t)t * count + bc];
    for (int i = tid; i < f.m; i += FINISH_ROWS) f.rec_x[(size_t)blockIdx.x * f.m + i] = f.X[(size_t)bc * f.m + i];
    FinishRec &rec = f.rec[blockIdx.x];
    if (tid == 0) {
        rec.value = bv; rec.index = f.index_base + bc;
        if (blockIdx.x == 0) { rec.ties = *f.ties; *f.ties = 0ull; }
    }
    const Done d = { &rec.seq, f.seq };
    signal_done(d, 0);
}

}  // namespace

hipError_t launch_finish_rows(const FinishRowsArgs &f, hipStream_t s)
{
    if (f.count <= 0) return hipSuccess;
    hipLaunchKernelGGL(finish_rows_kernel, dim3((unsigned)((f.count + FINISH_ROWS - 1) / FINISH_ROWS)), dim3(FINISH_ROWS), 0, s, f);
    return hipGetLastError();
}

// The margin of one type, as any_margin_kernel forms it, in the payoffs' own units.
static float half_margin_of(int m, int n, int ks, const float *B)
{
    std::vector<double> sum((size_t)n, 0.0);
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < n; ++j) {
            const float b = B[(size_t)i * n + j];
            sum[j] += (double)b * b;
        }
    return (float)(half_margin(ks) * std::sqrt(*std::max_element(sum.begin(), sum.end())));
}

// Two half-precision parts of a number hold 22 bits or more, and fewer products of them take fewer matrix instructions
// that round than six of bf16 parts.  Their sums decide where the greatest stands clear of the next by all that the parts
// leave out and the instructions round (half_margin: rigorous, some hundred times what the sums are off by as a rule);
// elsewhere sums in 64 bits, rounded once, do (exact_column, exact_actions), so that every best response is the one of
// the true sums rounded to 32 bits.
// Four products where m <= 48: a third k-step costs little, and the margin is half as wide.  Up to 32 leader actions six
// products are as fast.  Sixteen follower actions or fewer take their leader payoffs off the matrix cores, which nothing
// watches: six products.
// Payoffs of very different sizes (forbidden actions at -10^3 beside -2 to 2), payoffs with a large part in common and
// equal columns put many values within the margin; from about an eighth of the tiles on six products are the faster
// ones on the shapes with the least matrix work (200000 rows, K = 20, normal payoffs plus 30, 100, 200, 400, us, these and
// six products: m = 60, n = 100 290, 356, 385, 476, and 350, 387, 389, 422, the second with a share of 0.27; m = 40, n = 24
// 117, 131, 156, and 105, 111, 122 from 100 on).
bool any_half_suits(int m, int n, int K, const float *B)
{
    if (m <= 32 || n <= 16 || !any_supported(m, n)) return false;
    if (greatest_of((size_t)K * m * n, B) >= kHalfMost) return false;
    const int ks = any_geometry(m, n, K, 2).ks;
    return twice_summed(m, n, K, B, [=](int t) { return half_margin_of(m, n, ks, B + (size_t)t * m * n); }, 64, true) <= 0.125;
}

// m <= 128 products below 2^(e - 126) 2^(b + 1) come to 2^127 at most (e, b: exponents of the row, biased, and of the
// greatest payoff); infinities and what is no number are never below the end.
int row_end_of(size_t elems, const float *B)
{
    const float most = greatest_of(elems, B);
    return most > 0.0f ? std::min(255, 246 - std::ilogb(most)) : 255;
}

bool any_supported(int m, int n) { return m <= 128 && (long long)m * n > 64; }

AnyGeo any_geometry(int m, int n, int K, int terms)
{
    AnyGeo q{};
    static const int steps[] = { 1, 2, 3, 4, 6, 8 };
    q.terms = terms;
    q.ks = 8;
    for (int k : steps)
        if (16 * k >= m) { q.ks = k; break; }
    if (terms == 3 && q.ks != 2 && q.ks != 4) q.ks = q.ks == 1 ? 2 : q.ks == 3 ? 4 : 8;      // (fewer instantiations)
    const int parts = payoff_parts(terms), lbytes = terms == 1 ? 2 : 4;
    q.tile_bytes = parts * q.ks * 1024;
    q.form = n <= 8 ? 8 : n <= 16 ? 16 : n <= 32 ? 1 : n <= 64 && any_impl::two_tiles(terms, q.ks) ? 2
             : n <= 96 && n > 64 && any_impl::three_tiles(terms, q.ks) ? 3
             : n <= 128 && n > 96 && any_impl::four_tiles(terms, q.ks) ? 4 : 0;
    q.nq = 1; q.lead_off = -1;
    // Two stage buffers per workgroup, and as many workgroups on a compute unit of 160 KiB as the registers
    // allow: 26 KiB a stage for two or three, 19 for four.  Beyond that the row tiles come in pieces and the
    // leader column is gathered from L2; but one candidate tile a wavefront and two row tiles a type are too
    // little to hide a gather of 256 bytes behind: types that need up to 36 KiB with their leader rows go in one
    // piece there, for two workgroups (us, three and two: m = 120, n = 40, K = 30 bf16, 260000 rows 276 and 206;
    // m = 100, n = 60, K = 16 bf16 170 and 138; m = 60, n = 40, K = 20, 130000 rows 153 and 126; but m = 45,
    // n = 60, K = 20 f32, 260000 rows 197 and 210; m = 90, n = 70, K = 20 bf16, 20000 rows 40 and 45).
    const int waves = any_impl::occupancy(terms, q.ks, q.form, true);
    const bool gather = any_impl::tiles_per_wave(terms, q.ks, q.form, true) == 1 && n <= 64 && 16 * q.ks * lbytes >= 256;
    const int cap = (waves >= 4 ? 19 : 26) * 1024, most = waves >= 3 && !gather ? cap : 36 * 1024;
    if (q.form >= 8) {
        q.tpg = 1;
        q.units = (K + 32 / q.form - 1) / (32 / q.form);
        q.rec_bytes = 2 * q.tile_bytes;
    } else {
        q.tpg = (n + 31) / 32;
        q.units = K;
        q.lead_stride = 16 * q.ks * lbytes + 16;         // (16 bytes more: rows spread over the banks)
        const long long whole = (long long)q.tpg * q.tile_bytes + roundup(n * q.lead_stride, 1024);
        if (whole <= most) {
            q.lead_off = q.tpg * q.tile_bytes;
            q.rec_bytes = (int)whole;
        } else {
            q.rec_bytes = q.tpg * q.tile_bytes;
            q.stt = cap / q.tile_bytes > 1 ? cap / q.tile_bytes & ~1 : 1;      // tiles go in pairs
            if (q.stt > q.tpg || (q.form >= 2 && q.form <= 4)) q.stt = q.tpg;       // (32 KiB at most)
            q.nq = (q.tpg + q.stt - 1) / q.stt;
        }
    }
    q.ups = 1;
    if (q.nq == 1) {
        q.ups = cap / q.rec_bytes > 1 ? cap / q.rec_bytes : 1;
        if (q.ups > q.units) q.ups = q.units;
        q.stt = q.tpg;
        q.buf_bytes = q.ups * q.rec_bytes;
    } else {
        q.buf_bytes = q.stt * q.tile_bytes;
    }
    q.resident = std::max(2, std::min(waves, 160 * 1024 / (2 * q.buf_bytes + 1024)));
    q.resident_cut = terms == 1 ? q.resident : std::min(q.resident, any_impl::occupancy(terms, q.ks, q.form, false));
    return q;
}

const char *any_name(const AnyGeo &q) { return q.terms == 1 ? "mfma_bf16" : q.terms == 3 ? "mfma_split3" : "mfma_split6"; }

void any_pack_sizes(const GameView &g, size_t *Bbytes, size_t *ATbytes)
{
    *Bbytes = (size_t)g.any.units * g.any.rec_bytes + (g.any.terms == 2 ? (size_t)g.K * g.n * 16 * g.any.ks * 4 : 0);
    *ATbytes = g.any.form >= 8 ? 16 : (size_t)g.K * g.n * 16 * g.any.ks * (g.any.terms == 1 ? 2 : 4);
}

hipError_t launch_any_pack(const GameView &g, const float *A, const float *B, void *Bpack, void *ATpack, float *margin,
                           float *scale, hipStream_t s)
{
    size_t bb, ab;
    if (g.any.terms == 2) {
        hipLaunchKernelGGL(any_margin_kernel, dim3((unsigned)g.K), dim3(256), 0, s, g.m, g.n, half_margin(g.any.ks), B,
                           scale, margin);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    any_pack_sizes(g, &bb, &ab);
    const size_t pieces = bb / 16;
    size_t blocks = (pieces + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(any_pack_kernel, dim3((unsigned)blocks), dim3(256), 0, s, g.any, g.m, g.n, g.K, A, B, scale,
                       (uint4 *)Bpack, pieces);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || g.any.form >= 8) return e;
    blocks = (ab / 4 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(any_pack_lead_kernel, dim3((unsigned)blocks), dim3(256), 0, s, g.any, g.m, g.n, g.K, A, ATpack);
    return hipGetLastError();
}

hipError_t any_prepare(const GameView &g)
{
    if (2 * g.any.buf_bytes <= 48 * 1024) return hipSuccess;
    // (the most that any game takes on this kernel: the limit is the kernel's, not the game's)
    const int most = 2 * std::max(36 * 1024, 2 * g.any.tile_bytes);
    for (bool many : { false, true })
        if (hipError_t e = hipFuncSetAttribute((const void *)kernel_for(g.any, many), hipFuncAttributeMaxDynamicSharedMemorySize, most))
            return e;
    return hipSuccess;
}

constexpr int CUS = 256;

static int tiles_of(const AnyGeo &q, bool many) { return any_impl::tiles_per_wave(q.terms, q.ks, q.form, many); }
static long long blocks_of(const AnyGeo &q, long long count, bool many)
{
    const long long rows = 32LL * any_impl::WAVES * tiles_of(q, many);
    return (count + rows - 1) / rows;
}

// An uncut launch of `blocks` blocks for three workgroups a compute unit that takes one round of three and
// a last one of one: two rounds of two are full, and where a wavefront has three parts of a row they are
// faster (us, 768 workgroups and 512: m = 30, n = 50, K = 20, 210000 rows 144 and 128; m = 60, n = 30, K = 20,
// 100000 rows 90 and 82; whole numbers, m = 20, n = 140, K = 20, 210000 rows 191 and 179; but m = 16,
// n = 40, K = 30 bf16, 210000 rows 90 and 100).
static bool one_left_over(const AnyGeo &q, long long blocks)
{
    return q.resident == 3 && q.form < 8 && blocks > 3 * CUS && blocks <= 4 * CUS;
}

// Which of two kinds of kernel takes a launch (see two_kinds).  Long bf16 rows: the one for two workgroups where
// one would be left over, as it takes twice the rows in one round (us: m = 96, n = 60, K = 16, 130000 rows 82
// and 69; m = 128, n = 20, K = 30 99 and 88), and where LDS holds two only (see any_geometry).
static bool many_kind(const AnyGeo &q, long long count, bool cut)
{
    if (!any_impl::two_kinds(q.terms, q.ks, q.form)) return true;
    if (q.resident < 3 || (cut && q.terms != 1)) return false;
    const long long blocks = blocks_of(q, count, true);
    return cut || !(one_left_over(q, blocks) || (q.terms != 1 && blocks <= 2 * CUS));
}

// Workgroups on a compute unit of an uncut launch.
static int side_by_side(const AnyGeo &q, long long count)
{
    return !many_kind(q, count, false) || (q.terms != 1 && one_left_over(q, blocks_of(q, count, true))) ? 2 : q.resident;
}

// Time that `side` workgroups of a compute unit take for a block each, two being one.  (One takes no less: it
// waits for its own loads, and rarely is every unit left with one.)
static double round_time(long long side) { return side <= 0 ? 0.0 : side <= 2 ? 1.0 : side == 3 ? 1.3 : 1.65; }

long long any_num_blocks(const GameView &g, long long count)
{
    // At most one resident set, and always the whole of it: with the grid cut to the workgroups that share
    // the blocks evenly, some compute units held one workgroup and the others two (m = 16, n = 40, K = 30
    // bf16: 140000 rows 106 -> 96 us, 270000 rows 151 -> 134; m = 20, n = 12, K = 12: 400000 rows 78 -> 71).
    // All the workgroups that the registers allow, not two a compute unit (three or four, row tiles one
    // by one, us): the same 140000
    // rows 81 -> 70, 1000000 rows 348 -> 281; m = 12, n = 100, K = 30, 100000 rows 101 -> 89; m = 40, n = 80,
    // K = 50, 100000 rows 310 -> 261; m = 20, n = 20, K = 8, 270000 rows 51 -> 45; m = 9, n = 15, K = 20 bf16,
    // 1000000 rows 96 -> 74.
    const AnyGeo &q = g.any;
    return std::max(1LL, std::min<long long>(blocks_of(q, count, many_kind(q, count, false)), CUS * side_by_side(q, count)));
}

long long any_max_blocks(const GameView &g, long long count)
{
    return std::max(1LL, std::min<long long>(blocks_of(g.any, count, true), CUS * g.any.resident));
}

// Workgroups of a launch cut over the types, 1 when it is not to be cut.
int any_shares(const GameView &g, long long count)
{
    const AnyGeo &q = g.any;
    const long long blocks = blocks_of(q, count, many_kind(q, count, true)), pairs = blocks * q.units;
    if (q.units < 2) return 1;
    const double work = 20.0 + 1.5 * products(q) * q.ks * q.tpg;
    // Workgroups side by side: the time of a share, which begins with a block's rows (all that are resident,
    // two a compute unit, us: m = 60, n = 30, K = 20 bf16, 30000 rows 33 and 31; m = 16, n = 40, K = 30 bf16,
    // 20000 rows 26 and 28; m = 60, n = 100, K = 20, three products, 10000 rows 40 and 43).
    auto share_time = [&](int r) {
        const double each = (double)pairs / (CUS * r);
        return (0.5 * (each + std::ceil(each)) + (4.0 + 6.0 * q.ks) / work) * round_time(r);
    };
    int side = 1;
    for (int r = 2; r <= q.resident_cut; ++r)
        if (share_time(r) < share_time(side)) side = r;
    const int shares = (int)std::min<long long>(pairs, CUS * side);
    // Far fewer blocks of candidates than compute units, or packed types (the per-type outputs of a cut
    // launch are most of their cost).
    if (blocks < 128 || (q.form >= 8 && blocks < 256)) return shares;
    if (q.form >= 8 || (count + FINISH_ROWS - 1) / FINISH_ROWS * (g.m + g.K) > (1LL << 16)) return 1;
    // Otherwise what decides is how full the compute units are.  In units of the time a compute unit takes for
    // two blocks and all types side by side: uncut, the fullest one takes as many rounds as it has blocks for,
    // later ones shorter (they start one by one) and one block left over 0.8; cut, all take the same, more for
    // the outputs where a type is little work, and 12 us for another launch that sums them (the unit is about
    // 0.09 us per type and unit of `work`).  Uncut and cut, us: m = 50, n = 100, K = 24 bf16, 50000 rows 62 and
    // 52, 200000 rows 129 and 146; m = 30, n = 50, K = 20, 50000 rows 60 and 48, 100003 rows 67 and 72; m = 30,
    // n = 70, K = 20, whole numbers, 35000 rows 45 and 35, 140000 rows 82 and 87; m = 90, n = 100, K = 10, 70001
    // rows 121 and 94; m = 24, n = 24, K = 20, 50000 rows 48 and 38, 140000 rows 59 and 66; m = 12, n = 90, K = 30
    // bf16, 140000 rows 65 and 82.  Over 12 shapes of two to seven row tiles and 7 sizes from 20000 to 200000 rows the
    // choice takes 1 % longer than the better one on average, and 17 % at most (m = 45, n = 60, K = 20 bf16, 200000
    // rows 86, uncut 73).
    const bool many = many_kind(q, count, false);
    const int tiles = tiles_of(q, many), tiles_cut = tiles_of(q, many_kind(q, count, true)), full = side_by_side(q, count);
    const long long uncut_blocks = blocks_of(q, count, many), all = CUS * full;
    const long long sets = uncut_blocks / all, rest = (uncut_blocks % all + CUS - 1) / CUS;
    const double later = rest == 1 ? 0.8 : 0.82 * round_time(rest);
    const double rounds = sets == 0 ? round_time(rest) : round_time(full) * (1.0 + 0.82 * (double)(sets - 1)) + later;
    const double uncut = rounds * (tiles > tiles_cut ? 1.75 : 1.0);            // (twice the rows in a block)
    const double cut = 12.0 / (0.09 * work * q.units) + (0.94 + 9.0 / work) * round_time(side) * blocks / (CUS * side);
    return cut < 0.95 * uncut ? shares : 1;
}

long long any_row_blocks(const GameView &g, long long count)
{
    const int shares = any_shares(g, count);
    return shares > 1 ? shares : any_num_blocks(g, count);
}

hipError_t launch_sweep_any(const GameView &g, const SweepArgs &a, int shares, hipStream_t s)
{
    if (a.count <= 0) return hipSuccess;
    const bool many = many_kind(g.any, a.count, shares > 1);
    any_impl::any_kernel_t k = kernel_for(g.any, many);
    if (!k) return hipErrorNotSupported;
    any_impl::AnyArgs args{ g, a };
    const long long pairs = blocks_of(g.any, a.count, many) * g.any.units;
    if (shares > 1 && (a.V_out || a.blk_v || shares > pairs || pairs > 0x7FFFFFFFLL)) return hipErrorInvalidValue;
    args.a.slice_stages = shares > 1 ? (int)(pairs / shares) : 0;
    const long long nx = shares > 1 ? shares : any_num_blocks(g, a.count);
    if (nx > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((unsigned)nx), dim3(THREADS), (size_t)2 * g.any.buf_bytes, s, args);
    return hipGetLastError();
}

}  // namespace bsse
