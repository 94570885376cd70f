// Fused sweep for wide games with small whole-number payoffs (n = 256, m <= 128; integers 0..7, say): the follower
// product on the six-bit matrix instruction, three and a half times the rate of the bf16 one.
//
// Payoffs.  No difference of two actions notices what all payoffs of a leader action have in common, so the middle
// of their range is taken off; what is left, times a power of two per type, has to be one of the 63 values of the
// e2m3 format (whole numbers of a span up to 15 are).  A candidate row is cut into four e2m3 parts, each the nearest of
// what is left, in blocks of 32 components (one lane's slots of one instruction) whose greatest comes to 2 to 4;
// part k is scaled by 2^-5k through the instruction's block scales, so that nothing is rescaled and the four parts
// leave 2^-18 of the greatest or less.  Four parts are eight instructions per row tile and 128 leader actions, where
// two bf16 parts were sixteen of about the same length, and a row tile's fragments are 3 KiB instead of 8.
//
// Decisions.  The sums decide where the maximum stands clear of the next value by more than the row's remainder
// and the instructions' roundings can change (fp6_margins): then it is the maximum of the true sums.  Other columns sum
// three bf16 parts of the row, from the same fragments, as sweep_mfma.hip's settle does; ties go to the exact routine.
// Rows of few bits (multiples of 1/16, say), which tie often, have exact sums as they are and go there at once (m = 128,
// K = 32, 40000 such rows 933 us, without summing again 634, on bf16 parts alone 771).
//
// Layout as in sweep_mfma.hip: payoffs are the A operand, so a lane owns one candidate and half of a tile's rows.
// The row tiles of a type pass through two accumulators in turn; what stays is the maxima of the grid's rows and columns
// (ArgGrid).  The leader payoff is an fp32 chain over the unsplit half row and half-precision payoffs gathered from
// L2, requested when the best response is known and met during the next type.
// Workgroups of four wavefronts, two a compute unit, so that no barrier keeps the two wavefronts of a SIMD in step.
//
// Against two bf16 products (us): m = 128, n = 256, K = 256, 131072 rows 3225 and 2215; K = 100, 25000 rows 297 and 218;
// m = 100, K = 100, 66000 rows 835 and 510; m = 70, K = 30, 1000 rows 31 and 24.  Matrix and vector time still add up
// (a part less: 1788 of 2183, about 44 cycles an instruction); of the rest 4 % is the gather of leader columns and 2 %
// the columns that are summed again (0.9 % of the tiles).  Three parts would leave 25 % of the tiles to be summed again.
// Tiles in turn through two accumulators, maxima between the instructions: 2220 -> 2183 against two tiles at a time.
#include "bsse_internal.h"
#include "mfma_device.h"
#include "done_device.h"
#include <algorithm>
#include <cmath>
#include <limits.h>
#include <stdlib.h>
#include <string.h>

namespace bsse {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x6 __attribute__((ext_vector_type(6)));
typedef unsigned u32x16 __attribute__((ext_vector_type(16)));
typedef float f32x32 __attribute__((ext_vector_type(32)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef const void __attribute__((address_space(1))) *global_ptr;
typedef void __attribute__((address_space(3))) *lds_ptr;

constexpr int MP = 128, N = 256, HALF = MP / 2, TPG = N / 32, WAVES = 4, KS = 2, PARTS = 4;
constexpr int FRAG_BYTES = 1536;                 // one k-step of 64: sixteen bytes a lane, then eight
constexpr int TILE_BYTES = KS * FRAG_BYTES, REC_BYTES = TPG * TILE_BYTES;      // a record: one type
static_assert(REC_BYTES % (WAVES * 1024) == 0, "whole copies");

// Thirty-two numbers over 2^e (scale: 2^e) to e2m3, nearest even, and back.  The results must not share registers with
// the operands, which the instructions read while they write; the compiler's builtins do not say so.
__device__ __forceinline__ u32x6 to_fp6(const float *v, float scale)
{
    f32x16 even, odd;
#pragma unroll
    for (int e = 0; e < 16; ++e) { even[e] = v[2 * e]; odd[e] = v[2 * e + 1]; }
    u32x6 d;
    asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3" : "=&v"(d) : "v"(even), "v"(odd), "v"(scale));
    return d;
}
__device__ __forceinline__ f32x32 from_fp6(const u32x6 &p, float scale)
{
    f32x32 d;
    asm("v_cvt_scalef32_pk32_f32_fp6 %0, %1, %2" : "=&v"(d) : "v"(p), "v"(scale));
    return d;
}
// The payoffs of a fragment as bf16 (exact).
__device__ __forceinline__ u32x16 bf16_of_fp6(const u32x6 &p)
{
    u32x16 d;
    float one = 1.0f;
    asm("v_cvt_scalef32_pk32_bf16_fp6 %0, %1, %2" : "=&v"(d) : "v"(p), "v"(one));
    return d;
}
__device__ __forceinline__ i32x8 wide(const u32x6 &p)
{
    i32x8 r;
#pragma unroll
    for (int e = 0; e < 6; ++e) r[e] = (int)p[e];
    r[6] = r[7] = 0;
    return r;
}
// c += payoffs * row, the row's block scale in byte PART of `scales`
template <int PART> __device__ __forceinline__ f32x16 mfma_fp6(const i32x8 &payoffs, const u32x6 &x, const f32x16 &c, int scales)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(payoffs, wide(x), c, 2, 2, 0, 127, PART, scales);
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    const v2f ab = { a, b };
    return __builtin_bit_cast(unsigned, __builtin_convertvector(ab, v2bf));       // nearest, ties to even
}
__device__ __forceinline__ float bf16_lo(unsigned p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16_hi(unsigned p) { return __uint_as_float(p & 0xFFFF0000u); }

// What the instructions that go on with sums of full size lose: 2^-26 of the greatest of 65 terms each and 2^-24 of the
// sum are counted, two of them (the first parts' k-steps) and a sixteenth for those before; in |x|_2 |B_j|_2.  Measured
// on terms set to lose all they can, an instruction loses 5.1 2^-24 where this counts 17.25, which leaves room for second
// parts that come to more than a sixteenth of a row (to a third where one component of a block outweighs the others).
constexpr float kRounding = 2.125f * (65 * 0x1p-26f + 0x1p-24f);

// SLICED: workgroup row blockIdx.y walks its slice of the types and writes per-type outputs (see sweep_mfma.hip).
template <bool SLICED>
__global__ void __launch_bounds__(WAVES * 64, 2)
sweep_fp6_kernel(GameView g, SweepArgs a, int row_tiles)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // two stage buffers
    __shared__ float red_v[WAVES];
    __shared__ long long red_i[WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, col = lane & 31;
    const int m = g.m, K = g.K;
    const unsigned char *records = reinterpret_cast<const unsigned char *>(g.Bpack);
    const unsigned char *leaders = reinterpret_cast<const unsigned char *>(g.ATpack);
    const uniform_floats prior = (uniform_floats)g.prior;
    const long long wave_base = ((long long)blockIdx.x * WAVES + wave) * 32;
    const int begin = SLICED ? (int)blockIdx.y * a.slice_stages : 0;
    const int end = SLICED && begin + a.slice_stages < K ? begin + a.slice_stages : K;
    if (begin >= end) return;                            // whole workgroup
    (void)row_tiles;

    auto copy_stage = [&](int t) __attribute__((always_inline)) {
        const unsigned char *src = records + (size_t)t * REC_BYTES;
        unsigned char *dst = smem + (t & 1) * REC_BYTES;
#pragma unroll
        for (int i = 0; i < REC_BYTES / (WAVES * 1024); ++i) {
            const int chunk = i * WAVES + wave;
            __builtin_amdgcn_global_load_lds((global_ptr)(src + chunk * 1024 + lane * 16), (lds_ptr)(dst + chunk * 1024), 16, 0, 0);
        }
    };
    copy_stage(begin);

    // ---- the candidate row: the lane's half in fp32, its four parts, and what they leave
    const long long c = wave_base + col;
    const bool ok = c < a.count;                         // (past the end: the last row again)
    const unsigned valid32 = (unsigned)__builtin_amdgcn_ballot_w64(ok);
    float xf[HALF], reach, scale = 1.0f;                 // scale: of the row in its parts (leader payoffs take it as given)
    u32x6 x[KS][PARTS];
    int scales[KS];
    {
        load_half_row<HALF>(a.X + (ok ? c : a.count - 1) * (long long)m, h, m, xf);
        // The greatest component comes to 1 to 2 (2^-24 for the smallest numbers), so that rows of any size are alike, but
        // for those whose sums may be infinite, which are not for the parts.
        float row_most = 0.0f;
#pragma unroll
        for (int e = 0; e < HALF; ++e) row_most = fmaxf(row_most, fabsf(xf[e]));
        row_most = pair_max(row_most);
        const bool fits = (int)(__float_as_uint(row_most) >> 23) < g.any.row_end;
        const int up = 1 - __builtin_amdgcn_frexp_expf(row_most);
        if (fits) scale = __builtin_ldexpf(1.0f, up > 126 ? 126 : up < -126 ? -126 : up);
        float left = 0.0f, square = 0.0f;
        unsigned beyond = 0u;                            // what two parts leave of the row, any bit of it
        int least = 254;                                 // the smallest block's unit (a block of zeros has none)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            float r[32], most = 0.0f;
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                r[e] = xf[32 * s + e] * scale;
                most = fmaxf(most, fabsf(r[e]));
                square = fmaf(r[e], r[e], square);
            }
            // (blocks below 2^-90 have parts of zero and are all remainder)
            int ex = (int)(__float_as_uint(most) >> 23) - 1;             // biased exponent of the block's unit
            ex = ex < 37 ? 37 : ex > 187 ? 187 : ex;
            if (most > 0.0f) least = ex < least ? ex : least;
            scales[s] = ex | (ex - 5) << 8 | (ex - 10) << 16 | (ex - 15) << 24;
#pragma unroll
            for (int p = 0; p < PARTS; ++p) {
                const float unit = __uint_as_float((unsigned)(ex - 5 * p) << 23);
                x[s][p] = to_fp6(r, unit);
                const f32x32 back = from_fp6(x[s][p], unit);
#pragma unroll
                for (int e = 0; e < 32; ++e) r[e] -= back[e];            // exact
                if (p == 1)
#pragma unroll
                    for (int e = 0; e < 32; ++e) beyond |= __float_as_uint(r[e]) << 1;
            }
#pragma unroll
            for (int e = 0; e < 32; ++e) left = fmaf(r[e], r[e], left);
        }
        left = pair_sum(left); square = pair_sum(square);
        const float norm = __builtin_amdgcn_sqrtf(square);
        reach = fits ? __builtin_amdgcn_sqrtf(left) + kRounding * norm : INFINITY;
        // Rows that two parts hold are multiples of 2^-8 of their smallest block's unit, their products with payoffs of
        // 2^-11, and sums of these are exact while all terms together (7.5 |x|_1, |x|_1 <= sqrt(128) |x|_2) stay below
        // 2^24 of that (with room for the parts of one component having both signs): then the sums are the true ones.
        beyond = pair_or(beyond);
        const int other = __builtin_amdgcn_ds_bpermute(4 * (lane ^ 32), least);
        least = other < least ? other : least;
        if (fits && beyond == 0u && 90.0f * norm <= 0x1p13f * __uint_as_float((unsigned)least << 23)) reach = 0.0f;
    }

    // The lane's half of the row against its half of a leader column: two fp32 chains.
    auto leader_half = [&](const u32x4 *column) __attribute__((always_inline)) {
        float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int e = 0; e < HALF; e += 8) {
            const u32x4 w = column[e / 8];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f16x2 v = __builtin_bit_cast(f16x2, (unsigned)w[k]);
                l0 = fmaf(xf[e + 2 * k], (float)v[0], l0);
                l1 = fmaf(xf[e + 2 * k + 1], (float)v[1], l1);
            }
        }
        return l0 + l1;
    };
    auto column_of = [&](int t, int j) __attribute__((always_inline)) {
        return reinterpret_cast<const u32x4 *>(leaders + (((size_t)t * N + j) * MP + h * HALF) * 2);
    };
    // One row tile in three bf16 parts of the row, from its record in global memory: the first two in one sum, the
    // third in a sum of its own, as sweep_mfma.hip sums them.
    auto whole_tile = [&](int t, int tt) __attribute__((always_inline)) {
        f32x16 sum, rest;
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[e] = rest[e] = 0.0f;
        const unsigned char *tile = records + (size_t)t * REC_BYTES + tt * TILE_BYTES;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const u32x4 lo = *reinterpret_cast<const u32x4 *>(tile + s * FRAG_BYTES + lane * 16);
            const u32x2 hi = *reinterpret_cast<const u32x2 *>(tile + s * FRAG_BYTES + 1024 + lane * 8);
            const u32x6 f6 = { lo[0], lo[1], lo[2], lo[3], hi[0], hi[1] };
            const u32x16 b = bf16_of_fp6(f6);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                u32x4 p[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float va = xf[32 * s + 8 * k + 2 * e], vb = xf[32 * s + 8 * k + 2 * e + 1];
                    // (laundered: parts formed outside the loops would take the registers of the main path)
                    asm volatile("" : "+v"(va), "+v"(vb));
                    va *= scale; vb *= scale;
                    p[0][e] = pack_bf16(va, vb);
                    const float ra = va - bf16_lo(p[0][e]), rb = vb - bf16_hi(p[0][e]);
                    p[1][e] = pack_bf16(ra, rb);
                    p[2][e] = pack_bf16(ra - bf16_lo(p[1][e]), rb - bf16_hi(p[1][e]));
                }
                const u32x4 f = { b[4 * k], b[4 * k + 1], b[4 * k + 2], b[4 * k + 3] };
                const bf16x8 fb = __builtin_bit_cast(bf16x8, f);
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, __builtin_bit_cast(bf16x8, p[0]), sum, 0, 0, 0);
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, __builtin_bit_cast(bf16x8, p[1]), sum, 0, 0, 0);
                rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, __builtin_bit_cast(bf16x8, p[2]), rest, 0, 0, 0);
            }
        }
        return sum + rest;
    };
    unsigned tie_count = 0;                              // wave-uniform
    // The maximum of the whole sums in the candidate columns `multi`, over the row tiles `need`; returns the columns where
    // it is no unique one (sweep_mfma.hip).
    auto settle = [&](unsigned multi, unsigned need, int t, float &gmax, int &jstar) __attribute__((always_inline)) {
        float best = -INFINITY, w[16];
        unsigned btile = 0u;
        unsigned long long dup = 0ull;
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = -INFINITY;
#pragma unroll 1
        for (int tt = 0; tt < TPG; ++tt) {
            if (!(need >> tt & 1u)) continue;
            const f32x16 sum = whole_tile(t, tt);
            float u[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = sum[r];
            const float pm = vmax_chain16(-INFINITY, u);
            dup |= __builtin_amdgcn_ballot_w64(pm == best);
            keep_greater2(pm, (unsigned)(32 * tt), best, btile);
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = vmax2(w[r], u[r]);
        }
        const float gm = pair_max(best);
        const unsigned bm = bitmap16_pairs(w, gm), cnt = (unsigned)__builtin_popcount(bm), r = ffbh(bm) - 16u;
        const unsigned total = cnt ? (cnt << 16) | btile | ((r & 0xCu) << 1) | (r & 3u) | (4u * h) : 0u;
        const unsigned pair = pair_add_u32(total);
        if ((multi >> col) & 1u) { gmax = gm; jstar = (int)(pair & 0xFFFFu) & (N - 1); }
        return multi & ((unsigned)__builtin_amdgcn_ballot_w64((pair >> 16) != 1u) | (unsigned)(dup | (dup >> 32)));
    };
    // The maximisers of the whole sums, all of them in the row tiles `need`, in ascending order: the leader's payoff
    // decides, then the lower action.
    auto exact_type = [&](unsigned columns, unsigned need, int t, float gmax, float &l_out, int &j_out) __attribute__((always_inline)) {
        float lbest = kNotANumber;                       // (no maximiser: no sum is a number)
        int jbest = 0, nmatch = 0;
#pragma unroll 1
        for (int tt = 0; tt < TPG; ++tt) {
            if (!(need >> tt & 1u)) continue;
            const f32x16 sum = whole_tile(t, tt);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = 4 * q + rr, j = tt * 32 + acc_row_base(r) + 4 * hh;
                        const unsigned long long meq = __builtin_amdgcn_ballot_w64(sum[r] == gmax);
                        const unsigned hit = (unsigned)(hh ? (meq >> 32) : meq) & columns;
                        if (hit == 0u) continue;                               // wave-uniform
                        const float l = pair_sum(leader_half(column_of(t, j)));
                        if ((hit >> col) & 1u) {
                            if (nmatch == 0 || l > lbest) { lbest = l; jbest = j; }
                            ++nmatch;
                        }
                    }
        }
        if ((columns >> col) & 1u) { l_out = lbest; j_out = jbest; }
        tie_count += __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(nmatch >= 2));
    };

    float V = 0.0f;
    // The type before: its leader columns on their way, and the exact routine's answer in the columns `exact`.
    u32x4 column[HALF / 8];
    unsigned exact = 0u;
    float l_exact = 0.0f;
    int js = 0;
    const bool stores = SLICED || a.br_out;              // (vector stores count among the loads that a wait counts)
    auto finish = [&](int t) __attribute__((always_inline)) {
        float l = pair_sum(leader_half(column));
        if (exact != 0u && ((exact >> col) & 1u)) l = l_exact;
        V = fmaf(prior[t], l, V);
        if constexpr (SLICED) {
            if (h == 0 && ok) {
                a.l_out[c * a.l_sc + t * a.l_st] = l;
                if (a.br_out) a.br_out[c * a.br_sc + t * a.br_st] = js;
            }
        } else if (a.br_out) {
            if (h == 0 && ok) a.br_out[c * K + t] = js;
        }
    };

#pragma unroll 1
    for (int t = begin; t < end; ++t) {
        // The own copies of this stage have landed (behind them only the eight loads of a leader column are under way),
        // then everyone's, and everyone is done with the other buffer.
        if (t == begin || stores) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 1 < end) copy_stage(t + 1);
        const unsigned char *stage = smem + (t & 1) * REC_BYTES;
        float R[2 * TPG], C[8];
        // Two sets of fragments and of accumulators take turns: a tile's maxima and the next one's LDS reads run under
        // its successor's and its own matrix instructions.
        f32x16 acc[2];
        i32x8 f[2][KS];
        auto read = [&](int tt) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const unsigned char *p = stage + tt * TILE_BYTES + s * FRAG_BYTES;
                const u32x4 lo = *reinterpret_cast<const u32x4 *>(p + lane * 16);
                const u32x2 hi = *reinterpret_cast<const u32x2 *>(p + 1024 + lane * 8);
                const u32x6 f6 = { lo[0], lo[1], lo[2], lo[3], hi[0], hi[1] };
                f[tt & 1][s] = wide(f6);
            }
        };
        auto rows_of = [&](int tt) __attribute__((always_inline)) {
            float u[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = acc[tt & 1][r];
            vmax8x2(R[2 * tt], u, R[2 * tt + 1], u + 8);
        };
        auto columns_of = [&](int tt) __attribute__((always_inline)) {
            float u[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = acc[tt & 1][r];
            if (tt == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) C[e] = vmax2(u[e], u[e + 8]);
            } else {
                vmax_into8(C, u, u + 8);
            }
        };
        read(0);
        static_for<0, TPG, 1>([&](auto ttc) {
            constexpr int tt = decltype(ttc)::value, b = tt & 1;
            if constexpr (tt + 1 < TPG) read(tt + 1);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;
            // small parts first
            auto part = [&](auto pc) __attribute__((always_inline)) {
                constexpr int p = decltype(pc)::value;
#pragma unroll
                for (int s = 0; s < KS; ++s) acc[b] = mfma_fp6<p>(f[b][s], x[s][p], acc[b], scales[s]);
                __builtin_amdgcn_sched_barrier(0);
            };
            part(std::integral_constant<int, 3>{});
            part(std::integral_constant<int, 2>{});
            if constexpr (tt == 0) {
                if (t > begin) finish(t - 1);
            } else {
                // (four instructions of eight passes stand behind the last one of the tile before)
                asm volatile("" : "+v"(acc[b ^ 1]));
                rows_of(tt - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            part(std::integral_constant<int, 1>{});
            if constexpr (tt > 0) columns_of(tt - 1);
            __builtin_amdgcn_sched_barrier(0);
            part(std::integral_constant<int, 0>{});
        });
        // (the wait states between the last instruction and the asm below, which the compiler does not look into)
        asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[(TPG - 1) & 1]));
        rows_of(TPG - 1);
        columns_of(TPG - 1);
        const float most = vmax2(vmax3(vmax3(C[0], C[1], C[2]), vmax3(C[3], C[4], C[5]), C[6]), C[7]);
        float gmax = pair_max(most);
        const float floor = fmaf(-reach, prior[K + t], gmax);
        const unsigned map = pair_or(grid_map<TPG>(R, C, floor, 4u * h));
        js = (int)(grid_action<TPG>(map) & (N - 1));             // (any action where the column is not settled)
        const unsigned multi = (unsigned)__builtin_amdgcn_ballot_w64(__builtin_popcount(map) != 2);
        exact = 0u;
        if (multi != 0u) {
            // the tiles with a value from the threshold on, two grid rows each (columns without one take them all)
            unsigned need = 0u;
            const unsigned rows = (multi >> col) & 1u ? map >> (32 - 2 * TPG) : 0u;
#pragma unroll
            for (int k = 0; k < TPG; ++k)
                if (__builtin_amdgcn_ballot_w64((rows >> (2 * (TPG - 1 - k)) & 3u) != 0u) != 0ull) need |= 1u << k;
            if ((multi & (unsigned)__builtin_amdgcn_ballot_w64(rows == 0u)) != 0u) need = (1u << TPG) - 1u;
            const unsigned known = multi & (unsigned)__builtin_amdgcn_ballot_w64(reach == 0.0f);      // (maxima of true sums)
            exact = known;
            if (multi != known) exact |= settle(multi & ~known, need, t, gmax, js);
            exact &= valid32;
            if (exact != 0u) exact_type(exact, need, t, gmax, l_exact, js);
        }
        const u32x4 *from = column_of(t, js);
#pragma unroll
        for (int e = 0; e < HALF / 8; ++e) column[e] = from[e];
    }
    finish(end - 1);

    // ---- outputs
    float v = V == V ? V : -INFINITY;
    if (!SLICED && a.V_out && h == 0 && ok) a.V_out[c] = v;
    if (a.blk_v) {
        float bv = ok ? v : -INFINITY;
        long long bi = ok ? a.index_base + c : LLONG_MAX;
#pragma unroll
        for (int d = 16; d >= 1; d >>= 1) {              // both lane halves hold the same values
            const float ov = __shfl_xor(bv, d, 64);
            const long long oi = __shfl_xor(bi, d, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { red_v[wave] = bv; red_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < WAVES; ++w)
                if (red_v[w] > bv || (red_v[w] == bv && red_i[w] < bi)) { bv = red_v[w]; bi = red_i[w]; }
            a.blk_v[blockIdx.x] = bv;
            a.blk_i[blockIdx.x] = bi;
        }
    }
    if (a.tie_counter && lane == 0 && tie_count) atomicAdd(a.tie_counter, (unsigned long long)tie_count);
    if constexpr (SLICED)
        if (a.done.flag) signal_done(a.done, blockIdx.y * gridDim.x + blockIdx.x);
}

// e2m3 code of v, or -1: one sign bit, two of exponent, three of mantissa; eighths below 2, quarters below 4, halves
// up to 7.5.
// (from a table: which of the three spans a payoff is in no branch predictor knows)
struct Codes {
    signed char of[61];
    constexpr Codes() : of()
    {
        for (int q = 0; q <= 60; ++q) {
            const int e = q < 16 ? 0 : q < 32 ? 1 : 2;   // (below 1 the exponent field is 0, then 1)
            of[q] = (signed char)((q & ((1 << e) - 1)) != 0 ? -1 : e == 0 ? q : (e + 1) * 8 + ((q >> e) - 8));
        }
    }
};
constexpr Codes kCodes;
inline int fp6_code(double v)
{
    const double eighths = std::fabs(v) * 8.0;
    if (!(eighths <= 60.0)) return -1;
    const int q = (int)eighths;
    if ((double)q != eighths || kCodes.of[q] < 0) return -1;
    return kCodes.of[q] | (v < 0 ? 32 : 0);
}

// a + b, and whether that is the true sum (Knuth's two-sum leaves nothing over)
bool sum_is_exact(double a, double b, double *s)
{
    *s = a + b;
    const double back = *s - a;
    return (a - (*s - back)) + (b - back) == 0.0;
}

// The middle of the payoffs' range over the actions for each leader action of a type (mid[m]), and the power of two that
// brings what is left to 7.5 at most.
double type_scale(int m, const float *B, double *mid)
{
    double width = 0.0;
    for (int i = 0; i < m; ++i) {
        const float *row = B + (size_t)i * N;
        float lo = row[0], hi = row[0];
        for (int j = 1; j < N; ++j) { lo = row[j] < lo ? row[j] : lo; hi = row[j] > hi ? row[j] : hi; }
        mid[i] = 0.5 * ((double)lo + hi);
        width = std::fmax(width, (double)hi - mid[i]);
    }
    if (width == 0.0) return 1.0;
    int e;
    std::frexp(width / 7.5, &e);                         // width <= 7.5 * 2^e
    if (std::ldexp(7.5, e - 1) >= width) --e;
    return std::ldexp(1.0, -e);
}

}  // namespace

sweep_fn_t fp6_kernel(bool sliced) { return sliced ? sweep_fp6_kernel<true> : sweep_fp6_kernel<false>; }
int fp6_record_bytes() { return REC_BYTES; }

bool fp6_suits(int m, int n, int K, const float *A, const float *B)
{
    if (m > MP || n != N) return false;
    // leader payoffs have to be half-precision numbers, none of them subnormal
    auto half = [](float v) {
        const float w = std::fabs(v);
        uint32_t b; memcpy(&b, &v, 4);
        return v == 0.0f || (w >= 0x1p-14f && w <= 65504.0f && (b & 0x1FFFu) == 0u);
    };
    double mid[MP];
    for (int t = 0; t < K; ++t) {
        const float *Bt = B + (size_t)t * m * N, *At = A + (size_t)t * m * N;
        for (int i = 0; i < m * N; ++i)
            if (!half(At[i])) return false;
        const double scale = type_scale(m, Bt, mid);
        for (int i = 0; i < m; ++i) {
            // The codes have to be the payoffs less the middle, not what 53 bits leave of them: beside a payoff of -2^60
            // the numbers 0 to 7 are one and the same.  (Where no payoff but zero is below 2^-28 of the greatest, 53 bits
            // hold all: their last bits are 2^-23 of the least or more, the middle's half of that.  Asked of every payoff
            // the two-sums took 25 ms of m = 128, K = 256.)
            const float *row = Bt + (size_t)i * N;
            float lo = row[0], hi = row[0], least = INFINITY;
            for (int j = 0; j < N; ++j) {
                const float v = row[j], w = v == 0.0f ? INFINITY : std::fabs(v);
                lo = v < lo ? v : lo; hi = v > hi ? v : hi; least = w < least ? w : least;
            }
            const bool plain = least >= 0x1p-28f * std::fmax(std::fabs(lo), std::fabs(hi));
            double rest;
            if (!sum_is_exact(lo, hi, &rest)) return false;
            for (int j = 0; j < N; ++j) {
                if (plain) rest = row[j] - mid[i];
                else if (!sum_is_exact(row[j], -mid[i], &rest)) return false;
                if (fp6_code(rest * scale) < 0) return false;
            }
        }
    }
    return true;
}

// Fragments [type][row tile][k-step]: lane 32 h + r holds row r of the tile, leader actions 64 h + 32 s + 0..31, as 32
// codes of six bits, the first sixteen bytes of all lanes and then the last eight; leader payoffs [K][n][128] in half
// precision.
void fp6_pack(int m, int K, const float *A, const float *B, unsigned char *Bpack, unsigned short *ATpack)
{
    double mid[MP];
    for (int t = 0; t < K; ++t) {
        const float *Bt = B + (size_t)t * m * N;
        const double scale = type_scale(m, Bt, mid);
        for (int i = 0; i < m; ++i) {
            const int h = i / HALF, s = i % HALF / 32, bit = 6 * (i % 32);
            for (int j = 0; j < N; ++j) {
                const double v = (Bt[(size_t)i * N + j] - mid[i]) * scale;
                const unsigned code = (unsigned)fp6_code(v);
                unsigned char *frag = Bpack + (size_t)t * REC_BYTES + j / 32 * TILE_BYTES + s * FRAG_BYTES;
                const int lane = 32 * h + j % 32;
                for (int b = bit / 8; b <= (bit + 5) / 8; ++b) {
                    unsigned char *at = b < 16 ? frag + lane * 16 + b : frag + 1024 + lane * 8 + (b - 16);
                    const int shift = bit - 8 * b;
                    *at |= (unsigned char)(shift >= 0 ? code << shift : code >> -shift);
                }
            }
            for (int j = 0; j < N; ++j) {
                const _Float16 v = (_Float16)A[((size_t)t * m + i) * N + j];
                memcpy(&ATpack[((size_t)t * N + j) * MP + i], &v, 2);
            }
        }
    }
}

// margin[t]: a row of remainder r and rounding q (`reach` in the kernel: r + q) changes no difference of two payoffs by
// more than this times r + q, by Cauchy and Schwarz over both columns; 2 % for the roundings of the bound.
void fp6_margins(int m, int K, const float *B, float *margin)
{
    double mid[MP], square[N];
    for (int t = 0; t < K; ++t) {
        const float *Bt = B + (size_t)t * m * N;
        const double scale = type_scale(m, Bt, mid);
        for (int j = 0; j < N; ++j) square[j] = 0.0;
        for (int i = 0; i < m; ++i)
            for (int j = 0; j < N; ++j) {
                const double v = (Bt[(size_t)i * N + j] - mid[i]) * scale;
                square[j] += v * v;
            }
        double most = 0.0;
        for (int j = 0; j < N; ++j) most = std::fmax(most, square[j]);
        margin[t] = (float)(2.04 * std::sqrt(most));
    }
}

}  // namespace bsse
