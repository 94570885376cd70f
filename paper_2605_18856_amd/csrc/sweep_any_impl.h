// Fused sweep on the bf16 matrix cores for games of any shape with m <= 128 (not installed; one
// translation unit per TERMS instantiates it).
//
// The tile orientation, the partner-lane exchanges, the tie rule and the split of fp32 operands into
// bf16 parts are those of sweep_mfma.hip; what differs is that n and K are run-time numbers.
//   * The follower actions of a type are padded to whole row tiles.  A padded row never wins: its
//     accumulator starts at minus infinity (the C operand of the tile's first instruction) and its
//     payoffs are zero.
//   * FORM 0 (n > 128, and where no other suits) walks the row tiles of a type, one or two at a time (PAIRS), and keeps, per lane,
//     the eight column maxima of the tiles' grid over all of them and, for the tile or pair that holds
//     the running maximum, its number and its two or four row maxima; when the type is done a bit for
//     each that reaches the maximum names the action (unit_map).  Nothing depends on the number of
//     tiles, so registers do not grow with n.
//   * FORM 1 (16 < n <= 32) has one tile per type, a grid of four by four; FORM 2, 3 and 4 (n up to 64, 96
//     and 128) have two, three and four, side by side in registers.
//   * FORM 8 and FORM 16 (n <= 8, n <= 16) put four or two whole types into one row tile, the rows
//     permuted so that each lane holds every action of its types: no exchange is needed to find the
//     best response.  The leader payoffs of all the actions come off the matrix cores too and the one
//     at the best response is picked under the masks of the arg-max compares.
// The leader payoff of FORM 0 to 4 is an fp32 dot product (bf16 pairs in bf16 storage) with the
// column of A at the best response, from LDS where a whole type fits a stage, else from L2.
//
// Rows past the end of the candidates repeat the last one: they behave like any other row (no
// special case, no detour through the exact routine) and are left out of every output.
//
// A launch can be cut over the types (few candidates: workgroups walking all types would leave the chip
// idle): every workgroup then takes an equal share of the (block of candidates, unit) pairs, in order, and
// writes per-type leader payoffs; finish_rows_kernel sums them in type order, so a row's value has the
// same bits however the launch was cut.
#pragma once
#include "bsse_internal.h"
#include "mfma_device.h"
#include "done_device.h"
#include <limits.h>

namespace bsse {
namespace any_impl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef const void __attribute__((address_space(1))) *global_ptr;
typedef void __attribute__((address_space(3))) *lds_ptr;

constexpr int WAVES = 4, THREADS = WAVES * 64;

// Kernels of two kinds, for three workgroups on a compute unit (`many`) and for two: splits with two k-steps,
// which spill 15 to 29 registers at a block's start with three wavefronts a SIMD, and long bf16 rows, which
// have one candidate tile a wavefront with three and two with two.  The others have one kernel.
constexpr bool two_kinds(int terms, int ks, int form)
{
    return terms == 1 ? (ks == 6 && form == 0) || (ks == 8 && form < 3) : (form == 0 || form == 2) && ks == 2;
}
// Whether types of two, three or four row tiles keep them all in registers and in one stage (FORM 2, 3, 4): one wait
// for the matrix unit and one grid arg-max a type, and nothing carried from tile to tile.  Where it takes a wavefront
// one candidate tile in place of two, what it gives depends on the room that is left (1000000 rows, us, tile by tile
// and at once: m = 30, n = 50, K = 20 bf16 233 and 180; m = 60, n = 40, K = 20 651 and 584; m = 12, n = 90, K = 30
// bf16 393 and 297; m = 50, n = 100, K = 24 bf16, 600000 rows 386 and 330; m = 60, n = 66, K = 40, whole numbers,
// 300000 rows 474 and 407).  Not where it was slower: m = 55, n = 85, K = 24 bf16, 600000 rows 276 and 287; m = 45,
// n = 100, K = 20, 100003 rows 119 and 123, whole numbers 125 and 134; m = 30, n = 70, K = 20 618 and 639.
constexpr bool two_tiles(int terms, int ks) { return terms != 6 || ks <= 4; }
constexpr bool three_tiles(int terms, int ks) { return terms == 2 ? ks <= 4 : terms == 1 ? ks != 4 : terms == 3; }
constexpr bool four_tiles(int terms, int ks) { return terms == 1 || (terms == 3 && ks <= 2); }
// NT: 32-candidate tiles per wavefront.  Two let one fragment read serve two instructions; with
// three parts of a long row in registers there is room for one.
constexpr int tiles_per_wave(int terms, int ks, int form, bool many)
{
    if (form == 3 || form == 4) return 1;
    return ks <= (terms == 1 ? 4 : 2) || (terms == 1 && two_kinds(terms, ks, form) && !many) ? 2 : 1;
}
// Wavefronts per SIMD that the register allocation is held to; with one wavefront of every workgroup on each
// SIMD also the workgroups that a compute unit holds.  These kernels are bound by vector instructions, and a
// SIMD issues more of them the more wavefronts it chooses from (one, an instruction in 8 cycles; two, in 5.7;
// four, in 4.9): as many as fit without spilling in the loop over the types (row tiles one by one, us, 1000000 rows: m = 45,
// n = 100, K = 24 bf16 587 with two and 442 with three; m = 60, n = 100, K = 20, three products 1039 and 830).
constexpr int occupancy(int terms, int ks, int form, bool many)
{
    if (two_kinds(terms, ks, form)) return many ? 3 : 2;
    if (form == 3 || form == 4) return terms == 1 ? (ks <= 4 ? 4 : 3) : ks <= 2 ? 3 : 2;
    if (terms == 2) return ks == 1 && form == 1 ? 4 : ks <= 4 ? 3 : 2;
    if (form == 2 && terms == 1) return ks <= 2 ? 4 : 3;
    if (form == 0 || form == 2) return terms == 1 || ks <= 4 ? 3 : 2;
    if (form == 1) return terms == 1 ? (ks <= 4 ? 4 : 3) : ks == 1 ? 4 : ks <= 4 ? 3 : 2;
    return terms == 1 ? (ks <= 2 ? 4 : 3) : ks == 3 ? 4 : ks <= 4 ? 3 : 2;
}

// K-steps whose fragments are requested ahead of the one that is multiplied, as many as the registers hold (0: the
// compiler's order, as good with one row tile; half-precision parts have their own).
constexpr int fragments_ahead(int terms, int ks, int form, bool many)
{
    if (form < 2 || form >= 8 || terms == 2) return 0;
    if (terms == 1) return form != 4 ? 3 : ks == 3 ? 0 : ks == 6 ? 1 : 3;
    return (two_kinds(terms, ks, form) && many) || (terms == 6 && ks == 4) ? 0 : 1;
}

// The same within one row tile (FORM 0; us: m = 90, n = 150, K = 6 bf16, 300000 rows 130 and 122, 5000 rows 34.0 and
// 32.5; m = 50, n = 200, K = 12 bf16, 70001 rows 69 and 66; six products have enough to do meanwhile).
constexpr int tile_ahead(int terms, int ks, bool many)
{
    if (terms == 1) return ks < 4 ? ks - 1 : 3;
    return terms == 3 && (ks == 4 || (ks == 2 && !many)) ? 1 : 0;
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

// the nearest half-precision numbers, ties to even
__device__ __forceinline__ unsigned pack_half(float a, float b)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef _Float16 v2h __attribute__((ext_vector_type(2)));
    const v2f ab = { a, b };
    return __builtin_bit_cast(unsigned, __builtin_convertvector(ab, v2h));
}
__device__ __forceinline__ float half_of(unsigned p, int k)
{
    typedef _Float16 v2h __attribute__((ext_vector_type(2)));
    return (float)__builtin_bit_cast(v2h, p)[k];
}

__device__ __forceinline__ f32x16 mfma_half(const u32x4 &a, const unsigned *x, const f32x16 &c)
{
    const u32x4 b = { x[0], x[1], x[2], x[3] };
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma_bf16(const u32x4 &a, const unsigned *x, const f32x16 &c)
{
    const u32x4 b = { x[0], x[1], x[2], x[3] };
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The map of a type of several row tiles (grid_map's, over the columns of all its tiles and the rows of the
// one or two that lead): bits 16 to 27 stay free for the number of the leading tile.
constexpr unsigned kUnitTiles = 0xFFFu;
template <int ROWS> __device__ __forceinline__ unsigned unit_map(const float *R, const float *C, float floor, unsigned h4)
{
    unsigned r, c1, c0;
    if constexpr (ROWS == 4) {
        bits4x2<false, false>(r, R[0], R[1], R[2], R[3], c1, C[7], C[6], C[5], C[4], floor);
        c0 = bits4(C[3], C[2], C[1], C[0], floor);
    } else {
        bits4x2<false, false>(c1, C[7], C[6], C[5], C[4], c0, C[3], C[2], C[1], C[0], floor);
        r = (R[0] >= floor ? 2u : 0u) + (R[1] >= floor ? 1u : 0u);
    }
    return (r << (32 - ROWS)) | (((c1 << 8) | c0) << h4);
}

// Maximum of sixteen values.
__device__ __forceinline__ float vmax16(const float *u)
{
    const float a = vmax3(vmax3(u[0], u[1], u[2]), u[3], u[4]), b = vmax3(vmax3(u[8], u[9], u[10]), u[11], u[12]);
    const float c = vmax3(a, u[5], u[6]), d = vmax3(b, u[13], u[14]);
    return vmax2(vmax3(c, u[7], d), u[15]);
}

// Eight follower payoffs u against their maximum g with the leader payoffs w beside them, from the
// highest position down: l = w[j] wherever u[j] holds g, so that after the last block l belongs to the
// lowest position that does.  TOP: the first block of a chain (l starts as w[7]).  n_eq += how many
// (lane, position) pairs of the wavefront hold g.  Compare masks in scalar register pairs, counted on
// the scalar unit.
template <bool TOP>
__device__ __forceinline__ void argmax8_chain(const float *u, const float *w, float g, float &l, unsigned &n_eq)
{
    unsigned long long m0, m1, m2, m3, m4, m5, m6, m7;
    unsigned c, t;
    float lv = TOP ? w[7] : l;
#define BSSE_ACC(k) "s_bcnt1_i32_b64 %[t], %[m" #k "]\n\ts_add_u32 %[c], %[c], %[t]\n\t"
#define BSSE_SEL(k) "v_cndmask_b32 %[l], %[l], %[w" #k "], %[m" #k "]\n\t"
#define BSSE_CMP(k) "v_cmp_eq_f32 %[m" #k "], %[u" #k "], %[g]\n\t"
    if constexpr (TOP) {
        asm(BSSE_CMP(6) BSSE_CMP(5) BSSE_CMP(4) BSSE_CMP(3) BSSE_CMP(2) BSSE_CMP(1) BSSE_CMP(0) BSSE_CMP(7)
            BSSE_SEL(6) BSSE_SEL(5) BSSE_SEL(4) BSSE_SEL(3) BSSE_SEL(2) BSSE_SEL(1) BSSE_SEL(0)
            "s_bcnt1_i32_b64 %[c], %[m7]\n\t"
            BSSE_ACC(6) BSSE_ACC(5) BSSE_ACC(4) BSSE_ACC(3) BSSE_ACC(2) BSSE_ACC(1) BSSE_ACC(0)
            : [l] "+v"(lv), [c] "=&s"(c), [t] "=&s"(t), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2),
              [m3] "=&s"(m3), [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7)
            : [u0] "v"(u[0]), [u1] "v"(u[1]), [u2] "v"(u[2]), [u3] "v"(u[3]), [u4] "v"(u[4]), [u5] "v"(u[5]),
              [u6] "v"(u[6]), [u7] "v"(u[7]), [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]),
              [w4] "v"(w[4]), [w5] "v"(w[5]), [w6] "v"(w[6]), [g] "v"(g)
            : "scc");
    } else {
        asm(BSSE_CMP(7) BSSE_CMP(6) BSSE_CMP(5) BSSE_CMP(4) BSSE_CMP(3) BSSE_CMP(2) BSSE_CMP(1) BSSE_CMP(0)
            BSSE_SEL(7) BSSE_SEL(6) BSSE_SEL(5) BSSE_SEL(4) BSSE_SEL(3) BSSE_SEL(2) BSSE_SEL(1) BSSE_SEL(0)
            "s_bcnt1_i32_b64 %[c], %[m7]\n\t"
            BSSE_ACC(6) BSSE_ACC(5) BSSE_ACC(4) BSSE_ACC(3) BSSE_ACC(2) BSSE_ACC(1) BSSE_ACC(0)
            : [l] "+v"(lv), [c] "=&s"(c), [t] "=&s"(t), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2),
              [m3] "=&s"(m3), [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7)
            : [u0] "v"(u[0]), [u1] "v"(u[1]), [u2] "v"(u[2]), [u3] "v"(u[3]), [u4] "v"(u[4]), [u5] "v"(u[5]),
              [u6] "v"(u[6]), [u7] "v"(u[7]), [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]),
              [w4] "v"(w[4]), [w5] "v"(w[5]), [w6] "v"(w[6]), [w7] "v"(w[7]), [g] "v"(g)
            : "scc");
    }
#undef BSSE_ACC
#undef BSSE_SEL
#undef BSSE_CMP
    l = lv;
    n_eq += c;
}

// FIRST + ... of leaves FIRST to FIRST + COUNT (a power of two, of which the first LEAVES are there), two by two.
template <int FIRST, int COUNT, int LEAVES, class F> __device__ __forceinline__ double sum_of_eights(F &&leaf)
{
    if constexpr (COUNT == 1) return leaf(std::integral_constant<int, FIRST>{});
    else if constexpr (FIRST + COUNT / 2 >= LEAVES) return sum_of_eights<FIRST, COUNT / 2, LEAVES>(leaf);
    else {
        const double lower = sum_of_eights<FIRST, COUNT / 2, LEAVES>(leaf);
        return lower + sum_of_eights<FIRST + COUNT / 2, COUNT / 2, LEAVES>(leaf);
    }
}

// Folds `n` workgroup records (greatest value, lowest index among equals); every thread of the
// workgroup gets the result.
__device__ __forceinline__ void fold_records(const float *v, const long long *i, int n, float &bv, long long &bi)
{
    __shared__ float fv[WAVES];
    __shared__ long long fi[WAVES];
    bv = -INFINITY; bi = LLONG_MAX;
    for (int b = threadIdx.x; b < n; b += THREADS) {
        const float x = v[b];
        const long long k = i[b];
        if (x > bv || (x == bv && k < bi)) { bv = x; bi = k; }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const float ov = __shfl_xor(bv, d, 64);
        const long long oi = __shfl_xor(bi, d, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) { fv[threadIdx.x >> 6] = bv; fi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = fv[0]; bi = fi[0];
    for (int w = 1; w < WAVES; ++w)
        if (fv[w] > bv || (fv[w] == bv && fi[w] < bi)) { bv = fv[w]; bi = fi[w]; }
}

// Kernel arguments.  What the inner loop needs is read from the argument; everything else (outputs,
// records) through `late`, at the point of use: a pointer the compiler cannot see through keeps those
// fields out of the scalar registers of the loop, where they were spilled to vector lanes.
struct AnyArgs {
    GameView g;
    SweepArgs a;
};
typedef const AnyArgs __attribute__((address_space(4))) *late_args;
struct TypeOutput { unsigned c; int t; bool live; int32_t br; float l; };
__device__ __forceinline__ late_args late()
{
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (late_args)p;
}

// TERMS: 1 = operands rounded to bf16 (bf16 storage), 3 / 6 = fp32 operands as three bf16 parts
// against payoffs that are bf16 numbers / payoffs in three parts; 2 = fp32 operands as two half-precision
// parts each, three or four products of them (see any_half_suits).  KS: k-steps of 16 leader actions.
// FORM: see the top of the file.
template <int TERMS, int KS, int FORM, bool MANY>
__global__ void __launch_bounds__(THREADS, occupancy(TERMS, KS, FORM, MANY)) sweep_any_kernel(AnyArgs args)
{
    constexpr int NT = tiles_per_wave(TERMS, KS, FORM, MANY);
    constexpr bool FILTER = TERMS == 2;                  // values too near each other are summed in bf16 parts
    constexpr int XP = TERMS == 1 ? 1 : FILTER ? 2 : 3;  // parts of a candidate component
    constexpr int PA = TERMS == 6 ? 3 : FILTER ? 2 : 1;  // parts of a payoff
    constexpr int HALF = 8 * KS;                         // leader actions per lane half
    constexpr bool NARROW = FORM >= 8;
    static_assert(!(FILTER && NARROW), "leader payoffs off the matrix cores take all six products");
    constexpr bool XF = FILTER || (!NARROW && TERMS != 1 && KS <= 2);   // the fp32 half row stays in registers
    static_assert((FORM != 3 && FORM != 4) || NT == 1, "one wait names up to four accumulators");
    constexpr int WHOLE = FORM < 8 ? FORM : 0;           // row tiles of a type, where all are held at once
    constexpr int TPT = NARROW ? 32 / (NARROW ? FORM : 32) : 1;          // types per unit
    constexpr bool UNSCALE = XP == 3 && !XF;             // leader payoffs come from the split row: see load_rows
    constexpr bool PAIRS = FORM == 0 && TERMS == 1 && KS <= 2;      // row tiles two at a time: fewer vector instructions
                                                         // per tile where these outweigh the matrix time
    const AnyGeo &q = args.g.any;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // two stage buffers
    __shared__ float red_v[WAVES];
    __shared__ unsigned red_c[WAVES];
    __shared__ __attribute__((aligned(16))) float cinit[2][16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, col = lane & 31;
    const int partner_addr = 4 * (lane ^ 32);
    const int m = args.g.m, n = args.g.n, K = args.g.K;
    const unsigned count = (unsigned)args.a.count;       // <= 2^31 per launch
    const unsigned char *records = reinterpret_cast<const unsigned char *>(args.g.Bpack);
    const unsigned char *ATpack = reinterpret_cast<const unsigned char *>(args.g.ATpack);
    const uniform_floats prior = (uniform_floats)args.g.prior;
    const bool per_type = args.a.br_out || args.a.l_out; // per-type outputs are wanted
    constexpr unsigned PER_WG = WAVES * NT * 32;
    const unsigned nblk = (count + PER_WG - 1) / PER_WG;
    // Units [u0, u1) of block blk are worked on, `left` of them in all from there on.  Uncut: all units of
    // every gridDim.x-th block.  Cut: the workgroup's share of the pairs (block, unit); the first ones take
    // one more where the shares are not whole.  (There are at least as many pairs as workgroups.)
    unsigned blk = blockIdx.x, step = gridDim.x;
    int u0 = 0, left;
    if (const int share = args.a.slice_stages) {
        const int more = (int)nblk * q.units - share * (int)gridDim.x, w = (int)blockIdx.x;
        const int from = w * share + (w < more ? w : more);
        left = share + (w < more ? 1 : 0);
        blk = (unsigned)(from / q.units);
        u0 = from - (int)blk * q.units;
        step = 1u;
    } else {
        left = (int)((nblk - 1u - blk) / step + 1u) * q.units;
    }
    int u1 = u0 + left < q.units ? u0 + left : q.units;

    // a stage: `ups` whole units from `first` on (short of `end`), or (nq > 1) `stt` row tiles of one unit
    auto copy_stage = [&](int first, int end, int qq, int buf) __attribute__((always_inline)) {
        const unsigned char *src = records + (size_t)first * q.rec_bytes;
        int bytes;
        if (q.nq == 1) {
            const int nu = end - first < q.ups ? end - first : q.ups;
            bytes = nu * q.rec_bytes;
        } else {
            src += (size_t)qq * q.stt * q.tile_bytes;
            bytes = (q.tpg - qq * q.stt < q.stt ? q.tpg - qq * q.stt : q.stt) * q.tile_bytes;
        }
        unsigned char *dst = smem + buf * q.buf_bytes;
        for (int chunk = wave; chunk < (bytes >> 10); chunk += WAVES)
            __builtin_amdgcn_global_load_lds((global_ptr)(src + chunk * 1024 + lane * 16),
                                             (lds_ptr)(dst + chunk * 1024), 16, 0, 0);
    };
    copy_stage(u0, u1, 0, 0);

    // the one row of a fold launch: the winner among the records of an earlier launch
    const float *X = args.a.X;
    {
        const late_args p = late();
        if (p->a.fold_n > 0) {
            float bv;
            long long bi;
            fold_records(p->a.fold_v, p->a.fold_i, p->a.fold_n, bv, bi);
            const bool has = bi != LLONG_MAX;
            if (has) X += (bi - p->a.index_base) * m;
            if (blockIdx.x == 0 && tid == 0) {
                RunningBest r;
                r.value = has ? bv : 0.0f; r.has = has ? 1 : 0; r.index = has ? bi : -1; r.ties = *p->a.fold_ties;
                *p->a.fold_ties = 0ull;
                *p->a.fold_run = r;
            }
        }
        if (p->a.row_host && blockIdx.x == 0)
            for (int i = tid; i < m; i += THREADS) p->a.row_host[i] = X[i];
    }

    // C operand of the first instruction on a type's last row tile: minus infinity where the row is
    // padding (NARROW: in every tile, the row's action being its register index modulo FORM).  In LDS,
    // one copy per lane half, where sixteen registers are worth more than the reads.
    if (tid < 32) {
        const int r = tid & 15, hh = tid >> 4;
        cinit[hh][r] = (NARROW ? r % (FORM >= 8 ? FORM : 8) : (q.tpg - 1) * 32 + acc_row_base(r) + 4 * hh) < n ? 0.0f : -INFINITY;
    }
    const bool padded = NARROW ? n != FORM : n != 32 * q.tpg;

    unsigned x[NT][XP][KS * 4];
    float xf[NT][XF ? HALF : 1];
    float unscale[UNSCALE ? NT : 1];
    float norm[FILTER ? NT : 1];                         // of the row as it is split; infinite where the filter does not apply
    unsigned valid32[NT];
    [[maybe_unused]] unsigned zero32[NT];                // FILTER: valid rows of zeros
    // Rows of 16-byte multiples and others alike are read sixteen bytes a lane (the hardware asks for
    // four-byte alignment only); where a piece would reach past its row it is read ending with the row
    // and shifted.  All of a wavefront's pieces are requested before the first is used.  (Component by
    // component, k-step after k-step, the rows of m = 50 cost 128 requests of 64 lines each and eight
    // round trips per wavefront: 70001 rows, n = 100, K = 24 bf16, uncut: 105 -> 103 us; cut in five, each
    // slice reading the rows again: 93 -> 85.)
    // The parts of a component are exact from 2^-109 (they may be subnormal bf16 numbers) to the greatest
    // number (the first part does not round up to infinity).  A row whose greatest component is below
    // 2^-60 is split 2^64 times greater: its follower payoffs are compared with each other alone, and a
    // leader payoff that comes off the split row is scaled back.
    const bool vec4 = (m & 3) == 0;                      // no piece reaches past its row
    typedef f32x4 f32x4_dword __attribute__((aligned(4)));
    auto load_rows = [&](unsigned first) __attribute__((always_inline)) {
        // (laundered: the bounds masks are then formed here, not kept across the loop over blocks)
        int m_here = m;
        asm volatile("" : "+s"(m_here));
        const int m = m_here;
        float raw[NT][HALF];
        auto row_of = [&](int ct) __attribute__((always_inline)) {
            const unsigned c = first + ct * 32 + col;
            return X + (size_t)(c < count ? c : count - 1u) * m;
        };
        if (m >= 4) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const float *row = row_of(ct);
#pragma unroll
                for (int e = 0; e < HALF; e += 4) {
                    const int i = h * HALF + e;
                    const f32x4 t = *reinterpret_cast<const f32x4_dword *>(row + (i < m ? (i < m - 4 ? i : m - 4) : 0));
#pragma unroll
                    for (int k = 0; k < 4; ++k) raw[ct][e + k] = t[k];
                }
            }
            if (!vec4) {
#pragma unroll
                for (int ct = 0; ct < NT; ++ct)
#pragma unroll
                    for (int e = 0; e < HALF; e += 4) {
                        const int over = h * HALF + e + 4 - m;       // components past the end of the row
                        float (&r)[HALF] = raw[ct];
                        if (over == 1) { r[e] = r[e + 1]; r[e + 1] = r[e + 2]; r[e + 2] = r[e + 3]; }
                        if (over == 2) { r[e] = r[e + 2]; r[e + 1] = r[e + 3]; }
                        if (over == 3) { r[e] = r[e + 3]; }
                    }
            }
        } else {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const float *row = row_of(ct);
#pragma unroll
                for (int e = 0; e < HALF; ++e) raw[ct][e] = e < 4 ? row[e < m ? e : 0] : 0.0f;      // (m <= 3)
            }
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            valid32[ct] = (unsigned)__builtin_amdgcn_ballot_w64(first + ct * 32 + col < count);
            float scale = 1.0f;
            [[maybe_unused]] float rest = 1.0f;
            if constexpr (FILTER) {
                // the greatest component comes to 2^14 or more: what the parts leave of smaller ones is below 2^-39 of
                // it.  Rows that may have infinite sums are not for the filter.
                float most = 0.0f;
#pragma unroll
                for (int e = 0; e < HALF; ++e) most = fmaxf(most, fabsf(raw[ct][e]));
                most = fmaxf(most, pair_other(most, partner_addr));
                const int shift = 15 - __builtin_amdgcn_frexp_expf(most);      // (in two factors: 2^163 for the smallest)
                rest = shift > 64 ? 0x1p64f : 1.0f;
                scale = __builtin_ldexpf(1.0f, shift > 64 ? shift - 64 : shift);
                norm[ct] = (int)(__float_as_uint(most) >> 23) < late()->g.any.row_end ? 0.0f : INFINITY;
                bool zero = true;                        // (not from `most`, which passes over what is no number)
#pragma unroll
                for (int k = 0; k < HALF; ++k) zero = zero && !(h * HALF + k < m && raw[ct][k] != 0.0f);
                const unsigned long long zeros = __builtin_amdgcn_ballot_w64(zero);
                zero32[ct] = (unsigned)zeros & (unsigned)(zeros >> 32) & valid32[ct];
            }
            if constexpr (XP == 3) {
                float most = 0.0f;                       // (what `raw` holds past the row is of the row)
#pragma unroll
                for (int e = 0; e < HALF; ++e) most = fmaxf(most, fabsf(raw[ct][e]));
                most = fmaxf(most, pair_other(most, partner_addr));
                scale = most < 0x1p-60f ? 0x1p64f : 1.0f;
                if constexpr (UNSCALE) unscale[ct] = most < 0x1p-60f ? 0x1p-64f : 1.0f;
            }
#pragma unroll
            for (int e = 0; e < HALF; e += 2) {
                const int i = h * HALF + e, k = e / 2;
                float va = i < m ? raw[ct][e] : 0.0f, vb = i + 1 < m ? raw[ct][e + 1] : 0.0f;
                if constexpr (XF) { xf[ct][e] = va; xf[ct][e + 1] = vb; }
                if constexpr (XP == 3) { va *= scale; vb *= scale; }
                if constexpr (FILTER) {
                    va = va * scale * rest; vb = vb * scale * rest;
                    norm[ct] = fmaf(va, va, fmaf(vb, vb, norm[ct]));
                    const unsigned p = pack_half(va, vb);
                    x[ct][0][k] = p;
                    x[ct][XP - 1][k] = pack_half(va - half_of(p, 0), vb - half_of(p, 1));
                    continue;
                }
                constexpr float MOST = 0x1.FEp127f;      // the greatest bf16 number
                const unsigned p0 = XP == 3 ? pack_bf16(__builtin_amdgcn_fmed3f(va, -MOST, MOST), __builtin_amdgcn_fmed3f(vb, -MOST, MOST))
                                            : pack_bf16(va, vb);
                x[ct][0][k] = p0;
                if constexpr (XP == 3) {
                    // (the differences are exact: x = p0 + p1 + p2)
                    const float ra = va - bf16_lo(p0), rb = vb - bf16_hi(p0);
                    const unsigned p1 = pack_bf16(ra, rb);
                    x[ct][XP - 2][k] = p1;
                    x[ct][XP - 1][k] = pack_bf16(ra - bf16_lo(p1), rb - bf16_hi(p1));
                }
            }
            if constexpr (FILTER) norm[ct] = __builtin_amdgcn_sqrtf(norm[ct] + pair_other(norm[ct], partner_addr));
        }
    };

    // One row tile against the wavefront's candidate tiles: fragments [k-step][part][lane].  The order
    // of the products is fixed (small parts first within a k-step), so every way of reaching a tile
    // gives the same bits.
    // The C operand of a tile's first instruction.
    auto start_of = [&](f32x16 &c, bool last) __attribute__((always_inline)) {
        if (last) {
            const f32x4 *p = reinterpret_cast<const f32x4 *>(cinit[h]);
#pragma unroll
            for (int r = 0; r < 16; ++r) c[r] = p[r / 4][r % 4];
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) c[r] = 0.0f;
        }
    };
    // FILTER: small products first, beside which nothing is rounded that counts; the fragments of the great ones stay
    // in registers meanwhile (see any_half_suits for the number of products).  Candidate tiles [CT, CT + NTS).
    auto half_tiles = [&](auto ct0, auto nts, f32x16 *acc, auto fr, bool last) __attribute__((always_inline)) {
        constexpr int CT = decltype(ct0)::value, NTS = decltype(nts)::value;
#pragma unroll
        for (int ct = 0; ct < NTS; ++ct) start_of(acc[ct], last);
        u32x4 f0[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            f0[s] = fr[s * PA * 64];
            const u32x4 f1 = fr[(s * PA + PA - 1) * 64];
#pragma unroll
            for (int ct = 0; ct < NTS; ++ct) {
                if constexpr (KS == 3) acc[ct] = mfma_half(f1, &x[CT + ct][XP - 1][4 * s], acc[ct]);
                acc[ct] = mfma_half(f0[s], &x[CT + ct][XP - 1][4 * s], acc[ct]);
                acc[ct] = mfma_half(f1, &x[CT + ct][0][4 * s], acc[ct]);
            }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int ct = 0; ct < NTS; ++ct) acc[ct] = mfma_half(f0[s], &x[CT + ct][0][4 * s], acc[ct]);
    };
    auto tile_mfma = [&](f32x16 (&acc)[NT], auto fr, bool last) __attribute__((always_inline)) {
        if constexpr (FILTER) {
            half_tiles(std::integral_constant<int, 0>{}, std::integral_constant<int, NT>{}, acc, fr, last);
            return;
        }
        constexpr int HERE = NARROW || WHOLE > 0 ? 0 : tile_ahead(TERMS, KS, MANY);
        [[maybe_unused]] u32x4 ring[HERE + 1][PA];
        auto read = [&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i < KS)
#pragma unroll
                for (int p = 0; p < PA; ++p) ring[i % (HERE + 1)][p] = fr[(i * PA + p) * 64];
        };
        if constexpr (HERE > 0) static_for<0, HERE, 1>([&](auto ic) { read(ic); });
        static_for<0, KS, 1>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            u32x4 f[PA];
            if constexpr (HERE > 0) {
                read(std::integral_constant<int, s + HERE>{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < PA; ++p) f[p] = ring[s % (HERE + 1)][p];
            } else {
#pragma unroll
                for (int p = 0; p < PA; ++p) f[p] = fr[(s * PA + p) * 64];
            }
            auto product = [&](int pb, int px, bool first) __attribute__((always_inline)) {
                if (s == 0 && first) {
                    f32x16 zero;
#pragma unroll
                    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
                    if (last) {
                        const f32x4 *c = reinterpret_cast<const f32x4 *>(cinit[h]);
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
#pragma unroll
                            for (int r = 0; r < 16; ++r) acc[ct][r] = c[r / 4][r % 4];
                            acc[ct] = mfma_bf16(f[pb], &x[ct][px][4 * s], acc[ct]);
                        }
                    } else {
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) acc[ct] = mfma_bf16(f[pb], &x[ct][px][4 * s], zero);
                    }
                } else {
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) acc[ct] = mfma_bf16(f[pb], &x[ct][px][4 * s], acc[ct]);
                }
            };
            if constexpr (TERMS == 6) {
                product(2, 0, true); product(1, 1, false); product(0, 2, false);
                product(1, 0, false); product(0, 1, false); product(0, 0, false);
            } else if constexpr (TERMS == 3) {
                product(0, 2, true); product(0, 1, false); product(0, 0, false);
            } else {
                product(0, 0, true);
            }
            if constexpr (HERE > 0) __builtin_amdgcn_sched_barrier(0);
        });
    };
    // All row tiles of a type at once (FORM 2 to 4), in the same order.  The fragments of AHEAD k-steps are under way
    // while one is multiplied, in the order written: left to the compiler, which saves registers, every matrix
    // instruction waited for a read of LDS issued just before it (us: m = 50, n = 100, K = 24 bf16, 300000 rows 182 and
    // 173, 70001 rows 71.5 and 69.8; m = 90, n = 80, K = 10 bf16 118 and 112; m = 60, n = 40, K = 20, whole numbers,
    // 1000000 rows 435 and 424; up to 32 actions and with six products it makes no difference).
    constexpr int AHEAD = fragments_ahead(TERMS, KS, FORM, MANY);
    auto whole_mfma = [&](f32x16 (&acc)[WHOLE ? WHOLE : 1][NT], auto fr) __attribute__((always_inline)) {
        constexpr int STEPS = WHOLE * KS, RING = AHEAD + 1;
        u32x4 f[RING][PA];
        auto read = [&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i < STEPS)
#pragma unroll
                for (int p = 0; p < PA; ++p) f[i % RING][p] = fr[(i * PA + p) * 64];
        };
        static_for<0, AHEAD, 1>([&](auto ic) { read(ic); });
        static_for<0, STEPS, 1>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value, tt = i / KS, s = i % KS;
            read(std::integral_constant<int, i + AHEAD>{});
            if constexpr (s == 0)
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) start_of(acc[tt][ct], tt == WHOLE - 1);
            __builtin_amdgcn_sched_barrier(0);
            auto product = [&](int pb, int px) __attribute__((always_inline)) {
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) acc[tt][ct] = mfma_bf16(f[i % RING][pb], &x[ct][px][4 * s], acc[tt][ct]);
            };
            if constexpr (TERMS == 6) {
                product(PA - 1, 0); product(1 % PA, 1 % XP); product(0, XP - 1);
                product(1 % PA, 0); product(0, 1 % XP); product(0, 0);
            } else if constexpr (TERMS == 3) {
                product(0, XP - 1); product(0, 1 % XP); product(0, 0);
            } else {
                product(0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // The asm blocks below read accumulators, and the compiler's hazard handling does not look into
    // inline asm: the wait states a vector read of a fresh MFMA result needs are explicit, with the
    // accumulators as operands so that nothing that reads them can be scheduled above the wait.
    auto settle = [&](f32x16 (&acc)[NT]) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NT == 2) asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0]), "+v"(acc[NT - 1]));
        else asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0]));
    };

    float V[NT];
    unsigned tie_count = 0;                              // wave-uniform
    float best_v = -INFINITY;
    unsigned best_c = 0xFFFFFFFFu;

    // the lane's half of the candidate row against its half of leader column (t, j); two chains
    auto half_dot = [&](int ct, auto column) __attribute__((always_inline)) {
        float l0 = 0.0f, l1 = 0.0f;
        if constexpr (TERMS == 1) {
            u32x4 cr[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) cr[s] = column[s];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const unsigned w0 = cr[s][0], w1 = cr[s][1], w2 = cr[s][2], w3 = cr[s][3];
                asm volatile("v_dot2c_f32_bf16 %0, %2, %6\n\t"
                             "v_dot2c_f32_bf16 %1, %3, %7\n\t"
                             "v_dot2c_f32_bf16 %0, %4, %8\n\t"
                             "v_dot2c_f32_bf16 %1, %5, %9"
                             : "+v"(l0), "+v"(l1)
                             : "v"(x[ct][0][4 * s]), "v"(x[ct][0][4 * s + 1]), "v"(x[ct][0][4 * s + 2]),
                               "v"(x[ct][0][4 * s + 3]), "v"(w0), "v"(w1), "v"(w2), "v"(w3));
            }
            // (three wait states between a dot result and another kind of vector instruction)
            asm volatile("s_nop 2" : "+v"(l0), "+v"(l1));
        } else {
#pragma unroll
            for (int e = 0; e < HALF; e += 4) {
                const u32x4 raw = column[e / 4];
                const f32x4 r = __builtin_bit_cast(f32x4, raw);
                float v[4];
                if constexpr (XF) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = xf[ct][e + k];
                } else {
                    // the component from its three parts, exact: p1 + p2 is what p0 left of it
#pragma unroll
                    for (int k = 0; k < 4; k += 2) {
                        const unsigned p0 = x[ct][0][(e + k) / 2], p1 = x[ct][XP - 2][(e + k) / 2], p2 = x[ct][XP - 1][(e + k) / 2];
                        v[k] = bf16_lo(p0) + (bf16_lo(p1) + bf16_lo(p2));
                        v[k + 1] = bf16_hi(p0) + (bf16_hi(p1) + bf16_hi(p2));
                    }
                }
                l0 = fmaf(v[0], r[0], l0); l1 = fmaf(v[1], r[1], l1);
                l0 = fmaf(v[2], r[2], l0); l1 = fmaf(v[3], r[3], l1);
            }
        }
        return l0 + l1;
    };
    constexpr int LBYTES = TERMS == 1 ? 2 : 4;           // bytes of a leader payoff
    auto lead_global = [&](int t, int j) __attribute__((always_inline)) {
        return reinterpret_cast<const u32x4 *>(ATpack + (((size_t)t * n + j) * (2 * HALF) + h * HALF) * LBYTES);
    };
    auto pair_total = [&](int ct, float part) __attribute__((always_inline)) {
        const float other = pair_other(part, partner_addr);
        const float l = h ? other + part : part + other; // (lower half) + (upper half)
        return UNSCALE ? l * unscale[UNSCALE ? ct : 0] : l;
    };

    // Per-type outputs of type t of candidate c.  Everything the stores need is read at once: pointers and
    // strides one after another, each behind its own wait, held a wavefront up eight times a type (m = 50,
    // n = 100, K = 24 bf16, 70001 rows: 77.3 -> 74.5 us).
    auto put_type = [&](auto n_outputs, auto output) __attribute__((always_inline)) {
        const late_args o = late();
        int32_t *const br_out = o->a.br_out;
        float *const l_out = o->a.l_out;
        const long long l_sc = o->a.l_sc, l_st = o->a.l_st, br_sc = o->a.br_sc, br_st = o->a.br_st;
#pragma unroll
        for (int k = 0; k < decltype(n_outputs)::value; ++k) {
            const TypeOutput v = output(k);
            if (v.live && br_out) br_out[(size_t)v.c * br_sc + v.t * br_st] = v.br;
            if (v.live && l_out) l_out[(size_t)v.c * l_sc + v.t * l_st] = v.l;
        }
    };

    // Exact routine for one (candidate tile, type) of FORM 0 to 4: the type's tiles once more from the
    // records in global memory (same instructions, same bits), the exact maximisers in ascending
    // action order; the leader's payoff decides and then the lower action.  Sums of minus infinity, and sums
    // that are not numbers, count as the least finite number here: where a row has no others, all of its
    // actions are maximisers and its leader payoffs say what the row is worth.
    auto exact_type = [&](int ct, int t, float gm, float &l_out, int &j_out) __attribute__((always_inline)) {
        constexpr float LEAST = -3.402823466e38f;
        const float gmax = fmaxf(gm, LEAST);
        float lbest = 0.0f;
        int jbest = 0, nmatch = 0;
#pragma unroll 1
        for (int tt = 0; tt < q.tpg; ++tt) {
            f32x16 acc[NT];
            tile_mfma(acc, reinterpret_cast<const u32x4 *>(records + (size_t)t * q.rec_bytes + (size_t)tt * q.tile_bytes) + lane,
                      padded && tt == q.tpg - 1);
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = 4 * q4 + rr;
                        const int j = tt * 32 + acc_row_base(r) + 4 * hh;
                        const unsigned long long meq = __builtin_amdgcn_ballot_w64(fmaxf(acc[ct][r], LEAST) == gmax);
                        const unsigned hit = (unsigned)(hh ? (meq >> 32) : meq);
                        if (hit == 0u || j > n - 1) continue;               // wave-uniform
                        const float l = pair_total(ct, half_dot(ct, lead_global(t, j)));
                        if ((hit >> col) & 1u) {
                            if (nmatch == 0 || l > lbest) { lbest = l; jbest = j; }
                            ++nmatch;
                        }
                    }
        }
        l_out = lbest; j_out = jbest;
        tie_count += __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(nmatch >= 2 && gmax > LEAST) & valid32[ct]);
    };

    // FILTER: what the sums in 64 bits of a row with greatest component `most` are multiplied with before they are rounded:
    // those of a row below 2^-60 do not end as subnormal numbers (the six products split such rows 2^64 times greater).
    constexpr float kTinyRow = 0x1p-60f;
    auto rounded_up = [](float most) __attribute__((always_inline)) { return most < kTinyRow ? 0x1p64f : 1.0f; };
    auto from_lane = [](double v, auto lanes) __attribute__((always_inline)) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)u, decltype(lanes)::value, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), decltype(lanes)::value, 0xf, 0xf, false);
        return __builtin_bit_cast(double, (unsigned long long)(unsigned)hi << 32 | (unsigned)lo);
    };
    // FILTER: the best responses of the candidate columns `columns`, where several values are within the margin of the
    // maximum, by the same rule.  The half-precision sums once more say which actions they are (from `floor` on, in any of
    // the columns); their sums are taken in 64 bits and rounded once.  For ties, and where many columns come at once.
    auto exact_actions = [&](auto ctc, unsigned columns, int t, float gm, float floor, const u32x4 *fr, int &j_out) __attribute__((always_inline)) {
        constexpr int ct = decltype(ctc)::value;
        constexpr float LEAST = -3.402823466e38f;
        const bool mine = (columns >> col) & 1u;
        if (!(gm > LEAST)) floor = -INFINITY;            // (nothing but minus infinity and no numbers: every action)
        const float *payoffs = reinterpret_cast<const float *>(records + (size_t)q.units * q.rec_bytes) + (size_t)t * n * (2 * HALF);
        float cur = LEAST;
        int jbest = 0, nmatch = 0;
#pragma unroll 1
        for (int tt = 0; tt < q.tpg; ++tt) {
            f32x16 acc;
            half_tiles(ctc, std::integral_constant<int, 1>{}, &acc, fr + (size_t)tt * (PA * KS * 64), padded && tt == q.tpg - 1);
            __builtin_amdgcn_sched_barrier(0);
            unsigned near = 0u;                          // a bit for each row of the tile, as rows are numbered
#pragma unroll
            for (int r = 0; r < 16; ++r) near |= acc[r] < floor ? 0u : 1u << acc_row_base(r);
            near = mine ? near << (4 * h) : 0u;
            if (__builtin_amdgcn_ballot_w64(near != 0u) == 0ull) continue;
            const unsigned own = pair_or(near);          // a column weighs its own, whatever is near in the others
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) near |= (unsigned)__shfl_xor((int)near, d, 64);
            if (n - tt * 32 < 32) near &= (1u << (n - tt * 32)) - 1u;
#pragma unroll 1
            for (unsigned rest = (unsigned)__builtin_amdgcn_readfirstlane((int)near); rest != 0u; rest &= rest - 1u) {
                const int j = tt * 32 + __builtin_ctz(rest);
                // (the payoffs in one request, spread over the lanes; eight after eight by every lane, a round trip each, a tie
                // held a short launch up by another 6 us: m = 128, n = 32, K = 6, 10000 rows 35.0 -> 29.3, 25 without one)
                const float *b = payoffs + (size_t)j * (2 * HALF);
                const int at = lane < HALF ? lane : HALF - 1;
                const float b0 = b[at], b1 = b[HALF + at];
                float most = 0.0f;
                // (laundered, and eight at a time: numbers in 64 bits kept across the loop would take the main path's registers)
                const double sum = sum_of_eights<0, HALF <= 32 ? 4 : 8, HALF / 8>([&](auto leaf) __attribute__((always_inline)) {
                    constexpr int e = 8 * decltype(leaf)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    double eight = 0.0;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        float xe = xf[ct][XF ? e + k : 0];
                        asm volatile("" : "+v"(xe));
                        most = fmaxf(most, fabsf(xe));
                        const unsigned lower = __builtin_amdgcn_readlane(__float_as_uint(b0), e + k), upper = __builtin_amdgcn_readlane(__float_as_uint(b1), e + k);
                        eight = fma((double)xe, (double)__uint_as_float(h ? upper : lower), eight);
                    }
                    return eight;
                });
                const float up = rounded_up(fmaxf(most, pair_other(most, partner_addr)));
                const float u = fmaxf((float)((sum + __shfl_xor(sum, 32, 64)) * (double)up), LEAST);      // (the same in both lanes)
                const bool weighs = (own >> (j & 31)) & 1u;
                if (weighs && u > cur) { cur = u; nmatch = 0; }
                const bool equal = weighs && u == cur, again = equal && nmatch > 0;
                bool better = equal && nmatch == 0;
                if (__builtin_amdgcn_ballot_w64(again) != 0ull) {
                    const float l0 = pair_total(ct, half_dot(ct, lead_global(t, jbest))), l1 = pair_total(ct, half_dot(ct, lead_global(t, j)));
                    better = better || (again && l1 > l0);
                }
                if (equal) ++nmatch;
                if (better) jbest = j;
            }
        }
        if (mine) j_out = jbest;
        tie_count += __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(nmatch >= 2 && cur > LEAST) & columns);
    };

    // FILTER: one candidate column by the same sums, over the actions that the maps of its two lanes leave open (FORM 0:
    // in all row tiles where a bit of `units` says that a lane has several): an answer if one of them alone has the
    // greatest, else -1.  A column in 250 or 100 comes here, in short launches the last wavefront of them all, so what
    // counts is the chain of latencies and the code, which is cold: sixteen lanes hold the row and an action's payoffs,
    // eight components each, and four actions go side by side.  (All actions of the type in the lanes, each lane along
    // its own, were sixteen round trips where n = 255, us: m = 128, n = 255, K = 4, 1000 rows 38.2 -> 32.2, 30000 rows 71.6
    // -> 58.7; m = 128, n = 100, K = 10, 3000 rows 29.4 -> 26.1; m = 50, n = 90, K = 2, 10000 rows 22.1 -> 20.2; m = 60,
    // n = 100, K = 20, 30000 rows 61.6 -> 59.6; exact_actions for every column 58 where that took 49, 20000 rows.)
    auto exact_column = [&](unsigned c, int t, unsigned map0, unsigned map1, unsigned units) __attribute__((always_inline)) {
        constexpr float LEAST = -3.402823466e38f;
        int lane_here = lane;                            // (laundered: what follows from it is not kept across the main loop)
        asm volatile("" : "+v"(lane_here));
        const int lane = lane_here, leaf = lane & 7, i0 = leaf < HALF / 8 ? (lane >> 3 & 1) * HALF + 8 * leaf : 2 * HALF;
        typedef f32x4 f32x4_dword __attribute__((aligned(4)));
        const float *row = X + (size_t)(c < count ? c : count - 1u) * m;
        // (a piece that would reach past the row ends with it, and counts from where it should have begun)
        int from[2];
        float xe[2][4], most = 0.0f;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int i = i0 + 4 * p;
            from[p] = i < m - 4 ? i : m - 4;
            const f32x4 r = *reinterpret_cast<const f32x4_dword *>(row + from[p]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                xe[p][k] = from[p] + k < i ? 0.0f : r[k];
                most = fmaxf(most, fabsf(xe[p][k]));
            }
        }
        const float up = rounded_up(__builtin_amdgcn_ballot_w64(most >= kTinyRow) != 0ull ? kTinyRow : 0.0f);
        const float *payoffs = reinterpret_cast<const float *>(records + (size_t)q.units * q.rec_bytes) + (size_t)t * n * (2 * HALF);
        float best = -INFINITY;                          // of the actions that the sixteen lanes had
        int jbest = 0;
        bool again = false;
#pragma unroll 1
        for (int j0 = 0; j0 < n; j0 += 64) {
            const int jl = j0 + lane;
            const unsigned map = jl & 4 ? map1 : map0;
            bool open;
            if constexpr (FORM == 0) open = (map >> (jl & 15) & 1u) != 0u && ((units >> (jl >> 2 & 1) & 1u) != 0u || ((map >> 16 & kUnitTiles) == (unsigned)jl >> 5 && (map >> (31 - (jl >> 4 & 1)) & 1u) != 0u));
            else if constexpr (FORM == 1) open = jl < 32 && (map0 >> (31 - (jl >> 3 & 31)) & map0 >> (jl & 7) & 1u) != 0u;
            else open = (map0 >> (31 - (jl >> 4 & 31)) & map0 >> (jl & 15) & 1u) != 0u;
            unsigned long long rest = __builtin_amdgcn_ballot_w64(open && jl < n);
#pragma unroll 1
            while (rest != 0ull) {
                int j = -1;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const int next = rest != 0ull ? j0 + __builtin_ctzll(rest) : -1;
                    rest &= rest - 1ull;
                    j = lane >> 4 == a ? next : j;
                }
                const float *b = payoffs + (size_t)(j < 0 ? 0 : j) * (2 * HALF);
                const f32x4 b0 = *reinterpret_cast<const f32x4_dword *>(b + from[0]), b1 = *reinterpret_cast<const f32x4_dword *>(b + from[1]);
                double sum = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) sum = fma((double)xe[k / 4][k % 4], (double)(k < 4 ? b0 : b1)[k % 4], sum);
                // (both partners add the same two: pairs, fours and eights of lanes by their order in the row)
                sum += from_lane(sum, std::integral_constant<int, 0xB1>{});      // quad_perm 1 0 3 2
                sum += from_lane(sum, std::integral_constant<int, 0x4E>{});      // quad_perm 2 3 0 1
                sum += from_lane(sum, std::integral_constant<int, 0x141>{});     // the other four of eight
                sum += from_lane(sum, std::integral_constant<int, 0x140>{});     // the other half of the row
                const float u = fmaxf((float)(sum * (double)up), LEAST);
                again = j >= 0 ? u == best || (again && u < best) : again;
                if (j >= 0 && u > best) { best = u; jbest = j; }
            }
        }
        auto of = [&](int l) __attribute__((always_inline)) { return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(best), l)); };
        const float greatest = fmaxf(fmaxf(of(0), of(16)), fmaxf(of(32), of(48)));
        const unsigned long long at = __builtin_amdgcn_ballot_w64(best == greatest), twice = __builtin_amdgcn_ballot_w64(best == greatest && again);
        const int j = __builtin_amdgcn_readlane(jbest, (int)__builtin_ctzll(at | 1ull << 63));
        return greatest > LEAST && twice == 0ull && __builtin_popcountll(at) == 16 ? j : -1;
    };

    int buf = 0;
    for (;;) {
        const int nsu = (u1 - u0 + q.ups - 1) / q.ups;   // groups of units, nq stages each
        const unsigned first = (blk * WAVES + wave) * (NT * 32);
        load_rows(first);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) V[ct] = 0.0f;
        // state of the type in progress (FORM 0)
        // (a unit is one row tile, or two at a time: its grid rows as far as they hold the best value so far,
        // and the columns over all units)
        constexpr int UNIT = PAIRS ? 2 : 1;
        typedef ArgGrid<WHOLE == 3 ? 4 : WHOLE ? WHOLE : 2> Grid;
        constexpr int ROWS = WHOLE ? Grid::ROWS : 2 * UNIT;
        float best[NT], R[NT][ROWS], C[NT][Grid::COLS];
        unsigned btile[NT];
        [[maybe_unused]] unsigned long long dup[NT];
        [[maybe_unused]] float second[NT];               // FILTER: the greatest maximum of a unit beside the leading one's

#pragma unroll 1
        for (int su = 0; su < nsu; ++su) {
#pragma unroll 1
            for (int qq = 0; qq < q.nq; ++qq) {
                // own copies of this stage have landed; then everyone's have, and everyone is done with
                // the other buffer, which takes the next stage
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                {
                    int su2 = su, qq2 = qq + 1;
                    if (qq2 == q.nq) { qq2 = 0; ++su2; }
                    if (su2 < nsu) copy_stage(u0 + su2 * q.ups, u1, qq2, buf ^ 1);
                    else if (const int rest = left - (u1 - u0)) copy_stage(0, rest < q.units ? rest : q.units, 0, buf ^ 1);
                }
                const unsigned char *sb = smem + buf * q.buf_bytes;
                buf ^= 1;
                const int ub = u0 + su * q.ups;
                const int nu = u1 - ub < q.ups ? u1 - ub : q.ups;
#pragma unroll 1
                for (int ui = 0; ui < nu; ++ui) {
                    const int u = ub + ui;
                    const u32x4 *fr = reinterpret_cast<const u32x4 *>(sb + ui * q.rec_bytes) + lane;
                    if constexpr (NARROW) {
                        f32x16 uf[NT], wl[NT];
                        tile_mfma(uf, fr, padded);
                        tile_mfma(wl, fr + PA * KS * 64, false);
                        settle(uf); settle(wl);
                        constexpr int PT = TPT / 2;      // types per lane
                        float gm[NT][PT], l[NT][PT];
                        unsigned n_eq = 0;
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
                            float uu[16], ww[16];
#pragma unroll
                            for (int r = 0; r < 16; ++r) { uu[r] = uf[ct][r]; ww[r] = wl[ct][r]; }
                            if constexpr (FORM == 16) {
                                gm[ct][0] = vmax16(uu);
                                argmax8_chain<true>(uu + 8, ww + 8, gm[ct][0], l[ct][0], n_eq);
                                argmax8_chain<false>(uu, ww, gm[ct][0], l[ct][0], n_eq);
                            } else {
#pragma unroll
                                for (int p = 0; p < PT; ++p) {
                                    const float *v = uu + 8 * (p & 1);
                                    gm[ct][p] = vmax2(vmax3(vmax3(vmax3(v[0], v[1], v[2]), v[3], v[4]), v[5], v[6]), v[7]);
                                    argmax8_chain<true>(v, ww + 8 * (p & 1), gm[ct][p], l[ct][p], n_eq);
                                }
                            }
                        }
                        unsigned js[NT][PT];
                        const bool exact = n_eq != 64u * NT * PT;          // wave-uniform
                        if (exact || per_type) {
                            // several maximisers in some lane (or none), or the action itself is wanted:
                            // maximisers in ascending order, the leader's payoff decides, then the lower
                            // action; a lane with one maximiser keeps what it had
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct)
#pragma unroll
                                for (int p = 0; p < PT; ++p) {
                                    float lbest = kNotANumber;      // (no sum is a number)
                                    unsigned jbest = 0;
                                    int nm = 0;
#pragma unroll
                                    for (int j = 0; j < (FORM == 16 ? 16 : 8); ++j)
                                        if (uf[ct][8 * p + j] == gm[ct][p] && j < n) {
                                            const float lj = wl[ct][8 * p + j];
                                            if (nm == 0 || lj > lbest) { lbest = lj; jbest = (unsigned)j; }
                                            ++nm;
                                        }
                                    l[ct][p] = lbest; js[ct][p] = jbest;
                                    const bool live = TPT * u + PT * h + p < K && ((valid32[ct] >> col) & 1u) && gm[ct][p] > -INFINITY;
                                    tie_count += __builtin_popcountll(__builtin_amdgcn_ballot_w64(live && nm >= 2));
                                }
                        }
                        // the value in type order: the partner lane holds the other half's types
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
                            float lo[PT];
                            if constexpr (UNSCALE)
#pragma unroll
                                for (int p = 0; p < PT; ++p) l[ct][p] *= unscale[UNSCALE ? ct : 0];
#pragma unroll
                            for (int p = 0; p < PT; ++p) lo[p] = pair_other(l[ct][p], partner_addr);
#pragma unroll
                            for (int k = 0; k < TPT; ++k) {
                                const int t = TPT * u + k;
                                if (t >= K) break;       // (uniform; a padded type's payoff may be infinite)
                                const float lk = (k / PT == h) ? l[ct][k % PT] : lo[k % PT];
                                V[ct] = fmaf(prior[t], lk, V[ct]);
                            }
                        }
                        if (per_type)
                            put_type(std::integral_constant<int, NT * PT>{}, [&](int k) __attribute__((always_inline)) {
                                const int ct = k / PT, p = k % PT, t = TPT * u + PT * h + p;
                                const unsigned c = first + ct * 32 + col;
                                return TypeOutput{ c, t, c < count && t < K, (int32_t)js[ct][p], l[ct][p] };
                            });
                    } else {
                        // ---- FORM 0 to 4: one type
                        if (qq == 0) {
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct) {
                                // (not minus infinity: a lane whose rows of a tile are all padding must
                                // not count as a tie with the start value)
                                best[ct] = second[ct] = -3.402823466e38f; btile[ct] = 0u; dup[ct] = 0ull;
                                if constexpr (FORM == 0) {
#pragma unroll
                                    for (int r = 0; r < ROWS; ++r) R[ct][r] = -INFINITY;
#pragma unroll
                                    for (int c = 0; c < Grid::COLS; ++c) C[ct][c] = -INFINITY;
                                }
                            }
                        }
                        if constexpr (FORM == 1) {       // (by itself: as one of an array the tile costs registers)
                            f32x16 acc[NT];
                            tile_mfma(acc, fr, padded);
                            settle(acc);
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct) {
                                float v[1][16];
#pragma unroll
                                for (int r = 0; r < 16; ++r) v[0][r] = acc[ct][r];
                                best[ct] = grid_maxima<1>(v, R[ct], C[ct]);
                            }
                        } else if constexpr (WHOLE > 0) {
                            f32x16 acc[WHOLE][NT];
                            if constexpr (AHEAD == 0) {
#pragma unroll
                                for (int tt = 0; tt < WHOLE; ++tt) tile_mfma(acc[tt], fr + tt * (PA * KS * 64), padded && tt == WHOLE - 1);
                            } else {
                                whole_mfma(acc, fr);
                            }
                            constexpr int LAST = WHOLE - 1;      // (one wait for all of them)
                            __builtin_amdgcn_sched_barrier(0);
                            if constexpr (WHOLE * NT == 2) asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0][0]), "+v"(acc[LAST][0]));
                            else if constexpr (NT == 2)
                                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0][0]), "+v"(acc[0][NT - 1]), "+v"(acc[LAST][0]), "+v"(acc[LAST][NT - 1]));
                            else if constexpr (WHOLE == 3)
                                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0][0]), "+v"(acc[1][0]), "+v"(acc[LAST][0]));
                            else
                                asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0][0]), "+v"(acc[1][0]), "+v"(acc[LAST - 1][0]), "+v"(acc[LAST][0]));
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct) {
                                float v[WHOLE][16];
#pragma unroll
                                for (int tt = 0; tt < WHOLE; ++tt)
#pragma unroll
                                    for (int r = 0; r < 16; ++r) v[tt][r] = acc[tt][ct][r];
                                if constexpr (WHOLE == 3) {      // a grid of four row tiles, one of them empty
                                    grid_rows<3>(v, R[ct]);
                                    R[ct][ROWS - 2] = R[ct][ROWS - 1] = -INFINITY;
                                    vmax4x4(C[ct], v[0], v[0] + 8, v[1], v[1] + 8);
                                    vmax4x4(C[ct] + 4, v[0] + 4, v[0] + 12, v[1] + 4, v[1] + 12);
                                    vmax_into8(C[ct], v[WHOLE - 1], v[WHOLE - 1] + 8);
                                    best[ct] = vmax2(vmax3(R[ct][0], R[ct][1], R[ct][2]), vmax3(R[ct][3], R[ct][ROWS - 4], R[ct][ROWS - 3]));
                                } else {
                                    best[ct] = grid_maxima<WHOLE>(v, R[ct], C[ct]);
                                }
                            }
                        } else {
                            const int tb = qq * q.stt;
                            const int te = tb + q.stt < q.tpg ? tb + q.stt : q.tpg;
                            auto merge = [&](int ct, const float *r, int tt) __attribute__((always_inline)) {
                                const float pm = ROWS == 2 ? vmax2(r[0], r[1]) : vmax2(vmax3(r[0], r[1], r[ROWS - 2]), r[ROWS - 1]);
                                // (second <= best: the middle one is what the greater of the two leaves)
                                if constexpr (FILTER) second[ct] = __builtin_amdgcn_fmed3f(pm, best[ct], second[ct]);
                                else dup[ct] |= __builtin_amdgcn_ballot_w64(pm == best[ct]);
                                keep_greater_rows<ROWS>(pm, (unsigned)tt, r, best[ct], btile[ct], R[ct]);
                            };
#pragma unroll 1
                            for (int tt = tb; tt < te; tt += UNIT) {
                                f32x16 a0[NT], a1[PAIRS ? NT : 1];
                                const u32x4 *f0 = fr + (size_t)(tt - tb) * (PA * KS * 64);
                                tile_mfma(a0, f0, padded && tt == q.tpg - 1);
                                bool two = false;
                                if constexpr (PAIRS) if (tt + 1 < te) {
                                    two = true;
                                    tile_mfma(a1, f0 + PA * KS * 64, padded && tt + 1 == q.tpg - 1);
                                    settle(a0); settle(a1);
#pragma unroll
                                    for (int ct = 0; ct < NT; ++ct) {
                                        float v0[16], v1[16];
#pragma unroll
                                        for (int r = 0; r < 16; ++r) { v0[r] = a0[ct][r]; v1[r] = a1[ct][r]; }
                                        float r[4];
                                        vmax8x2(r[0], v0, r[1], v0 + 8);
                                        vmax8x2(r[2], v1, r[3], v1 + 8);
                                        vmax_into8(C[ct], v0, v0 + 8);
                                        vmax_into8(C[ct], v1, v1 + 8);
                                        merge(ct, r, tt);
                                    }
                                }
                                if (!two) {
                                    settle(a0);
#pragma unroll
                                    for (int ct = 0; ct < NT; ++ct) {
                                        float v0[16];
#pragma unroll
                                        for (int r = 0; r < 16; ++r) v0[r] = a0[ct][r];
                                        float r[ROWS];
                                        vmax8x2(r[0], v0, r[1], v0 + 8);
                                        if constexpr (PAIRS) r[2] = r[3] = -INFINITY;
                                        vmax_into8(C[ct], v0, v0 + 8);
                                        merge(ct, r, tt);
                                    }
                                }
                            }
                            if (qq + 1 < q.nq) continue;             // the type goes on in the next stage
                        }
                        // ---- epilogue of type t = u: both candidate tiles stage by stage
                        const int t = u;
                        const float pt = prior[t], reach = FILTER ? prior[K + t] : 0.0f;
                        float gm[NT], floor[NT];
                        unsigned map[NT], map_other[NT];
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) gm[ct] = pair_other(best[ct], partner_addr);
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
                            gm[ct] = vmax2(gm[ct], best[ct]);
                            // Values from `floor` on count as maximisers: with products missing that is what they
                            // and the roundings can change below the maximum.
                            floor[ct] = FILTER ? fmaf(-norm[FILTER ? ct : 0], reach, gm[ct]) : gm[ct];
                            // FORM 0: a unique maximiser of the pair sits in this lane's leading unit, whose
                            // first tile goes with the bits, or the columns are marked in dup
                            if constexpr (WHOLE > 0) {
                                map[ct] = grid_map<WHOLE == 3 ? 4 : WHOLE>(R[ct], C[ct], floor[ct], 4u * h);
                            } else {
                                map[ct] = unit_map<ROWS>(R[ct], C[ct], floor[ct], 4u * h);
                                map[ct] = map[ct] ? map[ct] | (btile[ct] << 16) : 0u;
                            }
                            map_other[ct] = (unsigned)__builtin_amdgcn_ds_bpermute(partner_addr, (int)map[ct]);
                        }
                        float l[NT];
                        int js[NT];
                        bool clean[NT];
                        [[maybe_unused]] unsigned columns[NT], maps[NT];      // FILTER: those without a value that stands clear
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
                            const unsigned both = map[ct] | map_other[ct];
                            constexpr unsigned BITS = WHOLE ? 0xFFFFFFFFu : ~(kUnitTiles << 16);
                            unsigned long long multi = __builtin_amdgcn_ballot_w64(__builtin_popcount(both & BITS) != 2);
                            if constexpr (FORM == 0) multi |= FILTER ? __builtin_amdgcn_ballot_w64(second[ct] >= floor[ct]) : dup[ct];
                            columns[ct] = (unsigned)(multi | (multi >> 32)) & valid32[ct];
                            if constexpr (FILTER) {
                                maps[ct] = FORM == 0 ? map[ct] : both;
                                // rows of zeros: all actions tie and are worth the same, and the map says the first
                                columns[ct] &= ~zero32[ct];
                                tie_count += __builtin_popcount(zero32[ct]);
                            }
                            clean[ct] = multi == 0ull;               // wave-uniform
                            // (a wavefront that is not clean may hold any bits, and its gather is issued
                            // all the same)
                            const unsigned j = WHOLE ? grid_action<WHOLE == 3 ? 4 : WHOLE ? WHOLE : 1>(both) : grid_action<2>(both) + 32u * ((both >> 16) & kUnitTiles);
                            js[ct] = j < (unsigned)n ? (int)j : 0;
                        }
                        if constexpr (FILTER) {
                            // (bit h: lane half h of the column has values from the threshold on in several units)
                            auto units = [&](int ct, int c) __attribute__((always_inline)) {
                                const unsigned long long several = __builtin_amdgcn_ballot_w64(second[ct] >= floor[ct]) >> c;
                                return ((unsigned)several & 1u) | ((unsigned)(several >> 32) & 1u) << 1;
                            };
                            unsigned long long few = columns[0] | (NT == 2 ? (unsigned long long)columns[NT - 1] << 32 : 0ull);
                            if (__builtin_popcountll(few) <= 4)
#pragma unroll 1
                                for (; few != 0ull; few &= few - 1ull) {
                                    const int c = __builtin_ctzll(few);
                                    const bool other = NT == 2 && c >= 32;
                                    const unsigned of = other ? maps[NT - 1] : maps[0];
                                    const int j = exact_column(first + c, t, (unsigned)__builtin_amdgcn_readlane((int)of, c % 32),
                                                               FORM == 0 ? (unsigned)__builtin_amdgcn_readlane((int)of, c % 32 + 32) : 0u,
                                                               FORM == 0 ? units(other ? NT - 1 : 0, c % 32) : 0u);
                                    if (j < 0) continue;
#pragma unroll
                                    for (int ct = 0; ct < NT; ++ct) {
                                        if (c / 32 != ct) continue;
                                        columns[ct] &= ~(1u << (c % 32));
                                        js[ct] = col == c % 32 ? j : js[ct];
                                    }
                                }
                            static_for<0, NT, 1>([&](auto ctc) __attribute__((always_inline)) {
                                constexpr int ct = decltype(ctc)::value;
                                if (columns[ct] != 0u)
                                    exact_actions(ctc, columns[ct], t, gm[ct], floor[ct],
                                                  q.nq == 1 ? fr : reinterpret_cast<const u32x4 *>(records + (size_t)t * q.rec_bytes) + lane,
                                                  js[ct]);
                            });
                        }
                        float part[NT];
                        if (q.lead_off >= 0) {
                            const lds_byte *lb = (const lds_byte *)sb + (unsigned)(ui * q.rec_bytes + q.lead_off + h * HALF * LBYTES);
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct)
                                part[ct] = half_dot(ct, (const __attribute__((address_space(3))) u32x4 *)(lb + (unsigned)(js[ct] * q.lead_stride)));
                        } else {
#pragma unroll
                            for (int ct = 0; ct < NT; ++ct) part[ct] = half_dot(ct, lead_global(t, js[ct]));
                        }
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) l[ct] = pair_total(ct, part[ct]);
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct) {
                            if constexpr (!FILTER)
                                if (!clean[ct]) exact_type(ct, t, gm[ct], l[ct], js[ct]);
                            V[ct] = fmaf(pt, l[ct], V[ct]);
                        }
                        if (per_type)
                            put_type(std::integral_constant<int, NT>{}, [&](int ct) __attribute__((always_inline)) {
                                const unsigned c = first + ct * 32 + col;
                                return TypeOutput{ c, t, h == 0 && c < count, js[ct], l[ct] };
                            });
                    }
                }
            }
        }
        // ---- outputs of the block
        float *V_out = late()->a.V_out;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const unsigned c = first + ct * 32 + col;
            float v = V[ct];
            if (!(v == v)) v = -INFINITY;
            if (V_out && h == 0 && c < count) V_out[c] = v;
            // (a lane meets its candidates in ascending order: strictly greater replaces)
            v = c < count ? v : -INFINITY;
            keep_greater2(v, c, best_v, best_c);
        }
        left -= u1 - u0;
        if (left == 0) break;
        blk += step; u0 = 0; u1 = left < q.units ? left : q.units;
    }

    const late_args o = late();
    if (o->a.blk_v) {
        if (best_c == 0xFFFFFFFFu) {                     // no value above minus infinity: the first row, as on the other paths
            const unsigned c = (blockIdx.x * WAVES + wave) * (NT * 32) + col;
            best_c = c < count ? c : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int d = 16; d >= 1; d >>= 1) {              // both lane halves hold the same values
            const float ov = __shfl_xor(best_v, d, 64);
            const unsigned oc = __shfl_xor(best_c, d, 64);
            if (ov > best_v || (ov == best_v && oc < best_c)) { best_v = ov; best_c = oc; }
        }
        if (lane == 0) { red_v[wave] = best_v; red_c[wave] = best_c; }
        __syncthreads();
        if (tid == 0) {
            for (int k = 1; k < WAVES; ++k)
                if (red_v[k] > best_v || (red_v[k] == best_v && red_c[k] < best_c)) { best_v = red_v[k]; best_c = red_c[k]; }
            o->a.blk_v[blockIdx.x] = best_v;
            o->a.blk_i[blockIdx.x] = best_c == 0xFFFFFFFFu ? LLONG_MAX : o->a.index_base + (long long)best_c;
        }
    }
    if (o->a.tie_counter && lane == 0 && tie_count) atomicAdd(o->a.tie_counter, (unsigned long long)tie_count);
    if (o->a.done.flag) {
        const Done d = { o->a.done.flag, o->a.done.seq };
        signal_done(d, blockIdx.x);
    }
}

typedef void (*any_kernel_t)(AnyArgs);

template <int KS> any_kernel_t any_kernel_half_form(int form, bool many)
{
    if (form == 1) return sweep_any_kernel<2, KS, 1, true>;
    if constexpr (three_tiles(2, KS))
        if (form == 3) return sweep_any_kernel<2, KS, 3, true>;
    if (form == 2) return many ? sweep_any_kernel<2, KS, 2, true> : sweep_any_kernel<2, KS, 2, !two_kinds(2, KS, 2)>;
    return many ? sweep_any_kernel<2, KS, 0, true> : sweep_any_kernel<2, KS, 0, !two_kinds(2, KS, 0)>;
}

template <int TERMS, int KS>
any_kernel_t any_kernel_form(int form, bool many)
{
    switch (form) {
    case 0: return many ? sweep_any_kernel<TERMS, KS, 0, true> : sweep_any_kernel<TERMS, KS, 0, !two_kinds(TERMS, KS, 0)>;
    case 1: return many ? sweep_any_kernel<TERMS, KS, 1, true> : sweep_any_kernel<TERMS, KS, 1, !two_kinds(TERMS, KS, 1)>;
    case 2:
        if constexpr (two_tiles(TERMS, KS)) return many ? sweep_any_kernel<TERMS, KS, 2, true> : sweep_any_kernel<TERMS, KS, 2, !two_kinds(TERMS, KS, 2)>;
        break;
    case 4:
        if constexpr (four_tiles(TERMS, KS)) return sweep_any_kernel<TERMS, KS, 4, true>;
        break;
    case 3:
        if constexpr (three_tiles(TERMS, KS)) return sweep_any_kernel<TERMS, KS, 3, true>;
        break;
    case 8: return sweep_any_kernel<TERMS, KS, 8, true>;
    case 16: return sweep_any_kernel<TERMS, KS, 16, true>;
    }
    return nullptr;
}

}  // namespace any_impl
}  // namespace bsse
