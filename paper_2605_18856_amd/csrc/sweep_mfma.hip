// Fused sweep, matrix-core paths (steps 2-5): fp32 MFMA 32x32x2 and bf16 MFMA 32x32x16 with
// fp32 accumulation.
//
// The follower step is the skinny product  U^T = Bcat^T * X^T  with Bcat^T = all (type, action)
// rows [K*n][m] and X^T = [m][candidates]; U is never written.  The product is oriented so
// that a 32x32 MFMA tile has 32 (type, action) rows as its M dimension and 32 candidates as
// its N dimension: in the accumulator layout every lane then owns ONE candidate (column
// lane%32) and 16 of the tile's 32 rows (rows 8*(r/4) + 4*(lane/32) + r%4 for register r), so
// the arg-max over follower actions runs down a lane's own registers and needs a single
// exchange with the partner lane (lane ^ 32) per (candidate, type).
//
// Contraction index.  Lane half h = lane/32 supplies the k-slots of its half in both MFMA
// operands; this kernel maps them to leader actions i = h*MP/2 + slot, so each lane keeps a
// contiguous half of its candidate's row in registers for the whole pass over types, and the
// same registers serve the leader-payoff dot product  x . A_t[:, j*]  (each lane sums its
// half, the partner adds the other).  Payoffs are pre-packed on the host in exactly the
// per-lane fragment order, so staging a row tile into LDS is a flat copy and the operand
// reads are conflict-free.
//
// Ties.  The accumulators of a whole type stay in registers.  With n >= 32 the arg-max comes from the maxima
// of the rows and columns of a grid of them (ArgGrid), with fewer actions from a max3 chain, one exchange
// with the partner lane and a compare pass whose sum carries the maximising action and the number of
// maximisers.  Anything other than one maximiser per candidate sends the wavefront through an exact
// routine for that type, which recomputes the same MFMA tiles (bit-identical) and walks the exact
// maximisers in ascending action order comparing leader payoffs.
#include "bsse_internal.h"
#include <algorithm>
#include <vector>
#include "mfma_device.h"
#include "done_device.h"
#include <limits.h>
#include <stdlib.h>
#include <string.h>
#include <math.h>

namespace bsse {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned bf16_bits_rne(float v)
{
    unsigned b = __float_as_uint(v);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return b >> 16;
}

// ------------------------------------------------------------------------------------------
// Per-dtype pieces.  HALF = MP/2 leader actions per lane; a "fragment" is what one lane feeds
// to one MFMA.
template <typename T, int MP> struct Path;

template <int MP> struct Path<float, MP> {
    static constexpr int KSTEPS = MP / 2;      // 32x32x2: one k-slot per lane half
    static constexpr int HALF = MP / 2;
    typedef float frag;                        // one fp32 per lane per MFMA
    typedef float xreg;                        // register holding candidate components
    static constexpr int XREGS = HALF;
    static constexpr int FRAG_BYTES = 4;

    __device__ static __forceinline__ f32x16 mfma(frag a, const xreg *x, int s, f32x16 c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, x[s], c, 0, 0, 0);
    }
    // x registers from HALF fp32 values
    __device__ static __forceinline__ void pack_x(const float *v, xreg *x)
    {
#pragma unroll
        for (int e = 0; e < HALF; ++e) x[e] = v[e];
    }
    // sum over this lane's half of x[i] * col[i]; col points at the lane's half of the column
    template <typename BP>      // BP: byte pointer, global (generic) or LDS address space
    __device__ static __forceinline__ float half_dot(const xreg *x, BP col)
    {
        typedef typename std::conditional<std::is_same<BP, const lds_byte *>::value,
                                          const __attribute__((address_space(3))) float *, const float *>::type FP;
        typedef typename std::conditional<std::is_same<BP, const lds_byte *>::value,
                                          const __attribute__((address_space(3))) f32x4 *, const f32x4 *>::type VP;
        const FP c = (FP)col;
        float l = 0.0f;
        if constexpr (HALF % 4 == 0) {
#pragma unroll
            for (int e = 0; e < HALF; e += 4) {
                const f32x4 v = *(VP)(c + e);
                l = fmaf(x[e], v[0], l); l = fmaf(x[e + 1], v[1], l);
                l = fmaf(x[e + 2], v[2], l); l = fmaf(x[e + 3], v[3], l);
            }
        } else {
#pragma unroll
            for (int e = 0; e < HALF; ++e) l = fmaf(x[e], c[e], l);
        }
        return l;
    }
};

template <int MP> struct Path<__bf16, MP> {
    static_assert(MP % 16 == 0, "bf16 path needs m_pad % 16 == 0");
    static constexpr int KSTEPS = MP / 16;     // 32x32x16: eight k-slots per lane half
    static constexpr int HALF = MP / 2;
    typedef u32x4 frag;                        // eight bf16 per lane per MFMA
    typedef unsigned xreg;                     // two bf16 per register
    static constexpr int XREGS = HALF / 2;
    static constexpr int FRAG_BYTES = 16;

    __device__ static __forceinline__ f32x16 mfma(frag a, const xreg *x, int s, f32x16 c)
    {
        u32x4 b = { x[4 * s], x[4 * s + 1], x[4 * s + 2], x[4 * s + 3] };
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    __device__ static __forceinline__ void pack_x(const float *v, xreg *x)
    {
#pragma unroll
        for (int e = 0; e < HALF; e += 2)
            x[e / 2] = bf16_bits_rne(v[e]) | (bf16_bits_rne(v[e + 1]) << 16);
    }
    template <typename BP>
    __device__ static __forceinline__ float half_dot(const xreg *x, BP col)
    {
        // l += x.lo*c.lo + x.hi*c.hi on packed bf16 pairs, fp32 accumulate.  Issued as asm on
        // plain 32-bit words: going through the bf16-pair builtin, a bit-cast of an element
        // extracted from a clang vector was seen to reuse element 0 for all four words of a load.
        typedef typename std::conditional<std::is_same<BP, const lds_byte *>::value,
                                          const __attribute__((address_space(3))) u32x4 *, const u32x4 *>::type VP;
        const VP c = (VP)col;
        float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int e = 0; e < XREGS; e += 4) {
            const u32x4 v = c[e / 4];
            const unsigned w0 = v[0], w1 = v[1], w2 = v[2], w3 = v[3];
            asm("v_dot2c_f32_bf16 %0, %2, %6\n\t"
                "v_dot2c_f32_bf16 %1, %3, %7\n\t"
                "v_dot2c_f32_bf16 %0, %4, %8\n\t"
                "v_dot2c_f32_bf16 %1, %5, %9\n\t"
                "s_nop 2"       // a dot result needs three wait states before another kind of
                                // vector instruction reads it; the compiler cannot see into asm
                : "+v"(l0), "+v"(l1)
                : "v"(x[e]), "v"(x[e + 1]), "v"(x[e + 2]), "v"(x[e + 3]), "v"(w0), "v"(w1), "v"(w2), "v"(w3));
        }
        const float l = l0 + l1;
        return l;
    }
    // The same sum in two steps -- the lane's half of the column into registers, then the dot
    // product -- so that a caller can put other work between the reads and their use.  Same
    // instruction sequence on the same values as half_dot, hence the same bits.
    typedef u32x4 colregs[XREGS / 4];
    __device__ static __forceinline__ void gather_half(const lds_byte *col, colregs &c)
    {
        const __attribute__((address_space(3))) u32x4 *p = (const __attribute__((address_space(3))) u32x4 *)col;
#pragma unroll
        for (int e = 0; e < XREGS / 4; ++e) c[e] = p[e];
    }
    __device__ static __forceinline__ float half_dot_regs(const xreg *x, const colregs &c)
    {
        float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int e = 0; e < XREGS; e += 4) {
            const unsigned w0 = c[e / 4][0], w1 = c[e / 4][1], w2 = c[e / 4][2], w3 = c[e / 4][3];
            // (a dot result feeding the next dot needs no wait states; the three that another kind
            // of vector instruction needs follow the last group only)
            asm volatile("v_dot2c_f32_bf16 %0, %2, %6\n\t"
                         "v_dot2c_f32_bf16 %1, %3, %7\n\t"
                         "v_dot2c_f32_bf16 %0, %4, %8\n\t"
                         "v_dot2c_f32_bf16 %1, %5, %9"
                         : "+v"(l0), "+v"(l1)
                         : "v"(x[e]), "v"(x[e + 1]), "v"(x[e + 2]), "v"(x[e + 3]), "v"(w0), "v"(w1), "v"(w2), "v"(w3));
        }
        asm volatile("s_nop 2" : "+v"(l0), "+v"(l1));
        return l0 + l1;
    }
    // Two candidate tiles at once: the four accumulation chains are interleaved (a dot product
    // feeding the next one of its chain waits for it), each chain as in half_dot_regs.
    __device__ static __forceinline__ void half_dot_regs2(const xreg *xa, const colregs &ca, const xreg *xb,
                                                          const colregs &cb, float &la, float &lb)
    {
        float a0 = 0.0f, a1 = 0.0f, b0 = 0.0f, b1 = 0.0f;
#pragma unroll
        for (int e = 0; e < XREGS; e += 4) {
            const unsigned p0 = ca[e / 4][0], p1 = ca[e / 4][1], p2 = ca[e / 4][2], p3 = ca[e / 4][3];
            const unsigned q0 = cb[e / 4][0], q1 = cb[e / 4][1], q2 = cb[e / 4][2], q3 = cb[e / 4][3];
            asm volatile("v_dot2c_f32_bf16 %0, %4, %8\n\t"
                         "v_dot2c_f32_bf16 %2, %12, %16\n\t"
                         "v_dot2c_f32_bf16 %1, %5, %9\n\t"
                         "v_dot2c_f32_bf16 %3, %13, %17\n\t"
                         "v_dot2c_f32_bf16 %0, %6, %10\n\t"
                         "v_dot2c_f32_bf16 %2, %14, %18\n\t"
                         "v_dot2c_f32_bf16 %1, %7, %11\n\t"
                         "v_dot2c_f32_bf16 %3, %15, %19"
                         : "+v"(a0), "+v"(a1), "+v"(b0), "+v"(b1)
                         : "v"(xa[e]), "v"(xa[e + 1]), "v"(xa[e + 2]), "v"(xa[e + 3]), "v"(p0), "v"(p1), "v"(p2), "v"(p3),
                           "v"(xb[e]), "v"(xb[e + 1]), "v"(xb[e + 2]), "v"(xb[e + 3]), "v"(q0), "v"(q1), "v"(q2), "v"(q3));
        }
        asm volatile("s_nop 2" : "+v"(a0), "+v"(a1), "+v"(b0), "+v"(b1));
        la = a0 + a1;
        lb = b0 + b1;
    }
    // The same sum when the column holds three identical blocks (payoffs that are bf16 numbers,
    // against the three parts of x): each 16 bytes of the first block are loaded once and used
    // for all three parts, instead of gathering the same values three times.
    template <typename BP>
    __device__ static __forceinline__ float half_dot_rep3(const xreg *x, BP col)
    {
        typedef typename std::conditional<std::is_same<BP, const lds_byte *>::value,
                                          const __attribute__((address_space(3))) u32x4 *, const u32x4 *>::type VP;
        static_assert(XREGS % 12 == 0, "three blocks of whole 16-byte pieces");
        constexpr int BLOCK = XREGS / 3;
        const VP c = (VP)col;
        float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int e = 0; e < BLOCK; e += 4) {
            const u32x4 v = c[e / 4];
            const unsigned w0 = v[0], w1 = v[1], w2 = v[2], w3 = v[3];
#pragma unroll
            for (int term = 0; term < 3; ++term) {
                const int b = term * BLOCK + e;
                asm("v_dot2c_f32_bf16 %0, %2, %6\n\t"
                    "v_dot2c_f32_bf16 %1, %3, %7\n\t"
                    "v_dot2c_f32_bf16 %0, %4, %8\n\t"
                    "v_dot2c_f32_bf16 %1, %5, %9\n\t"
                    "s_nop 2"
                    : "+v"(l0), "+v"(l1)
                    : "v"(x[b]), "v"(x[b + 1]), "v"(x[b + 2]), "v"(x[b + 3]), "v"(w0), "v"(w1), "v"(w2), "v"(w3));
            }
        }
        const float l = l0 + l1;
        return l;
    }
};

// ------------------------------------------------------------------------------------------
// Stage records.  The packed follower payoffs are cut into "stages" of STAGE_TILES 32-row
// tiles; when AT_LDS, the leader-payoff rows of the types a stage covers follow its tiles, so
// that one flat asynchronous copy (global_load_lds) brings everything a stage needs into LDS.
// Leader rows in LDS are padded by 16 bytes so that gathers of different rows spread over
// banks.  The record size is rounded to what one sweep of all wavefronts copies (1 KiB each).
// terms == 6: the six products take the payoffs' parts 0 1 0 2 1 0, and a tile holds the three once (mp / 2
// slots): half the stage copies, and four fragment reads instead of six for the products that are always
// summed.  2^20 rows, K = 16, us: m = n = 32 175 -> 165, n = 64 291 -> 268,
// m = n = 16 101 -> 93.
struct Geometry {
    int tile_bytes, tpg, types, ts, ats, at_bytes, rec_bytes;
};
// terms == 6 (both operands split into bf16 parts) with leader rows in LDS: the leader rows are kept
// as plain fp32 (mp / terms values and 16 bytes of padding per action), not as parts.
// terms == 3 (payoffs that are bf16 numbers against the three parts of the candidate): the three
// blocks of a row tile's fragments would be identical, so a tile holds one block (mp / 3 slots)
// and every fragment read serves three matrix instructions.
__host__ __device__ constexpr Geometry make_geometry(int esz, int mp, int n, int stage_tiles,
                                                     int waves, bool at_lds, int terms = 1)
{
    Geometry q{};
    q.tile_bytes = 32 * (terms == 3 ? mp / 3 : terms == 6 ? mp / 2 : mp) * esz;
    q.tpg = n >= 32 ? n / 32 : 1;
    q.types = n >= 32 ? 1 : 32 / n;
    q.ts = stage_tiles >= q.tpg ? (stage_tiles / q.tpg) * q.types : 0;     // whole types per stage
    q.ats = (terms == 6 && at_lds) ? (mp / terms + 4) * 4 / esz : mp + 16 / esz;   // in elements of esz
    q.at_bytes = at_lds ? q.ts * n * q.ats * esz : 0;
    const int unit = waves * 1024;
    q.rec_bytes = (stage_tiles * q.tile_bytes + q.at_bytes + unit - 1) / unit * unit;
    return q;
}

// dynamic LDS of sweep_wide_kernel: two fragment buffers and two leader-row buffers
__host__ __device__ constexpr int wide_lds_bytes(int esz, int mp, int n, int waves)
{
    const Geometry q = make_geometry(esz, mp, n, n / 32, waves, true);
    return 2 * (q.tpg * q.tile_bytes) + 2 * ((q.at_bytes + 1023) / 1024 * 1024);
}

typedef const void __attribute__((address_space(1))) *global_ptr;
typedef void __attribute__((address_space(3))) *lds_ptr;

// What the filter of the split kernels scales a row's later parts by before it takes their norms, and the
// least norm and margin it works with (see filter_margins).
constexpr float kScale1 = 0x1p9f, kScale2 = 0x1p18f, kLeastNorm = 0x1p-30f, kLeastMargin = 0x1p-90f;

// ------------------------------------------------------------------------------------------
// T: float | __bf16.  MP: padded m.  N: follower actions (8, 16 or a multiple of 32).
// NT: 32-candidate tiles per wavefront.  WAVES: wavefronts per workgroup.
// STAGE_TILES: row tiles per LDS stage.  OCC: wavefronts per SIMD the register allocation is
// held to.  AT_LDS: leader-payoff rows travel with the stage (else they are gathered from
// global memory / L2).
//
// A "group" is the set of row tiles that holds whole types: N/32 tiles of one type when
// N >= 32, one tile of 32/N types otherwise.  The accumulators of a whole group stay in
// registers (N/2 per lane and candidate tile when N >= 32), so the arg-max is passes over
// registers.  N >= 32: the maxima of a grid's rows and columns, one exchange with the partner
// lane for the pair's maximum, then a bit for each row and column that reaches it, both lanes'
// (grid_map).  N < 32: a max3 chain and the exchange, then a compare pass that adds
// (action + 2^16) for every register equal to the maximum: the sum carries the maximising action
// and the number of maximisers.  Anything other than one maximiser per candidate means an exact
// tie somewhere in the tile (FILTER: or values too near each other, which settle sums whole
// first) and sends the wavefront through the exact routine for that type.
//
// Stages are double-buffered: the copy of stage s+1 is issued (asynchronously, straight into
// LDS) before the work on stage s and awaited after it, one workgroup barrier per stage.
//
// SLICED: the launch is two-dimensional and workgroup row blockIdx.y walks only its slice of the
// stages (whole groups), writing the per-type leader payoffs instead of the value; used to
// re-evaluate a few rows against many types with the whole chip.  The per-candidate instruction
// sequence does not depend on NT, OCC or SLICED, so every instantiation of a packing gives the
// same bits for the same row.
template <typename T, int MP, int N, int NT, int WAVES, int STAGE_TILES, int OCC, bool AT_LDS, int TERMS,
          bool SLICED, int PF, bool FILTER>
__global__ void __launch_bounds__(WAVES * 64, OCC)
sweep_mfma_kernel(GameView g, SweepArgs a, int row_tiles)
{
    static_assert(TERMS == 1 || TERMS == 3 || TERMS == 6, "1 = operands as stored; 3, 6 = split fp32");
    static_assert(TERMS == 1 || std::is_same<T, __bf16>::value, "split terms run on the bf16 path");
    static_assert(MP % TERMS == 0, "MP is TERMS blocks of the padded m");
    constexpr int MP_BASE = MP / TERMS, HALF_BASE = MP_BASE / 2;
    typedef Path<T, MP> P;
    typedef typename P::frag frag;
    typedef typename P::xreg xreg;
    constexpr int KS = P::KSTEPS, HALF = P::HALF;
    constexpr Geometry G = make_geometry((int)sizeof(T), MP, N, STAGE_TILES, WAVES, AT_LDS, TERMS);
    constexpr int TPG = G.tpg, TYPES = G.types;
    static_assert(N == 8 || N == 16 || N % 32 == 0, "unsupported action count");
    static_assert(STAGE_TILES % TPG == 0 || TPG % STAGE_TILES == 0, "stage/group mismatch");
    static_assert(!AT_LDS || STAGE_TILES >= TPG, "leader rows in LDS need whole types per stage");
    constexpr int REP = TERMS == 3 ? 3 : 1;             // part products per stored fragment
    constexpr int KF = KS / REP;                        // fragment k-steps per row tile
    constexpr int TILE_FRAGS = (TERMS == 6 ? KF / 2 : KF) * 64;         // fragments per row tile
    // FILTER (split operands): the products that decide nearly every arg-max are summed first, (p0,B0) (p0,B1)
    // (p1,B0) of six and p0 and p1 of three; then the small others (of three in a sum of their own, which
    // is added: the margin is a third), which are left out where the maximum stands clear of the
    // next value by more than they can change (see filter_margins).  Matrix and vector time add up in
    // these kernels, and the products were half of it: m = n = 32, K = 16, 2^20 rows 215 -> 171 us, n = 64
    // 376 -> 284; m = 128, n = 256, K = 256, 131072 rows 4120 -> 3200, of which 1 % for the rows that are
    // not clear (0.8 % of the tiles).
    constexpr int MAIN_KF = FILTER && TERMS == 6 ? KF / 2 : KF, MAIN_REP = FILTER && TERMS == 3 ? 2 : REP;
    static_assert(!FILTER || (TERMS > 1 && STAGE_TILES >= TPG && N >= 32), "split operands, whole types per stage");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ float red_v[WAVES];
    __shared__ long long red_i[WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, col = lane & 31;
    const int m = g.m, K = g.K;
    const unsigned char *records = reinterpret_cast<const unsigned char *>(g.Bpack);
    const unsigned char *ATpack = reinterpret_cast<const unsigned char *>(g.ATpack);
    const long long wave_base = ((long long)blockIdx.x * WAVES + wave) * (NT * 32);
    const int nstages = (row_tiles + STAGE_TILES - 1) / STAGE_TILES;
    // the stages this workgroup walks: all of them, or slice blockIdx.y of them
    const int stage_begin = SLICED ? (int)blockIdx.y * a.slice_stages : 0;
    const int stage_end = SLICED && stage_begin + a.slice_stages < nstages
                              ? stage_begin + a.slice_stages : nstages;
    if (SLICED && stage_begin >= stage_end) return;                     // whole workgroup

    auto prefetch = [&](int st) __attribute__((always_inline)) {
        const unsigned char *src = records + (size_t)st * G.rec_bytes;
        unsigned char *dst = smem + (st & 1) * G.rec_bytes;
#pragma unroll
        for (int i = 0; i < G.rec_bytes / (WAVES * 1024); ++i) {
            const int chunk = i * WAVES + wave;
            __builtin_amdgcn_global_load_lds((global_ptr)(src + chunk * 1024 + lane * 16),
                                             (lds_ptr)(dst + chunk * 1024), 16, 0, 0);
        }
    };
    // own copies have landed; then everyone's have, and everyone is done with the old stage
    auto stage_sync = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    prefetch(stage_begin);

    // ---- candidate rows into registers: lane (col, h) keeps its half of the leader actions,
    // x[c][h*HALF_BASE .. (h+1)*HALF_BASE); on the split path each component becomes TERMS
    // bf16 parts, laid out as TERMS blocks of HALF_BASE to match the packed payoffs
    // Split path: three bf16 parts per component are stored once each (p0, p1, p2 as blocks of
    // XB registers); the six k-slot blocks (p0,B0) (p0,B1) (p1,B0) (p0,B2) (p1,B1) (p2,B0) of the
    // packed payoffs pick them in x_mfma.  Where the leader rows are in LDS they are fp32, and
    // so is the lane's half of the candidate row that meets them (xf).
    constexpr bool LEAD_F32 = TERMS == 6 && AT_LDS;
    constexpr int XB = TERMS > 1 ? HALF_BASE / 2 : P::XREGS;            // registers per part
    constexpr int XS = TERMS > 1 ? 3 * XB : P::XREGS;                   // registers stored per tile
    constexpr int SPT = KS / TERMS;                                     // k-steps per block
    auto x_mfma = [](const frag &fr, const xreg *xc, int s, const f32x16 &c) __attribute__((always_inline)) {
        if constexpr (TERMS == 6) {
            constexpr int xsel6[6] = { 0, 0, 1, 0, 1, 2 };
            return P::mfma(fr, xc + xsel6[s / SPT] * XB + 4 * (s % SPT), 0, c);
        } else {
            return P::mfma(fr, xc, s, c);
        }
    };
    // stored fragment of k-step s (of a tile)
    auto stored = [](int s) __attribute__((always_inline)) {
        constexpr int bsel6[6] = { 0, 1, 0, 2, 1, 0 };
        return (TERMS == 6 ? bsel6[s / SPT] * SPT + s % SPT : s) * 64;
    };
    xreg x[NT][XS];
    float xf[NT][LEAD_F32 ? HALF_BASE : 1];
    float norm[FILTER ? NT : 1];              // of the row, and of what its later parts can weigh
    unsigned valid32[NT];                     // bit c set iff candidate c of the tile exists
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        // (columns past the end repeat the last row: they behave like any other and are left out of
        // every output; as rows of zeros they tied everywhere and sent their tile through the exact
        // routine for every type -- 54 us instead of 11 for 1000 rows of m = n = 32, K = 16)
        const long long c = wave_base + ct * 32 + col;
        const bool ok = c < a.count;
        float vb[HALF_BASE];
        const float *row = a.X + (ok ? c : a.count - 1) * (long long)m + h * HALF_BASE;
        if (m == MP_BASE && HALF_BASE % 4 == 0 && ((uintptr_t)a.X & 15) == 0) {
#pragma unroll
            for (int e = 0; e < HALF_BASE; e += 4) {
                const f32x4 q = *(const f32x4 *)(row + e);
                vb[e] = q[0]; vb[e + 1] = q[1]; vb[e + 2] = q[2]; vb[e + 3] = q[3];
            }
        } else if constexpr (TERMS != 3) {
            load_half_row<HALF_BASE>(row - h * HALF_BASE, h, m, vb);
        } else {
            // (component by component: at the register limit, m = 100, n = 256, K = 100, 65536 rows take
            // 908 us like this and 916 in pieces)
#pragma unroll
            for (int e = 0; e < HALF_BASE; ++e) {
                const bool in = h * HALF_BASE + e < m;
                const float t = row[in ? e : -h * HALF_BASE];
                vb[e] = in ? t : 0.0f;
            }
        }
        if constexpr (TERMS == 1) {
            P::pack_x(vb, x[ct]);
        } else {
            // x = p0 + p1 + p2 with bf16 parts (the subtractions are exact in fp32)
            float v[3 * HALF_BASE];
#pragma unroll
            for (int e = 0; e < HALF_BASE; ++e) {
                float part[3];
                part[0] = __uint_as_float(bf16_bits_rne(vb[e]) << 16);
                const float r1 = vb[e] - part[0];
                part[1] = __uint_as_float(bf16_bits_rne(r1) << 16);
                const float r2 = r1 - part[1];
                part[2] = __uint_as_float(bf16_bits_rne(r2) << 16);
#pragma unroll
                for (int q = 0; q < 3; ++q) v[q * HALF_BASE + e] = part[q];
            }
#pragma unroll
            for (int e = 0; e < 3 * HALF_BASE; e += 2)
                x[ct][e / 2] = bf16_bits_rne(v[e]) | (bf16_bits_rne(v[e + 1]) << 16);
            if constexpr (FILTER) {
                float sq[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    sq[q] = 0.0f;
#pragma unroll
                    for (int e = 0; e < XB; ++e) {
                        const bf16x2 pv = __builtin_bit_cast(bf16x2, x[ct][q * XB + e]);
                        sq[q] = __builtin_amdgcn_fdot2_f32_bf16(pv, pv, sq[q], false);
                    }
                }
                const float first = TERMS == 6 ? pair_sum(sq[0]) : 0.25f * pair_sum(sq[0]);
                const float second = TERMS == 6 ? kScale1 * kScale1 * pair_sum(sq[1]) : 0.0f;
                norm[ct] = fmaxf(__builtin_amdgcn_sqrtf(fmaxf(first, fmaxf(second, kScale2 * kScale2 * pair_sum(sq[2])))), kLeastNorm);
            }
            if constexpr (LEAD_F32) {
#pragma unroll
                for (int e = 0; e < HALF_BASE; ++e) xf[ct][e] = vb[e];
            }
        }
        valid32[ct] = (unsigned)__builtin_amdgcn_ballot_w64(ok);
    }

    float V[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) V[ct] = 0.0f;
    unsigned tie_count = 0;                   // wave-uniform
    const uniform_floats prior = (uniform_floats)g.prior;
    // per-register constants of the compare pass: the action a register stands for within its
    // row tile and type (lane half included) plus 2^16
    [[maybe_unused]] unsigned creg[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        creg[r] = (unsigned)((N >= 32 ? acc_row_base(r) : acc_row_base(r) % N) + 4 * h) + 65536u;

    // Leader-payoff half sum over a column gathered from global memory.  With three part products
    // the column's three blocks are identical, and one is read.
    auto leader_half = [&](const xreg *xc, const unsigned char *colp) __attribute__((always_inline)) {
        if constexpr (TERMS == 3 && !AT_LDS) return P::half_dot_rep3(xc, colp);
        else return P::half_dot(xc, colp);
    };
    // fp32 leader rows (LEAD_F32): the lane's HALF_BASE components against its half of the row,
    // two fused multiply-add chains; the same sequence from LDS and from global memory.
    auto leader_half_f32 = [&](const float *xc, auto row) __attribute__((always_inline)) {
        float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int e = 0; e < (LEAD_F32 ? HALF_BASE : 0); e += 4) {
            const f32x4 r = row[e / 4];
            l0 = fmaf(xc[e], r[0], l0); l1 = fmaf(xc[e + 1], r[1], l1);
            l0 = fmaf(xc[e + 2], r[2], l0); l1 = fmaf(xc[e + 3], r[3], l1);
        }
        return l0 + l1;
    };
    // One row tile, whose fragments are at `tile`, against one candidate tile, small products and all.
    auto rest_of = [&](const xreg *xc, const frag *tile, f32x16 r) __attribute__((always_inline)) {
#pragma unroll
        for (int s = TERMS == 6 ? KF / 2 : 0; s < KF; ++s) r = x_mfma(tile[stored(s) + lane], xc, TERMS == 3 ? 2 * KF + s : s, r);
        return r;
    };
    auto whole_tile = [&](const xreg *xc, const frag *tile) __attribute__((always_inline)) {
        f32x16 sum;
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[e] = 0.0f;
#pragma unroll
        for (int s = 0; s < MAIN_KF; ++s) {
            const frag af = tile[stored(s) + lane];
#pragma unroll
            for (int q = 0; q < MAIN_REP; ++q) sum = x_mfma(af, xc, q * KF + s, sum);
        }
        if constexpr (FILTER && TERMS == 3) sum += rest_of(xc, tile, f32x16{});
        else if constexpr (FILTER) sum = rest_of(xc, tile, sum);
        return sum;
    };
    // Exact routine for one (candidate tile, type): recomputes the type's tiles one at a time
    // from the packed records in global memory (same instruction sequence, hence the same
    // bits), visits the exact maximisers in ascending action order, lets the leader's payoff
    // decide and then the lower action, in the candidate columns of the mask `columns`.
    auto exact_type = [&](int ct, unsigned columns, int group, int ti, int t, float gmax, float &l_out,
                          int &j_out) __attribute__((always_inline)) {
        float lbest = kNotANumber;               // (no maximiser: no sum is a number)
        int jbest = 0, nmatch = 0;
        const unsigned char *ATt = ATpack + (size_t)t * N * MP * sizeof(T);
#pragma unroll 1
        for (int tt = 0; tt < TPG; ++tt) {
            const int gt = group * TPG + tt;
            const f32x16 acc1 = whole_tile(x[ct], reinterpret_cast<const frag *>(
                records + (size_t)(gt / STAGE_TILES) * G.rec_bytes + (size_t)(gt % STAGE_TILES) * G.tile_bytes));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = 4 * q + rr;
                        const int rb = acc_row_base(r);
                        if (N < 32 && rb / N != ti) continue;
                        const int j = (N >= 32 ? tt * 32 + rb : rb % N) + 4 * hh;
                        const unsigned long long meq = __builtin_amdgcn_ballot_w64(acc1[r] == gmax);
                        const unsigned hit = (unsigned)(hh ? (meq >> 32) : meq) & columns;
                        if (hit == 0u) continue;                       // wave-uniform
                        float lh;
                        if constexpr (LEAD_F32)
                            lh = leader_half_f32(xf[ct], reinterpret_cast<const f32x4 *>(
                                     reinterpret_cast<const float *>(ATpack) + ((size_t)t * N + j) * MP_BASE + h * HALF_BASE));
                        else
                            lh = leader_half(x[ct], ATt + ((size_t)j * MP + h * HALF) * sizeof(T));
                        const float l = pair_sum(lh);
                        if ((hit >> col) & 1u) {
                            if (nmatch == 0 || l > lbest) { lbest = l; jbest = j; }
                            ++nmatch;
                        }
                    }
        }
        if (!FILTER || ((columns >> col) & 1u)) { l_out = lbest; j_out = jbest; }
        tie_count += __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(nmatch >= 2));
    };

    // accumulators of the current group, all NT candidate tiles
    f32x16 acc[NT][TPG];
    auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int tt = 0; tt < TPG; ++tt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ct][tt][r] = 0.0f;
    };
    // MFMAs of NTILES consecutive row tiles (fragments in LDS at `base`; tt0 = index of the first
    // one within the group) against all NT candidate tiles.  The fragment reads are software-
    // pipelined in chunks of PF k-steps where that was measured to pay: the
    // reads of chunk q+1 are issued before the MFMAs of chunk q, so the LDS latency runs under the
    // matrix pipe instead of in front of it.
    auto mfma_run = [&](const frag *base, auto ntiles_c, auto tt0_c) __attribute__((always_inline)) {
        constexpr int NTILES = decltype(ntiles_c)::value, TT0 = decltype(tt0_c)::value;
        if constexpr (PF == 0) {               // reads where they are used; the compiler schedules
#pragma unroll
            for (int tt = 0; tt < NTILES; ++tt)
#pragma unroll
                for (int ks = 0; ks < MAIN_KF; ++ks) {
                    const frag af = base[(size_t)tt * TILE_FRAGS + stored(ks) + lane];
#pragma unroll
                    for (int q = 0; q < MAIN_REP; ++q)
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct)
                            acc[ct][TT0 + tt] = x_mfma(af, x[ct], q * KF + ks, acc[ct][TT0 + tt]);
                }
            return;
        }
        static_assert(PF == 0 || TERMS != 6, "fragments are read ahead in the order of the k-steps");
        static_assert(PF == 0 || KF % (PF ? PF : 1) == 0, "fragment chunk must divide the k-steps of a tile");
        constexpr int C = PF ? PF : 1;
        constexpr int NCH = NTILES * KF / C;
        frag fb[2][C];
        const frag *lane_base = base + lane;
#pragma unroll
        for (int e = 0; e < C; ++e) fb[0][e] = lane_base[(size_t)e * 64];
        static_for<0, NCH, 1>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if constexpr (q + 1 < NCH) {
#pragma unroll
                for (int e = 0; e < C; ++e) {
                    constexpr int f0 = (q + 1) * C;
                    const int f = f0 + e;                                    // flat (tile, k-step)
                    fb[(q + 1) & 1][e] = lane_base[(size_t)(f / KF) * TILE_FRAGS + (size_t)(f % KF) * 64];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, C, 1>([&](auto ec) {
                constexpr int f = q * C + decltype(ec)::value;
                constexpr int tt = TT0 + f / KF, ks = f % KF;
#pragma unroll
                for (int p = 0; p < MAIN_REP; ++p)
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct)
                        acc[ct][tt] = x_mfma(fb[q & 1][decltype(ec)::value], x[ct], p * KF + ks, acc[ct][tt]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // FILTER: the maximum of the whole sums for the candidate columns `multi` of a tile, where several values
    // are within the margin of the greatest.  `need`: the row tiles that hold such a value in one of these
    // columns (no other can hold their maximum).  Returns the columns where it is no unique one (ties).
    auto settle = [&](int ct, unsigned multi, unsigned need, auto tiles_of_group, float &gmax, int &jstar) __attribute__((always_inline)) {
        float best = -INFINITY, w[16];
        unsigned btile = 0u;
        unsigned long long dup = 0ull;
        auto tile_sums = [&](int tt, float (&u)[16]) __attribute__((always_inline)) {
            f32x16 sum = whole_tile(x[ct], tiles_of_group + (size_t)tt * TILE_FRAGS);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 15" : "+v"(sum));
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = sum[r];
        };
        if constexpr (TPG == 1) {
            tile_sums(0, w);
            best = vmax_chain16(best, w);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = -INFINITY;
#pragma unroll 1
            for (int tt = 0; tt < TPG; ++tt) {
                if (!(need >> tt & 1u)) continue;
                float u[16];
                tile_sums(tt, u);
                const float pm = vmax_chain16(-INFINITY, u);
                dup |= __builtin_amdgcn_ballot_w64(pm == best);
                keep_greater2(pm, (unsigned)(32 * tt), best, btile);
#pragma unroll
                for (int r = 0; r < 16; ++r) w[r] = vmax2(w[r], u[r]);
            }
        }
        const float gm = pair_max(best);
        const unsigned bm = bitmap16_pairs(w, gm), cnt = (unsigned)__builtin_popcount(bm), r = ffbh(bm) - 16u;
        const unsigned total = cnt ? (cnt << 16) | btile | ((r & 0xCu) << 1) | (r & 3u) | (4u * h) : 0u;
        const unsigned pair = pair_add_u32(total);
        if ((multi >> col) & 1u) { gmax = gm; jstar = (int)(pair & 0xFFFFu) & (N - 1); }
        return multi & ((unsigned)__builtin_amdgcn_ballot_w64((pair >> 16) != 1u) | (unsigned)(dup | (dup >> 32)));
    };
    // second half of a type's epilogue: leader payoff at the best response (fast path: one row
    // gather and a dot product; otherwise the exact routine), value accumulation, outputs
    // (ties: the candidate columns without a unique maximiser, per tile)
    // READ_AHEAD: the column at the best response is requested as soon as that is known, and met after the
    // arg-max of the other candidate tile: fetch and meet.  (m = n = 32, K = 16, 2^22 rows 600 -> 590 us; n = 64, 2^20
    // rows 267 -> 262; m = 16, n = 32 bf16 85 -> 83.  Three products spill; with one tile there is no other.)
    constexpr bool READ_AHEAD = NT > 1 && N >= 32 && AT_LDS && TERMS != 3 && std::is_same<T, __bf16>::value;
    constexpr int COL16 = READ_AHEAD ? (LEAD_F32 ? HALF_BASE / 4 : HALF / 8) : 1;       // 16-byte pieces of a lane's half
    auto fetch = [&](int ti, int js, const lds_byte *at_lds, u32x4 (&column)[COL16]) __attribute__((always_inline)) {
        const auto *p = (const __attribute__((address_space(3))) u32x4 *)(
            at_lds + (unsigned)((ti * N + js) * G.ats * sizeof(T) + h * COL16 * 16));
#pragma unroll
        for (int e = 0; e < COL16; ++e) column[e] = p[e];
    };
    auto meet = [&](int ct, const u32x4 (&column)[COL16]) __attribute__((always_inline)) {
        if constexpr (!READ_AHEAD) return 0.0f;
        else if constexpr (LEAD_F32) return leader_half_f32(xf[ct], reinterpret_cast<const f32x4 *>(column));
        else return P::half_dot_regs(x[ct], column);
    };
    auto leader_part = [&](int group, int ti, int t, float pt, const lds_byte *at_lds, const float *gmax,
                           const int *jstar, const unsigned *ties, const auto &column) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            float l;
            int js = jstar[ct];
            if (FILTER || READ_AHEAD || ties[ct] == 0u) {
                float part;
                if constexpr (READ_AHEAD)
                    part = meet(ct, column[ct]);
                else if constexpr (LEAD_F32)
                    part = leader_half_f32(xf[ct], (const __attribute__((address_space(3))) f32x4 *)(
                               at_lds + (unsigned)(((ti * N + js) * G.ats) * sizeof(T) + h * HALF_BASE * sizeof(float))));
                else if constexpr (AT_LDS)
                    part = P::half_dot(x[ct], at_lds + (unsigned)(((ti * N + js) * G.ats + h * HALF) * sizeof(T)));
                else
                    part = leader_half(x[ct], ATpack + (((size_t)t * N + js) * MP + h * HALF) * sizeof(T));
                l = pair_sum(part);
            }
            if (ties[ct] != 0u) exact_type(ct, (FILTER ? ties[ct] : 0xFFFFFFFFu) & valid32[ct], group, ti, t, gmax[ct], l, js);
            V[ct] = fmaf(pt, l, V[ct]);
            if constexpr (SLICED) {
                const long long c = wave_base + ct * 32 + col;
                if (h == 0 && c < a.count) {
                    a.l_out[c * a.l_sc + t * a.l_st] = l;
                    if (a.br_out) a.br_out[c * a.br_sc + t * a.br_st] = js;
                }
            } else if (a.br_out) {
                const long long c = wave_base + ct * 32 + col;
                if (h == 0 && c < a.count) a.br_out[c * K + t] = js;
            }
        }
    };
    // per-type epilogue of a finished group; at_lds = LDS rows of the group's first type; rest = its row
    // tiles, for products that were left out
    auto epilogue = [&](int group, const lds_byte *at_lds, auto rest) __attribute__((always_inline)) {
        // The asm blocks below read the accumulators, and the compiler's hazard handling does not
        // look into inline asm: the wait states a vector read of a fresh MFMA result needs (passes
        // + 3: 11 for the 8-pass bf16 MFMA, 19 for the 16-pass fp32 one) are put here explicitly.
        __builtin_amdgcn_sched_barrier(0);
        // The statements behind it tie the accumulators to the wait: asm that is not volatile moves above
        // one that names nothing it reads.
        asm volatile("s_nop 15");
        if constexpr (std::is_same<T, float>::value) asm volatile("s_nop 3");
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int tt = 0; tt < TPG; ++tt) asm volatile("" : "+v"(acc[ct][tt]));
        static_for<0, TYPES, 1>([&](auto tic) {
            constexpr int ti = decltype(tic)::value;
            const int t = group * TYPES + ti;
            if (t >= K) return;                                         // padded type rows
            const float pt = prior[t], reach = FILTER ? prior[K + t] : 0.0f;
            float gmax[NT];
            int jstar[NT];
            unsigned ties[NT];
            u32x4 column[NT][COL16];
            [[maybe_unused]] unsigned maps[NT];
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                // Values from `floor` on count as maximisers.  While products are missing that is the maximum
                // less what they can change: where one value stands alone it is the maximum of the whole
                // sums too.
                const float room = FILTER ? -norm[FILTER ? ct : 0] * reach : 0.0f;
                typedef ArgGrid<TPG> Grid;
                float gm;
                unsigned map = 0u, multi;                 // multi: columns where no value stands alone
                if constexpr (N >= 32) {
                    // whole row tiles belong to the type
                    float u[TPG][16];
#pragma unroll
                    for (int tt = 0; tt < TPG; ++tt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) u[tt][r] = acc[ct][tt][r];
                    float R[Grid::ROWS], C[Grid::COLS];
                    gm = pair_max(grid_maxima<TPG, SLICED>(u, R, C));
                    map = pair_or(grid_map<TPG>(R, C, FILTER ? gm + room : gm, 4u * h));
                    jstar[ct] = (int)(grid_action<TPG>(map) & (N - 1));       // (any action where the row is not settled)
                    multi = (unsigned)__builtin_amdgcn_ballot_w64(__builtin_popcount(map) != 2);
                } else {
                    // lane maximum over this type's registers
                    float pm = -INFINITY, pend[2];
                    unsigned total = 0u;
                    int np = 0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        if (acc_row_base(r) / N != ti) continue;
                        pend[np++] = acc[ct][0][r];
                        if (np == 2) { pm = vmax3(pm, pend[0], pend[1]); np = 0; }
                    }
                    if (np == 1) pm = vmax2(pm, pend[0]);
                    gm = pair_max(pm);
                    const float floor = FILTER ? gm + room : gm;
                    // compare pass over the type's registers of the tile
                    static_for<0, 4, 1>([&](auto qc) {
                        constexpr int r = 4 * decltype(qc)::value;
                        if constexpr (acc_row_base(r) / N == ti)
                            match4(acc[ct][0][r], acc[ct][0][r + 1], acc[ct][0][r + 2], acc[ct][0][r + 3],
                                   floor, creg[r], creg[r + 1], creg[r + 2], creg[r + 3], total);
                    });
                    const unsigned pair = pair_add_u32(total);
                    jstar[ct] = (int)(pair & 0xFFFFu);
                    multi = (unsigned)__builtin_amdgcn_ballot_w64((pair >> 16) != 1u);
                }
                gmax[ct] = gm;
                ties[ct] = multi;
                maps[ct] = map;
                if constexpr (READ_AHEAD) fetch(ti, jstar[ct], at_lds, column[ct]);
            }
            if constexpr (FILTER) {
                unsigned any = 0u;
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) any |= ties[ct];
                if (any != 0u) {
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) {
                        const unsigned multi = ties[ct];
                        if (multi == 0u) continue;
                        unsigned need = 1u;
                        if constexpr (TPG > 1) {
                            // the tiles with a value from the threshold on, two grid rows each (columns without
                            // one, whose sums are infinite or no numbers, take them all)
                            constexpr int ROWS = ArgGrid<TPG>::ROWS;
                            need = 0u;
                            const unsigned rows = (multi >> col) & 1u ? maps[ct] >> (32 - ROWS) : 0u;
#pragma unroll
                            for (int k = 0; k < TPG; ++k)
                                if (__builtin_amdgcn_ballot_w64((rows >> (2 * (TPG - 1 - k)) & 3u) != 0u) != 0ull) need |= 1u << k;
                            if ((multi & (unsigned)__builtin_amdgcn_ballot_w64(rows == 0u)) != 0u) need = (1u << TPG) - 1u;
                        }
                        ties[ct] = settle(ct, multi, need, rest, gmax[ct], jstar[ct]);
                        if constexpr (READ_AHEAD) fetch(ti, jstar[ct], at_lds, column[ct]);
                    }
                }
            }
            leader_part(group, ti, t, pt, at_lds, gmax, jstar, ties, column);
        });
    };

    stage_sync();                              // the first stage is in LDS
    const int groups = row_tiles / TPG;
    // Two roles where the epilogue reads nothing from LDS (leader rows gathered from global memory),
    // a stage holds whole types and one workgroup fills the compute unit: the late half of the
    // wavefronts passes the barrier that ends a stage BEFORE the stage's last epilogue, the early half
    // after it, so that behind every barrier the two wavefronts of a SIMD are one epilogue apart
    // -- one on the matrix pipe, one on the vector unit -- instead of wanting the same unit at the
    // same time (measured on the m=128 n=256 three-term variant: 4 %; with a barrier per row tile
    // the late half held the early half up instead, and on the wide bf16 kernel it gained nothing).
    constexpr bool ROLES = !AT_LDS && !SLICED && WAVES == 8 && STAGE_TILES >= TPG;
    const bool late = ROLES && wave >= WAVES / 2;
    if constexpr (STAGE_TILES >= TPG) {
        constexpr int GPS = STAGE_TILES / TPG;                          // groups per stage
#pragma unroll 1
        for (int st = stage_begin; st < stage_end; ++st) {
            if (st + 1 < stage_end) prefetch(st + 1);
            const unsigned char *buf = smem + (st & 1) * G.rec_bytes;
            const frag *tiles = reinterpret_cast<const frag *>(buf);
            const int g0 = st * GPS;
            const int ng = groups - g0 < GPS ? groups - g0 : GPS;
#pragma unroll 1
            for (int gi = 0; gi < ng; ++gi) {
                zero_acc();
                const frag *gt = tiles + (size_t)(gi * TPG) * TILE_FRAGS;
                mfma_run(gt, std::integral_constant<int, TPG>{}, std::integral_constant<int, 0>{});
                if (ROLES && late && gi == ng - 1) stage_sync();
                // (with two roles the stage's buffer may be overwritten by now)
                const lds_byte *at = (const lds_byte *)buf + (unsigned)(STAGE_TILES * G.tile_bytes + gi * TYPES * N * G.ats * sizeof(T));
                epilogue(g0 + gi, at, ROLES ? reinterpret_cast<const frag *>(records + (size_t)st * G.rec_bytes) + (size_t)(gi * TPG) * TILE_FRAGS : gt);
            }
            if (!(ROLES && late) || ng <= 0) stage_sync();      // (every wavefront: one barrier per stage)
        }
    } else {
        constexpr int SPG = TPG / STAGE_TILES;                          // stages per group
        int st = stage_begin;                                           // a multiple of SPG
        const int group_end = stage_end / SPG < groups ? stage_end / SPG : groups;
#pragma unroll 1
        for (int gr = stage_begin / SPG; gr < group_end; ++gr) {
            zero_acc();
            static_for<0, SPG, 1>([&](auto ssc) {
                constexpr int ss = decltype(ssc)::value;
                if (st + 1 < stage_end) prefetch(st + 1);
                const frag *tiles = reinterpret_cast<const frag *>(smem + (st & 1) * G.rec_bytes);
                mfma_run(tiles, std::integral_constant<int, STAGE_TILES>{},
                         std::integral_constant<int, ss * STAGE_TILES>{});
                if constexpr (ss == SPG - 1) epilogue(gr, nullptr, tiles);
                stage_sync();
                ++st;
            });
        }
    }

    // ---- outputs
    if (!SLICED && a.V_out) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const long long c = wave_base + ct * 32 + col;
            float v = V[ct];
            if (!(v == v)) v = -INFINITY;
            if (h == 0 && c < a.count) a.V_out[c] = v;
        }
    }
    if (a.blk_v) {
        float bv = -INFINITY;
        long long bi = LLONG_MAX;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const long long c = wave_base + ct * 32 + col;
            float v = V[ct];
            if (!(v == v)) v = -INFINITY;
            if (c < a.count && (v > bv || (v == bv && a.index_base + c < bi))) { bv = v; bi = a.index_base + c; }
        }
#pragma unroll
        for (int d = 16; d >= 1; d >>= 1) {          // both lane halves hold the same values
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


// ------------------------------------------------------------------------------------------
// The same sweep for wide games (N a multiple of 32 with two or four row tiles per type; leader
// rows in LDS; one type per stage).  Every wavefront sweeps TWO pairs of candidate tiles against
// each staged type, one pair after the other, so a workgroup of four wavefronts covers 512
// candidates per copy of the packed payoffs: stage copies (global memory -> LDS) slow the matrix
// pipe down roughly in proportion to the bytes a compute unit copies, and this halves them.  The
// fragments and the leader rows of a stage have LDS buffers of their own, two each; the one
// workgroup barrier per type stands at the start of the type, behind it the other buffers are free
// and the copies issued one type ago have landed, so a copy has a whole type to arrive.
// Epilogue: both candidate tiles of a pair advance together, stage by stage, so that every
// exchange with the partner lane (through the LDS crossbar) and every gather is in flight while
// the other tile's vector work is issued: the maxima of the grid's rows and columns, the map of
// those that hold the pair's maximum, the leader column at its two bits; anything but two bits
// goes to the exact routine.  Arithmetic, operand order, packing and the exact-tie routine are
// those of sweep_mfma_kernel: the same bits per candidate.
// FULL: rows of MP components; shorter ones have a kernel of their own (two registers of it are
// spilled where it loads its rows, none in the loop over the types).
template <typename T, int MP, int N, int WAVES, int PF, bool FULL>
__global__ void __launch_bounds__(WAVES * 64, 2)
sweep_wide_kernel(GameView g, SweepArgs a, int row_tiles)
{
    constexpr int NT = 2, NP = 2;              // candidate tiles per pass, passes per staged type
    typedef Path<T, MP> P;
    typedef typename P::frag frag;
    typedef typename P::xreg xreg;
    constexpr int KS = P::KSTEPS, HALF = P::HALF;
    constexpr Geometry G = make_geometry((int)sizeof(T), MP, N, N / 32, WAVES, true);
    constexpr int TPG = G.tpg;
    static_assert(N % 32 == 0 && (TPG == 2 || TPG == 4) && G.ts == 1, "one type of two or four row tiles per stage");
    static_assert(std::is_same<T, __bf16>::value, "bf16 matrix cores");
    constexpr int TILE_FRAGS = KS * 64;
    constexpr int FRAG_BYTES = TPG * G.tile_bytes;                      // the stage's fragments
    constexpr int LROW_CHUNKS = (G.at_bytes + 1023) / 1024;             // its leader rows, in 1 KiB copies
    constexpr int LROW_BYTES = LROW_CHUNKS * 1024;
    static_assert(FRAG_BYTES % (WAVES * 1024) == 0 && FRAG_BYTES + LROW_BYTES <= G.rec_bytes, "record layout");
    constexpr int NCH = TPG * KS / PF;                                  // fragment chunks per type
    static_assert(PF > 0 && KS % PF == 0 && NCH % 2 == 0, "chunk 0 of every pass lands in the same registers");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // F[2], then L[2]
    __shared__ float red_v[WAVES];
    __shared__ long long red_i[WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, col = lane & 31;
    const int m = g.m, K = g.K;
    const unsigned char *records = reinterpret_cast<const unsigned char *>(g.Bpack);
    const unsigned char *ATpack = reinterpret_cast<const unsigned char *>(g.ATpack);
    const long long wave_base = ((long long)blockIdx.x * WAVES + wave) * (NP * NT * 32);
    const int partner_addr = 4 * (lane ^ 32);
    (void)row_tiles;

    auto copy_stage = [&](int st, int buf) __attribute__((always_inline)) {
        const unsigned char *src = records + (size_t)st * G.rec_bytes;
        unsigned char *dstF = smem + buf * FRAG_BYTES;
        unsigned char *dstL = smem + 2 * FRAG_BYTES + buf * LROW_BYTES;
#pragma unroll
        for (int i = 0; i < FRAG_BYTES / (WAVES * 1024); ++i) {
            const int chunk = i * WAVES + wave;
            __builtin_amdgcn_global_load_lds((global_ptr)(src + chunk * 1024 + lane * 16),
                                             (lds_ptr)(dstF + chunk * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < (LROW_CHUNKS + WAVES - 1) / WAVES; ++i) {
            const int chunk = i * WAVES + wave;
            if (chunk < LROW_CHUNKS)                                     // wave-uniform
                __builtin_amdgcn_global_load_lds((global_ptr)(src + FRAG_BYTES + chunk * 1024 + lane * 16),
                                                 (lds_ptr)(dstL + chunk * 1024), 16, 0, 0);
        }
    };
    copy_stage(0, 0);

    // ---- candidate rows into registers (as in sweep_mfma_kernel), both passes
    constexpr int HALF_BASE = MP / 2;
    xreg x[NP][NT][P::XREGS];
    unsigned valid32[NP][NT];
#pragma unroll
    for (int ps = 0; ps < NP; ++ps)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const long long c = wave_base + (ps * NT + ct) * 32 + col;
            const bool ok = c < a.count;                     // (past the end: the last row again)
            float vb[HALF_BASE];
            const float *row = a.X + (ok ? c : a.count - 1) * (long long)m + h * HALF_BASE;
            if constexpr (FULL) {                            // (rows are then 16-byte aligned)
#pragma unroll
                for (int e = 0; e < HALF_BASE; e += 4) {
                    const f32x4 q = *(const f32x4 *)(row + e);
                    vb[e] = q[0]; vb[e + 1] = q[1]; vb[e + 2] = q[2]; vb[e + 3] = q[3];
                }
            } else {
                load_half_row<HALF_BASE>(row - h * HALF_BASE, h, m, vb);
            }
            P::pack_x(vb, x[ps][ct]);
            valid32[ps][ct] = (unsigned)__builtin_amdgcn_ballot_w64(ok);
        }

    float V[NP][NT];
#pragma unroll
    for (int ps = 0; ps < NP; ++ps)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) V[ps][ct] = 0.0f;
    unsigned tie_count = 0;                   // wave-uniform

    // Exact routine for one (candidate tile, type), as in sweep_mfma_kernel: the type's tiles once
    // more from the packed records in global memory (same instructions, same bits), the exact
    // maximisers in ascending action order, the leader's payoff decides and then the lower action.
    auto exact_type = [&](const xreg *xc, unsigned valid, int t, float gmax, float &l_out, int &j_out) __attribute__((always_inline)) {
        float lbest = kNotANumber;               // (no maximiser: no sum is a number)
        int jbest = 0, nmatch = 0;
        const unsigned char *ATt = ATpack + (size_t)t * N * MP * sizeof(T);
#pragma unroll 1
        for (int tt = 0; tt < TPG; ++tt) {
            const frag *afrags = reinterpret_cast<const frag *>(
                records + (size_t)t * G.rec_bytes + (size_t)tt * G.tile_bytes);
            f32x16 acc1;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc1[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < KS; ++s) acc1 = P::mfma(afrags[s * 64 + lane], xc, s, acc1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = 4 * q + rr;
                        const int j = tt * 32 + acc_row_base(r) + 4 * hh;
                        const unsigned long long meq = __builtin_amdgcn_ballot_w64(acc1[r] == gmax);
                        const unsigned hit = (unsigned)(hh ? (meq >> 32) : meq) & valid;
                        if (hit == 0u) continue;                       // wave-uniform
                        const float l = pair_sum(P::half_dot(xc, ATt + ((size_t)j * MP + h * HALF) * sizeof(T)));
                        if ((hit >> col) & 1u) {
                            if (nmatch == 0 || l > lbest) { lbest = l; jbest = j; }
                            ++nmatch;
                        }
                    }
        }
        l_out = lbest; j_out = jbest;
        tie_count += __builtin_popcount((unsigned)__builtin_amdgcn_ballot_w64(nmatch >= 2));
    };

    f32x16 acc[NT][TPG];
    frag fb[2][PF];
    auto read_chunk = [&](const frag *lane_base, auto qc, frag (&dst)[PF]) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int e = 0; e < PF; ++e) {
            constexpr int f0 = q * PF;
            const int f = f0 + e;                                        // flat (tile, k-step)
            dst[e] = lane_base[(size_t)(f / KS) * TILE_FRAGS + (size_t)(f % KS) * 64];
        }
    };
    // MFMAs of one type for one pair of candidate tiles; chunk 0 of the fragments is already in
    // fb[0]; chunk q+1 is read before the MFMAs of chunk q are issued.
    auto mfma_type = [&](const frag *lane_base, const xreg (*xp)[P::XREGS]) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int tt = 0; tt < TPG; ++tt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ct][tt][r] = 0.0f;
        static_for<0, NCH, 1>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if constexpr (q + 1 < NCH) read_chunk(lane_base, std::integral_constant<int, q + 1>{}, fb[(q + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, PF, 1>([&](auto ec) {
                constexpr int f = q * PF + decltype(ec)::value;
                constexpr int tt = f / KS, ks = f % KS;
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) acc[ct][tt] = P::mfma(fb[q & 1][decltype(ec)::value], xp[ct], ks, acc[ct][tt]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Epilogue of type t for one pair of candidate tiles (rows xp, validity masks vp, values Vp);
    // leader rows of the type in Lt.
    auto epilogue = [&](int t, float pt, const lds_byte *Lt, const xreg (*xp)[P::XREGS], const unsigned *vp,
                        float *Vp, long long cbase) __attribute__((always_inline)) {
        // The asm blocks read the accumulators, and the compiler's hazard handling does not look into
        // inline asm: the wait states a vector read of a fresh MFMA result needs (passes + 3 = 11) are
        // explicit, and the accumulators are tied to them.
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15");
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int tt = 0; tt < TPG; ++tt) asm volatile("" : "+v"(acc[ct][tt]));
        // stage 1: the maxima of the grid's rows and columns; the lane maximum goes to the partner lane
        typedef ArgGrid<TPG> Grid;
        float R[NT][Grid::ROWS], C[NT][Grid::COLS], pm[NT], pm_other[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            float u[TPG][16];
#pragma unroll
            for (int tt = 0; tt < TPG; ++tt)
#pragma unroll
                for (int r = 0; r < 16; ++r) u[tt][r] = acc[ct][tt][r];
            pm[ct] = grid_maxima<TPG>(u, R[ct], C[ct]);
            pm_other[ct] = pair_other(pm[ct], partner_addr);
            __builtin_amdgcn_sched_barrier(0);
        }
        // stage 2: the pair's maximum; the map of the rows and columns that hold it goes to the partner
        float gm[NT];
        unsigned map[NT], map_other[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            gm[ct] = vmax2(pm[ct], pm_other[ct]);
            map[ct] = grid_map<TPG>(R[ct], C[ct], gm[ct], 4u * h);
            map_other[ct] = (unsigned)__builtin_amdgcn_ds_bpermute(partner_addr, (int)map[ct]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // stage 3: the action, the gather of its leader column, and whether the tile is clean
        int js[NT];
        bool clean[NT];
        typename P::colregs cr[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const unsigned both = map[ct] | map_other[ct];
            // (masked: a wavefront that is not clean may hold any bits here, and the gather is issued
            // before that is known)
            const unsigned jg = grid_action<TPG>(both) & (unsigned)(N - 1);
            js[ct] = (int)jg;
            P::gather_half(Lt + (unsigned)((jg * G.ats + h * HALF) * sizeof(T)), cr[ct]);
            clean[ct] = __builtin_amdgcn_ballot_w64(__builtin_popcount(both) != 2) == 0ull;      // wave-uniform
            __builtin_amdgcn_sched_barrier(0);
        }
        // stage 4: leader payoffs (each lane its half, the partner the other) and the value
        float l[NT];
        if (clean[0] && clean[1]) {
            float part[NT], part_other[NT];
            P::half_dot_regs2(xp[0], cr[0], xp[1], cr[1], part[0], part[1]);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) part_other[ct] = pair_other(part[ct], partner_addr);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
                l[ct] = h ? part_other[ct] + part[ct] : part[ct] + part_other[ct];      // (lower half) + (upper half)
        } else {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                if (clean[ct]) {
                    const float part = P::half_dot_regs(xp[ct], cr[ct]);
                    const float other = pair_other(part, partner_addr);
                    l[ct] = h ? other + part : part + other;
                } else {
                    exact_type(xp[ct], vp[ct], t, gm[ct], l[ct], js[ct]);
                }
            }
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            Vp[ct] = fmaf(pt, l[ct], Vp[ct]);
            if (a.br_out) {
                const long long c = cbase + ct * 32 + col;
                if (h == 0 && c < a.count) a.br_out[c * K + t] = js[ct];
            }
        }
    };

    const frag *F0 = reinterpret_cast<const frag *>(smem) + lane;
    const frag *F1 = reinterpret_cast<const frag *>(smem + FRAG_BYTES) + lane;
    const lds_byte *L0 = (const lds_byte *)smem + (unsigned)(2 * FRAG_BYTES);
#pragma unroll 1
    for (int t = 0; t < K; ++t) {
        // own copies of this type's stage have landed; then everyone's have, and everyone is done with
        // the previous type, whose buffers take the next type's stage
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t + 1 < K) copy_stage(t + 1, (t + 1) & 1);
        const float pt = ((uniform_floats)g.prior)[t];
        const frag *Ft = (t & 1) ? F1 : F0;
        const lds_byte *Lt = L0 + (unsigned)((t & 1) * LROW_BYTES);
        read_chunk(Ft, std::integral_constant<int, 0>{}, fb[0]);
#pragma unroll
        for (int ps = 0; ps < NP; ++ps) {
            mfma_type(Ft, x[ps]);
            if (ps + 1 < NP) read_chunk(Ft, std::integral_constant<int, 0>{}, fb[0]);   // the next pass's first fragments
            epilogue(t, pt, Lt, x[ps], valid32[ps], V[ps], wave_base + ps * NT * 32);
        }
    }

    // ---- outputs (as in sweep_mfma_kernel)
    if (a.V_out) {
#pragma unroll
        for (int ps = 0; ps < NP; ++ps)
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const long long c = wave_base + (ps * NT + ct) * 32 + col;
                float v = V[ps][ct];
                if (!(v == v)) v = -INFINITY;
                if (h == 0 && c < a.count) a.V_out[c] = v;
            }
    }
    if (a.blk_v) {
        float bv = -INFINITY;
        long long bi = LLONG_MAX;
#pragma unroll
        for (int ps = 0; ps < NP; ++ps)
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const long long c = wave_base + (ps * NT + ct) * 32 + col;
                float v = V[ps][ct];
                if (!(v == v)) v = -INFINITY;
                if (c < a.count && (v > bv || (v == bv && a.index_base + c < bi))) { bv = v; bi = a.index_base + c; }
            }
#pragma unroll
        for (int d = 16; d >= 1; d >>= 1) {          // both lane halves hold the same values
            const float ov = __shfl_xor(bv, d, 64);
            const long long oi = __shfl_xor(bi, d, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { red_v[wave] = bv; red_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            for (int w2 = 1; w2 < WAVES; ++w2)
                if (red_v[w2] > bv || (red_v[w2] == bv && red_i[w2] < bi)) { bv = red_v[w2]; bi = red_i[w2]; }
            a.blk_v[blockIdx.x] = bv;
            a.blk_i[blockIdx.x] = bi;
        }
    }
    if (a.tie_counter && lane == 0 && tie_count) atomicAdd(a.tie_counter, (unsigned long long)tie_count);
}

// ------------------------------------------------------------------------------------------
// Instantiation table.
struct Variant {
    int mode;                    // 0 fp32 MFMA, 1 bf16 MFMA on rounded operands, 2 bf16 MFMA on split fp32
    int terms;                   // 1, or the number of part products of the split (3 or 6)
    int mp_base, n, nt, waves, stage_tiles;
    bool at_lds;
    bool cut;                    // part products are left out where they decide nothing (see mfma_filter)
    void (*kernel)(GameView, SweepArgs, int);     // null when `wide` sweeps this packing
    void (*sliced)(GameView, SweepArgs, int);     // one candidate tile per wavefront, types sliced
    Geometry geo;
    const char *name;
    void (*wide)(GameView, SweepArgs, int);       // sweep_wide_kernel for this packing and rows of m_pad components, or null
    void (*wide_part)(GameView, SweepArgs, int);  // the same for shorter rows
    int wide_lds;                                 // its dynamic LDS bytes
    int side;                                     // workgroups a compute unit holds where that is one or two, else 0
    bool fp6;                                     // sweep_fp6.hip
};

// (A few rows on six products wait for latencies, not for matrix instructions: they leave nothing out.)
#define BSSE_VARIANT(T, MODE, TERMSv, MPB, Nv, NTv, Wv, STv, OCCv, ATL, PFv, CUTv, NAME)             \
    { MODE, TERMSv, MPB, Nv, NTv, Wv, STv, ATL, CUTv,                                                \
      sweep_mfma_kernel<T, MPB * TERMSv, Nv, NTv, Wv, STv, OCCv, ATL, TERMSv, false, PFv, CUTv>,     \
      sweep_mfma_kernel<T, MPB * TERMSv, Nv, 1, Wv, STv, 1, ATL, TERMSv, true, PFv, CUTv && TERMSv != 6>, \
      make_geometry((int)sizeof(T), MPB * TERMSv, Nv, STv, Wv, ATL, TERMSv), NAME, nullptr, nullptr, 0, Wv == 8 ? 1 : 0, false }
// A packing that sweep_wide_kernel also takes (one type per stage, leader rows in LDS, NT = 2)
#define BSSE_VARIANT_WIDE(T, MODE, MPB, Nv, Wv, PFv, NAME)                                           \
    { MODE, 1, MPB, Nv, 2, Wv, Nv / 32, true, false,                                                 \
      nullptr,                                                                                       \
      sweep_mfma_kernel<T, MPB, Nv, 1, Wv, Nv / 32, 1, true, 1, true, PFv, false>,                   \
      make_geometry((int)sizeof(T), MPB, Nv, Nv / 32, Wv, true), NAME,                               \
      sweep_wide_kernel<T, MPB, Nv, Wv, PFv, true>, sweep_wide_kernel<T, MPB, Nv, Wv, PFv, false>, wide_lds_bytes((int)sizeof(T), MPB, Nv, Wv), 1, false }

// The six-bit kernel for the games of (<=128, 256) with three products: a type per stage, two workgroups a compute unit.
Variant fp6_variant()
{
    Geometry q{};
    q.tpg = 8; q.types = q.ts = 1; q.rec_bytes = fp6_record_bytes();
    return { 2, 3, 128, 256, 1, 4, 8, false, true, fp6_kernel(false), fp6_kernel(true), q, "mfma_split3", nullptr, nullptr, 0, 2, true };
}

const Variant kVariants[] = {
    // fp32 MFMA (the last number: k-steps per fragment read-ahead chunk, 0 = the fragment reads are left
    // where they are used; the last flag: small part products are left out where they decide nothing.  n = 16
    // with six products keeps them: there are few to leave out (100 -> 106 us for 2^20 rows of m = 16, K = 16))
    BSSE_VARIANT(float, 0, 1, 8, 8, 4, 4, 1, 2, true, 0, false, "mfma_f32"),
    BSSE_VARIANT(float, 0, 1, 16, 16, 4, 4, 2, 2, true, 0, false, "mfma_f32"),
    BSSE_VARIANT(float, 0, 1, 32, 32, 4, 4, 4, 2, true, 0, false, "mfma_f32"),
    BSSE_VARIANT(float, 0, 1, 32, 64, 2, 4, 4, 2, true, 0, false, "mfma_f32"),
    BSSE_VARIANT(float, 0, 1, 128, 256, 1, 4, 2, 2, false, 0, false, "mfma_f32"),
    // bf16 MFMA, operands rounded to bf16
    // Candidate tiles a wavefront and wavefronts a SIMD: these kernels issue vector instructions most of the
    // time, and more wavefronts issue more of them, as long as registers and two stages in LDS allow it
    // (2^20 rows, K = 16, us: m = 16, n = 32 bf16, four tiles 91, two 85, one 92; m = 32, n = 16, four 118,
    // two 111, one 103; three products, two tiles a wavefront and one row tile a stage, four wavefronts a SIMD
    // 145, three 186, four tiles and two wavefronts 184; six products with n = 32 spill with four wavefronts,
    // 200, and with one tile wait for LDS, 199; 170 as they are)
    BSSE_VARIANT(__bf16, 1, 1, 16, 32, 2, 4, 2, 4, true, 0, false, "mfma_bf16"),
    BSSE_VARIANT(__bf16, 1, 1, 32, 16, 1, 4, 2, 4, false, 0, false, "mfma_bf16"),
    BSSE_VARIANT_WIDE(__bf16, 1, 64, 128, 8, 4, "mfma_bf16"),
    // bf16 MFMA on fp32 operands split into bf16 parts
    BSSE_VARIANT(__bf16, 2, 6, 16, 16, 2, 4, 2, 2, true, 0, false, "mfma_split6"),
    BSSE_VARIANT(__bf16, 2, 6, 32, 32, 2, 4, 1, 3, true, 0, true, "mfma_split6"),
    BSSE_VARIANT(__bf16, 2, 3, 32, 32, 2, 4, 1, 4, true, 0, true, "mfma_split3"),
    BSSE_VARIANT(__bf16, 2, 6, 32, 64, 2, 4, 2, 2, true, 0, true, "mfma_split6"),
    // (for games where the small products decide too often; behind those that leave them out)
    BSSE_VARIANT(__bf16, 2, 6, 32, 32, 2, 4, 1, 3, true, 0, false, "mfma_split6"),
    BSSE_VARIANT(__bf16, 2, 6, 32, 64, 2, 4, 2, 2, true, 0, false, "mfma_split6"),
    // (one fragment ahead: the next one's LDS read runs under two matrix instructions; two ahead spill.  Six
    // registers are spilled as it is, three read back per type, and four of m = n = 32 with three products)
    BSSE_VARIANT(__bf16, 2, 3, 128, 256, 1, 8, 8, 2, false, 1, true, "mfma_split3"),
    // the same games with small whole-number payoffs (fp6_suits)
    fp6_variant(),
};
constexpr int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));
constexpr int kSmallVariant = 1000;          // the small-game kernel (sweep_small.hip)

int row_tiles_for(const Variant &v, int K)
{
    if (v.n >= 32) return K * (v.n / 32);
    const int tpt = 32 / v.n;
    return (K + tpt - 1) / tpt;
}

// bf16 parts of a value: hi, mid, lo with v = hi + mid + lo up to the rounding of lo
void bf16_parts(float v, float part[3])
{
    auto rne = [](float f) {
        uint32_t b; memcpy(&b, &f, 4);
        b += 0x7FFFu + ((b >> 16) & 1u);
        b &= 0xFFFF0000u;
        memcpy(&f, &b, 4);
        return f;
    };
    part[0] = rne(v);
    const float r1 = v - part[0];
    part[1] = rne(r1);
    const float r2 = r1 - part[1];
    part[2] = rne(r2);
}

}  // namespace

int mfma_select(int m, int n, int K, int mode, bool exact)
{
    if (mode == 0 && small_supported(m, n, K, 0)) return kSmallVariant;
    int best = -1;
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        if (v.fp6 || v.mode != mode || v.n != n || v.mp_base < m) continue;
        if (v.terms == 3 && !exact) continue;
        // smallest padded m wins; among equals, fewer terms
        if (best < 0 || v.mp_base < kVariants[best].mp_base ||
            (v.mp_base == kVariants[best].mp_base && v.terms < kVariants[best].terms))
            best = i;
    }
    return best;
}

const char *mfma_variant_name(int variant)
{
    if (variant == kSmallVariant) return "mfma_small_split6";
    return (variant >= 0 && variant < kNumVariants) ? kVariants[variant].name : "";
}

bool mfma_is_six_bit(int variant) { return variant >= 0 && variant < kNumVariants && kVariants[variant].fp6; }
bool mfma_is_small(int variant) { return variant == kSmallVariant; }

long long mfma_num_blocks(int variant, long long count)
{
    if (variant == kSmallVariant) return small_num_blocks(count);
    const Variant &v = kVariants[variant];
    const long long per = (long long)v.nt * 32 * v.waves * (v.wide ? 2 : 1);     // candidates per workgroup record
    return (count + per - 1) / per;
}

// The limit of the static scratch is one of candidates too: n <= 32 with one or three products count 512 to a
// record, of which the workgroups may take as few as 128, and the six-bit kernel 256, of which they take 128.
long long mfma_limit_blocks(int variant, long long count)
{
    const Variant &v = kVariants[variant];
    if (v.fp6) return (count + 255) / 256;
    return v.n <= 32 && v.terms != 6 ? (count + 511) / 512 : mfma_num_blocks(variant, count);
}

// Kernels of eight wavefronts fill a compute unit with one workgroup: the time of `blocks` blocks of rows and
// all types, cut into `slices`, in types of one candidate tile a wavefront.  A slice begins with its rows
// (two types' time).
static long long cut_time(long long blocks, int K, int slices, int side)
{
    return (blocks * slices + 256 * side - 1) / (256 * side) * ((K + slices - 1) / slices + 2);
}

// Stages per type slice of a sliced launch: 32 candidates per wavefront, whole groups per slice.
// Workgroups of four wavefronts: few rows are cut into about 1024 slices, four a compute unit (two thirds
// to one half of the time of 256: m = n = 32, K = 16, 10000 rows 21 -> 19 us; three products, 30000 rows
// 27 us with 512 and 24 with 1024).  Of eight: the number with the least time (m = 128, n = 256, K = 100,
// 40000 rows 593 -> 468 us; cut finer than rounds of 256 workgroups ask for, 1000 rows 37 -> 43).
static int stages_per_slice(const Variant &v, int K, long long count)
{
    const int nstages = (row_tiles_for(v, K) + v.stage_tiles - 1) / v.stage_tiles;
    const long long per = 32LL * v.waves, blocks = (count + per - 1) / per;
    int slices = 1;
    if (!v.side) {
        slices = blocks >= 1024 ? 1 : (int)(1024 / blocks);
    } else if (blocks < 4096 * v.side) {
        const int all = 256 * v.side;
        slices = blocks >= all ? 1 : (int)std::min<long long>(all / blocks, K);          // one round
        for (int s = slices + 1; s <= K && s <= 16; ++s)
            if (cut_time(blocks, K, s, v.side) < cut_time(blocks, K, slices, v.side)) slices = s;
    }
    const int spg = v.geo.tpg > v.stage_tiles ? v.geo.tpg / v.stage_tiles : 1;       // stages per group
    return ((nstages + slices - 1) / slices + spg - 1) / spg * spg;
}

int mfma_slices(const GameView &g, long long count)
{
    if (g.variant < 0 || g.variant >= kNumVariants) return 1;
    const Variant &v = kVariants[g.variant];
    const int nstages = (row_tiles_for(v, g.K) + v.stage_tiles - 1) / v.stage_tiles;
    const int sps = stages_per_slice(v, g.K, count);
    return (nstages + sps - 1) / sps;
}

long long mfma_row_blocks(const GameView &g, long long count)
{
    const long long per = 32LL * kVariants[g.variant].waves;
    return (count + per - 1) / per * mfma_slices(g, count);
}

// A workgroup of the unsliced kernel walks every type, whatever the number of rows: where they do not fill
// the chip, the same rows spread over types finish sooner, although one candidate tile per wavefront reads
// every fragment for 32 candidates only.  Workgroups of four wavefronts: up to 512 of them with one candidate
// tile each (40000 rows, us, whole and cut: m = n = 32, K = 16 39 and 30; n = 64 48 and 36; three products
// 40 and 25; m = 16, n = 32 bf16 29 and 21; m = n = 16 30 and 23; 100000 rows 43 and 52).  With K = 2 to 128 and
// 1000 to 200000 rows that is within 4 % of the better one, but for n = 64 and K = 64 or more (50000 rows, K = 64
// 110 and 123, K = 128 198 and 226).  Of eight: fewer whole workgroups than half the compute units, or where
// that is less time: the wide kernel takes its four candidate tiles in that of 2.5 here, and a type takes about
// n (0.0104 + 3.3e-5 terms m) us, a fit to times with the small products left out, in which `terms` counts
// them (us, whole or uncut in slices, and now: m = 64, n = 128, K = 64 bf16, 66000 rows 204 and 152; m = 128,
// n = 256, K = 100, 66000 rows 1187 and 829, 140000 rows 1859 and 1528; with fewer types the fit asks too much of
// the cut: K = 16, 40000 rows 132 whole, as it goes, and 106).
bool mfma_few_rows(const GameView &g, long long count)
{
    if (g.variant < 0 || g.variant >= kNumVariants) return false;
    const Variant &v = kVariants[g.variant];
    const long long per = 32LL * v.waves, blocks = (count + per - 1) / per, whole = mfma_num_blocks(g.variant, count);
    if (!v.side) return blocks <= 512 && mfma_slices(g, count) > 1;
    if (blocks >= 4096 * v.side) return false;
    const int slices = mfma_slices(g, count);
    if (whole <= 128 * v.side && (v.wide || slices > 1)) return true;
    const double type = v.n * (0.0104 + 3.3e-5 * v.terms * v.mp_base);
    const double outputs = (12.0 + 2e-6 * (double)count * g.K) / type;
    const long long all = 256 * v.side;
    return (double)cut_time(blocks, g.K, slices, v.side) + outputs < 0.95 * (v.wide ? 2.5 : 1.0) * (double)((whole + all - 1) / all * g.K);
}

// Once per game, on the game's device: kernels whose two stage buffers exceed the default 48 KiB of
// dynamic LDS get their limit raised here, not at every launch.
hipError_t mfma_prepare(int variant)
{
    if (variant == kSmallVariant) return hipSuccess;
    if (variant < 0 || variant >= kNumVariants) return hipErrorNotSupported;
    const Variant *v = &kVariants[variant];
    // (the most that any number of types takes on this kernel: the limit is the kernel's, not the game's)
    const size_t lds = (size_t)v->geo.rec_bytes * 2;
    if (v->wide && v->wide_lds > 48 * 1024) {
        for (const void *k : { (const void *)v->wide, (const void *)v->wide_part })
            if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, v->wide_lds); e != hipSuccess) return e;
    }
    if (lds <= 48 * 1024) return hipSuccess;
    hipError_t e = hipSuccess;
    if (v->kernel) e = hipFuncSetAttribute((const void *)v->kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)v->sliced, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    return e;
}

hipError_t launch_sweep_mfma(const GameView &g, const SweepArgs &a, hipStream_t s)
{
    if (a.count <= 0) return hipSuccess;
    if (g.variant == kSmallVariant) return launch_sweep_small(g, a, s);
    if (g.variant < 0 || g.variant >= kNumVariants) return hipErrorNotSupported;
    const Variant *v = &kVariants[g.variant];
    const int tiles = row_tiles_for(*v, g.K);
    const int nstages = (tiles + v->stage_tiles - 1) / v->stage_tiles;
    const size_t lds = (size_t)v->geo.rec_bytes * (nstages > 1 ? 2 : 1);
    auto kernel = a.l_out ? v->sliced : v->kernel;     // (mfma_prepare has raised their LDS limit)
    if (!a.l_out) {
        const long long blocks = mfma_num_blocks(g.variant, a.count);
        if (v->wide)       // (every wavefront sweeps two pairs of candidate tiles)
            hipLaunchKernelGGL((g.m == v->mp_base ? v->wide : v->wide_part), dim3((unsigned)blocks), dim3(v->waves * 64), (size_t)v->wide_lds, s, g, a, tiles);
        else
            hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(v->waves * 64), lds, s, g, a, tiles);
        return hipGetLastError();
    }
    // type-sliced evaluation
    const long long per = 32LL * v->waves, blocks = (a.count + per - 1) / per;
    if (a.blk_v || a.V_out || blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    SweepArgs b = a;
    b.slice_stages = stages_per_slice(*v, g.K, a.count);
    const int slices = (nstages + b.slice_stages - 1) / b.slice_stages;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, (unsigned)slices), dim3(v->waves * 64), lds, s, g, b,
                       tiles);
    return hipGetLastError();
}

// The filter's margins: per type t a number a_t such that in a row of norm r (as the kernels compute it) the
// products they leave out change no difference of two follower payoffs by r * a_t or more.
//
// Left out of six are (p0,B2) (p1,B1) (p2,B0) with p, B the parts of row and payoffs, of three p2 alone.
// By Cauchy and Schwarz |sum_i p_i B_ij| <= |p|_2 |B_j|_2.  For six, r bounds |p0|_2,
// 2^9 |p1|_2 and 2^18 |p2|_2, which are about equal for rows of ordinary numbers; for three, |p0|_2 / 2 and
// 2^18 |p2|_2, and the payoffs count from the middle of their range over the actions, which no difference
// notices.  Matrix instructions lose at most 8 2^-24 of the sum of their absolute products, which over all k-steps is
// |x|_2 |B_j|_2 at most, and 6 2^-24 of the sum that they go on with, each (measured with terms set for it): 2^-21 of
// |x|_2 |B_j|_2 is taken for each that goes on with the sum of the others (six: three a k-step, two k-steps or more).
// A sum of its own (three) comes to 2^-16 of that, and its addition rounds to 2^-24: 2^-23 is taken.  Both payoffs of a
// difference move: twice all that, and 2 % for the roundings of r, of a_t and of the threshold.  Rows and payoffs so
// small that parts underflow meet the two least values.
static void filter_margins(const Variant &v, int m, int n, int K, const float *B, float *margin)
{
    const int parts = v.terms == 6 ? 3 : 1;
    constexpr int MOST_N = 256;                              // of the variants
    for (int t = 0; t < K; ++t) {
        // squared norms of the actions' columns: parts 0, 1, 2, and centred
        double sum[4][MOST_N] = {};
        for (int i = 0; i < m; ++i) {
            const float *row = B + ((size_t)t * m + i) * n;
            if (parts == 1) {
                float lo = row[0], hi = row[0];
                for (int j = 1; j < n; ++j) { lo = row[j] < lo ? row[j] : lo; hi = row[j] > hi ? row[j] : hi; }
                const double mid = 0.5 * ((double)lo + hi);
                for (int j = 0; j < n; ++j) {
                    const double b = row[j], c = b - mid;
                    sum[0][j] += b * b; sum[3][j] += c * c;
                }
            } else {
                for (int j = 0; j < n; ++j) {
                    float part[3];
                    bf16_parts(row[j], part);
                    for (int q = 0; q < 3; ++q) sum[q][j] += (double)part[q] * part[q];
                }
            }
        }
        double norm[4] = { 0, 0, 0, 0 };
        for (int q = 0; q < 4; ++q) {
            for (int j = 0; j < n; ++j) norm[q] = norm[q] > sum[q][j] ? norm[q] : sum[q][j];
            norm[q] = sqrt(norm[q]);
        }
        const double left_out = parts == 1 ? norm[3] / kScale2 : norm[2] + norm[1] / kScale1 + norm[0] / kScale2;
        const double rounding = norm[0] * (parts == 1 ? 2 * 0x1p-23 : v.mp_base / 16 * 3 * 0x1p-21);
        const double a = 2 * 1.02 * (left_out + 1.01 * rounding);       // (|x|_2 is within 2^-8 of |p0|_2)
        margin[t] = (float)(a > kLeastMargin ? (a < 0x1p127 ? a : 0x1p127) : kLeastMargin);
    }
}

// The share of (candidate tile, type) pairs that a filter with these margins sums twice and that would not
// have been for a tie of equal columns, which every kernel does (and the filter's exact routine looks at the
// tied candidates only; `ties`: these count too): from the gaps between the greatest two payoffs in 64 pairs of up to eight types and
// rows of the flat Dirichlet distribution.  A gap is below the margin a sixteenth as often as below sixteen
// margins, of which 64 pairs show enough.
double twice_summed(int m, int n, int K, const float *B, const std::function<float(int)> &margin, int pairs,
                    bool ties)
{
    constexpr int PAIRS = 64;                                           // at most
    const int types = K < 8 ? K : 8, rows = pairs / types;
    float norm[PAIRS];
    std::vector<float> rows_of_x((size_t)rows * m), u(n);
    float *x[PAIRS];
    uint64_t state = 0;
    for (int r = 0; r < rows; ++r) {
        float sum = 0.0f, square = 0.0f;
        x[r] = rows_of_x.data() + (size_t)r * m;
        for (int i = 0; i < m; ++i) {
            uint64_t z = state += 0x9E3779B97F4A7C15ull;                // splitmix64
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            x[r][i] = -logf(((float)((z ^ (z >> 31)) >> 41) + 0.5f) * 0x1p-23f);
            sum += x[r][i]; square += x[r][i] * x[r][i];
        }
        for (int i = 0; i < m; ++i) x[r][i] /= sum;
        norm[r] = sqrtf(square) / sum;
    }
    double share = 0.0;
    for (int q = 0; q < types; ++q) {
        const int t = (int)((long long)q * K / types);
        const float room = margin(t);
        int near = 0, tied = 0;
        for (int r = 0; r < rows; ++r) {
            float first = -INFINITY, second = -INFINITY;
            const float *Bt = B + (size_t)t * m * n;
            int done = 0;
            for (; done + 16 <= n; done += 16) {                        // (sixteen sums in registers)
                float sum[16] = {};
                for (int i = 0; i < m; ++i)
                    for (int k = 0; k < 16; ++k) sum[k] += x[r][i] * Bt[(size_t)i * n + done + k];
                for (int k = 0; k < 16; ++k) u[done + k] = sum[k];
            }
            for (; done < n; ++done) {
                u[done] = 0.0f;
                for (int i = 0; i < m; ++i) u[done] += x[r][i] * Bt[(size_t)i * n + done];
            }
            for (int j = 0; j < n; ++j) {
                second = u[j] > first ? first : u[j] > second ? u[j] : second;
                first = u[j] > first ? u[j] : first;
            }
            tied += first == second;
            near += first > second && first - second < 16.0f * norm[r] * room;
        }
        const double clear = ties ? 1.0 : 1.0 - (double)tied / rows;
        if (ties) near += 16 * tied;
        share += (pow(clear, 32.0) - pow(std::max(0.0, clear - near / 16.0 / rows), 32.0)) / types;
    }
    return share;
}

// Games with equal columns tie in most tiles, which three parts settle sooner (every eighth column twice, K = 64, 65536
// rows 1820 us and 2170 on the six-bit instruction).
bool six_bit_suits(int m, int n, int K, const float *A, const float *B)
{
    return fp6_suits(m, n, K, A, B) && twice_summed(m, n, K, B, [](int) { return 0.0f; }, 64, true) <= 0.25;
}

// The margins grow with the payoffs, the gaps with what tells them apart: payoffs with a large part in common
// make the filter sum most tiles twice, at the pace of one chain.  From about a quarter of them on, six
// products sum everything at once (m = n = 32 and n = 64, K = 16, 2^20 rows, normal payoffs plus 0, 10, 30,
// 100 and 1000, us, filter and whole sums: 182 and 213, 190 and 210, 207 and 210, 259 and 211, 303 and 225; 265
// and 360, 322 and 356, 378 and 356, 486 and 365, 588 and 385; share 0.01, 0.11, 0.27, 0.65, 1).  Three products
// have no other variant: payoffs that are bf16 numbers differ by 2^-8 of their size if they differ (whole
// numbers 248..255 in place of 0..7: 143 -> 150 us, and 443 -> 507 for m = 128, n = 256, where all products at
// once took 203 and 623).
int mfma_filter(int variant, int m, int n, int K, const float *A, const float *B, float *margin)
{
    if (variant < 0 || variant >= kNumVariants || !kVariants[variant].cut) return variant;
    const Variant &v = kVariants[variant];
    if (v.terms == 3 && v.n == 256 && six_bit_suits(m, n, K, A, B)) {
        fp6_margins(m, K, B, margin);
        for (int i = 0; i < kNumVariants; ++i)
            if (kVariants[i].fp6) return i;
    }
    filter_margins(v, m, n, K, B, margin);
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &w = kVariants[i];
        if (w.mode == v.mode && w.terms == v.terms && w.mp_base == v.mp_base && w.n == v.n && !w.cut)
            return twice_summed(m, n, K, B, [=](int t) { return margin[t]; }, 64, false) > 0.25 ? i : variant;
    }
    return variant;
}

// Host packing.
// The contraction index of a variant runs over MP = terms * mp_base slots.  Lane half h owns
// slots h*MP/2 .. (h+1)*MP/2; within a half, slot = term * mp_base/2 + (i - h*mp_base/2) for the
// leader actions i of that half, and the value stored at (term, i) is part q(term) of the payoff:
// the payoff itself when terms == 1, parts (0,1,0,2,1,0) for six terms, (0,0,0) for three (whose
// fragments hold the first block only: the kernel uses each for all three terms; those of six terms hold
// parts 0, 1 and 2 once).
// Bpack = stage records (see Geometry): per stage, STAGE_TILES row tiles, each laid out as
// [k-step][lane 0..63][fragment], where lane = 32*h + rowInTile supplies the slots
// h*MP/2 + (elements per lane)*s + e of (type, action) row 32*tile + rowInTile; then, when the
// variant keeps leader rows in LDS, the rows [type slot][action][MP + pad] of the types the
// stage covers, in the same slot order.  Rows past K*n and actions past m are zero.
// ATpack = [K][n][MP] leader payoffs in slot order (zero padded), so that a lane's half of a
// column is contiguous; used by the global gather and by the exact routine.  Six-term variants that
// keep leader rows in LDS carry them as plain fp32 instead, in the stage records ([type slot]
// [action][mp_base + 4]) and in ATpack ([K][n][mp_base]).
void mfma_pack(int variant, int m, int n, int K, const float *A, const float *B, void **Bpack,
               size_t *Bbytes, void **ATpack, size_t *ATbytes, int *m_pad, int *n_pad)
{
    *Bpack = nullptr; *ATpack = nullptr; *Bbytes = 0; *ATbytes = 0;
    if (variant == kSmallVariant) {
        *m_pad = 8; *n_pad = n;
        small_pack(m, n, K, A, B, Bpack, Bbytes, ATpack, ATbytes);
        return;
    }
    if (variant < 0 || variant >= kNumVariants) return;
    const Variant *v = &kVariants[variant];
    const Geometry &G = v->geo;
    const int MP = v->mp_base * v->terms, half = MP / 2, half_base = v->mp_base / 2;
    const bool bf = v->mode != 0;
    const int epl = bf ? 8 : 1;                            // k-slots per lane per MFMA
    const int ks = half / epl / (v->terms == 3 ? 3 : v->terms == 6 ? 2 : 1);         // stored fragments per tile and lane
    const int tiles = row_tiles_for(*v, K);
    const int nstages = (tiles + v->stage_tiles - 1) / v->stage_tiles;
    const size_t esz = bf ? 2 : 4;
    static const int bsel6[6] = { 0, 1, 0, 2, 1, 0 };
    *m_pad = v->mp_base; *n_pad = n;
    if (v->fp6) {
        *Bbytes = (size_t)K * G.rec_bytes; *ATbytes = (size_t)K * n * v->mp_base * 2;
        *Bpack = calloc(*Bbytes, 1); *ATpack = calloc(*ATbytes, 1);
        if (*Bpack && *ATpack) fp6_pack(m, K, A, B, (unsigned char *)*Bpack, (unsigned short *)*ATpack);
        return;
    }
    *Bbytes = (size_t)nstages * G.rec_bytes;
    const bool lead_f32 = v->terms == 6 && v->at_lds;       // leader rows as plain fp32
    *ATbytes = lead_f32 ? (size_t)K * n * v->mp_base * sizeof(float) : (size_t)K * n * MP * esz;
    unsigned char *pb = (unsigned char *)calloc(*Bbytes, 1);
    unsigned char *pa = (unsigned char *)calloc(*ATbytes, 1);
    if (!pb || !pa) { free(pb); free(pa); return; }
    auto put = [&](unsigned char *base, size_t idx, float val) {
        if (bf) {
            uint32_t b; memcpy(&b, &val, 4);
            b += 0x7FFFu + ((b >> 16) & 1u);
            const uint16_t hb = (uint16_t)(b >> 16);
            memcpy(base + idx * 2, &hb, 2);
        } else {
            memcpy(base + idx * 4, &val, 4);
        }
    };
    // value stored at slot `li` (within lane half hh) of payoff matrix M (type t, action j)
    auto slot_value = [&](const float *M, int t, int j, int hh, int li, bool fragment) -> float {
        const int term = li / half_base, i = hh * half_base + li % half_base;
        if (t >= K || i >= m) return 0.0f;
        const float val = M[((size_t)t * m + i) * n + j];
        if (v->terms == 1) return val;
        float part[3];
        bf16_parts(val, part);
        return part[v->terms == 3 ? 0 : fragment ? term : bsel6[term]];
    };
    for (int tile = 0; tile < tiles; ++tile) {
        unsigned char *tb = pb + (size_t)(tile / v->stage_tiles) * G.rec_bytes +
                            (size_t)(tile % v->stage_tiles) * G.tile_bytes;
        for (int s = 0; s < ks; ++s)
            for (int lane = 0; lane < 64; ++lane) {
                const int hh = lane / 32, row = tile * 32 + lane % 32;
                const int t = row / n, j = row % n;
                for (int e = 0; e < epl; ++e)
                    put(tb, ((size_t)s * 64 + lane) * epl + e, slot_value(B, t, j, hh, epl * s + e, true));
            }
    }
    if (v->at_lds)
        for (int st = 0; st < nstages; ++st) {
            unsigned char *ab = pb + (size_t)st * G.rec_bytes + (size_t)v->stage_tiles * G.tile_bytes;
            for (int q = 0; q < G.ts; ++q) {
                const int t = st * G.ts + q;
                if (t >= K) break;
                for (int j = 0; j < n; ++j) {
                    if (lead_f32) {
                        float *row = reinterpret_cast<float *>(ab + ((size_t)q * n + j) * G.ats * esz);
                        for (int i = 0; i < v->mp_base; ++i) row[i] = i < m ? A[((size_t)t * m + i) * n + j] : 0.0f;
                        continue;
                    }
                    for (int hh = 0; hh < 2; ++hh)
                        for (int li = 0; li < half; ++li)
                            put(ab, ((size_t)q * n + j) * G.ats + hh * half + li, slot_value(A, t, j, hh, li, false));
                }
            }
        }
    for (int t = 0; t < K; ++t)
        for (int j = 0; j < n; ++j) {
            if (lead_f32) {
                float *row = reinterpret_cast<float *>(pa) + ((size_t)t * n + j) * v->mp_base;
                for (int i = 0; i < v->mp_base; ++i) row[i] = i < m ? A[((size_t)t * m + i) * n + j] : 0.0f;
                continue;
            }
            for (int hh = 0; hh < 2; ++hh)
                for (int li = 0; li < half; ++li)
                    put(pa, ((size_t)t * n + j) * MP + hh * half + li, slot_value(A, t, j, hh, li, false));
        }
    *Bpack = pb; *ATpack = pa;
}

}  // namespace bsse
