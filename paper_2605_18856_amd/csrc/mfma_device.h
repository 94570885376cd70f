// Device helpers shared by the matrix-core sweep kernels (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

namespace bsse {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A number that is none, as an inline constant (the usual bit pattern costs a register).
#define kNotANumber __uint_as_float(0xFFFFFFFFu)

// Row of a 32x32 MFMA accumulator tile held in register r of a lane, without the lane-half
// term 4*(lane/32): lane l holds column l%32 and rows 8*(r/4) + 4*(l/32) + r%4.
__device__ __host__ constexpr int acc_row_base(int r) { return 8 * (r / 4) + (r % 4); }

// max(a, b, c) / max(a, b) as single instructions.  (fmaxf() makes the compiler canonicalise
// every operand first -- one extra VALU instruction per input.)  NaN inputs are outside the
// contract; v_max3_f32 returns a non-NaN operand when there is one.
__device__ __forceinline__ float vmax3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ float vmax2(float a, float b)
{
    float d;
    asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

// Per-type numbers that every lane reads, through the scalar data cache.  (A plain load is a vector one
// behind inline asm that clobbers memory, and waiting for it waits for the stage copies in flight.)
typedef const float __attribute__((address_space(4))) *uniform_floats;
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

// Partner-lane helpers built on v_permlane32_swap: the two results hold, in every lane, the
// value of the lane with the same column in the lower half and in the upper half, so any
// commutative combination of them is the pair's result, identical in both lanes.
__device__ __forceinline__ float pair_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return vmax2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// The partner lane's value, through the LDS crossbar (no LDS memory is touched): this keeps
// the exchange off the vector ALU, where a swap costs two copies, the swap and a select.
// partner_addr = 4 * (lane ^ 32).
__device__ __forceinline__ float pair_other(float v, int partner_addr)
{
    return __uint_as_float((unsigned)__builtin_amdgcn_ds_bpermute(partner_addr, (int)__float_as_uint(v)));
}
__device__ __forceinline__ float pair_sum(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Compile-time loop: f(integral_constant<int, I>) for I = Begin, Begin+Step, ... (Step may be
// negative), so that loop indices can feed immediate operands.
template <int I, int End, int Step, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr ((Step > 0 && I < End) || (Step < 0 && I > End)) {
        f(std::integral_constant<int, I>{});
        static_for<I + Step, End, Step>(f);
    }
}

// Four steps of the "which register holds the maximum" pass:
//     sum += sum_k (u_k >= gmax ? c_k : 0),   k = 0..3
// (gmax: the maximum, or the maximum less a margin)
// where c_k = (action of register k) + 2^16, so that after all registers sum & 0xFFFF is the
// maximising action and sum >> 16 the number of maximisers (the action is only meaningful
// when that number is one; callers send every other case through an exact routine).
// Ten vector instructions for four values, nothing on the scalar unit.  Written as one asm
// block for two reasons: the four compare masks live in three scalar pairs plus vcc only
// inside the block (left to the scheduler, masks of many steps were kept alive and spilled),
// and every select stands three instructions behind its compare, which satisfies the two wait
// states this part needs between a vector write of a scalar register and a vector read of it.
__device__ __forceinline__ void match4(float u0, float u1, float u2, float u3, float gmax,
                                       unsigned c0, unsigned c1, unsigned c2, unsigned c3,
                                       unsigned &sum)
{
    unsigned t0, t1, t2, t3;
    unsigned long long m0, m1, m2;
    asm("v_cmp_ge_f32 %[m0], %[u0], %[g]\n\t"
        "v_cmp_ge_f32 %[m1], %[u1], %[g]\n\t"
        "v_cmp_ge_f32 %[m2], %[u2], %[g]\n\t"
        "v_cmp_ge_f32 vcc, %[u3], %[g]\n\t"
        "v_cndmask_b32 %[t0], 0, %[c0], %[m0]\n\t"
        "v_cndmask_b32 %[t1], 0, %[c1], %[m1]\n\t"
        "v_cndmask_b32 %[t2], 0, %[c2], %[m2]\n\t"
        "v_cndmask_b32 %[t3], 0, %[c3], vcc\n\t"
        "v_add3_u32 %[s], %[s], %[t0], %[t1]\n\t"
        "v_add3_u32 %[s], %[s], %[t2], %[t3]"
        : [s] "+v"(sum), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3),
          [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2)
        : [u0] "v"(u0), [u1] "v"(u1), [u2] "v"(u2), [u3] "v"(u3), [g] "v"(gmax),
          [c0] "v"(c0), [c1] "v"(c1), [c2] "v"(c2), [c3] "v"(c3)
        : "vcc");
}

// Four fp32 values as three bf16 parts each, x = x1 + x2 + x3: every part is the nearest bf16 of
// what is left, and what is left is formed exactly (a bf16 dot product with -1 in one slot and 0
// in the other subtracts one packed value from an fp32 number; the difference has at most 16
// significant bits).  p12 = (x1[0..3], x2[0..3]) and p31 = (x3[0..3], x1[0..3]) as eight bf16 each,
// the k-slot order of the small-game kernel's matrix instructions.
__device__ __forceinline__ void split_parts(const f32x4 &x, unsigned (&p12)[4], unsigned (&p31)[4])
{
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    // (-1, 0) and (0, -1) as packed bf16, kept in scalar registers as plain bit patterns: written
    // as constants they may be encoded as an inline operand of the dot instruction, and what that
    // operand expands to for a bf16 instruction is not something to rely on
    unsigned bits_lo = 0x0000BF80u, bits_hi = 0xBF800000u;
    asm("" : "+s"(bits_lo), "+s"(bits_hi));
    const v2bf minus_lo = __builtin_bit_cast(v2bf, bits_lo), minus_hi = __builtin_bit_cast(v2bf, bits_hi);
    // (a plain conversion, not inline asm: the compiler has to see the instruction to keep the
    // wait states between it and the dot products around it)
    auto pack = [](float a, float b) __attribute__((always_inline)) {
        typedef float v2f __attribute__((ext_vector_type(2)));
        const v2f ab = { a, b };
        return __builtin_bit_cast(unsigned, __builtin_convertvector(ab, v2bf));
    };
    auto rest = [&](unsigned packed, float a, float b, float &ra, float &rb) __attribute__((always_inline)) {
        const v2bf pv = __builtin_bit_cast(v2bf, packed);
        ra = __builtin_amdgcn_fdot2_f32_bf16(pv, minus_lo, a, false);
        rb = __builtin_amdgcn_fdot2_f32_bf16(pv, minus_hi, b, false);
    };
    float r[4], q[4];
    p12[0] = pack(x[0], x[1]); p12[1] = pack(x[2], x[3]);
    rest(p12[0], x[0], x[1], r[0], r[1]); rest(p12[1], x[2], x[3], r[2], r[3]);
    p12[2] = pack(r[0], r[1]); p12[3] = pack(r[2], r[3]);
    rest(p12[2], r[0], r[1], q[0], q[1]); rest(p12[3], r[2], r[3], q[2], q[3]);
    p31[0] = pack(q[0], q[1]); p31[1] = pack(q[2], q[3]);
    p31[2] = p12[0]; p31[3] = p12[1];
}

// Eight follower payoffs u with their maximum g, and the eight leader payoffs w beside them:
// l = w at the lowest position where u holds g; n_eq = how many (lane, position) pairs of the
// wavefront hold g (64 exactly when every lane has one maximiser); with WANT_IDX also that
// position.  Compare masks in scalar pairs, selects from the highest position down, the count on
// the scalar unit, every select at least two instructions behind its compare.
template <bool WANT_IDX>
__device__ __forceinline__ void argmax8_pick(const float (&u)[8], const float (&w)[8], float g, float &l,
                                             unsigned &idx, unsigned &n_eq)
{
    unsigned long long m0, m1, m2, m3, m4, m5, m6, m7;
    unsigned c, t;
    float lv;
    asm("v_cmp_eq_f32 %[m6], %[u6], %[g]\n\t"
        "v_cmp_eq_f32 %[m5], %[u5], %[g]\n\t"
        "v_cmp_eq_f32 %[m4], %[u4], %[g]\n\t"
        "v_cmp_eq_f32 %[m3], %[u3], %[g]\n\t"
        "v_cmp_eq_f32 %[m2], %[u2], %[g]\n\t"
        "v_cmp_eq_f32 %[m1], %[u1], %[g]\n\t"
        "v_cmp_eq_f32 %[m0], %[u0], %[g]\n\t"
        "v_cmp_eq_f32 %[m7], %[u7], %[g]\n\t"
        "v_cndmask_b32 %[l], %[w7], %[w6], %[m6]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w5], %[m5]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w4], %[m4]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w3], %[m3]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w2], %[m2]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w1], %[m1]\n\t"
        "v_cndmask_b32 %[l], %[l], %[w0], %[m0]\n\t"
        "s_bcnt1_i32_b64 %[c], %[m0]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m1]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m2]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m3]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m4]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m5]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m6]\n\t"
        "s_add_u32 %[c], %[c], %[t]\n\t"
        "s_bcnt1_i32_b64 %[t], %[m7]\n\t"
        "s_add_u32 %[c], %[c], %[t]"
        : [l] "=&v"(lv), [c] "=&s"(c), [t] "=&s"(t), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2),
          [m3] "=&s"(m3), [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7)
        : [u0] "v"(u[0]), [u1] "v"(u[1]), [u2] "v"(u[2]), [u3] "v"(u[3]), [u4] "v"(u[4]), [u5] "v"(u[5]),
          [u6] "v"(u[6]), [u7] "v"(u[7]), [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]),
          [w4] "v"(w[4]), [w5] "v"(w[5]), [w6] "v"(w[6]), [w7] "v"(w[7]), [g] "v"(g)
        : "scc");
    l = lv; n_eq = c;
    if constexpr (WANT_IDX) {
        // (evaluation mode only: the position itself, by the same rule)
        unsigned i = 7u;
#pragma unroll
        for (int j = 6; j >= 0; --j) i = u[j] == g ? (unsigned)j : i;
        idx = i;
    }
}

// (bv, bc) <- (v, c) in the lanes where v > bv; the mask in a scalar register pair.
__device__ __forceinline__ void keep_greater2(float v, unsigned c, float &bv, unsigned &bc)
{
    unsigned long long m;
    asm("v_cmp_gt_f32 %[m], %[v], %[bv]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32 %[bv], %[bv], %[v], %[m]\n\t"
        "v_cndmask_b32 %[bc], %[bc], %[c], %[m]"
        : [bv] "+v"(bv), [bc] "+v"(bc), [m] "=&s"(m)
        : [v] "v"(v), [c] "v"(c));
}

// (bv, bc, br[]) <- (v, c, r[]) in the lanes where v > bv; the mask in a scalar register pair.
template <int N> __device__ __forceinline__ void keep_greater_rows(float v, unsigned c, const float *r, float &bv, unsigned &bc, float *br)
{
    static_assert(N == 2 || N == 4, "rows of one or two row tiles");
    unsigned long long m;
#define BSSE_KEEP                                                               \
        "v_cmp_gt_f32 %[m], %[v], %[bv]\n\t"                                    \
        "s_nop 1\n\t"                                                           \
        "v_cndmask_b32 %[bv], %[bv], %[v], %[m]\n\t"                            \
        "v_cndmask_b32 %[bc], %[bc], %[c], %[m]\n\t"                            \
        "v_cndmask_b32 %[b0], %[b0], %[r0], %[m]\n\t"                           \
        "v_cndmask_b32 %[b1], %[b1], %[r1], %[m]\n\t"
    if constexpr (N == 2)
        asm(BSSE_KEEP
            : [bv] "+v"(bv), [bc] "+v"(bc), [b0] "+v"(br[0]), [b1] "+v"(br[1]), [m] "=&s"(m)
            : [v] "v"(v), [c] "v"(c), [r0] "v"(r[0]), [r1] "v"(r[1]));
    else
        asm(BSSE_KEEP
            "v_cndmask_b32 %[b2], %[b2], %[r2], %[m]\n\t"
            "v_cndmask_b32 %[b3], %[b3], %[r3], %[m]"
            : [bv] "+v"(bv), [bc] "+v"(bc), [b0] "+v"(br[0]), [b1] "+v"(br[1]), [b2] "+v"(br[2]), [b3] "+v"(br[3]), [m] "=&s"(m)
            : [v] "v"(v), [c] "v"(c), [r0] "v"(r[0]), [r1] "v"(r[1]), [r2] "v"(r[2]), [r3] "v"(r[3]));
#undef BSSE_KEEP
}

// number of leading zero bits; 0xFFFFFFFF for zero
__device__ __forceinline__ unsigned ffbh(unsigned x)
{
    unsigned r;
    asm("v_ffbh_u32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
// number of trailing zero bits; 0xFFFFFFFF for zero
__device__ __forceinline__ unsigned ffbl(unsigned x)
{
    unsigned r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
// Maximum of sixteen on top of p, in one block: the compiler pads every boundary between two asm
// statements with a no-op, so fewer, larger blocks save issue slots in the epilogue.
__device__ __forceinline__ float vmax_chain16(float p, const float *u)
{
    asm("v_max3_f32 %0, %0, %1, %2\n\t"
        "v_max3_f32 %0, %0, %3, %4\n\t"
        "v_max3_f32 %0, %0, %5, %6\n\t"
        "v_max3_f32 %0, %0, %7, %8\n\t"
        "v_max3_f32 %0, %0, %9, %10\n\t"
        "v_max3_f32 %0, %0, %11, %12\n\t"
        "v_max3_f32 %0, %0, %13, %14\n\t"
        "v_max3_f32 %0, %0, %15, %16"
        : "+v"(p)
        : "v"(u[0]), "v"(u[1]), "v"(u[2]), "v"(u[3]), "v"(u[4]), "v"(u[5]), "v"(u[6]), "v"(u[7]),
          "v"(u[8]), "v"(u[9]), "v"(u[10]), "v"(u[11]), "v"(u[12]), "v"(u[13]), "v"(u[14]), "v"(u[15]));
    return p;
}


// ---- the arg-max over whole row tiles ----------------------------------------------------
// A lane's TPG * 16 sums of one type (value r of row tile tt: action 32 tt + 8 (r / 4) + 4 h + r % 4) are
// taken as a grid of ROWS x COLS, action = 2 COLS * row + (position of the column): the maximum of every grid
// row and of every column, then a map with one bit for each of them that reaches the threshold.  One value
// alone there sets one row bit and one column bit; any second one, in the lane or in its partner (whose
// column bits lie elsewhere), sets a third, so a candidate has its unique maximiser exactly when the map of
// both lanes has two bits, and the places of its highest and lowest bit are the action.
// Vector instructions are what bounds these epilogues (each costs about 4.9 cycles beside the matrix
// instructions, whatever its kind): for four row tiles 64 + 4 for the maxima, 32 for sixteen values against
// the threshold and 8 for the map's bits.  Maxima per tile (32) and per position over the tiles (32), with
// four compares and selects for the tile, sixteen values against the threshold and a lane-wise count,
// took 13 more: m = 64, n = 128, K = 64 bf16, 2^22 rows 4.90 -> 4.75 ms; m = 128, n = 256, K = 256, 131072
// rows 3.29 -> 3.19 ms; one row tile (16 maxima and 8 compares in place of 8 and 16): m = 16, n = 32, K = 16
// bf16, 2^20 rows 104 -> 92 us.
template <int TPG> struct ArgGrid {
    static constexpr int ROWS = TPG == 1 ? 4 : 2 * TPG, COLS = TPG == 1 ? 4 : 8;
};
// Maximum of sixteen values, two independent streams interleaved: a wavefront that is alone in its epilogue
// (its neighbour on the SIMD being busy with matrix instructions) issues dependent vector instructions at
// about half rate.
__device__ __forceinline__ void vmax16x2(float &pa, const float *ua, float &pb, const float *ub)
{
#define BSSE_U4(x, a, b, c, d) [x##a] "v"(x[a]), [x##b] "v"(x[b]), [x##c] "v"(x[c]), [x##d] "v"(x[d])
#define BSSE_MX(a, b)                                                           \
        "v_max3_f32 %[pa], %[pa], %[ua" #a "], %[ua" #b "]\n\t"                  \
        "v_max3_f32 %[pb], %[pb], %[ub" #a "], %[ub" #b "]\n\t"
#define BSSE_MX_FIRST                                                           \
        "v_max3_f32 %[pa], %[ua0], %[ua1], %[ua2]\n\t"                          \
        "v_max3_f32 %[pb], %[ub0], %[ub1], %[ub2]\n\t"
    asm(BSSE_MX_FIRST BSSE_MX(3, 4) BSSE_MX(5, 6) BSSE_MX(7, 8) BSSE_MX(9, 10) BSSE_MX(11, 12) BSSE_MX(13, 14)
        "v_max_f32 %[pa], %[pa], %[ua15]\n\t"
        "v_max_f32 %[pb], %[pb], %[ub15]"
        : [pa] "=&v"(pa), [pb] "=&v"(pb)
        : BSSE_U4(ua, 0, 1, 2, 3), BSSE_U4(ua, 4, 5, 6, 7), BSSE_U4(ua, 8, 9, 10, 11),
          BSSE_U4(ua, 12, 13, 14, 15), BSSE_U4(ub, 0, 1, 2, 3), BSSE_U4(ub, 4, 5, 6, 7),
          BSSE_U4(ub, 8, 9, 10, 11), BSSE_U4(ub, 12, 13, 14, 15));
}
// The same for eight values.
__device__ __forceinline__ void vmax8x2(float &pa, const float *ua, float &pb, const float *ub)
{
    asm(BSSE_MX_FIRST BSSE_MX(3, 4) BSSE_MX(5, 6)
        "v_max_f32 %[pa], %[pa], %[ua7]\n\t"
        "v_max_f32 %[pb], %[pb], %[ub7]"
        : [pa] "=&v"(pa), [pb] "=&v"(pb)
        : BSSE_U4(ua, 0, 1, 2, 3), BSSE_U4(ua, 4, 5, 6, 7), BSSE_U4(ub, 0, 1, 2, 3), BSSE_U4(ub, 4, 5, 6, 7));
#undef BSSE_MX_FIRST
#undef BSSE_MX
}
// w[i] = max(a[i], b[i], c[i], d[i]), i = 0..3
__device__ __forceinline__ void vmax4x4(float *w, const float *a, const float *b, const float *c, const float *d)
{
    asm("v_max3_f32 %[w0], %[a0], %[b0], %[c0]\n\t"
        "v_max3_f32 %[w1], %[a1], %[b1], %[c1]\n\t"
        "v_max3_f32 %[w2], %[a2], %[b2], %[c2]\n\t"
        "v_max3_f32 %[w3], %[a3], %[b3], %[c3]\n\t"
        "v_max_f32 %[w0], %[w0], %[d0]\n\t"
        "v_max_f32 %[w1], %[w1], %[d1]\n\t"
        "v_max_f32 %[w2], %[w2], %[d2]\n\t"
        "v_max_f32 %[w3], %[w3], %[d3]"
        : [w0] "=&v"(w[0]), [w1] "=&v"(w[1]), [w2] "=&v"(w[2]), [w3] "=&v"(w[3])
        : BSSE_U4(a, 0, 1, 2, 3), BSSE_U4(b, 0, 1, 2, 3), BSSE_U4(c, 0, 1, 2, 3), BSSE_U4(d, 0, 1, 2, 3));
#undef BSSE_U4
}
// Maxima of the grid's rows, and of its columns.
template <int TPG> __device__ __forceinline__ void grid_rows(const float (&u)[TPG][16], float *R)
{
    if constexpr (TPG == 1) {
        float s[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e][q] = u[0][4 * q + e];
        vmax4x4(R, s[0], s[1], s[2], s[3]);
    } else {
#pragma unroll
        for (int t = 0; t < TPG; ++t) vmax8x2(R[2 * t], u[t], R[2 * t + 1], u[t] + 8);
    }
}
template <int TPG> __device__ __forceinline__ void grid_columns(const float (&u)[TPG][16], float *C)
{
    if constexpr (TPG == 1) {
        vmax4x4(C, u[0], u[0] + 4, u[0] + 8, u[0] + 12);
    } else if constexpr (TPG == 2) {
        vmax4x4(C, u[0], u[0] + 8, u[1], u[1] + 8);
        vmax4x4(C + 4, u[0] + 4, u[0] + 12, u[1] + 4, u[1] + 12);
    } else {
        float s[8][2 * TPG];
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int k = 0; k < 2 * TPG; ++k) s[c][k] = u[k / 2][8 * (k % 2) + c];
#pragma unroll
        for (int c = 0; c < 8; c += 2) {
            if constexpr (TPG == 4) vmax8x2(C[c], s[c], C[c + 1], s[c + 1]);
            else vmax16x2(C[c], s[c], C[c + 1], s[c + 1]);
        }
    }
}
// c[i] = max(c[i], a[i], b[i]), i = 0..7
__device__ __forceinline__ void vmax_into8(float *c, const float *a, const float *b)
{
#define BSSE_STEP(i) "v_max3_f32 %[c" #i "], %[c" #i "], %[a" #i "], %[b" #i "]\n\t"
#define BSSE_INOUT(i) [c##i] "+v"(c[i])
#define BSSE_IN(i) [a##i] "v"(a[i]), [b##i] "v"(b[i])
    asm(BSSE_STEP(0) BSSE_STEP(1) BSSE_STEP(2) BSSE_STEP(3) BSSE_STEP(4) BSSE_STEP(5) BSSE_STEP(6) BSSE_STEP(7)
        : BSSE_INOUT(0), BSSE_INOUT(1), BSSE_INOUT(2), BSSE_INOUT(3), BSSE_INOUT(4), BSSE_INOUT(5), BSSE_INOUT(6), BSSE_INOUT(7)
        : BSSE_IN(0), BSSE_IN(1), BSSE_IN(2), BSSE_IN(3), BSSE_IN(4), BSSE_IN(5), BSSE_IN(6), BSSE_IN(7));
#undef BSSE_STEP
#undef BSSE_INOUT
#undef BSSE_IN
}
// Both sets; returns the lane's maximum (from the smaller set).  COLS_FIRST: the eight column maxima before
// the rows', which for eight row tiles saves the registers that are spilled otherwise (m = 128, n = 256, 2000
// rows cut over K = 100 types: 51.0 us, rows first 53.0) but is slower in long launches (65536 rows of m = 100:
// 685 us, rows first 672).
template <int TPG, bool COLS_FIRST = false>
__device__ __forceinline__ float grid_maxima(const float (&u)[TPG][16], float *R, float *C)
{
    if constexpr (COLS_FIRST) grid_columns<TPG>(u, C);
    grid_rows<TPG>(u, R);
    if constexpr (!COLS_FIRST) grid_columns<TPG>(u, C);
    if constexpr (TPG <= 2) return vmax2(vmax3(R[0], R[1], R[2]), R[3]);
    float most;
    asm("v_max3_f32 %0, %1, %2, %3\n\t"
        "v_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\t"
        "v_max_f32 %0, %0, %8"
        : "=&v"(most)
        : "v"(C[0]), "v"(C[1]), "v"(C[2]), "v"(C[3]), "v"(C[4]), "v"(C[5]), "v"(C[6]), "v"(C[7]));
    return most;
}
// Two bit streams of four values each against a threshold, the first value in the highest bit; a stream
// that goes on shifts what it has by four.  One compare and one add-with-carry (bits + bits + carry) a
// value, a select for the first of a stream; the eight compares precede the eight that read their masks,
// which also keeps the two wait states between a vector write of a scalar register and a vector read of it.
// Every mask in a scalar register pair (a vector instruction that takes its mask or carry from vcc issues
// several times slower on this part than one that takes it from a scalar pair).
template <bool GO_ON_A, bool GO_ON_B>
__device__ __forceinline__ void bits4x2(unsigned &a, float a0, float a1, float a2, float a3, unsigned &b, float b0,
                                        float b1, float b2, float b3, float g)
{
    unsigned long long m0, m1, m2, m3, m4, m5, m6, m7;
#define BSSE_ADDC(b, m) "v_addc_co_u32_e64 %[" #b "], %[" #m "], %[" #b "], %[" #b "], %[" #m "]\n\t"
#define BSSE_FIRST(b, m) "v_cndmask_b32_e64 %[" #b "], 0, 1, %[" #m "]\n\t"
#define BSSE_BITS(A, IN_A, B, IN_B)                                             \
    asm("v_cmp_ge_f32 %[m0], %[a0], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m4], %[b0], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m1], %[a1], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m5], %[b1], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m2], %[a2], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m6], %[b2], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m3], %[a3], %[g]\n\t"                                   \
        "v_cmp_ge_f32 %[m7], %[b3], %[g]\n\t"                                   \
        A(a, m0) B(b, m4) BSSE_ADDC(a, m1) BSSE_ADDC(b, m5) BSSE_ADDC(a, m2) BSSE_ADDC(b, m6) BSSE_ADDC(a, m3)    \
        BSSE_ADDC(b, m7)                                                        \
        : [a] IN_A(a), [b] IN_B(b), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3),                \
          [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7)        \
        : [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3), [b0] "v"(b0), [b1] "v"(b1), [b2] "v"(b2),        \
          [b3] "v"(b3), [g] "v"(g))
    if constexpr (GO_ON_A && GO_ON_B) BSSE_BITS(BSSE_ADDC, "+v", BSSE_ADDC, "+v");
    else if constexpr (GO_ON_A) BSSE_BITS(BSSE_ADDC, "+v", BSSE_FIRST, "=&v");
    else BSSE_BITS(BSSE_FIRST, "=&v", BSSE_FIRST, "=&v");
#undef BSSE_BITS
}
// One such stream.
__device__ __forceinline__ unsigned bits4(float a0, float a1, float a2, float a3, float g)
{
    unsigned a;
    unsigned long long m0, m1, m2, m3;
    asm("v_cmp_ge_f32 %[m0], %[a0], %[g]\n\t"
        "v_cmp_ge_f32 %[m1], %[a1], %[g]\n\t"
        "v_cmp_ge_f32 %[m2], %[a2], %[g]\n\t"
        "v_cmp_ge_f32 %[m3], %[a3], %[g]\n\t"
        BSSE_FIRST(a, m0) BSSE_ADDC(a, m1) BSSE_ADDC(a, m2) BSSE_ADDC(a, m3)
        : [a] "=&v"(a), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3)
        : [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3), [g] "v"(g));
    return a;
#undef BSSE_FIRST
#undef BSSE_ADDC
}
// The lane's map: grid row k at bit 31 - k, column 4 i + e at bit 8 i + e + 4 h (h4 = 4 h: the lane's half).
template <int TPG>
__device__ __forceinline__ unsigned grid_map(const float *R, const float *C, float floor, unsigned h4)
{
    unsigned r, c;
    if constexpr (TPG == 1) {
        bits4x2<false, false>(r, R[0], R[1], R[2], R[3], c, C[3], C[2], C[1], C[0], floor);
    } else {
        unsigned c1, c0;
        if constexpr (TPG == 2) {
            bits4x2<false, false>(r, R[0], R[1], R[2], R[3], c1, C[7], C[6], C[5], C[4], floor);
            c0 = bits4(C[3], C[2], C[1], C[0], floor);
        } else {
            bits4x2<false, false>(r, R[0], R[1], R[2], R[3], c1, C[7], C[6], C[5], C[4], floor);
            bits4x2<true, false>(r, R[4], R[5], R[6], R[7], c0, C[3], C[2], C[1], C[0], floor);
            if constexpr (TPG == 8) {
                unsigned r0 = r, r1;
                bits4x2<true, false>(r0, R[8], R[9], R[10], R[11], r1, R[12], R[13], R[14], R[15], floor);
                r = (r0 << 4) | r1;
            }
        }
        c = (c1 << 8) | c0;
    }
    return (r << (32 - ArgGrid<TPG>::ROWS)) | (c << h4);
}
// The action of a map of both lanes with two bits (the callers mask it where it may have others).
template <int TPG> __device__ __forceinline__ unsigned grid_action(unsigned map)
{
    return (ffbh(map) << (TPG == 1 ? 3 : 4)) | ffbl(map);
}

// Sixteen values as two interleaved streams of eight (u[0..7] and u[8..15]) against one maximum:
// returns the 16-bit map with bit 15 - r set iff u[r] >= gmax.  Every compare mask in a scalar register
// pair (a vector instruction that takes its mask or carry from vcc issues several times slower on this
// part than one that takes it from a scalar pair).
__device__ __forceinline__ unsigned bitmap16_pairs(const float *u, float gmax)
{
    unsigned ba = 0u, bb = 0u;
    unsigned long long m0, m1, m2, m3, m4, m5, m6, m7;
#define BSSE_BM4S(a, b, c, d, e, f, g, h)                                       \
        "v_cmp_ge_f32 %[m0], %[u" #a "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m1], %[u" #e "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m2], %[u" #b "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m3], %[u" #f "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m4], %[u" #c "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m5], %[u" #g "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m6], %[u" #d "], %[g]\n\t"                              \
        "v_cmp_ge_f32 %[m7], %[u" #h "], %[g]\n\t"                              \
        "v_addc_co_u32_e64 %[ba], %[m0], %[ba], %[ba], %[m0]\n\t"               \
        "v_addc_co_u32_e64 %[bb], %[m1], %[bb], %[bb], %[m1]\n\t"               \
        "v_addc_co_u32_e64 %[ba], %[m2], %[ba], %[ba], %[m2]\n\t"               \
        "v_addc_co_u32_e64 %[bb], %[m3], %[bb], %[bb], %[m3]\n\t"               \
        "v_addc_co_u32_e64 %[ba], %[m4], %[ba], %[ba], %[m4]\n\t"               \
        "v_addc_co_u32_e64 %[bb], %[m5], %[bb], %[bb], %[m5]\n\t"               \
        "v_addc_co_u32_e64 %[ba], %[m6], %[ba], %[ba], %[m6]\n\t"               \
        "v_addc_co_u32_e64 %[bb], %[m7], %[bb], %[bb], %[m7]\n\t"
    asm(BSSE_BM4S(0, 1, 2, 3, 8, 9, 10, 11) BSSE_BM4S(4, 5, 6, 7, 12, 13, 14, 15)
        : [ba] "+v"(ba), [bb] "+v"(bb), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3),
          [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7)
        : [u0] "v"(u[0]), [u1] "v"(u[1]), [u2] "v"(u[2]), [u3] "v"(u[3]), [u4] "v"(u[4]),
          [u5] "v"(u[5]), [u6] "v"(u[6]), [u7] "v"(u[7]), [u8] "v"(u[8]), [u9] "v"(u[9]),
          [u10] "v"(u[10]), [u11] "v"(u[11]), [u12] "v"(u[12]), [u13] "v"(u[13]), [u14] "v"(u[14]),
          [u15] "v"(u[15]), [g] "v"(gmax));
#undef BSSE_BM4S
    return (ba << 8) | bb;
}

// (a | b) over the two lanes of a candidate
__device__ __forceinline__ unsigned pair_or(unsigned v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return r[0] | r[1];
}
// (a + b) over the two lanes of a candidate, same value in both (integers)
__device__ __forceinline__ unsigned pair_add_u32(unsigned v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return r[0] + r[1];
}

// Half h (HALF components from h * HALF on) of the candidate row of m numbers at `row`, zeros from m on.
// Sixteen bytes a request (the hardware asks for four-byte alignment only); where a piece would reach
// past the row it is read ending with the row and shifted.  One request per component touched 64 cache
// lines each time: 2^21 rows of m = 27, n = 32, K = 16 took 496 us and take 473; 2^20 rows of m = 50,
// n = 128, K = 40 bf16 853 and 820.
template <int HALF>
__device__ __forceinline__ void load_half_row(const float *row, int h, int m, float (&v)[HALF])
{
    typedef f32x4 f32x4_dword __attribute__((aligned(4)));
    static_assert(HALF % 4 == 0, "whole pieces");
    if (m >= 4) {
#pragma unroll
        for (int e = 0; e < HALF; e += 4) {
            const int i = h * HALF + e;
            const f32x4 t = *reinterpret_cast<const f32x4_dword *>(row + (i < m ? (i < m - 4 ? i : m - 4) : 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) v[e + k] = t[k];
        }
        if ((m & 3) != 0) {
#pragma unroll
            for (int e = 0; e < HALF; e += 4) {
                const int over = h * HALF + e + 4 - m;       // components past the end of the row
                if (over == 1) { v[e] = v[e + 1]; v[e + 1] = v[e + 2]; v[e + 2] = v[e + 3]; }
                if (over == 2) { v[e] = v[e + 2]; v[e + 1] = v[e + 3]; }
                if (over == 3) { v[e] = v[e + 3]; }
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < HALF; ++e) v[e] = e < 4 ? row[e < m ? e : 0] : 0.0f;      // (m <= 3: all in the first half)
    }
#pragma unroll
    for (int e = 0; e < HALF; ++e) v[e] = h * HALF + e < m ? v[e] : 0.0f;
}

}  // namespace bsse
