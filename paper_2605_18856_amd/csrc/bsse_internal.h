// Internal declarations shared by the translation units of libbsse (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <functional>

namespace bsse {

// Record geometry of the any-shape matrix-core kernel (see sweep_any_impl.h).  A unit is one type
// (forms 1, 2, 3, 4: that many row tiles, n > 16; form 0: any number) or one row tile of several types (form 8, 16: n <= 8, n <= 16).
struct AnyGeo {
    int terms;            // 1, 3 or 6 part products of bf16 parts; 2: three or four of half-precision parts, and behind the
                          // records in Bpack the payoffs as given, [type][action][16 * ks], zero padded
    int ks;               // k-steps of 16 leader actions
    int form;
    int tpg;              // row tiles per type (forms 0 to 4)
    int units;
    int tile_bytes;       // fragments of one row tile
    int rec_bytes;        // one unit: fragments, then leader rows (or leader fragments, forms 8 and 16)
    int lead_off;         // offset of the leader rows in a record; -1: gathered from global memory
    int lead_stride;      // bytes from one leader row to the next in a record
    int ups;              // units per LDS stage
    int stt, nq;          // a unit too large for a stage: stt row tiles per stage, nq stages
    int buf_bytes;        // one of the two stage buffers
    int resident;         // workgroups that a compute unit holds
    int resident_cut;     // the same of the kernel for launches cut over the types
    int row_end;          // terms 2, and the six-bit kernel: rows whose greatest component has this biased exponent or more may have infinite sums
};

// Device view of one game, passed to kernels by value.  All pointers are device memory
// owned by the handle.
struct GameView {
    int m, n, K;
    int x_bf16;           // 1: round each candidate component to bf16 before use
    const float *B;       // [K][m][n]  follower payoffs, row-major (VALU path)
    const float *AT;      // [K][n][m]  leader payoffs, one follower action's column contiguous
    const float *prior;   // [K], then [K] margins of the split kernels' filter (see filter_margins)
    // MFMA paths (null when the shape has no MFMA packing)
    const void *Bpack;    // follower payoffs in MFMA A-operand fragment order
    const void *ATpack;   // leader payoffs [K][n][m_pad] in the contraction's k order
    int m_pad;            // m rounded up to the MFMA k granularity
    int n_pad;            // n rounded up to the row-tile granularity (see sweep_mfma.hip)
    int variant;          // matrix-core kernel variant chosen at create (see mfma_select)
    AnyGeo any;           // variant kAnyVariant
};

// Completion flags of a call in pinned host memory: workgroup b of its last launch stores `seq` into
// flag[b] once its results are there (see done_device.h).  flag == nullptr: nobody waits.
struct Done {
    unsigned *flag;
    unsigned seq;
};

// Running best over chunks, in device memory.
struct RunningBest {
    float value;
    int   has;               // 0 until a chunk has been merged
    long long index;
    unsigned long long ties; // tie evaluations of all merged chunks
};

// Small-game kernel, sweep mode.  Workgroup b keeps its own running best over the chunks of a
// sweep in slot b (read and rewritten by that workgroup alone, so chunk launches need no grid
// stage and no synchronisation); a one-workgroup kernel folds the slots when the result is asked
// for.  A slot belongs to the current sweep when its epoch matches.
struct SmallSlot {
    float value;
    unsigned epoch;
    long long index;         // global candidate index
    unsigned br[2];          // packed best responses (three bits per type; one word per lane half)
    unsigned pad[2];
    float x[8];              // the row itself
};

struct SmallSweep {
    SmallSlot *slots;        // [small_num_slots()]; nullptr outside the small-game sweep
    unsigned epoch;
    const unsigned *epoch_now;   // where the epoch is read instead (a launch that a graph may replay), or nullptr
};

// Fold of the slots into the result of the sweep.
struct FinishArgs {
    const SmallSlot *slots;  // up to three sets, small_num_slots() apart
    int used[3];             // slots of each set that a launch of this sweep may have written
    unsigned epoch;
    const unsigned *epoch_now;
    int first;               // != 0: first fold of this sweep (the tie count restarts)
    unsigned long long *tie_counter;
    RunningBest *run;        // device
    RunningBest *run_host;   // device-visible pinned host memory
    float *x_host;           // [m] row of the best (pinned host)
    float *win_v;            // its value (pinned host)
    int32_t *win_br;         // [K] its best responses (pinned host)
    Done done;
};

// One sweep launch.  Either (V_out, br_out) [evaluation mode: per-candidate outputs] or
// (blk_v, blk_i) [sweep mode: one record per workgroup] is used.
struct SweepArgs {
    const float *X;          // [count][m] fp32
    long long count;
    long long index_base;    // global index of row 0
    float *V_out;            // [count]            (evaluation mode, nullable)
    int32_t *br_out;         // [count][K]         (evaluation mode, nullable)
    float *blk_v;            // [nblocks]          (sweep mode)
    long long *blk_i;        // [nblocks] global candidate index, LLONG_MAX if none
    unsigned long long *tie_counter;  // += number of (candidate,type) evaluations with a tie
    // Evaluation mode only: l_out [count][K] receives the leader payoffs l_t[j*_t] at the best
    // responses.  In the general matrix-core kernel this selects the type-sliced instantiation:
    // for few rows the launch is split over the types as well (one workgroup walking every type
    // would leave the chip idle); the value comes from launch_finish_rows or, for one row, from the
    // host, which sum l_out in type order (term by term the sum of the unsliced kernel).
    float *l_out;
    int slice_stages;        // LDS stages per slice; any-shape kernel: (block, unit) pairs per workgroup, rounded
                             // down, 0 uncut (set by the launcher)
    // l_out / br_out element (c, t) sits at c * _sc + t * _st (unsliced general and wide kernel: br_out
    // at c * K + t).
    long long l_sc, l_st, br_sc, br_st;
    Done done;               // evaluation mode: a flag per workgroup (blockIdx.y * gridDim.x + blockIdx.x)
    // Any-shape kernel, one row (count == 1): with fold_n > 0 the row is the winner of fold_n
    // workgroup records of an earlier launch over the rows X; the winner and the tie counter's value
    // (which is cleared) go to fold_run.  row_host (nullable) receives the row evaluated.
    const float *fold_v;
    const long long *fold_i;
    int fold_n;
    unsigned long long *fold_ties;
    RunningBest *fold_run;
    float *row_host;
    // Small-game kernel only, gen != 0: X is not read; row c is the flat-Dirichlet row
    // gen_first + c of the generator keyed (gen_k0, gen_k1), produced in registers with the
    // arithmetic of the generation kernel (sweep mode only).
    int gen;
    unsigned gen_k0, gen_k1;
    long long gen_first;
    SmallSweep small;        // small-game kernel, sweep mode
};

// Running best of one prior of a prior batch.
struct PriorBest {
    float value;
    int   has;
    long long index;
};

enum PathKind { PATH_VALU = 1, PATH_MFMA_F32 = 2, PATH_MFMA_BF16 = 3, PATH_MFMA_SPLIT = 4 };

// --- launchers (each validates nothing: the API layer has checked shapes) ----------------
// Number of workgroup records the sweep-mode launch of `count` candidates writes.
long long valu_num_blocks(long long count);
hipError_t launch_sweep_valu(const GameView &g, const SweepArgs &a, bool eval, hipStream_t s);

// Short rows on the vector unit (see sweep_tiny.hip): m <= 24, payoffs [K][n][tiny_pad(m)] in g.B and
// g.AT, g.m_pad = tiny_pad(m).
constexpr int kTinyVariant = 3000;
// One launch that leaves the workgroups' winners in pinned host memory (sweep mode without blk_v).
struct TinyRecs {
    struct FinishRec *rec;   // [workgroups]
    float *rec_x;            // [workgroups][m]
    int32_t *rec_br;         // [workgroups][K]
    unsigned seq;            // stored into a record last (see Done)
};
int tiny_pad(int m);                   // 0: not for this kernel
long long tiny_num_blocks(long long count);
int tiny_slices(const GameView &g, long long count);
long long tiny_row_blocks(const GameView &g, long long count);
// slices > 1 (evaluation mode): l_out and br_out only.
hipError_t launch_sweep_tiny(const GameView &g, const SweepArgs &a, bool eval, int slices, const TinyRecs &r, hipStream_t s);

// Matrix-core variants.  mode: 0 = fp32 MFMA on fp32 payoffs, 1 = bf16 MFMA on bf16-rounded
// operands, 2 = bf16 MFMA on fp32 operands split into bf16 parts.  `exact` = every payoff is
// exactly representable in bf16 (lets mode 2 use three terms instead of six).  Returns a
// variant id >= 0, or -1 when the shape has no such kernel.
int mfma_select(int m, int n, int K, int mode, bool exact);
const char *mfma_variant_name(int variant);
long long mfma_num_blocks(int variant, long long count);
long long mfma_limit_blocks(int variant, long long count);        // the same as the limit of the static scratch counts them
hipError_t launch_sweep_mfma(const GameView &g, const SweepArgs &a, hipStream_t s);
hipError_t mfma_prepare(int variant);   // per game, on its device, before the first launch
// Type slices of a launch with l_out; whether `count` candidates are so few that a sweep or an
// evaluation is a launch with l_out and then launch_finish_rows.
int mfma_slices(const GameView &g, long long count);
long long mfma_row_blocks(const GameView &g, long long count);      // workgroups of such a launch
bool mfma_few_rows(const GameView &g, long long count);
bool mfma_is_small(int variant);       // the small-game kernel: launch_finish_small applies
// Host-side packing of payoffs for a variant; returns malloc'ed buffers (caller frees).
void mfma_pack(int variant, int m, int n, int K, const float *A, const float *B, void **Bpack,
               size_t *Bbytes, void **ATpack, size_t *ATbytes, int *m_pad, int *n_pad);

// Margins [K] of the filter of variants with split operands (others leave `margin` as it is).  Returns the variant
// that sweeps this game: the one without a filter where that is the faster one.
int mfma_filter(int variant, int m, int n, int K, const float *A, const float *B, float *margin);

// Small whole-number payoffs, n = 256, on the six-bit matrix instruction (see sweep_fp6.hip): a variant of the general
// matrix-core kernel's table.  fp6_pack: Bpack [K][fp6_record_bytes()] and ATpack [K][n][128], both zeroed.
typedef void (*sweep_fn_t)(GameView, SweepArgs, int);
sweep_fn_t fp6_kernel(bool sliced);
int fp6_record_bytes();
bool mfma_is_six_bit(int variant);
bool fp6_suits(int m, int n, int K, const float *A, const float *B);
void fp6_pack(int m, int K, const float *A, const float *B, unsigned char *Bpack, unsigned short *ATpack);
void fp6_margins(int m, int K, const float *B, float *margin);
bool six_bit_suits(int m, int n, int K, const float *A, const float *B);         // whether they are swept by it

// The share of (candidate tile, type) pairs that a filter with margin(t) sums twice, from `pairs` (8 to 64) pairs of
// types and rows (see sweep_mfma.hip).
double twice_summed(int m, int n, int K, const float *B, const std::function<float(int)> &margin, int pairs, bool ties);

// Small-game matrix-core kernel (n = 8, m = 8, K in {4, 8, 12, 16}, fp32); part of the MFMA path.
bool small_supported(int m, int n, int K, int storage);
long long small_num_blocks(long long count);
hipError_t launch_sweep_small(const GameView &g, const SweepArgs &a, hipStream_t s);
int small_num_slots();
hipError_t launch_finish_small(const GameView &g, const FinishArgs &f, hipStream_t s);
void small_pack(int m, int n, int K, const float *A, const float *B, void **Bpack, size_t *Bbytes,
                void **ATpack, size_t *ATbytes);

// Any-shape matrix-core kernel (m <= 128; see sweep_any.hip).
constexpr int kAnyVariant = 2000;
bool any_supported(int m, int n);
AnyGeo any_geometry(int m, int n, int K, int terms);
void any_pack_sizes(const GameView &g, size_t *Bbytes, size_t *ATbytes);
// Fragments and leader rows from the payoffs as given to create (device, fp32 [K][m][n]).
// terms 2: also the filter's margins, into margin [K], and the payoffs' scales [K] (scratch).
hipError_t launch_any_pack(const GameView &g, const float *A, const float *B, void *Bpack, void *ATpack, float *margin,
                           float *scale, hipStream_t s);
// Whether an fp32 game of this shape is swept in half-precision parts (terms 2).
bool any_half_suits(int m, int n, int K, const float *B);
// AnyGeo::row_end of a game (m <= 128).
int row_end_of(size_t elems, const float *B);
hipError_t any_prepare(const GameView &g);
const char *any_name(const AnyGeo &q);
long long any_num_blocks(const GameView &g, long long count);     // workgroups (= records) of an uncut launch
long long any_max_blocks(const GameView &g, long long count);     // the most that one of up to `count` candidates has
// Workgroups that share a launch over `count` candidates cut over the types (1: it is not to be cut).
int any_shares(const GameView &g, long long count);
long long any_row_blocks(const GameView &g, long long count);       // workgroups of a launch cut like that
// shares > 1: l_out (and br_out) only; the value comes from launch_finish_rows.
hipError_t launch_sweep_any(const GameView &g, const SweepArgs &a, int shares, hipStream_t s);

// Values of rows whose per-type leader payoffs l (type-major, [K][count]) a sliced launch left
// (here and below on the any-shape path and for the general matrix-core kernel alike):
// V[c] = sum_t prior[t] * l[t][c] in type order.  V_out: [count], nullable.  blk_v / blk_i: one record
// per workgroup of FINISH_ROWS rows, nullable.  With rec: the same records in pinned host memory, each
// with the row and the best responses (br type-major, [K][count]) of the workgroup's winner.
constexpr int FINISH_ROWS = 256;
struct FinishRec { float value; unsigned seq; long long index; unsigned long long ties; };
struct FinishRowsArgs {
    const float *l, *prior, *X;
    const int32_t *br;
    long long count, index_base;
    int K, m;
    float *V_out, *blk_v;
    long long *blk_i;
    FinishRec *rec;
    float *rec_x;            // [workgroups][m]
    int32_t *rec_br;         // [workgroups][K]
    unsigned long long *ties;   // read into record 0 and cleared
    unsigned seq;            // stored into a record last (see Done)
};
hipError_t launch_finish_rows(const FinishRowsArgs &f, hipStream_t s);

// first != 0: the running best is replaced, not merged (start of a sweep).  tie_counter (the
// chunk's count, left by the sweep kernel) is folded into run->ties and cleared.  The merged
// record is also written to run_host and the row of a new best to x_host (pinned host memory; for a
// handle's own sweep run and best_x are these).
hipError_t launch_reduce_merge(const float *blk_v, const long long *blk_i, long long nblocks,
                               const float *X, long long index_base, int m, int first,
                               unsigned long long *tie_counter, RunningBest *run,
                               RunningBest *run_host, float *best_x, float *x_host, hipStream_t s);

// dst = src (device-visible pinned host memory) by a kernel: a few words cost less than a copy command.
hipError_t launch_copy_words(const void *src, void *dst, size_t words, hipStream_t s);
// *p = 0 by a one-thread kernel (a fill node that is safe to capture in a graph).
hipError_t launch_clear_u64(unsigned long long *p, hipStream_t s);
// A new sweep on the small-game kernel, in stream order: the next epoch, no ties counted.
hipError_t launch_new_epoch(unsigned *epoch, unsigned long long *tie_counter, RunningBest *run, hipStream_t s);
// Nothing but the completion flag 0.
hipError_t launch_signal(const Done &d, hipStream_t s);
// Zero `bytes` (a multiple of 16) at the 16-byte aligned device address p, by a kernel.
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s);

// Prior batch (see prior_batch.hip): V_p[c] = sum_t priT[t][p] * L[t][c] and the arg-max over c for each
// of P priors, merged into run[P].
struct PriorFoldArgs {
    const float *L;          // [K][ld], 16-byte aligned, readable up to the next multiple of four of count
    unsigned count, ld;      // ld: a multiple of four
    int K;
    const float *priT;       // [K][prior_batch_ld(P)], zero from P on
    long long index_base;
    int first;               // != 0: run is replaced, not merged
    PriorBest *run;          // [P]
    float *rows;             // last launch of a batch (else nullptr): [P][m] rows of the running bests,
    const float *X;          // out of these,
    int m;
    PriorBest *run_host;     // the running bests once more,
    const unsigned long long *ties;
    unsigned long long *ties_host;   // and the tie count
    // set by the launcher
    const float *blk_v;      // [P][nblocks]
    unsigned slice, nblocks;
    int ldp;
};
int prior_batch_blocks(long long count, int P);
int prior_batch_ld(int P);
// blk_v: workspace of prior_batch_blocks(a.count, P) * P records.
hipError_t launch_prior_batch(PriorFoldArgs a, int P, float *blk_v, hipStream_t s);

// Top-k reduction (see topk.hip) of `sets` sets of `count` values each, one behind the other, over the
// rows X in the same order: the k <= min(256, count) best of each set, best first.
struct TopkArgs {
    const float *V;
    unsigned long long *heads;   // workspace of topk_heads_bytes (nullptr when that is 0)
    const float *X;
    unsigned count;
    int k, m;
    long long index_base;    // global index of element 0 of a set
    float *val;              // [sets][k]
    long long *idx;          // [sets][k]
    float *rows;             // [sets][k][m] their rows
    float *rows_host;        // the same once more, nullable
};
size_t topk_heads_bytes(long long count, int sets);
hipError_t launch_topk(const TopkArgs &args, int sets, hipStream_t s);

// Profiles that candidates realise, and their programs on the device (see realised.hip).  A profile is
// named by the key (topk_device.h) of its best candidate.
struct LpArgs {
    const float *A, *B, *prior;  // payoffs as given to create, [K][m][n]
    int m, n_act, K;
    const int32_t *br;           // [count][K]
    const unsigned long long *sel;   // the profiles to solve
    const unsigned *n;           // distinct profiles; min(*n, most) are in sel
    unsigned most;
    double *v, *x;               // [most] optimum, [most][m] vertex
    int *rc;                     // [most] as solve_profile_lp returns
};
struct LpBest { double value; unsigned profiles, solved; int found, failed; };
unsigned profile_table_slots(long long count);
hipError_t launch_profiles(const float *V, const int32_t *br, long long count, int K, unsigned *slots,
                           unsigned long long *best, unsigned *n, unsigned long long *list, unsigned most,
                           unsigned long long *sel, hipStream_t s);
bool lp_on_device(int m, int n, int K);
hipError_t launch_profile_lps(const LpArgs &a, LpBest *out, double *x_host, int32_t *profile_host, const Done &done, hipStream_t s);

// Host code: the linear program of one pure follower profile (see profile_lp.hip).  Returns 0 with
// x_out[m] (on the simplex) and *value_out, 1 when the profile is a best response nowhere, 2 when
// the simplex method hit its iteration limit.  May throw std::bad_alloc.
int solve_profile_lp(int m, int n, int K, const float *A, const float *B, const float *prior,
                     const int32_t *profile, double *x_out, double *value_out);

// centre (device [m], nullable) and radius: the generated set shrunk towards the centre, each
// component fl(fl(radius * t) + fl(fl(1 - radius) * centre[i])); centre == nullptr: the plain set.
// sets > 1: that many sets one behind the other, set s around row s of centre and with seed + s.
hipError_t launch_lattice(const unsigned long long *table, int m, int N, long long count,
                          const float *centre, float radius, int sets, float *out, hipStream_t s);
hipError_t launch_dirichlet(uint64_t seed, long long first, long long count, int m,
                            const float *centre, float radius, int sets, float *out, hipStream_t s);

}  // namespace bsse
