// Prior-robustness batch: the sweep for P priors at once.
//
// A follower's best response does not depend on the prior, so the leader payoffs at the best
// responses, L[t][c] = l_t[j*_t(x_c)], are computed once by the sweep kernels (evaluation mode
// with the per-type output, type-major) and every prior p only needs
//     V_p[c] = sum_t P[p][t] * L[t][c]        (fp32 fused multiply-adds, t ascending)
// and an arg-max over c (greatest value, lowest index).
//
// Candidates sit on the lanes, four consecutive ones in each, and PB_G priors are worked on at once: the
// payoffs come in as one 16-byte load per type and lane, the priors through scalar loads, and a step of
// t is 4 PB_G independent multiply-adds.  Nothing goes through LDS.  Only the greatest value is kept (two
// three-operand maxima per four candidates); the fold finds the lowest workgroup that reached it and
// looks its candidate up again, among those that workgroup had.  Bound by the vector unit:
// 2^20 candidates, K = 4, 101 priors: 22 us of the 12 that the multiply-adds alone take at one per lane
// and four cycles; with priors on the lanes and rows broadcast from LDS it was 52.
#include "bsse_internal.h"
#include "mfma_device.h"
#include <limits.h>

namespace bsse {

namespace {

constexpr int PB_T = 256;
constexpr int PB_G = 16;                 // priors per workgroup
constexpr int PB_STEP = 4 * PB_T;        // candidates per step of a workgroup

// priT: [K][P rounded up to PB_G].  blk_v: [P][gridDim.x] greatest values.  `slice` candidates per
// workgroup (a multiple of PB_STEP); L rows `ld` apart (a multiple of four, the rows 16-byte aligned).
// (With K a constant, the priors of up to four types in scalar registers for all of a workgroup's
// candidates, the call takes the same time: 109.4 us at K = 4, 2^20 candidates and 101 priors, 71-72 at 2.)
__global__ void __launch_bounds__(PB_T, 4)
prior_batch_kernel(const float *__restrict__ L, unsigned count, unsigned ld, int K, const float *__restrict__ priT, int P,
                   unsigned slice, float *__restrict__ blk_v)
{
    __shared__ float sv[PB_T / 64][PB_G];
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p0 = (int)blockIdx.y * PB_G, ldp = (P + PB_G - 1) / PB_G * PB_G;
    const unsigned first = blockIdx.x * slice, end = first + slice < count ? first + slice : count;
    float best[PB_G];
#pragma unroll
    for (int p = 0; p < PB_G; ++p) best[p] = -INFINITY;
    for (unsigned c = first + 4 * tid; c < end; c += PB_STEP) {
        float v[PB_G][4];
        const float *col = L + c;
        const float *pr = priT + p0;
        {
            const float4 l = *reinterpret_cast<const float4 *>(col);
#pragma unroll
            for (int p = 0; p < PB_G; ++p) {
                const float w = pr[p];
                v[p][0] = w * l.x; v[p][1] = w * l.y; v[p][2] = w * l.z; v[p][3] = w * l.w;
            }
        }
#pragma unroll 2
        for (int t = 1; t < K; ++t) {
            const float4 l = *reinterpret_cast<const float4 *>(col + (size_t)t * ld);
#pragma unroll
            for (int p = 0; p < PB_G; ++p) {
                const float w = pr[t * ldp + p];
                v[p][0] = fmaf(w, l.x, v[p][0]); v[p][1] = fmaf(w, l.y, v[p][1]);
                v[p][2] = fmaf(w, l.z, v[p][2]); v[p][3] = fmaf(w, l.w, v[p][3]);
            }
        }
        if (c + 3 >= count) {                            // (what lies behind the last candidate of a row of L)
#pragma unroll
            for (int p = 0; p < PB_G; ++p)
#pragma unroll
                for (unsigned q = 1; q < 4; ++q) v[p][q] = c + q < count ? v[p][q] : -INFINITY;
        }
        // (a maximum never is a value that is not a number)
#pragma unroll
        for (int p = 0; p < PB_G; ++p) best[p] = vmax3(vmax3(best[p], v[p][0], v[p][1]), v[p][2], v[p][3]);
    }
    // The wavefront's maxima of all priors together: in each of the first four steps a lane gives away the
    // half of its priors that its partner keeps (17 exchanges instead of 6 per prior); lane l ends with
    // prior l / 4.
    static_assert(PB_G == 16, "sixteen priors over sixteen groups of four lanes");
#pragma unroll
    for (int h = PB_G / 2; h >= 1; h >>= 1) {
        const bool upper = (lane & (4u * h)) != 0u;
#pragma unroll
        for (int p = 0; p < h; ++p) {
            const float keep = upper ? best[p + h] : best[p], give = upper ? best[p] : best[p + h];
            best[p] = vmax2(keep, __shfl_xor(give, 4 * h, 64));
        }
    }
    best[0] = vmax2(best[0], __shfl_xor(best[0], 2, 64));
    best[0] = vmax2(best[0], __shfl_xor(best[0], 1, 64));
    if ((lane & 3) == 0) sv[wave][lane >> 2] = best[0];
    __syncthreads();
    if (tid < PB_G && p0 + (int)tid < P) {
        float b = sv[0][tid];
#pragma unroll
        for (int w = 1; w < PB_T / 64; ++w) b = vmax2(b, sv[w][tid]);
        blk_v[(size_t)(p0 + tid) * gridDim.x + blockIdx.x] = b;
    }
}

// One workgroup per prior: the greatest value of its records, the lowest workgroup that reached it, and
// the lowest candidate of that workgroup that has it (the same sum once more); merged into the running
// best of the prior (greater value, then lower index; first != 0: replaced).  With rows: also the
// row of the running best (row 0 if there is none), and everything to pinned host memory.
__global__ void __launch_bounds__(PB_T) prior_fold_kernel(PriorFoldArgs a)
{
    __shared__ float sv[PB_T / 64];
    __shared__ unsigned sb[PB_T / 64];
    __shared__ long long win;
    const unsigned p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float bv = -INFINITY;
    unsigned bb = 0xFFFFFFFFu;
    for (unsigned b = tid; b < a.nblocks; b += PB_T) {
        const float v = a.blk_v[(size_t)p * a.nblocks + b];
        if (v > bv) { bv = v; bb = b; }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const float ov = __shfl_xor(bv, d, 64);
        const unsigned ob = __shfl_xor(bb, d, 64);
        if (ov > bv || (ov == bv && ob < bb)) { bv = ov; bb = ob; }
    }
    if (lane == 0) { sv[wave] = bv; sb[wave] = bb; }
    __syncthreads();
    bv = sv[0]; bb = sb[0];
#pragma unroll
    for (int w = 1; w < PB_T / 64; ++w)
        if (sv[w] > bv || (sv[w] == bv && sb[w] < bb)) { bv = sv[w]; bb = sb[w]; }
    // the candidate: no workgroup, none
    unsigned bc = 0xFFFFFFFFu;
    if (bb != 0xFFFFFFFFu) {
        const unsigned first = bb * a.slice, end = first + a.slice < a.count ? first + a.slice : a.count;
        for (unsigned c = first + 4 * tid; c < end; c += PB_STEP) {
            float v[4] = { 0.0f, 0.0f, 0.0f, 0.0f };
#pragma unroll 4
            for (int t = 0; t < a.K; ++t) {
                const float4 l = *reinterpret_cast<const float4 *>(a.L + (size_t)t * a.ld + c);
                const float w = a.priT[(size_t)t * a.ldp + p];
                v[0] = fmaf(w, l.x, v[0]); v[1] = fmaf(w, l.y, v[1]); v[2] = fmaf(w, l.z, v[2]); v[3] = fmaf(w, l.w, v[3]);
            }
#pragma unroll
            for (int q = 3; q >= 0; --q)
                if (v[q] == bv && c + q < a.count && c + q < bc) bc = c + q;
        }
    }
    __syncthreads();
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned oc = __shfl_xor(bc, d, 64);
        bc = oc < bc ? oc : bc;
    }
    if (lane == 0) sb[wave] = bc;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < PB_T / 64; ++w) bc = sb[w] < bc ? sb[w] : bc;
        PriorBest r = a.run[p];
        if (a.first) { r.value = 0.0f; r.has = 0; r.index = -1; }
        if (bc != 0xFFFFFFFFu && (!r.has || bv > r.value || (bv == r.value && a.index_base + bc < r.index))) {
            r.value = bv; r.index = a.index_base + bc; r.has = 1;
        }
        a.run[p] = r;
        if (a.rows) {
            a.run_host[p] = r;
            if (p == 0) *a.ties_host = *a.ties;
        }
        win = r.has ? r.index : 0;
    }
    if (!a.rows) return;
    __syncthreads();
    for (int i = tid; i < a.m; i += PB_T) a.rows[(size_t)p * a.m + i] = a.X[win * a.m + i];
}

// Candidates per workgroup.  Every workgroup ends with PB_G wavefront reductions, about as much work as
// three steps at K = 4: four steps where that still leaves a grid of twice the resident set
// (256 compute units, four workgroups each), down to one for fewer candidates; more for many, so that
// the fold has no more than 1024 records per prior.
unsigned pb_slice(long long count, int P)
{
    const long long groups = (P + PB_G - 1) / PB_G;
    long long steps = count * groups / (2048LL * PB_STEP);
    if (steps < 1) steps = 1;
    if (steps > 4) steps = 4;
    const long long least = (count + 1024LL * PB_STEP - 1) / (1024LL * PB_STEP);
    if (steps < least) steps = least;
    return (unsigned)(steps * PB_STEP);
}

}  // namespace

int prior_batch_blocks(long long count, int P)
{
    const long long slice = pb_slice(count, P);
    return (int)((count + slice - 1) / slice);
}
int prior_batch_ld(int P) { return (P + PB_G - 1) / PB_G * PB_G; }

hipError_t launch_prior_batch(PriorFoldArgs a, int P, float *blk_v, hipStream_t s)
{
    if (a.count == 0 || P <= 0) return hipSuccess;
    if (a.ld % 4 != 0 || a.ld < a.count || ((uintptr_t)a.L & 15) != 0) return hipErrorInvalidValue;
    a.slice = pb_slice(a.count, P);
    a.nblocks = (unsigned)prior_batch_blocks(a.count, P);
    a.ldp = prior_batch_ld(P);
    a.blk_v = blk_v;
    hipLaunchKernelGGL(prior_batch_kernel, dim3(a.nblocks, (unsigned)(a.ldp / PB_G)), dim3(PB_T), 0, s, a.L, a.count, a.ld, a.K,
                       a.priT, P, a.slice, blk_v);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(prior_fold_kernel, dim3(P), dim3(PB_T), 0, s, a);
    return hipGetLastError();
}

}  // namespace bsse
