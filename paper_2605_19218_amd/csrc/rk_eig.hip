// All eigenpairs of the query-weighted scatter C_q = (sigma sigma^T) .* C of every (b, h_kv) (step 5 of Alg. 1,
// Eq. 4, and the "Query-Weighted PCA" of Sec. 3.2), then rank, keep-mask, R_r and delta_mu (steps 14-16).
//
// Four launches, all arithmetic in double:
//   eig_tridiag      C_q = Q T Q^T by Householder reflections, one work-group per matrix, C_q in registers
//   eig_tri_vectors  eigenvalues of T by multisection, vectors of T by twisted factorisation, whole chip
//   eig_orth_back    one Newton-Schulz step on the vectors of T, then R = Q Z, rank, mask, keep_idx, R_r, whole chip
//   eig_finish       sums delta_mu; solves the (rare) matrices that the first three leave alone by parallel
//                    Jacobi, with their rank, mask, keep_idx, R_r and delta_mu
// The fp64 vector rate of this part equals its unpacked fp32 rate, so double costs registers and LDS width only; it
// buys vectors that need no iteration over the whole matrix.  A sweep of Jacobi is 127 dependent rounds on one compute
// unit and 8-10 sweeps are needed; the reduction is 126 dependent steps in all, and everything behind it is independent
// per eigenpair.  Measured (32 / 512 matrices): 86 + 31 + 20 + 5 us / 187 + 304 + 287 + 5 us against 756 us / 2.3 ms of the
// parallel Jacobi that solved every matrix before, with eigenvalues to their fp32 rounding (1e-7 of the spectrum
// against 8e-7).
#include <type_traits>

#include "rk_kernels.hpp"

namespace rk {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Scratch of one matrix (doubles).  A "spread" row of 128 numbers holds element j at eig_spread(j): the eight elements
// j = s + 16 m of lane s of a group of 16 are four pairs, and a pair of all 16 lanes is 256 contiguous bytes, so that a
// lane group reads or writes its row with four conflict-free 16-byte accesses.
constexpr int EIGW_V = 0;                          // [126][128] Householder vectors, spread rows
constexpr int EIGW_Z = EIGW_V + (D - 2) * D;       // [128][128] vectors of T, row c = column c of the result
constexpr int EIGW_DE = EIGW_Z + D * D;            // [128] pairs (d_i, e_{i-1}^2) of the scaled T
constexpr int EIGW_E = EIGW_DE + 2 * D;            // [128] e_i (e_127 unused)
constexpr int EIGW_TAU = EIGW_E + D;               // [128] H_k = I - tau_k v_k v_k^T
constexpr int EIGW_SCALE = EIGW_TAU + D;           // C_q = scale * (Q T Q^T)
constexpr int EIGW_T = EIGW_SCALE + 2;             // [8][16][16] -T_b of H_{16 b} ... H_{16 b + 15} = I - V_b T_b V_b^T
constexpr int EIGW_PART = EIGW_DE;                 // [8][128] fp32, in the place of T and tau: shares of R_r R_r^T mu
static_assert(2 * (EIGW_SCALE - EIGW_PART) >= 8 * D, "eight rows of 128 fp32 numbers");
constexpr int EIGW_TOTAL = EIGW_T + 8 * 256;

size_t eig_scratch_bytes(size_t U) { return U * EIGW_TOTAL * sizeof(double); }

__host__ __device__ constexpr int eig_spread(int j) { return (((j >> 5) * 16 + (j & 15)) << 1) | ((j >> 4) & 1); }

// 1 / x: hardware estimate and two Newton steps
__device__ __forceinline__ double rcp_f64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// ---------------------------------------------------------------------------
// Householder reduction, one work-group of five waves per matrix.  Threads 0 .. 255 hold the matrix: thread (rg, cg) =
// (tid / 16, tid % 16) has rows rg + 16 i and columns cg + 16 m, so the active part shrinks evenly over the threads in both
// directions, a row lies in the 16 consecutive lanes of a group, where sums are lane permutations, and a vector is
// read from LDS by rows exactly as by columns.  The fifth wave makes the reflections.  With x the part of row k behind the
// diagonal, the reflection's vector is v = x + s e with s = +-|x| and e its first place, so that A v = A x + s a, a = row
// k + 1.  A step has two barriers:
//   x is in LDS; every group forms A x on its rows -> LDS; meanwhile the fifth wave finds s and tau and keeps the
//   record                                                                                           -> barrier
//   p = A x + s a, A -= tau (v p^T + p v^T - tau (v^T p) v v^T), the first two products while v^T p is being summed, and the
//   group that owns row k + 2 hands it over; meanwhile the fifth wave applies the same to row k + 1 alone and publishes the
//   next x                                                                                           -> barrier
// What bounds a step is its dependent chain (two LDS round trips, two lane-group sums one behind the other, two barriers) and
// the instructions of one wave: a wave alone on its SIMD issues one about every seven cycles, and a taken branch costs some 36.
// So the steps come two to a loop iteration, and the last step of a block, whose row lies in the next place of a lane, is one of
// its own: no choice between places is left in the others.  32 matrices: 86 us, 512: 187; 93 with those choices, one step an iteration and
// the row handed over in front of A x; 106 with 512 threads of 4 x 8 elements (which read every vector twice as often) whose
// waves made the reflections between their own updates.  Tried: four steps an iteration (the same); 512 threads and the ninth
// wave (103 us: twice the LDS reads); 1024 threads of 2 x 8 elements (119 us: twice the sums and LDS reads per element); the reflection found
// between the barriers of the update, behind the sum v^T p (94 us); every lane group finding it for itself, with one barrier a step
// (114 us: the instructions of all that redundancy cost more than the barrier).
// status[2 u]: 1 for a matrix left to Jacobi (already diagonal to its threshold, zero, or not finite), else 0; status
// [2 u + 1] is cleared for the two kernels behind, which set it when a vector fails its check (they read the first flag
// only: the second may change while they run).
constexpr int TRI_HOLD = 256, TRI_THREADS = TRI_HOLD + 64;

struct TriShared {
    double xs[2][D];                    // spread: x of this step and of the next, zeros in front of its first place
    double ps[D];                       // spread: A x
    double row[2][D];                   // spread: row k + 1 before this step, and the next one
    f64x2 ts[D];                        // (tau, s)
    double d[D], e[D];
    double red[2][TRI_HOLD / 64];
};

// 8 - KB places of a spread vector
template <int KB>
__device__ __forceinline__ void tri_read(double (&x)[8], const double* s, int g)
{
#pragma unroll
    for (int q = KB >> 1; q < 4; ++q) {
        const f64x2 t = *(const f64x2*)(s + (q * 16 + g) * 2);
        x[2 * q] = t.x;
        x[2 * q + 1] = t.y;
    }
}

// The steps of a block all have row k + 1, and the first place of x, in place AT = KB of a lane, but for the last one: AT = KB + 1.
// x + s e
template <int AT>
__device__ __forceinline__ void tri_add_first(double (&x)[8], double s, int lead, int g)
{
    x[AT] += g + 16 * AT == lead ? s : 0.0;
}

// The x of step kn out of row kn, into LDS and x; the diagonal element beside it.
template <int KB, int AT>
__device__ __forceinline__ void tri_publish(const double (&row)[8], int kn, double (&x)[8], TriShared& S, int lane)
{
    const int cg = lane & 15;
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = m < AT ? 0.0 : m > AT || cg + 16 * m > kn ? row[m] : 0.0;
    if (lane < 16) {
        double* xb = S.xs[kn & 1];
#pragma unroll
        for (int q = KB >> 1; q < 4; ++q) *(f64x2*)(xb + (q * 16 + cg) * 2) = (f64x2){x[2 * q], x[2 * q + 1]};
        if (cg == (kn & 15)) S.d[kn] = row[AT];
    }
}

// Step k of the fifth wave, whose lane groups all hold the same: x of the step in v.
template <int KB, int AT>
__device__ __forceinline__ void tri_reflect_step(int k, double (&v)[8], TriShared& S, double* __restrict__ Vg, int lane)
{
    const int cg = lane & 15, kn = k + 1;                        // the first place of x, and the next row
    const double first = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v[AT]), kn & 15),
                                          __builtin_amdgcn_readlane(__double2loint(v[AT]), kn & 15));
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int m = AT; m < 8; ++m) {
        const double y = m == AT && cg + 16 * m == kn ? 0.0 : v[m];
        if (m & 1) s1 = fma(y, y, s1);
        else s0 = fma(y, y, s0);
    }
    const double sig = row16_sum_f64(s0 + s1);
    const double h = fma(first, first, sig);
    // |x| = h / sqrt(h): hardware estimate and one third-order step
    const double y = __builtin_amdgcn_rsq(h), t = h * y, r = fma(-t, y, 1.0);
    const double nrm = fma(t * r, fma(r, 0.375, 0.5), t);
    const bool act = sig > 1e-36;                                // else nothing to clear at double precision: H = I
    const double s = !act ? 0.0 : first >= 0.0 ? nrm : -nrm;                          // (|x| is NaN for x = 0)
    const double tau = act ? rcp_f64(fma(fabs(first), nrm, h)) : 0.0;                 // H = I - tau v v^T
    tri_add_first<AT>(v, s, kn, cg);
    if (lane == 0) {
        S.ts[k] = (f64x2){tau, s};
        S.e[k] = act ? -s : first;
    }
    if (lane < 16) {
#pragma unroll
        for (int q = KB >> 1; q < 4; ++q)
            *(f64x2*)(Vg + (size_t)k * D + (q * 16 + cg) * 2) = (f64x2){2 * q < KB ? 0.0 : v[2 * q], v[2 * q + 1]};
    }
    lds_barrier();
    // (the last step's row 126 and its diagonal element, which the matrix has as well, go unused)
    double p[8], row[8];
    tri_read<KB>(p, S.ps, cg);
    tri_read<KB>(row, S.row[kn & 1], cg);
    const double pk = fma(s, S.row[kn & 1][eig_spread(kn)], S.ps[eig_spread(kn)]);
#pragma unroll
    for (int m = AT; m < 8; ++m) p[m] = fma(s, row[m], p[m]);
    double d0 = 0.0, d1 = 0.0;
#pragma unroll
    for (int m = AT; m < 8; ++m) {
        if (m & 1) d1 = fma(v[m], p[m], d1);
        else d0 = fma(v[m], p[m], d0);
    }
    const double tl = -tau * (first + s), tp = -tau * pk;
#pragma unroll
    for (int m = AT; m < 8; ++m) row[m] = fma(tl, p[m], fma(tp, v[m], row[m]));
    const double c = -tau * tl * row16_sum_f64(d0 + d1);
#pragma unroll
    for (int m = AT; m < 8; ++m) row[m] = fma(c, v[m], row[m]);
    tri_publish<KB, AT>(row, kn, v, S, lane);
    lds_barrier();
}
// Steps 16 KB .. 16 KB + 15
template <int KB>
__device__ __forceinline__ void tri_reflect(double (&v)[8], TriShared& S, double* __restrict__ Vg, int lane)
{
#pragma unroll 1
    for (int k = 16 * KB; k < 16 * KB + 14; k += 2) {            // (a taken branch costs as much as eight instructions)
        tri_reflect_step<KB, KB>(k, v, S, Vg, lane);
        tri_reflect_step<KB, KB>(k + 1, v, S, Vg, lane);
    }
    if constexpr (KB < 7) {
        tri_reflect_step<KB, KB>(16 * KB + 14, v, S, Vg, lane);
        tri_reflect_step<KB, KB + 1>(16 * KB + 15, v, S, Vg, lane);
        tri_reflect<KB + 1>(v, S, Vg, lane);
    }
}

// Sums of p[KB ..] over the 16 lanes of a group.  With several rows the first steps halve the rows that a lane carries instead
// of adding all of them everywhere: H of N rows stay, lanes with the step's bit set taking row j + H where there is one.
// row: which of them this lane ends up with.
template <int N, int STEP>
__device__ __forceinline__ double tri_fold(const double (&t)[8], int cg)
{
    auto other = [](double x) {
        return STEP == 0 ? dpp_f64<0x128>(x)                     // row_ror 8: lane i takes from lane i ^ 8
             : STEP == 1 ? dpp_f64<0x141>(x)                     // row_half_mirror: lane i ^ 7
             : STEP == 2 ? dpp_f64<0x4E>(x) : dpp_f64<0xB1>(x);  // lane i ^ 2, lane i ^ 1
    };
    if constexpr (STEP == 4) {
        return t[0];
    } else {
        constexpr int H = N > 4 ? 4 : N > 2 ? 2 : 1;
        const bool up = (cg & (8 >> STEP)) != 0;
        double s[8];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const double a = t[j], b = j + H < N ? t[j + H] : 0.0;      // (by value: a choice between places becomes an index)
            if (j + H < N) s[j] = (up ? b : a) + other(up ? a : b);
            else s[j] = a + other(a);
        }
        return tri_fold<H, STEP + 1>(s, cg);
    }
}
template <int N>
__device__ __forceinline__ int tri_fold_row(int cg)
{
    const int b3 = (cg >> 3) & 1, b2 = (cg >> 2) & 1, b1 = (cg >> 1) & 1;
    if (N > 4) { const int j = 2 * b2 + b1; return j + (b3 && j + 4 < N ? 4 : 0); }
    if (N > 2) return b2 + (b3 && b2 + 2 < N ? 2 : 0);
    return N > 1 ? b3 : 0;
}

// Step k of the waves that hold the matrix: row and column places below KB are finished.
template <int KB, int AT>
__device__ __forceinline__ void tri_step(int k, double (&a)[8][8], TriShared& S, int rg, int cg, int wave, int mine)
{
    constexpr int N = 8 - KB;
    const int kn = k + 1;
    const bool live = KB < 7 || 112 + 4 * wave + 3 > k;                   // wave-uniform: some row of this wave is still active
    double v[8], vi[8];
    if (live) {
        tri_read<KB>(v, S.xs[k & 1], cg);
        tri_read<KB>(vi, S.xs[k & 1], rg);
        double p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) p[j] = 0.0;
#pragma unroll
        for (int m = KB; m < 8; ++m)
#pragma unroll
            for (int j = 0; j < N; ++j) p[j] = fma(a[KB + j][m], v[m], p[j]);
        S.ps[mine] = tri_fold<N, 0>(p, cg);                      // (several lanes store the same number)
    }
    lds_barrier();
    if (live) {
        double w[8], wi[8], r[8], ri[8];
        const f64x2 ts = S.ts[k];
        tri_read<KB>(w, S.ps, cg);
        tri_read<KB>(r, S.row[kn & 1], cg);
        tri_read<KB>(wi, S.ps, rg);
        tri_read<KB>(ri, S.row[kn & 1], rg);
        const double tau = ts.x;
        tri_add_first<AT>(v, ts.y, kn, cg);
        tri_add_first<AT>(vi, ts.y, kn, rg);
        double d0 = 0.0, d1 = 0.0;
#pragma unroll
        for (int m = KB; m < 8; ++m) {
            w[m] = fma(ts.y, r[m], w[m]);
            if (m & 1) d1 = fma(v[m], w[m], d1);
            else d0 = fma(v[m], w[m], d0);
        }
#pragma unroll
        for (int i = KB; i < 8; ++i) wi[i] = fma(ts.y, ri[i], wi[i]);
        // rows that are finished hold leftovers of v: whatever they become is never read
#pragma unroll
        for (int i = KB; i < 8; ++i) {
            const double tv = -tau * vi[i];
#pragma unroll
            for (int m = KB; m < 8; ++m) a[i][m] = fma(tv, w[m], a[i][m]);
        }
        const double nd = -tau * row16_sum_f64(d0 + d1);
#pragma unroll
        for (int i = KB; i < 8; ++i) {
            const double tw = -tau * fma(nd, vi[i], wi[i]);
#pragma unroll
            for (int m = KB; m < 8; ++m) a[i][m] = fma(tw, v[m], a[i][m]);
        }
        // row k + 2 for the next step, here where the fifth wave is the one to wait for
        if (rg == ((kn + 1) & 15)) {
            const bool far = KB < 7 && ((kn + 1) >> 4) > KB;
            constexpr int FAR = KB < 7 ? KB + 1 : KB;
            double* hand = S.row[(kn + 1) & 1];
#pragma unroll
            for (int q = KB >> 1; q < 4; ++q)
                *(f64x2*)(hand + (q * 16 + cg) * 2) = far ? (f64x2){a[FAR][2 * q], a[FAR][2 * q + 1]}
                                                          : (f64x2){a[KB][2 * q], a[KB][2 * q + 1]};
        }
    }
    lds_barrier();
}
// Steps 16 KB .. 16 KB + 15
template <int KB>
__device__ __forceinline__ void tri_block(double (&a)[8][8], TriShared& S, int rg, int cg, int wave)
{
    const int mine = eig_spread(rg + 16 * (KB + tri_fold_row<8 - KB>(cg)));
#pragma unroll 1
    for (int k = 16 * KB; k < 16 * KB + 14; k += 2) {
        tri_step<KB, KB>(k, a, S, rg, cg, wave, mine);
        tri_step<KB, KB>(k + 1, a, S, rg, cg, wave, mine);
    }
    if constexpr (KB < 7) {
        tri_step<KB, KB>(16 * KB + 14, a, S, rg, cg, wave, mine);
        tri_step<KB, KB + 1>(16 * KB + 15, a, S, rg, cg, wave, mine);
        tri_block<KB + 1>(a, S, rg, cg, wave);
    }
}

__global__ __launch_bounds__(TRI_THREADS) void eig_tridiag(const float* __restrict__ cov, const float* __restrict__ sigma,
                                                           double* __restrict__ scratch, int32_t* __restrict__ status)
{
    __shared__ __attribute__((aligned(16))) TriShared S;
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, rg = tid >> 4, cg = tid & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* C = cov + (size_t)u * D * D;
    double* W = scratch + (size_t)u * EIGW_TOTAL;

    double a[8][8];
    if (wave < TRI_HOLD / 64) {
        float cf[8][8];                     // every load is out before the first is used
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int m = 0; m < 8; ++m) cf[i][m] = C[(rg + 16 * i) * D + cg + 16 * m];
        float sr[8], sc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) sr[i] = sigma ? sigma[(size_t)u * D + rg + 16 * i] : 1.f;
#pragma unroll
        for (int m = 0; m < 8; ++m) sc[m] = sigma ? sigma[(size_t)u * D + cg + 16 * m] : 1.f;
        double all = 0.0, off = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const double x = (double)cf[i][m] * ((double)sr[i] * (double)sc[m]);
                a[i][m] = x;
                all = fma(x, x, all);
                off = rg + 16 * i == cg + 16 * m ? off : fma(x, x, off);
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            all += __shfl_xor(all, o);
            off += __shfl_xor(off, o);
        }
        if (lane == 0) { S.red[0][wave] = all; S.red[1][wave] = off; }
    }
    __syncthreads();
    double all = 0.0, off = 0.0;
    for (int w = 0; w < TRI_HOLD / 64; ++w) { all += S.red[0][w]; off += S.red[1][w]; }
    // uniform: left to Jacobi, whose threshold this is (2e-8 ||C_q||_F); NaN and infinities land here too
    if (!(off > 4e-16 * all) || !(all < 1e300)) {
        if (tid == 0) { status[2 * u] = 1; status[2 * u + 1] = 0; }
        return;
    }
    // scaled by a power of two to a Frobenius norm in [1/2, 1)
    const int ex = __builtin_amdgcn_frexp_exp(sqrt(all));
    if (wave < TRI_HOLD / 64) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int m = 0; m < 8; ++m) a[i][m] = ldexp(a[i][m], -ex);
        if (rg < 2)
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f64x2*)(S.row[rg] + (q * 16 + cg) * 2) = (f64x2){a[0][2 * q], a[0][2 * q + 1]};
        __syncthreads();
        __syncthreads();
        tri_block<0>(a, S, rg, cg, wave);
        if (rg == 14 && cg == 14) S.d[126] = a[7][7];
        if (rg == 14 && cg == 15) S.e[126] = a[7][7];
        if (rg == 15 && cg == 15) S.d[127] = a[7][7];
    } else {
        __builtin_amdgcn_s_setprio(3);      // its chain is the longer one, and it shares its SIMD with a wave of the others
        __syncthreads();
        double row[8], v[8];
        tri_read<0>(row, S.row[0], cg);
        tri_publish<0, 0>(row, 0, v, S, lane);
        __syncthreads();
        tri_reflect<0>(v, S, W + EIGW_V, lane);
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    // What the vectors are computed from: T plus a diagonal of up to 6.4e-11 (128 distinct multiples of 5e-13), which
    // separates eigenvalues that are equal to rounding (dead channels, rank-deficient Keys) by enough for
    // independent vectors and is a thousandth of the fp32 rounding of C; off-diagonals at least 1e-18, so T never splits.
    if (tid < D) {
        const double ep = tid > 0 ? S.e[tid - 1] : 0.0, en = tid < D - 1 ? S.e[tid] : 0.0;
        const double epf = fabs(ep) < 1e-18 ? 1e-18 : ep, enf = fabs(en) < 1e-18 ? 1e-18 : en;
        ((f64x2*)(W + EIGW_DE))[tid] = (f64x2){S.d[tid] + 5e-13 * (double)((37 * tid) & (D - 1)), tid > 0 ? epf * epf : 0.0};
        W[EIGW_E + tid] = enf;
        W[EIGW_TAU + tid] = tid < D - 2 ? S.ts[tid].x : 0.0;
    }
    if (tid == 0) {
        W[EIGW_SCALE] = ldexp(1.0, ex);
        status[2 * u] = 0;
        status[2 * u + 1] = 0;
    }
}

// ---------------------------------------------------------------------------
// Work-group -> (matrix, slice) of the two whole-chip kernels: the eight work-groups of a matrix get linear indices that
// agree modulo 8, so that they run on one XCD and share the matrix's scratch in its L2 (work-groups are dealt round-robin
// to the XCDs; eig_tridiag's work-group u is on the same one).
__device__ __forceinline__ void eig_slice(int& u, int& slice)
{
    const int slot = (int)blockIdx.x >> 3;
    slice = slot & 7;
    u = 8 * (slot >> 3) + ((int)blockIdx.x & 7);
}
static unsigned eig_slices(int U) { return 64u * (unsigned)((U + 7) / 8); }

__device__ __forceinline__ int row16_sum_i32(int v)
{
    v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);      // the lane permutations of row16_sum_f64
    v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);
    return v + __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true);
}

// Eigenpairs of T, four per wave, 16 lanes each; a work-group makes 16 of a matrix's 128.
// Eigenvalue by multisection: the 16 lanes count the eigenvalues below 16 points of the interval (sign changes of
// the three-term recurrence p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1}, division-free, rescaled every 16 steps: a step is at
// least a factor 5e-13 but for one, so 16 stay above 1e-250) and the interval shrinks 17-fold, eleven times, behind a first
// round in which the whole work-group counts below 256 points for all of its pairs: 2 / (257 17^11) = 2e-16.  T comes through
// the scalar cache, 8 rows ahead: one wave per SIMD has nobody else to hide a load behind.  (The recurrence from both ends at
// once, joined in the middle, took as long: a wave alone on its SIMD issues an instruction about every seven cycles, whatever
// it waits for.)
// Vector by twisted factorisation, again without a division in the chain: a lane of wave 0 runs (T - lambda) y = 0 from the
// top, one of wave 1 from the bottom, both rescaled every 8 steps (exponents kept per block of 8); the vector is the one above
// the row with the smallest twist gamma_i = (d_i - lambda) + e_{i-1} y_{i-1} / y_i + e_i x_{i+1} / x_i and the other below
// it.  A second round, at the Rayleigh-corrected eigenvalue, leaves a residual of a few 1e-16; only close neighbours need it.
// 32 matrices 30 us, 34 with twelve rounds of 17, both rounds of vectors always and chains that make their coefficients on the way.
constexpr int TV_PAIRS = 16, TV_SECT = 12, TV_LD = D + 2;
constexpr double TV_GAP = 5e-12;

// -T of reflections 16 b .. 16 b + 15 by one wave: their inner products G on the matrix cores (the order of the contraction
// is that of the record, from its first written pair on; a lane's row of V serves as both operands), then
// T_ij = -tau_j sum_{i <= l < j} T_il G_lj, a row of T per lane, lane groups alike.  G: 256 doubles of LDS.
__device__ __forceinline__ void tri_block_t(const double* __restrict__ W, double* __restrict__ Tout, double* __restrict__ G,
                                            int b, int lane)
{
    const int g = lane >> 4, n = lane & 15;
    const double* row = W + EIGW_V + (size_t)min(16 * b + n, D - 3) * D;      // (rows 126 and 127: tau is 0)
    f64x2 v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = *(const f64x2*)(row + max(8 * t, 32 * (b >> 1)) + 2 * g);
    const double tau = W[EIGW_TAU + 16 * b + n];
    f64x4 acc[2];
    acc[0] = acc[1] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 16; ++t)
        if (8 * t >= 32 * (b >> 1)) {
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t].x, v[t].x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t].y, v[t].y, acc[1], 0, 0, 0);
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) G[(4 * r + g) * 16 + n] = acc[0][r] + acc[1][r];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double T[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int l = 0; l < j; ++l) {
            if (l & 1) s1 = fma(T[l], G[l * 16 + j], s1);
            else s0 = fma(T[l], G[l * 16 + j], s0);
        }
        const double tj = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(tau), j),
                                           __builtin_amdgcn_readlane(__double2loint(tau), j));
        T[j] = j < n ? 0.0 : j == n ? tj : -tj * (s0 + s1);
    }
    if (g == 0)
#pragma unroll
        for (int j = 0; j < 16; j += 2) *(f64x2*)(Tout + n * 16 + j) = (f64x2){-T[j], -T[j + 1]};
}

__global__ __launch_bounds__(256, 2) void eig_tri_vectors(int U, const double* __restrict__ scratch,
                                                       double* __restrict__ Zout, float* __restrict__ lam_out,
                                                       int32_t* __restrict__ status)
{
    // coefficients of the two recurrences, in the order in which a lane walks them: (d, 1 / e ahead), e behind / e ahead
    __shared__ f64x2 sco[2][D];
    __shared__ __attribute__((aligned(16))) double sw[2][D];
    __shared__ double se[D];
    // y (from the top) and x (from the bottom); before a chain comes by, its coefficients (lambda - d) / e ahead
    __shared__ __attribute__((aligned(16))) double yx[TV_PAIRS][2][TV_LD];
    __shared__ int ys[TV_PAIRS][2][D / 8];           // their exponents, per block of 8 rows
    __shared__ double slam[TV_PAIRS];
    __shared__ double sg16[256];
    __shared__ __attribute__((aligned(16))) unsigned char first_counts[256];
    int u, slice;
    eig_slice(u, slice);
    if (u >= U || status[2 * u] != 0) return;
    const int tid = threadIdx.x, lane = tid & 63, s = lane & 15;
    const int pr = tid >> 4;                          // eigenpair of this work-group
    const int col = slice * TV_PAIRS + pr;            // result column: descending eigenvalues
    const int below = D - 1 - col;                    // eigenvalues below this one
    const double* W = scratch + (size_t)u * EIGW_TOTAL;
    const f64x2* __restrict__ de = (const f64x2*)(W + EIGW_DE);
    if (tid < D) {
        const int i = tid, r = D - 1 - i;
        const double d = de[i].x, e = W[EIGW_E + i], ep = W[EIGW_E + max(i - 1, 0)];
        // ahead of row i lies e_i from the top and e_{i-1} from the bottom; past the last row anything finite does
        const double ie = rcp_f64(i < D - 1 ? e : 1.0), iep = rcp_f64(i > 0 ? ep : 1.0);
        sco[0][i] = (f64x2){d, ie};
        sw[0][i] = i > 0 ? ep * ie : 0.0;
        sco[1][r] = (f64x2){d, iep};
        sw[1][r] = i < D - 1 ? e * iep : 0.0;
        se[i] = e;
    }

    // eigenvalues below x
    auto count = [&](double x) {
        double p0 = 0.0, p = 1.0;
        int changes = 0;
        uint32_t last = 0, sg = 0;
        f64x2 ca[8], cb[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) ca[i] = de[i];
        // Scalar loads complete out of order, so a wait for one batch is a wait for all that are out: the next batch is
        // requested right behind the first use of the present one.
        auto steps = [&](const f64x2 (&c)[8], f64x2 (&next)[8], int at) {
            double t = c[0].x - x;
            asm volatile("" : "+v"(t));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 8; ++i) next[i] = de[at + i];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double pn = fma(t, p, -(c[i].y * p0));
                p0 = p;
                p = pn;
                if (i < 7) t = c[i + 1].x - x;
                sg = __builtin_amdgcn_alignbit(sg, (uint32_t)__double2hiint(p), 31);     // (sg << 1) | sign
            }
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll 1
        for (int i0 = 0; i0 < D; i0 += 16) {
            steps(ca, cb, i0 + 8);
            steps(cb, ca, min(i0 + 16, D - 8));
            const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p0)));
            p = ldexp(p, -ex);
            p0 = ldexp(p0, -ex);
            // 16 signs of this block behind the last one of the block before it
            changes += __popc((sg ^ ((sg >> 1) | (last << 15))) & 0xffffu);
            last = sg & 1u;
            sg &= 0xffffu;
        }
        return changes;
    };
    double lo = -1.001, hi = 1.001;                   // the Frobenius norm is below 1
    double under = 2.0, over = -2.0;                  // of the points between this eigenvalue and its neighbours, the outermost
    int points = 256;                                 // of the first round: all of the work-group's, for all of its pairs
#pragma unroll 1
    for (int it = 0; it < TV_SECT; ++it) {
        const double wid = (hi - lo) * (1.0 / (points + 1)), x = fma(wid, (double)((it == 0 ? tid : s) + 1), lo);
        const int changes = count(x);
        int m;                                        // points with at most `below` eigenvalues under them
        if (it == 0) {
            first_counts[tid] = (unsigned char)changes;
            __syncthreads();
            const uint4 c = *(const uint4*)(first_counts + 16 * s);
            const uint32_t w[4] = {c.x, c.y, c.z, c.w};
            m = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) m += (int)((w[k >> 2] >> (8 * (k & 3))) & 0xffu) <= below;
            m = row16_sum_i32(m);
        } else {
            under = changes == below ? fmin(under, x) : under;
            over = changes == below + 1 ? fmax(over, x) : over;
            m = __popc((uint32_t)(__ballot(changes <= below) >> (lane & 48)) & 0xffffu);
        }
        const double nlo = fma(wid, (double)m, lo);
        hi = m == points ? hi : fma(wid, (double)(m + 1), lo);
        lo = nlo;
        points = 16;
    }
    double lam = 0.5 * (lo + hi);
#pragma unroll
    for (int o = 0; o < 4; ++o) {                                // the lane permutations of row16_sum_f64
        under = fmin(under, o == 0 ? dpp_f64<0xB1>(under) : o == 1 ? dpp_f64<0x4E>(under) : o == 2 ? dpp_f64<0x141>(under) : dpp_f64<0x140>(under));
        over = fmax(over, o == 0 ? dpp_f64<0xB1>(over) : o == 1 ? dpp_f64<0x4E>(over) : o == 2 ? dpp_f64<0x141>(over) : dpp_f64<0x140>(over));
    }
    if (s == 0) slam[pr] = lam;
    __syncthreads();
    // One round leaves a vector with a residual of some 5e-16, and that over the gap to the next eigenvalue in its direction:
    // 1e-4 at TV_GAP.  What of it keeps two vectors from being orthogonal the step in eig_orth_back squares (3.2e-5 was the most in 1008
    // glued tridiagonal matrices, 3.7e-6 with two rounds).  What turns two neighbours into each other stays, and stays below what the
    // shift of T's diagonal, up to 6.4e-11, does to such neighbours: over 32 matrices of 16384 rows the largest element of R is 4.0461e-2 from
    // the vectors of C_q itself with one round, 4.0460e-2 with two, and 1e-6 between them.  A nearer neighbour (of any pair
    // of this work-group; the neighbours of its first and last pair are only known to lie beyond a point) asks for the second round.
    const double above = (pr > 0 ? slam[max(pr - 1, 0)] : over) - lam, under_by = lam - (pr < TV_PAIRS - 1 ? slam[min(pr + 1, TV_PAIRS - 1)] : under);
    const int rounds = __syncthreads_or(!(above > TV_GAP) || !(under_by > TV_GAP)) ? 2 : 1;

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double (*yv)[TV_LD] = yx[pr];
    double zz[8];
    double norm2 = 1.0, gam = 0.0;
#pragma unroll 1
    for (int round = 0; round < rounds; ++round) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = s + 16 * m;
            const f64x2 c = sco[0][i];
            const double t = lam - c.x;
            yv[0][i] = t * c.y;
            yv[1][i] = t * sco[1][D - 1 - i].y;
        }
        __syncthreads();
        // Wave 0 runs the 16 chains from the top, wave 1 those from the bottom, each a wave alone on its SIMD, which issues an
        // instruction about every seven cycles: the coefficients come ready (by all waves, above) and two rows to an access,
        // and the vector takes their place.  With the coefficients made on the way a step took 62 cycles.
        auto chain = [&](auto direction) {
            constexpr int dir = decltype(direction)::value, stp = dir ? -2 : 2;
            double y0 = 0.0, y = 1.0;
            int exps = 0;
            double* at = yx[lane][dir] + (dir ? D - 2 : 0);
            f64x2 ca[2], cb[2], wa[2], wb[2];
            auto fetch = [&](f64x2 (&c)[2], f64x2 (&w)[2], int row) {     // rows row .. row + 3 of the walk
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    c[i] = *(const f64x2*)(yx[lane][dir] + (dir ? D - 2 - row - 2 * i : row + 2 * i));
                    w[i] = *(const f64x2*)(sw[dir] + row + 2 * i);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto steps = [&](const f64x2 (&c)[2], const f64x2 (&w)[2]) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const double y1 = fma(dir ? c[i].y : c[i].x, y, -(w[i].x * y0));
                    const double y2 = fma(dir ? c[i].x : c[i].y, y1, -(w[i].y * y));
                    *(f64x2*)at = dir ? (f64x2){y1, y} : (f64x2){y, y1};
                    at += stp;
                    y0 = y1;
                    y = y2;
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            fetch(ca, wa, 0);
#pragma unroll 1
            for (int b = 0; b < D / 8; ++b) {
                ys[lane][dir][dir ? D / 8 - 1 - b : b] = exps;
                fetch(cb, wb, 8 * b + 4);
                steps(ca, wa);
                fetch(ca, wa, min(8 * b + 8, D - 4));
                steps(cb, wb);
                const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(y), fabs(y0)));
                y = ldexp(y, -ex);
                y0 = ldexp(y0, -ex);
                exps += ex;
            }
        };
        if (wave == 0 && lane < TV_PAIRS) chain(std::integral_constant<int, 0>());
        if (wave == 1 && lane < TV_PAIRS) chain(std::integral_constant<int, 1>());
        // meanwhile the block reflector that eig_orth_back wants of reflections 16 slice .. + 15
        if (wave == 2 && round == 0) tri_block_t(W, Zout + (size_t)u * EIGW_TOTAL + EIGW_T + 256 * slice, sg16, slice, lane);
        __syncthreads();
        // the twist: smallest |gamma|, first row of equals
        double bg = __builtin_huge_val();
        int twist = 0;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = s + 16 * m, blk = i >> 3;
            double g = sco[0][i].x - lam;
            if (i > 0) {
                const double yb = ldexp(yv[0][max(i - 1, 0)], ys[pr][0][max(i - 1, 0) >> 3] - ys[pr][0][blk]);
                g = fma(se[max(i - 1, 0)], yb * rcp_f64(yv[0][i]), g);
            }
            if (i < D - 1) {
                const double xb = ldexp(yv[1][min(i + 1, D - 1)], ys[pr][1][min(i + 1, D - 1) >> 3] - ys[pr][1][blk]);
                g = fma(se[i], xb * rcp_f64(yv[1][i]), g);
            }
            if (fabs(g) < fabs(bg)) { bg = g; twist = i; }
        }
#pragma unroll
        for (int o = 0; o < 4; ++o) {                            // the lane permutations of row16_sum_f64
            const double og = o == 0 ? dpp_f64<0xB1>(bg) : o == 1 ? dpp_f64<0x4E>(bg) : o == 2 ? dpp_f64<0x141>(bg) : dpp_f64<0x140>(bg);
            const int ot = o == 0   ? __builtin_amdgcn_mov_dpp(twist, 0xB1, 0xf, 0xf, true)
                           : o == 1 ? __builtin_amdgcn_mov_dpp(twist, 0x4E, 0xf, 0xf, true)
                           : o == 2 ? __builtin_amdgcn_mov_dpp(twist, 0x141, 0xf, 0xf, true)
                                    : __builtin_amdgcn_mov_dpp(twist, 0x140, 0xf, 0xf, true);
            if (fabs(og) < fabs(bg) || (fabs(og) == fabs(bg) && ot < twist)) { bg = og; twist = ot; }
        }
        const double iy = rcp_f64(yv[0][twist]), ix = rcp_f64(yv[1][twist]);
        const int ey = ys[pr][0][twist >> 3], ex = ys[pr][1][twist >> 3];
        double n2 = 0.0;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = s + 16 * m;
            const double zi = i <= twist ? ldexp(yv[0][i] * iy, ys[pr][0][i >> 3] - ey)
                                         : ldexp(yv[1][i] * ix, ys[pr][1][i >> 3] - ex);
            zz[m] = zi;
            n2 = fma(zi, zi, n2);
        }
        norm2 = row16_sum_f64(n2);
        gam = bg;
        if (round + 1 < rounds) {
            lam += gam / norm2;
            __syncthreads();
        }
    }
    const double inv = 1.0 / sqrt(norm2);
    // residual |gamma| / ||z||: a few 1e-16 when all is well; anything else (NaN included) goes to Jacobi
    if (s == 0) {
        lam_out[(size_t)u * D + col] = (float)((lam + gam / norm2) * W[EIGW_SCALE]);
        if (!(fabs(gam) * inv < 1e-12)) status[2 * u + 1] = 1;
    }
    double* Zc = Zout + (size_t)u * EIGW_TOTAL + EIGW_Z + (size_t)col * D;
#pragma unroll
    for (int m = 0; m < 8; ++m) Zc[s + 16 * m] = zz[m] * inv;
}

// ---------------------------------------------------------------------------
// R = Q Z after one Newton-Schulz step Z <- Z (3 I - Z^T Z) / 2; 16 columns per work-group of 4 waves.
// The step is what makes independent vectors safe: neighbours a gap g apart come out orthogonal only to about
// 5e-16 / g (g above TV_GAP, one round of vectors) or 2e-17 / g (below it, two rounds), the step squares that defect, and because
// each vector is an eigenvector to 5e-16 the correction mixes close neighbours only and costs no residual.  A defect E leaves
// (3/4) E^2 behind, so what the step may be given is bounded by what the result is held to: an element above EIG_ORTH_MAX sends
// the matrix to Jacobi.  (1008 glued tridiagonal matrices, with up to 91 gaps between TV_GAP and 2e-11 each: 3.2e-5 at most above TV_GAP;
// 2.4e-4 below it, at gaps under 1e-13, the shift of 5e-13 undone; five, with gaps of 1e-14 and less, left to Jacobi, 21 when every
// vector took two rounds behind a coarser multisection.)
// Both products run on the fp64 matrix cores with all of Z in LDS; then Z's space takes the reflections, which were on
// their way in registers meanwhile.  They are applied 16 at a time as I - V T V^T, again on the matrix cores, with the 16
// columns of Z staying in result registers; T comes from eig_tri_vectors, where two waves have nothing else to do.
// Bound, of 36000 cycles: loading Z 6500, the products 6000 + 6600 (matrix pipe 4100 each), storing V 2800, reflections 13700
// (eight rounds of four dependent matrix steps, one exchange between the waves, eight more).  Four reflections at a time
// on the vector unit: 20000 + 2500 for their inner products (LDS-bound, every lane group reads all of V), 23 us; one at a time
// with loads where they are used: 56000 cycles in all, 27.7 us.  18 us for 32 matrices, 266 for 512 (547 at first);
// with the ranks, R_r and the products with mu 20 and 287, for 5 and 17 less in eig_finish (32 matrices gain, 512 lose 4 us by it).
constexpr double EIG_ORTH_MAX = 3e-4;
static_assert(0.75 * D * EIG_ORTH_MAX * EIG_ORTH_MAX <= 1e-5, "|R^T R - I| <= 1e-5, every column of E at its limit");
constexpr int OB_LD = D + 2, OB_MLD = 17;
constexpr size_t OB_LDS_BYTES = (size_t)(D * OB_LD + D * OB_MLD) * sizeof(double);

// Z <- H_{16 KB} ... H_{16 KB + 15} Z and on to block 0.  Wave w holds row tiles w and w + 4 of the 16 columns in result
// layout, whose register r is the right operand of contraction step r.  X = -T (V^T Z), Z += V X: V^T Z is summed over
// the waves in LDS (Wx: two buffers, so one barrier per block), the rest stays within the wave.
// T: -T of this block as left operand; that of the next block is on its way meanwhile.
__device__ __forceinline__ void ob_load_t(double (&T)[4], const double* __restrict__ Tg, int b, int g, int n)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) T[r] = Tg[256 * b + 16 * n + 4 * r + g];
}

template <int KB>
__device__ __forceinline__ void ob_block(f64x4 (&z)[2], const double (&T)[4], const double* __restrict__ Tg,
                                         const double* __restrict__ Vs, double* Wx, int wave, int g, int n)
{
    double T_next[4];
    ob_load_t(T_next, Tg, KB > 0 ? KB - 1 : 0, g, n);
    constexpr int Q0 = KB >= 4 ? 1 : 0;                   // block KB leaves the rows above 16 KB alone
    const double* V = Vs + 16 * KB * OB_LD + 16 * wave;
    double left[2][4], up[2][4];
#pragma unroll
    for (int q = Q0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) left[q][r] = V[n * OB_LD + 64 * q + 4 * r + g];
#pragma unroll
    for (int q = Q0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) up[q][r] = V[(4 * r + g) * OB_LD + 64 * q + n];
    f64x4 w[2];
    w[0] = w[1] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = Q0; q < 2; ++q) w[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(left[q][r], z[q][r], w[q], 0, 0, 0);
    f64x2* x = (f64x2*)Wx + (KB & 1) * 512 + 16 * g + n;
    x[128 * wave] = (f64x2){w[0][0] + w[1][0], w[0][1] + w[1][1]};
    x[128 * wave + 64] = (f64x2){w[0][2] + w[1][2], w[0][3] + w[1][3]};
    lds_barrier();
    const f64x2 lo = (x[0] + x[128]) + (x[256] + x[384]), hi = (x[64] + x[192]) + (x[320] + x[448]);
    const double s[4] = {lo.x, lo.y, hi.x, hi.y};
    f64x4 y = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) y = __builtin_amdgcn_mfma_f64_16x16x4f64(T[r], s[r], y, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = Q0; q < 2; ++q) z[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(up[q][r], y[r], z[q], 0, 0, 0);
    if constexpr (KB > 0) ob_block<KB - 1>(z, T_next, Tg, Vs, Wx, wave, g, n);
}

// Rank, mask, keep_idx, R_r and this slice's share of R_r R_r^T mu are made here as well, where the columns are in registers:
// the ranks while Z is on its way, and of R_r R_r^T mu 128 sums per slice, for eig_finish.
__global__ __launch_bounds__(256) void eig_orth_back(int U, double* __restrict__ scratch, float* __restrict__ R_out,
                                                     int32_t* __restrict__ status, int r, const float* __restrict__ lam,
                                                     const float* __restrict__ mu, uint8_t* __restrict__ mask_out,
                                                     int32_t* __restrict__ keep_out, float* __restrict__ Rr_out)
{
    extern __shared__ __attribute__((aligned(16))) double ob_lds[];
    double* Zs = ob_lds;                    // [128][130] all vectors of T; later the reflections, in natural order
    double* Ms = Zs + D * OB_LD;            // [128][17]; later the sums of ob_block (2048)
    int u, slice;
    eig_slice(u, slice);
    if (u >= U || status[2 * u] != 0) return;
    const int c0 = slice * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, n = lane & 15;
    double* W = scratch + (size_t)u * EIGW_TOTAL;
    float mu_row[8], lam_at[32];
    const float lam_own = lam[(size_t)u * D + c0 + n];
#pragma unroll
    for (int i = 0; i < 32; i += 4) {
        const f32x4_any l = *(const f32x4_any*)(lam + (size_t)u * D + 32 * g + i);
        lam_at[i] = l.x; lam_at[i + 1] = l.y; lam_at[i + 2] = l.z; lam_at[i + 3] = l.w;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) mu_row[i] = mu[(size_t)u * D + 16 * wave + 64 * (i >> 2) + 4 * (i & 3) + g];
    // every load of Z is out before the first is waited for; the reflections follow into registers and arrive under the
    // two products
    f64x2 stage[D * D / 512];
#pragma unroll
    for (int i = 0; i < D * D / 512; ++i) stage[i] = ((const f64x2*)(W + EIGW_Z))[tid + 256 * i];
    __builtin_amdgcn_sched_barrier(0);
    // rank of column c0 + n by value, ties to the lower column: a lane group counts over 32 of the others
    int rank = 0;
#pragma unroll
    for (int i = 0; i < 32; ++i)
        rank += (lam_at[i] > lam_own || (lam_at[i] == lam_own && 32 * g + i < c0 + n)) ? 1 : 0;
    rank += __shfl_xor(rank, 16);
    rank += __shfl_xor(rank, 32);
    const bool kept = rank < r;
    if (tid < 16) {
        mask_out[(size_t)u * D + c0 + n] = (uint8_t)kept;
        if (kept) keep_out[(size_t)u * r + rank] = c0 + n;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < D * D / 512; ++i) *(f64x2*)(Zs + ((tid >> 6) + 4 * i) * OB_LD + 2 * (tid & 63)) = stage[i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < D * D / 512; ++i) {
        const int k = (tid >> 6) + 4 * i;   // (rows 126 and 127 do not exist)
        stage[i] = ((const f64x2*)(W + EIGW_V))[min(k, D - 3) * (D / 2) + (tid & 63)];
    }
    double T[4];
    ob_load_t(T, W + EIGW_T, 7, g, n);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();

    // G = Z^T Z[:, c0 ..]: wave = rows 32 wave ..+31 of G.  A 16x16x4 step takes one contraction index per lane group;
    // two steps share a 16-byte read, so group g holds indices 8 t + 2 g + b of step pair t.
    // Result element r of lane (g, n) is row 4 r + g, column n.
    f64x4 acc[2];
    acc[0] = acc[1] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = 0; t < 16; ++t) {
        const int kk = 8 * t + 2 * g;
        const f64x2 bv = *(const f64x2*)(Zs + (c0 + n) * OB_LD + kk);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f64x2 av = *(const f64x2*)(Zs + (32 * wave + 16 * q + n) * OB_LD + kk);
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.x, acc[q], 0, 0, 0);
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, bv.y, acc[q], 0, 0, 0);
        }
    }
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 32 * wave + 16 * q + 4 * r + g;
            const double dev = acc[q][r] - (i == c0 + n ? 1.0 : 0.0);
            bad = bad || !(fabs(dev) < EIG_ORTH_MAX);
            Ms[i * OB_MLD + n] = (i == c0 + n ? 1.0 : 0.0) - 0.5 * dev;
        }
    if (bad) status[2 * u + 1] = 1;
    lds_barrier();

    // Z' = Z M for the 16 columns: row tiles wave and wave + 4
    f64x4 z[2];
    z[0] = z[1] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int t = 0; t < 32; ++t) {
        const int i = 4 * t + g;
        const double bv = Ms[i * OB_MLD + n];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            z[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(Zs[i * OB_LD + 16 * wave + 64 * q + n], bv, z[q], 0, 0, 0);
    }
    lds_barrier();
    // pairs left of block k / 32 of row k were not recorded
#pragma unroll
    for (int i = 0; i < D * D / 512; ++i) {
        const int k = (tid >> 6) + 4 * i, p = (tid & 63) >> 4;
        const bool there = k < D - 2 && p >= (k >> 5);
        double* d = Zs + k * OB_LD + 32 * p + (tid & 15);
        d[0] = there ? stage[i].x : 0.0;
        d[16] = there ? stage[i].y : 0.0;
    }
    lds_barrier();
    ob_block<7>(z, T, W + EIGW_T, Zs, Ms, wave, g, n);
    float* R = R_out + (size_t)u * D * D + c0 + n;
    float* Rk = Rr_out + (size_t)u * D * r + (kept ? rank : 0);
    double x[8], w = 0.0;                   // the columns as they are stored, and R^T mu
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 16 * wave + 64 * (i >> 2) + 4 * (i & 3) + g;
        const float f = (float)z[i >> 2][i & 3];
        R[row * D] = f;
        if (kept) Rk[row * r] = f;
        x[i] = (double)f;
        w = fma(x[i], (double)mu_row[i], w);
    }
    double* ws = Ms + 1024;                 // (ob_block<1>'s sums: everyone has read them before ob_block<0>'s barrier)
    ws[tid] = w;
    lds_barrier();
    w = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) w += ws[16 * i + n];
    w = kept ? w : 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] *= w;
    const double part = tri_fold<8, 0>(x, n);
    const int i = tri_fold_row<8>(n);
    if (!(n & 1)) ((float*)(W + EIGW_PART))[slice * D + 16 * wave + 64 * (i >> 2) + 4 * (i & 3) + g] = (float)part;
}

// ---------------------------------------------------------------------------
// Parallel two-sided Jacobi for the matrices that the reduction leaves alone, run by the work-group of eig_finish: a
// round-robin ordering (a sweep is 127 rounds of 64 disjoint pairs), A in LDS, the rows of V in registers.
// Pairs are taken by POSITION: position 2 k and 2 k + 1 form pair k, and after every round the rows and columns move
// to new positions (position 0 stays, 1 -> 2, even positions move up by two, 126 -> 127, odd positions move down by
// two): the 127 moving positions form one cycle, every two indices meet exactly once in 127 rounds, and after a sweep
// every index is back where it started, so eigenvalue c is the final A[c][c] and its vector is V[:, c].  Every thread
// reads and writes the same LDS addresses in every round: the rotated 2x2 block is written straight to its next
// position in a second copy of A, and only the part on or above the diagonal (by pair, then by position) is kept.
// V: lane k of a wave holds the elements at positions 2 k ("top") and 2 k + 1 ("bottom") of its rows, lane 0 its pair
// exchanged, so that the 127 moving positions form one ring through the registers: a round's movement is two
// whole-wave lane shifts and a select.
constexpr int EIG_THREADS = 1024;
constexpr int EIG_MAX_SWEEPS = 20;
constexpr int EIG_ROUNDS = D - 1;
constexpr int EIG_LD = D + 2;             // row stride of the LDS copies of A (even: a 2x2 block is two 8-byte reads)
constexpr size_t EIG_LDS_BYTES = (size_t)(2 * D * EIG_LD + 4 * 64 + 32 + D) * sizeof(float);

// LDS offset of the kept copy of element (r, c) = (c, r): pairs in ascending order, then positions
__device__ __forceinline__ constexpr int eig_upper(int r, int c)
{
    return ((r >> 1) < (c >> 1) || ((r >> 1) == (c >> 1) && r <= c)) ? r * (D + 2) + c : c * (D + 2) + r;
}

// position of a row / column after one round
__host__ __device__ constexpr int eig_next_pos(int p)
{
    return p == 0 ? 0 : p == 1 ? 2 : p == D - 2 ? D - 1 : (p & 1) ? p - 2 : p + 2;
}

// Rotation that annihilates the (p, q) element: t = tan, s = sin, tau = s / (1 + c).  One square
// root and hardware reciprocals with a Newton step each: the chain sits between the two barriers of
// every round, and the IEEE division and square-root sequences are several times as long.
// (s, tau) is applied as x' = x - s (y + tau x), y' = y + s (x - tau y), which is orthogonal to the
// accuracy of tau = s / (1 + c) alone, so a last-place error in t only moves the angle.
__device__ __forceinline__ float rcp_nr(float x)
{
    float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.f), r);
}
__device__ __forceinline__ void jacobi_params(float app, float aqq, float apq, float thr_skip, float& s, float& tau,
                                              float& t)
{
    s = 0.f; tau = 0.f; t = 0.f;
    if (fabsf(apq) > thr_skip) {
        // t = sgn(theta) / (|theta| + sqrt(theta^2 + 1)), theta = (aqq - app) / (2 apq), without forming theta
        const float al = aqq - app, be = 2.f * apq;
        const float h = __builtin_amdgcn_sqrtf(fmaf(al, al, be * be));
        t = (al >= 0.f) ? be * rcp_nr(al + h) : be * rcp_nr(al - h);
        const float d = fmaf(t, t, 1.f);
        float c = __builtin_amdgcn_rsqf(d);
        c = c * fmaf(-0.5f * d * c, c, 1.5f);          // one Newton step on 1/sqrt(d)
        s = t * c;
        tau = s * rcp_nr(1.f + c);
    }
}

// whole-wave lane shifts by one (data-parallel-primitive moves; the end lane has no source and keeps `keep`)
__device__ __forceinline__ float lane_from_below(float keep, float v)      // lane i <- lane i - 1; lane 0 keeps `keep`
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, keep), __builtin_bit_cast(int, v),
                                                                 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_from_above(float keep, float v)      // lane i <- lane i + 1; lane 63 keeps `keep`
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, keep), __builtin_bit_cast(int, v),
                                                                 0x130, 0xf, 0xf, false));
}

template <bool B>
struct EigBool { static constexpr bool value = B; };

constexpr int EIGV_ROWS = 9;                            // rows of V per wave (waves 1..15)
// Eigenvalues to lam_out [128] and vectors to R_out [128][128] (column c = vector of lam_out[c]); returns the number of
// sweeps, 20 = still above the threshold of 2e-8 ||C_q||_F.
__device__ __forceinline__ int jacobi_solve(const float* __restrict__ C, const float* __restrict__ sg,
                                            float* __restrict__ lam_out, float* __restrict__ R_out, float* sm)
{
    float* A2 = sm;                                   // [2][128][130]: the two copies of A
    float2* prm = (float2*)(A2 + 2 * D * EIG_LD);     // [2][64] (sin, sin / (1 + cos)) of this round and the next
    float* red = (float*)(prm + 128);                 // [32] reduction scratch
    constexpr int BUF = D * EIG_LD;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);          // 16 waves

    // load C_q = sigma_i sigma_j C_ij and ||C_q||_F^2
    float nrm = 0.f;
    for (int idx = tid; idx < D * D; idx += EIG_THREADS) {
        int i = idx >> 7, j = idx & 127;
        float v = C[idx];
        if (sg) v *= sg[i] * sg[j];
        A2[i * EIG_LD + j] = v;
        nrm = fmaf(v, v, nrm);
    }
    nrm = wave_sum(nrm);
    if (lane == 0) red[wave] = nrm;
    __syncthreads();
    float normF2 = 0.f;
    for (int w = 0; w < 16; ++w) normF2 += red[w];
    const float normF = sqrtf(normF2);
    const float thr_skip = 1e-12f * normF;
    const float tol2 = (2e-8f * 2e-8f) * normF2;
    __syncthreads();

    // The 2016 blocks above the diagonal as 32 wave-wide tasks, two per wave: task j covers row
    // pair j (63 - j blocks) in its first lanes and row pair 62 - j (j + 1 blocks) in the rest;
    // task 31 is the 32 blocks of row pair 31 alone.  A thread's two blocks never change.
    // Stores: one instruction stores an even column from lanes with bit 4 clear and an odd column from
    // the others (and the second instruction the other way round), so that the 32 lanes the LDS serves
    // together spread over all 32 banks instead of the 16 of one column parity.
    const bool hi16 = (lane & 16) != 0;
    int rd[2], rd1[2], pk[2], pkp[2], wa[2][2], wb[2][2];
    bool act[2];
#pragma unroll
    for (int ts = 0; ts < 2; ++ts) {
        const int j = ts == 0 ? wave : 31 - wave;
        const int split = 63 - j;
        const int k = lane < split ? j : 62 - j;
        const int kp = lane < split ? j + 1 + lane : 63 - j + (lane - split);
        act[ts] = !(j == 31 && lane >= 32);
        rd[ts] = 2 * k * EIG_LD + 2 * kp;
        rd1[ts] = rd[ts] + EIG_LD;
        asm volatile("" : "+v"(rd1[ts]));      // two 8-byte reads: measured at 7 cycles per wave against 10 for one two-address read
        pk[ts] = k;
        pkp[ts] = kp;
        const int r0 = eig_next_pos(2 * k), r1 = eig_next_pos(2 * k + 1);
        const int c0 = eig_next_pos(2 * kp), c1 = eig_next_pos(2 * kp + 1);
        // pairs (x0, x1) = (e00, e01) and (e10, e11): first store takes x0 in the low lanes and x1 in the
        // high lanes, second store the rest
        const int w00 = eig_upper(r0, c0), w01 = eig_upper(r0, c1), w10 = eig_upper(r1, c0), w11 = eig_upper(r1, c1);
        wa[ts][0] = hi16 ? w01 : w00; wb[ts][0] = hi16 ? w00 : w01;
        wa[ts][1] = hi16 ? w11 : w10; wb[ts][1] = hi16 ? w10 : w11;
    }
    // Wave 0, lane k, owns pair k: its diagonal block and its rotation.  The rotation of round n + 1 is
    // computed DURING round n, so that no wave ever waits for it: after round n the new diagonal
    // block of pair k holds the old (rotated) diagonal elements of pairs k - 1 and k + 1 -- known to
    // this wave -- and one off-diagonal element of the block (k - 1, k + 1), which the lane rotates
    // for itself from the current copy of A (lanes 0, 1 and 63 sit at the ends of the cycle and take
    // their three elements from the neighbouring places instead).
    const int lk = lane;
    const int lrow = lk <= 1 ? 0 : lk == 63 ? 62 : lk - 1;              // row pair of the look-ahead block
    const int lcol = lk == 0 ? 1 : lk == 63 ? 63 : lk + 1;              // its column pair
    const int lrd = 2 * lrow * EIG_LD + 2 * lcol;
    int lrd1 = lrd + EIG_LD;
    asm volatile("" : "+v"(lrd1));
    const int dn0 = eig_next_pos(2 * lk), dn1 = eig_next_pos(2 * lk + 1);
    float ps = 0.f, ptau = 0.f, dE00 = 0.f, dE11 = 0.f, dOff = 0.f;    // pair k: rotation and rotated diagonal block
    if (wave == 0) __builtin_amdgcn_s_setprio(3);     // its dependent chain is the critical path of every round (740 -> 727 us)
    if (wave == 0) {
        const int dg = 2 * lk * EIG_LD + 2 * lk;
        const float app = A2[dg], apq = A2[dg + 1], aqq = A2[dg + EIG_LD + 1];
        float tn;
        jacobi_params(app, aqq, apq, thr_skip, ps, ptau, tn);
        prm[lk] = make_float2(ps, ptau);
        dOff = (ps == 0.f) ? apq : 0.f;                    // left as it is when the rotation is skipped
        dE00 = app - tn * apq;
        dE11 = aqq + tn * apq;
    }
    __syncthreads();
    // Wave w >= 1 holds rows 9 (w - 1) .. + 8 of V (rows >= 128 are padding), lane k the elements at
    // positions 2 k and 2 k + 1
    float vtop[EIGV_ROWS], vbot[EIGV_ROWS];
    const int vrow0 = (wave - 1) * EIGV_ROWS;
#pragma unroll
    for (int i = 0; i < EIGV_ROWS; ++i) {
        {
            // lane 0 holds its pair exchanged (position 1 on top)
            vtop[i] = (wave > 0 && vrow0 + i == (lane == 0 ? 1 : 2 * lane)) ? 1.f : 0.f;
            vbot[i] = (wave > 0 && vrow0 + i == (lane == 0 ? 0 : 2 * lane + 1)) ? 1.f : 0.f;
        }
    }

    // One round: from copy FROM1 of A to the other one; rotations of this round in prm[FROM1].
    // Rotations are applied as x' = x - s (y + tau x), y' = y + s (x - tau y) with tau = s / (1 + c):
    // 1 - c is then carried to relative precision, so small angles (c rounding to 1) do not inflate
    // the column norms of V.
    auto round_step = [&](auto from1) {
        constexpr int F = decltype(from1)::value ? 1 : 0;
        const float* cur = A2 + F * BUF;
        float* nxt = A2 + (1 - F) * BUF;
        const float2* pcur = prm + 64 * F;
        float2* pnext = prm + 64 * (1 - F);
        if (wave == 0) {
            // this round's rotated diagonal blocks, at their next positions
            nxt[dn0 * EIG_LD + dn0] = dE00;
            nxt[dn1 * EIG_LD + dn1] = dE11;
            nxt[eig_upper(dn0, dn1)] = dOff;
            // next round's pair k
            const float2 ltop = *(const float2*)(cur + lrd), lbot = *(const float2*)(cur + lrd1);
            const float a00 = ltop.x, a01 = ltop.y, a10 = lbot.x, a11 = lbot.y;
            const float s1 = lane_from_below(ps, ps), tau1 = lane_from_below(ptau, ptau);      // pair k - 1 (lane 0: its own)
            const float s2 = lane_from_above(ps, ps), tau2 = lane_from_above(ptau, ptau);      // pair k + 1 (lane 63: its own)
            const float b00 = a00 - s1 * (a10 + tau1 * a00), b01 = a01 - s1 * (a11 + tau1 * a01);
            const float b10 = a10 + s1 * (a00 - tau1 * a10), b11 = a11 + s1 * (a01 - tau1 * a11);
            const float e00 = b00 - s2 * (b01 + tau2 * b00), e01 = b01 + s2 * (b00 - tau2 * b01);
            const float e11 = b11 + s2 * (b10 - tau2 * b11);
            const float apq = lk == 1 ? e11 : lk == 63 ? e00 : e01;
            const float below00 = lane_from_below(dE00, dE00), below11 = lane_from_below(dE11, dE11);
            const float app = lk == 1 ? below11 : below00;                 // lane 0: its own dE00
            const float aqq = lane_from_above(dE00, dE11);                 // lane 63: its own dE00
            float tn;
            jacobi_params(app, aqq, apq, thr_skip, ps, ptau, tn);
            pnext[lk] = make_float2(ps, ptau);
            dOff = (ps == 0.f) ? apq : 0.f;
            dE00 = app - tn * apq;
            dE11 = aqq + tn * apq;
        }
        float2 pv = make_float2(0.f, 0.f);
        if (wave != 0) {
            pv = pcur[lane];
            if (lane == 0) pv = make_float2(-pv.x, -pv.y);
        }
        float a[2][4];
        float2 p1[2], p2[2];
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) {
            const float2 top = *(const float2*)(cur + rd[ts]), bot = *(const float2*)(cur + rd1[ts]);
            a[ts][0] = top.x; a[ts][1] = top.y; a[ts][2] = bot.x; a[ts][3] = bot.y;
            p1[ts] = pcur[pk[ts]];
            p2[ts] = pcur[pkp[ts]];
        }
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) {
            const float s1 = p1[ts].x, tau1 = p1[ts].y, s2 = p2[ts].x, tau2 = p2[ts].y;
            const float a00 = a[ts][0], a01 = a[ts][1], a10 = a[ts][2], a11 = a[ts][3];
            // rows 2 k, 2 k + 1 : J^T from the left
            const float b00 = a00 - s1 * (a10 + tau1 * a00), b01 = a01 - s1 * (a11 + tau1 * a01);
            const float b10 = a10 + s1 * (a00 - tau1 * a10), b11 = a11 + s1 * (a01 - tau1 * a11);
            // columns 2 k', 2 k' + 1 : J from the right
            const float e00 = b00 - s2 * (b01 + tau2 * b00), e01 = b01 + s2 * (b00 - tau2 * b01);
            const float e10 = b10 - s2 * (b11 + tau2 * b10), e11 = b11 + s2 * (b10 - tau2 * b11);
            const float xa0 = hi16 ? e01 : e00, xb0 = hi16 ? e00 : e01;
            const float xa1 = hi16 ? e11 : e10, xb1 = hi16 ? e10 : e11;
            if (act[ts]) { nxt[wa[ts][0]] = xa0; nxt[wb[ts][0]] = xb0; nxt[wa[ts][1]] = xa1; nxt[wb[ts][1]] = xb1; }
        }
        if (wave != 0) {                      // V <- V J, then the columns move
            const bool lane0 = lane == 0;
#pragma unroll
            for (int i = 0; i < EIGV_ROWS; ++i) {
                const float x = vtop[i], y = vbot[i];
                const float xn = x - pv.x * (y + pv.y * x), yn = y + pv.x * (x - pv.y * y);
                const float b_dn = lane_from_above(xn, yn);
                vtop[i] = lane_from_below(b_dn, xn);
                vbot[i] = lane0 ? yn : b_dn;
            }
        }
        __syncthreads();
    };
    // One sweep that starts in copy START1 (and ends in the other one: 127 is odd).
    auto sweep_from = [&](auto start1) {
        constexpr bool S1 = decltype(start1)::value;
#pragma unroll 1
        for (int round = 0; round < EIG_ROUNDS - 1; round += 2) {
            round_step(EigBool<S1>{});
            round_step(EigBool<!S1>{});
        }
        round_step(EigBool<S1>{});
    };

    int sweeps_done = 0;
    for (int sweep = 0; sweep < EIG_MAX_SWEEPS; ++sweep) {
        // off-diagonal norm (every index is at its own position between sweeps)
        const float* cur = A2 + (sweeps_done & 1) * BUF;
        float off = 0.f;
        for (int idx = tid; idx < D * D; idx += EIG_THREADS) {
            int i = idx >> 7, j = idx & 127;
            float v = cur[i * EIG_LD + j];
            if (i < j) off = fmaf(2.f * v, v, off);             // only the upper triangle is kept
        }
        off = wave_sum(off);
        if (lane == 0) red[16 + wave] = off;
        __syncthreads();
        float off2 = 0.f;
        for (int w = 0; w < 16; ++w) off2 += red[16 + w];
        __syncthreads();
        if (!(off2 > tol2)) break;      // uniform across the block
        if (sweeps_done & 1) sweep_from(EigBool<true>{});
        else sweep_from(EigBool<false>{});
        ++sweeps_done;
    }

    const float* Af = A2 + (sweeps_done & 1) * BUF;
    if (tid < D) lam_out[tid] = Af[tid * EIG_LD + tid];
    if (wave != 0) {
#pragma unroll
        for (int i = 0; i < EIGV_ROWS; ++i)
            if (vrow0 + i < D)
                *(float2*)(R_out + (size_t)(vrow0 + i) * D + 2 * lane) =
                    lane == 0 ? make_float2(vbot[i], vtop[i]) : make_float2(vtop[i], vbot[i]);
    }
    __syncthreads();
    return sweeps_done;
}

// ---------------------------------------------------------------------------
// delta_mu = mu - R_r R_r^T mu (Alg. 1 steps 14 to 16), one work-group per matrix: for a solved matrix the sum of what
// eig_orth_back left (the work-groups of the other slices may still be running there, so the sum takes a launch).  A matrix
// that the reduction left alone is solved by Jacobi, and its rank, mask, keep_idx and R_r = R[:, keep] are made here too; R is
// staged in LDS (row stride 129) so that the column reads do not go to memory one by one.
// status NULL: every matrix is solved by Jacobi here.
// Bound: the launch and one memory round trip.  With the ranks, R_r and both products with mu made here, from R in memory, this
// kernel took 9.3 us for 32 matrices; the call is 6 us shorter so.
constexpr int EIGF_LD = D + 1;
constexpr int EIGF_THREADS = EIG_THREADS, EIGF_PARTS = EIGF_THREADS / D;
constexpr size_t EIGF_LDS_BYTES = (size_t)(D * EIGF_LD + EIGF_PARTS * D + 3 * D) * sizeof(float) + D * sizeof(int);
constexpr size_t EIGF_LDS_ALL = EIGF_LDS_BYTES > EIG_LDS_BYTES ? EIGF_LDS_BYTES : EIG_LDS_BYTES;
__global__ __launch_bounds__(EIGF_THREADS) void eig_finish(const float* __restrict__ cov, const float* __restrict__ sigma,
                                                           const int32_t* __restrict__ status,
                                                           const double* __restrict__ scratch, int r, float* R,
                                                           float* lam, uint8_t* __restrict__ mask_out,
                                                           int32_t* __restrict__ keep_out,
                                                           int32_t* __restrict__ sweeps_out,
                                                           const float* __restrict__ mu_in, float* __restrict__ Rr_out,
                                                           float* __restrict__ dmu_out)
{
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    const int u = blockIdx.x, tid = threadIdx.x;
    if (status) {                             // (everything is requested before the flags are looked at)
        const float* part = (const float*)(scratch + (size_t)u * EIGW_TOTAL + EIGW_PART) + (tid & (D - 1));
        float p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = part[i * D];
        const float m = mu_in[(size_t)u * D + (tid & (D - 1))];
        if ((status[2 * u] | status[2 * u + 1]) == 0) {
            if (tid < D) {
                double sum = 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) sum += (double)p[i];
                dmu_out[(size_t)u * D + tid] = (float)((double)m - sum);
            }
            if (tid == 0 && sweeps_out) sweeps_out[u] = 1;       // solved by the reduction
            return;
        }
    }
    const int sweeps = jacobi_solve(cov + (size_t)u * D * D, sigma ? sigma + (size_t)u * D : nullptr, lam + (size_t)u * D,
                                    R + (size_t)u * D * D, fsm);
    __threadfence_block();
    __syncthreads();
    if (tid == 0 && sweeps_out) sweeps_out[u] = sweeps;
    float* Vs = fsm;                          // [128][129]
    float* part = Vs + D * EIGF_LD;           // [parts][128] partial sums
    float* sw = part + EIGF_PARTS * D;        // [128] R_r^T mu
    float* smu = sw + D;                      // [128]
    int* skeep = (int*)(smu + D);             // [128]
    float* slam = (float*)(skeep + D);        // [128]
    const float* V = R + (size_t)u * D * D;
    for (int idx = tid; idx < D * D / 4; idx += EIGF_THREADS) {
        const float4 v = *(const float4*)(V + 4 * idx);
        float* d = Vs + (idx >> 5) * EIGF_LD + 4 * (idx & 31);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    }
    if (tid < D) smu[tid] = mu_in[(size_t)u * D + tid];
    if (tid < D) { slam[tid] = lam[(size_t)u * D + tid]; skeep[tid] = 0; }
    __syncthreads();
    if (tid < D) {                             // rank by value, ties to the lower column
        const float lc = slam[tid];
        int rank = 0;
        for (int i = 0; i < D; ++i) {
            const float li = slam[i];
            rank += (li > lc || (li == lc && i < tid)) ? 1 : 0;
        }
        mask_out[(size_t)u * D + tid] = (uint8_t)(rank < r);
        if (rank < r) {
            keep_out[(size_t)u * r + rank] = tid;
            skeep[rank] = tid;
        }
    }
    __syncthreads();
    for (int idx = tid; idx < D * r; idx += EIGF_THREADS) {
        int c = idx / r, j = idx - c * r;
        Rr_out[(size_t)u * D * r + idx] = Vs[c * EIGF_LD + skeep[j]];
    }
    const int pt = tid >> 7, x = tid & (D - 1);
    {                                          // w_j = sum_c V[c][keep_j] mu[c], the rows in EIGF_PARTS ranges
        float w = 0.f;
        if (x < r) {
            const int col = skeep[x];
            constexpr int RP = D / EIGF_PARTS;
            for (int c = RP * pt; c < RP * pt + RP; ++c) w = fmaf(Vs[c * EIGF_LD + col], smu[c], w);
        }
        part[pt * D + x] = w;
    }
    __syncthreads();
    if (tid < r) {
        float w = 0.f;
#pragma unroll
        for (int k = 0; k < EIGF_PARTS; ++k) w += part[k * D + tid];
        sw[tid] = w;
    }
    __syncthreads();
    {                                          // delta_mu[c] = mu[c] - sum_j V[c][keep_j] w_j, the kept columns in ranges
        float pr = 0.f;
        const int per = (r + EIGF_PARTS - 1) / EIGF_PARTS, j0 = min(pt * per, r), j1 = min(j0 + per, r);
        for (int j = j0; j < j1; ++j) pr = fmaf(Vs[x * EIGF_LD + skeep[j]], sw[j], pr);
        part[pt * D + x] = pr;
    }
    __syncthreads();
    if (tid < D) {
        float pr = 0.f;
#pragma unroll
        for (int k = 0; k < EIGF_PARTS; ++k) pr += part[k * D + tid];
        dmu_out[(size_t)u * D + tid] = smu[tid] - pr;
    }
}

__global__ __launch_bounds__(256) void gather_rotation_kernel(int r, const float* __restrict__ R,
                                                              const int32_t* __restrict__ keep_idx,
                                                              float* __restrict__ Rr)
{
    const int u = blockIdx.x;
    for (int idx = threadIdx.x; idx < D * r; idx += 256) {
        int c = idx / r, j = idx - c * r;
        int col = keep_idx[(size_t)u * r + j];
        col = min(max(col, 0), D - 1);
        Rr[(size_t)u * D * r + idx] = R[(size_t)u * D * D + c * D + col];
    }
}

// ---------------------------------------------------------------------------
hipError_t launch_eig(bool plain, int U, const float* cov, const float* sigma, const float* mu, int r, float* R,
                      float* lam, uint8_t* mask, int32_t* keep_idx, float* Rr, float* dmu, int32_t* sweeps,
                      void* scratch, int32_t* status, hipStream_t st)
{
    double* W = (double*)scratch;
    hipError_t e;
    if (!plain) {
        hipLaunchKernelGGL(eig_tridiag, dim3(U), dim3(TRI_THREADS), 0, st, cov, sigma, W, status);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(eig_tri_vectors, dim3(eig_slices(U)), dim3(256), 0, st, U, W, W, lam, status);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = allow_dynamic_lds((const void*)eig_orth_back, OB_LDS_BYTES);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(eig_orth_back, dim3(eig_slices(U)), dim3(256), OB_LDS_BYTES, st, U, W, R, status,
                           r, (const float*)lam, mu, mask, keep_idx, Rr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    e = allow_dynamic_lds((const void*)eig_finish, EIGF_LDS_ALL);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(eig_finish, dim3(U), dim3(EIGF_THREADS), EIGF_LDS_ALL, st, cov, sigma,
                       plain ? (const int32_t*)nullptr : status, (const double*)W, r, R, lam, mask,
                       keep_idx, sweeps, mu, Rr, dmu);
    return hipGetLastError();
}

hipError_t launch_gather_rotation(int U, int r, const float* R, const int32_t* keep_idx, float* Rr,
                                  hipStream_t st)
{
    hipLaunchKernelGGL(gather_rotation_kernel, dim3(U), dim3(256), 0, st, r, R, keep_idx, Rr);
    return hipGetLastError();
}

}  // namespace rk
