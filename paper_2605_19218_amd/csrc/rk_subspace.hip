// Cholesky-based subspace iteration (Alg. 1 steps 6-13, App. E): T rounds of W <- C_q V, G = W^T W, L = chol(G + rho I),
// V = W L^{-T}, one 512-thread work-group per (b, h_kv) and the whole loop in one launch (the paper's four kernels per
// iteration exist to cut dispatch count; here there is nothing to dispatch).  All arithmetic is fp64: the Gram matrix
// has the squared condition of C_q's leading block, which fp32 cannot factor.
//
// Everything but the 16 x 16 factorisations runs on the fp64 matrix cores (v_mfma_f64_16x16x4), whose rate equals the
// vector rate here, but whose operands come 256 FMA to a lane's double: the vector form of this kernel was bound by LDS
// reads and by one barrier per column (163 / 235 / 377 us at k = 32 / 64 / 96, T = 5, 32 heads; now 61 / 120 / 195 us).
// Lane (g, n) = (lane / 16, lane % 16).  A 16x16x4 step takes A[n][g], B[g][n]; result register r is D[4 r + g][n].
// A tile held in that result layout is therefore, register by register, the B operand of a product that contracts over
// its rows, and, read as its transpose, the A operand.  The whole round is arranged around that:
//   - wave w owns rows 16 w ..+15 of the basis and keeps 16 columns of C_q (= rows: it is symmetric) in registers for
//     good, as B operands; W^T = V^T C_q comes out as tiles Y_J[j][i] (j: column 16 J + j of W, i: row 16 w + i);
//   - G needs W the other way round: each wave passes its rows through LDS once and adds up its share of every tile
//     G_JI, J <= I (contracted over its 16 rows); the eight shares are summed in wave order;
//   - block elimination: G_JJ = L D L^T and T_J = D^{-1/2} L^{-1} by wave 0 (see sub_factor), H_IJ = G_IJ T_J^T,
//     G_KI -= H_KJ H_IJ^T, V_J^T = T_J Y_J, Y_K -= H_KJ V_J^T.  Tiles of G, T and H are all kept as [lane][r], in which
//     they are operands as they are.
// The bound is the product with C_q (KT x 8 K cycles of fp64 matrix work), then wave 0's chain of factorisations, which
// the other waves' updates run beside.
#include "rk_kernels.hpp"

namespace rk {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int SUB_THREADS = 512, SUB_WAVES = SUB_THREADS / 64;
constexpr int SUB_MAX_K = 104;

template <int KT>
struct SubCfg {
    static constexpr int NT = KT * (KT + 1) / 2;          // tiles of the Gram matrix
    static constexpr int LDW = 16 * KT + 1;               // row stride of the basis
    // tiles whose eight shares are in LDS at a time (next to all of G), in passes of equal size
    static constexpr int FIT = (20000 - NT * 256) / (SUB_WAVES * 256) < 8 ? (20000 - NT * 256) / (SUB_WAVES * 256) : 8;
    static constexpr int NP = (NT + FIT - 1) / FIT, TP = (NT + NP - 1) / NP;
    static constexpr int OFF_G = TP * SUB_WAVES * 256;    // G behind the shares; the basis overlays both
    static constexpr int MAIN = OFF_G + NT * 256 > D * LDW ? OFF_G + NT * 256 : D * LDW;
    static constexpr size_t LDS_BYTES = (size_t)(MAIN + 4 * D + D + 2) * sizeof(double);
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

__device__ __forceinline__ double sub_make(uint32_t lo, uint32_t hi) { return __hiloint2double((int)hi, (int)lo); }
// value of lane J of every row of 16 lanes, for all lanes of the row
template <int J>
__device__ __forceinline__ double sub_row_bcast(double v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x150 + J, 0xf, 0xf, true);      // DPP row_newbcast, which takes 64 bits at a time
}
// value of lane (G0, n) for every lane (., n): odd and even rows of 16 lanes exchanged, then the halves of the wave
template <int G0>
__device__ __forceinline__ uint32_t sub_group_bcast32(uint32_t v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t x = (G0 & 1) ? a[1] : a[0];            // rows (0, 0, 2, 2) or (1, 1, 3, 3)
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (G0 & 2) ? b[1] : b[0];
}
template <int G0>
__device__ __forceinline__ double sub_group_bcast(double v)
{
    return sub_make(sub_group_bcast32<G0>((uint32_t)__double2loint(v)), sub_group_bcast32<G0>((uint32_t)__double2hiint(v)));
}
// 1 / sqrt(a) for a > 0: hardware estimate and one third-order step
__device__ __forceinline__ double sub_rsqrt(double a)
{
    const double y = __builtin_amdgcn_rsq(a), r = fma(-(a * y), y, 1.0);
    return fma(y * r, fma(r, 0.375, 0.5), y);
}

// Steps J .. 15 of the elimination of [x | m] = [G_JJ | I] in one wave: lane (g, n) holds elements (n, 4 q + g) of both.
// Row n becomes (pivot times itself - G[n][J] times row J) / 2^e, 2^e the pivot's power of two, so that no reciprocal stands
// between one pivot and the next; the pivot's mantissa, in [1/2, 1), scales all the rows below alike, and `scale` keeps
// their product: what is left of m is scale times L^{-1}, and the pivots are scale times D.  (With the reciprocal, 1 / pivot, in
// the chain the kernel took 62 / 124 / 201 us at k = 32 / 64 / 96; with lanes' values moved by halves besides, 65 / 129 / 207.)
template <int J>
__device__ __forceinline__ void sub_eliminate(double (&x)[4], double (&m)[4], double& own, double& scale, bool& bad, int n)
{
    if constexpr (J < 16) {
        constexpr int QJ = J >> 2, GJ = J & 3;
        const int src = 16 * GJ + J;
        const double p = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x[QJ]), src),
                                          __builtin_amdgcn_readlane(__double2loint(x[QJ]), src));
        bad = bad || !(p > 0.0);
        own = n == J ? p : own;
        const double col = sub_group_bcast<GJ>(x[QJ]);
        const double keep = n > J ? __builtin_amdgcn_frexp_mant(p) : 1.0;
        const double f = n > J ? -ldexp(col, -__builtin_amdgcn_frexp_exp(p)) : 0.0;
        scale *= keep;
#pragma unroll
        for (int q = QJ; q < 4; ++q) x[q] = fma(f, sub_row_bcast<J>(x[q]), keep * x[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) m[q] = q <= QJ ? fma(f, sub_row_bcast<J>(m[q]), keep * m[q]) : keep * m[q];
        sub_eliminate<J + 1>(x, m, own, scale, bad, n);
    }
}

// T_J = D^{-1/2} L^{-1} of the tile in x (result layout; the tile is symmetric), stored as [lane][r] = T[n][4 r + g].
__device__ __forceinline__ void sub_factor(f64x4 x4, double* __restrict__ tile, int* __restrict__ flag, int lane)
{
    const int g = lane >> 4, n = lane & 15;
    double x[4], m[4], own = 1.0, scale = 1.0;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        x[q] = x4[q];
        m[q] = n == 4 * q + g ? 1.0 : 0.0;
    }
    sub_eliminate<0>(x, m, own, scale, bad, n);
    const double sc = sub_rsqrt(own * scale);
    ((f64x2*)tile)[2 * lane] = (f64x2){m[0] * sc, m[1] * sc};
    ((f64x2*)tile)[2 * lane + 1] = (f64x2){m[2] * sc, m[3] * sc};
    if (lane == 0 && bad) *flag = 1;
}

__device__ __forceinline__ f64x4 sub_tile(const double* __restrict__ t, int lane)
{
    const f64x2 a = ((const f64x2*)t)[2 * lane], b = ((const f64x2*)t)[2 * lane + 1];
    return (f64x4){a.x, a.y, b.x, b.y};
}
__device__ __forceinline__ void sub_tile_store(double* __restrict__ t, int lane, const f64x4& v)
{
    ((f64x2*)t)[2 * lane] = (f64x2){v[0], v[1]};
    ((f64x2*)t)[2 * lane + 1] = (f64x2){v[2], v[3]};
}
// c + a b: the four steps of a 16 x 16 x 16 product (a: A[n][4 r + g], b: B[4 r + g][n])
__device__ __forceinline__ f64x4 sub_mma(const f64x4& a, const f64x4& b, f64x4 c)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[r], c, 0, 0, 0);
    return c;
}
constexpr int sub_idx(int I, int J) { return I * (I + 1) / 2 + J; }      // tile G_JI, J <= I

template <int KT>
__global__ __launch_bounds__(SUB_THREADS) void subspace_iter(const float* __restrict__ cov, const float* __restrict__ sigma,
                                                             const float* __restrict__ mu, const float* __restrict__ V0,
                                                             int k, int T, double eps, float* __restrict__ Rr,
                                                             float* __restrict__ dmu, int32_t* __restrict__ status)
{
    typedef SubCfg<KT> Cfg;
    constexpr int LDW = Cfg::LDW, NT = Cfg::NT, TP = Cfg::TP;
    extern __shared__ __attribute__((aligned(16))) double sub_lds[];
    double* W = sub_lds;                                  // [128][LDW]
    double* P = sub_lds;                                  // [8][TP][256] shares
    double* G = sub_lds + Cfg::OFF_G;                     // [NT][256]
    double* part = sub_lds + Cfg::MAIN;                   // [4][128]
    double* tv = part + 4 * D;                            // [128]
    int* flag = (int*)(tv + D);

    const int u = blockIdx.x, tid = threadIdx.x;
    int lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* C = cov + (size_t)u * D * D;
    double c[32];                                         // C_q[4 s + g][16 wave + n]
    {
        float cf[32], sf[32];
#pragma unroll
        for (int s = 0; s < 32; ++s) {
            cf[s] = C[(16 * wave + n) * D + 4 * s + g];
            sf[s] = sigma ? sigma[(size_t)u * D + 4 * s + g] : 1.f;
        }
        const double sn = sigma ? (double)sigma[(size_t)u * D + 16 * wave + n] : 1.0;
#pragma unroll
        for (int s = 0; s < 32; ++s) c[s] = (double)cf[s] * ((double)sf[s] * sn);
    }
    for (int idx = tid; idx < D * 16 * KT; idx += SUB_THREADS) {
        const int i = idx / (16 * KT), j = idx - i * (16 * KT);
        W[i * LDW + j] = j < k ? (double)V0[(size_t)u * D * k + (size_t)i * k + j] : 0.0;    // padding columns stay zero
    }
    if (tid == 0) *flag = 0;
    lds_barrier();

    int fail = 0;
#pragma unroll 1
    for (int t = 0; t < T; ++t) {
        // The lane numbers are made opaque in every round: otherwise the LDS addresses derived from them (dozens) are
        // computed before the loop and held in registers, or spilled, through all of it.
        asm volatile("" : "+v"(lane), "+v"(g), "+v"(n));
        // ---- Y = (C_q V)^T for this wave's 16 rows ----
        f64x4 Y[KT];
#pragma unroll
        for (int J = 0; J < KT; ++J) Y[J] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 32; ++s)
#pragma unroll
            for (int J = 0; J < KT; ++J)
                Y[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[(4 * s + g) * LDW + 16 * J + n], c[s], Y[J], 0, 0, 0);
        lds_barrier();                                    // every wave has read the old basis
        // ---- this wave's rows the other way round: f_J[s] = W[16 wave + 4 s + g][16 J + n] ----
        f64x4 f[KT];
#pragma unroll
        for (int J = 0; J < KT; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) W[(16 * wave + n) * LDW + 16 * J + 4 * r + g] = Y[J][r];
        wave_lds_fence();
#pragma unroll
        for (int J = 0; J < KT; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) f[J][r] = W[(16 * wave + 4 * r + g) * LDW + 16 * J + n];
        lds_barrier();                                    // the basis is read: its space takes the shares of G
        asm volatile("" : "+v"(lane));
        // ---- G_JI = sum over the waves of f_J^T f_I, TP tiles at a time ----
#pragma unroll
        for (int p = 0; p < Cfg::NP; ++p) {
#pragma unroll
            for (int I = 0; I < KT; ++I)
#pragma unroll
                for (int J = 0; J <= I; ++J) {
                    const int q = sub_idx(I, J) - p * TP;
                    if (q >= 0 && q < TP)
                        sub_tile_store(P + (wave * TP + q) * 256, lane, sub_mma(f[J], f[I], (f64x4){0.0, 0.0, 0.0, 0.0}));
                }
            lds_barrier();
            for (int e = tid; e < TP * 128; e += SUB_THREADS)
                if (p * TP * 128 + e < NT * 128) {
                    f64x2 s = ((const f64x2*)P)[e];
#pragma unroll
                    for (int w = 1; w < SUB_WAVES; ++w) s += ((const f64x2*)P)[w * TP * 128 + e];
                    ((f64x2*)G)[p * TP * 128 + e] = s;
                }
            lds_barrier();
        }
        // ---- rho = eps tr(G) / k, identity in the padding, and the first block ----
        if (wave == 0) {
            double d[2], tr = 0.0;
            int at[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int a = lane + 64 * h, an = a & 15;
                at[h] = sub_idx(a >> 4, a >> 4) * 256 + (16 * (an & 3) + an) * 4 + (an >> 2);
                d[h] = a < k ? G[at[h]] : 0.0;
                tr += d[h];
            }
            tr = row16_sum_f64(tr);
            tr = (sub_group_bcast<0>(tr) + sub_group_bcast<1>(tr)) + (sub_group_bcast<2>(tr) + sub_group_bcast<3>(tr));
            const double rho = eps * tr / (double)k;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (lane + 64 * h < 16 * KT) G[at[h]] = lane + 64 * h < k ? d[h] + rho : 1.0;
            wave_lds_fence();
            sub_factor(sub_tile(G, lane), G, flag, lane);
        }
        lds_barrier();
        asm volatile("" : "+v"(lane), "+v"(g), "+v"(n));
        // ---- block elimination ----
#pragma unroll
        for (int J = 0; J < KT; ++J) {
            const f64x4 TJ = sub_tile(G + sub_idx(J, J) * 256, lane);
            if (J + 1 + wave < KT) {                      // H_IJ = G_IJ T_J^T, one I per wave, as (T_J G_JI)
                double* ht = G + ((J + 1 + wave) * (J + 2 + wave) / 2 + J) * 256;
                sub_tile_store(ht, lane, sub_mma(TJ, sub_tile(ht, lane), (f64x4){0.0, 0.0, 0.0, 0.0}));
            }
            Y[J] = sub_mma(TJ, Y[J], (f64x4){0.0, 0.0, 0.0, 0.0});                   // V_J^T
            if (J + 1 == KT) break;
            lds_barrier();
            // wave 0: the next diagonal block and its factor; the other waves: the other tiles G_KI, K <= I, in turn
            if (wave == 0) {
                const f64x4 h = -sub_tile(G + sub_idx(J + 1 < KT ? J + 1 : J, J) * 256, lane);
                double* gt = G + sub_idx(J + 1 < KT ? J + 1 : J, J + 1 < KT ? J + 1 : J) * 256;
                sub_factor(sub_mma(h, -h, sub_tile(gt, lane)), gt, flag, lane);
            } else {
                int turn = 0;
#pragma unroll
                for (int I = J + 1; I < KT; ++I)
#pragma unroll
                    for (int K = J + 1; K <= I; ++K) {
                        if (I == J + 1) continue;
                        if (turn % (SUB_WAVES - 1) == wave - 1) {
                            double* gt = G + sub_idx(I, K) * 256;
                            const f64x4 hk = -sub_tile(G + sub_idx(K, J) * 256, lane), hi = sub_tile(G + sub_idx(I, J) * 256, lane);
                            sub_tile_store(gt, lane, sub_mma(hk, hi, sub_tile(gt, lane)));
                        }
                        ++turn;
                    }
            }
#pragma unroll
            for (int K = J + 1; K < KT; ++K) Y[K] = sub_mma(-sub_tile(G + sub_idx(K, J) * 256, lane), Y[J], Y[K]);
            lds_barrier();
        }
        lds_barrier();                                    // G is dead, its space may take the basis again
        if (*flag) { fail = t + 1; break; }               // uniform; the rest of the round ran on meaningless numbers
#pragma unroll
        for (int J = 0; J < KT; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) W[(16 * wave + n) * LDW + 16 * J + 4 * r + g] = Y[J][r];
        lds_barrier();
    }

    // ---- outputs: R_k = V, delta_mu = mu - V V^T mu (Alg. 1 steps 14, 16) ----
    if (tid == 0 && status) status[u] = fail;
    if (fail) {
        // No basis (its place holds Gram tiles): R_k = 0 and delta_mu = mu, so that an empty sequence of a ragged batch, whose
        // Gram matrix is zero, stays finite when tokens are appended to it.
        for (int idx = tid; idx < D * k; idx += SUB_THREADS) Rr[(size_t)u * D * k + idx] = 0.f;
        if (tid < D) dmu[(size_t)u * D + tid] = mu[(size_t)u * D + tid];
        return;
    }
    for (int idx = tid; idx < D * k; idx += SUB_THREADS) {
        const int i = idx / k, j = idx - i * k;
        Rr[(size_t)u * D * k + idx] = (float)W[i * LDW + j];
    }
    const int pt = tid >> 7, x = tid & (D - 1);
    {
        double a = 0.0;
        if (x < k)
            for (int i = 32 * pt; i < 32 * pt + 32; ++i) a = fma(W[i * LDW + x], (double)mu[(size_t)u * D + i], a);
        part[pt * D + x] = a;
    }
    lds_barrier();
    if (tid < D) tv[tid] = (part[tid] + part[D + tid]) + (part[2 * D + tid] + part[3 * D + tid]);
    lds_barrier();
    {
        const int per = (k + 3) / 4, j0 = min(pt * per, k), j1 = min(j0 + per, k);
        double a = 0.0;
        for (int j = j0; j < j1; ++j) a = fma(W[x * LDW + j], tv[j], a);
        part[pt * D + x] = a;
    }
    lds_barrier();
    if (tid < D)
        dmu[(size_t)u * D + tid] = (float)((double)mu[(size_t)u * D + tid] -
                                           ((part[tid] + part[D + tid]) + (part[2 * D + tid] + part[3 * D + tid])));
}

int subspace_max_keep() { return SUB_MAX_K; }

template <int KT>
static hipError_t launch_subspace_kt(int U, const float* cov, const float* sigma, const float* mu, const float* V0, int k,
                                     int T, double eps, float* Rr, float* dmu, int32_t* status, hipStream_t st)
{
    const hipError_t e = allow_dynamic_lds((const void*)subspace_iter<KT>, SubCfg<KT>::LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(subspace_iter<KT>, dim3(U), dim3(SUB_THREADS), SubCfg<KT>::LDS_BYTES, st, cov, sigma, mu, V0, k, T,
                       eps, Rr, dmu, status);
    return hipGetLastError();
}

hipError_t launch_subspace(int U, const float* cov, const float* sigma, const float* mu, const float* V0, int k,
                           int T, double eps, float* Rr, float* dmu, int32_t* status, hipStream_t st)
{
    if (k < 1 || k > SUB_MAX_K) return hipErrorInvalidValue;
    switch ((k + 15) / 16) {
        case 1: return launch_subspace_kt<1>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 2: return launch_subspace_kt<2>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 3: return launch_subspace_kt<3>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 4: return launch_subspace_kt<4>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 5: return launch_subspace_kt<5>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 6: return launch_subspace_kt<6>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        case 7: return launch_subspace_kt<7>(U, cov, sigma, mu, V0, k, T, eps, Rr, dmu, status, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rk
