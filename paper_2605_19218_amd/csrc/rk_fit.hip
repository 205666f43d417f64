// Prefill-side rotation construction (Alg. 1 of the RotateK paper):
//   cov_partial_*   : per token chunk, S = sum x x^T and column sums   (Alg. 1 steps 1-3)
//   cov_finalize    : mu, C = S - n mu mu^T, reduced over chunks in fp64
//   sigma_window    : the query weights (step 4)
// The full eigendecomposition is in rk_eig.hip, the subspace iteration in rk_subspace.hip.
#include <mutex>
#include <set>
#include <utility>
#include "rk_kernels.hpp"

namespace rk {

hipError_t allow_dynamic_lds(const void* kernel, size_t bytes)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void*>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count({dev, kernel})) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done.insert({dev, kernel});
    return e;
}

// ---------------------------------------------------------------------------
// Plain covariance partial: 256 threads, thread (ty, tx) owns the 8x8 outputs
// (ty + 16 i, tx + 16 j); a 16-token tile is staged in LDS as fp32.
template <typename T>
__global__ __launch_bounds__(256) void cov_partial_generic(RowsDev rows, int Hkv, int n_chunks,
                                                           float* __restrict__ part_S,
                                                           float* __restrict__ part_sum)
{
    const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int u = b * Hkv + h;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int n_b = rows_count(rows, b);
    const int t0 = chunk * COV_CHUNK;
    const int t1 = min(t0 + COV_CHUNK, n_b);
    const T* base = (const T*)rows.data;

    __shared__ float tile[16][D];
    float acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    float csum = 0.f;

    for (int tt = t0; tt < t1; tt += 16) {
        {   // stage 16 rows x 128 channels; thread loads 8 consecutive channels of one row
            int rr = tt + ty;
            int c0 = tx * 8;
            if (rr < t1) {
                const T* src = base + rows_offset(rows, b, h, rr) + c0;
#pragma unroll
                for (int e = 0; e < 8; ++e) tile[ty][c0 + e] = ld_elem(src + e);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) tile[ty][c0 + e] = 0.f;
            }
        }
        __syncthreads();
        if (tid < D) {
#pragma unroll
            for (int t = 0; t < 16; ++t) csum += tile[t][tid];
        }
#pragma unroll 4
        for (int t = 0; t < 16; ++t) {
            float a[8], bb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) { a[i] = tile[t][ty + 16 * i]; bb[i] = tile[t][tx + 16 * i]; }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[i][j] = fmaf(a[i], bb[j], acc[i][j]);
        }
        __syncthreads();
    }
    float* S = part_S + ((size_t)u * n_chunks + chunk) * (D * D);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) S[(ty + 16 * i) * D + tx + 16 * j] = acc[i][j];
    if (tid < D) part_sum[((size_t)u * n_chunks + chunk) * D + tid] = csum;
}

// ---------------------------------------------------------------------------
// MFMA covariance partial (bf16 Keys): S = K^T K over a chunk (up to 2048 tokens, fewer on small inputs) with
// v_mfma_f32_32x32x16_bf16, contraction index = tokens.  The matrix core wants, per
// lane, 8 consecutive TOKENS of one channel, while memory holds 8 consecutive
// CHANNELS of one token.  No LDS staging is used: lane (g2, m) loads the 8x8 block
// (tokens 8 g2 ..+7) x (channels 8 (m%16) ..+7) as eight 16-byte row pieces and
// transposes it in registers with v_perm; lanes m and m+16 share a block and take
// the even / odd channels of it.  The channel held by MFMA row m of block cbk is
// therefore ch(cbk, m) = 8 (m % 16) + 2 cbk + m / 16 -- a permutation that is undone
// when the 128x128 partial is written.  Each wave accumulates the 10 upper-triangular
// 32x32 tiles for a quarter of the tokens (160 accumulator registers); the four waves are
// summed through LDS in a fixed order, each wave folding and storing a quarter.
constexpr int COVM_CHUNK = 2048;           // the longest chunk
constexpr int COVM_STAGES = 4;             // 16-token k-steps of loads in flight per wave (16 KB; 3 to 5 time alike, 6 and 8 slower)
constexpr size_t COVM_LDS_BYTES = (size_t)(4 * 30 * 4 * 64 + 4 * D) * sizeof(float);   // 4 x 30 parked groups + column sums

// Eight rows that all exist, without a token list: plain loads, nothing for the compiler to predicate, one 64-bit add a row.
// covm_load clamps to row t_last (always a valid one); covm_zero_past clears what lies behind the end.
__device__ __forceinline__ void covm_load_full(uint4 (&r)[8], const bf16_t* __restrict__ row, int64_t st)
{
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        // read-once stream: non-temporal, so the rows do not displace each other in the L2
        const u32x4 v = __builtin_nontemporal_load((const u32x4*)row);
        r[jj] = make_uint4(v.x, v.y, v.z, v.w);
        row += st;
    }
}

// Token-list form: the row numbers of a k-step (eight per lane) and the rows they address are
// two loads in a chain.  The row numbers are requested a whole turn of the stage ring ahead of
// their rows, so that the wait for them does not drain the rows in flight.
__device__ __forceinline__ void covm_load_idx(int (&ix)[8], const int32_t* __restrict__ list, int tok0, int t_last)
{
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) ix[jj] = list[min(tok0 + jj, t_last)];
}
// The same for eight rows that all exist: two loads (a list's rows start at any entry: 4-byte alignment).  Eight single loads
// beside eight rows in each of four stages are more than a wave's counter of loads in flight holds.  (4 x 32 heads, up to
// 4128 of 8192 rows: prefill 216.9 -> 213.9 us.)
__device__ __forceinline__ void covm_load_idx_full(int (&ix)[8], const int32_t* __restrict__ list, int tok0)
{
    typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    const i32x4_any a = *(const i32x4_any*)(list + tok0), b = *(const i32x4_any*)(list + tok0 + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { ix[e] = a[e]; ix[4 + e] = b[e]; }
}
__device__ __forceinline__ void covm_load_rows(uint4 (&r)[8], const bf16_t* __restrict__ base, int64_t head_base,
                                               int64_t st, const int (&ix)[8], int o)
{
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) r[jj] = *(const uint4*)(base + head_base + (int64_t)ix[jj] * st + 8 * o);
}

template <bool GATHER>
__device__ __forceinline__ void covm_load(uint4 (&r)[8], const bf16_t* __restrict__ base, int64_t head_base,
                                          int64_t st, const int32_t* __restrict__ list, int tok0, int t_last, int o)
{
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) r[jj] = *(const uint4*)(base + row_off<GATHER>(head_base, st, list, min(tok0 + jj, t_last)) + 8 * o);
}
__device__ __forceinline__ void covm_zero_past(uint4 (&r)[8], int tok0, int t_end)
{
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) r[jj] = tok0 + jj < t_end ? r[jj] : make_uint4(0, 0, 0, 0);
}

__device__ __forceinline__ uint32_t dw(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

__device__ __forceinline__ void covm_step(const uint4 (&r)[8], uint32_t sel, f32x16 (&acc)[10], float (&csum)[4])
{
    bf16x8 frag[4];
#pragma unroll
    for (int cbk = 0; cbk < 4; ++cbk) {
        uint4 d;
        // token pair (2 tp, 2 tp + 1) of channel 2 cbk + parity: low or high halves of dword cbk
        d.x = __builtin_amdgcn_perm(dw(r[1], cbk), dw(r[0], cbk), sel);
        d.y = __builtin_amdgcn_perm(dw(r[3], cbk), dw(r[2], cbk), sel);
        d.z = __builtin_amdgcn_perm(dw(r[5], cbk), dw(r[4], cbk), sel);
        d.w = __builtin_amdgcn_perm(dw(r[7], cbk), dw(r[6], cbk), sel);
        frag[cbk] = __builtin_bit_cast(bf16x8, d);
        // column sums: v_dot2 of each token pair with (1, 1), fp32 accumulate
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        float s = csum[cbk];
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, d.x), one2, s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, d.y), one2, s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, d.z), one2, s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, d.w), one2, s, false);
        csum[cbk] = s;
    }
    int t = 0;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = bi; bj < 4; ++bj) {
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[bi], frag[bj], acc[t], 0, 0, 0);
            ++t;
        }
}

// End-of-chunk reduction over the four waves of a work-group.  park area: [wave][30][lane]
// 16-byte groups, wave w's group g (not one of its own) at slot g - (g > 10 w ? 10 : 0).
constexpr int COVM_OWN = 10, COVM_PARKED = 30;
__device__ __forceinline__ constexpr int covm_slot(int w, int g) { return w * COVM_PARKED + (g < COVM_OWN * w ? g : g - COVM_OWN); }

template <int W>
__device__ __forceinline__ void covm_park(const f32x16 (&acc)[10], f32x4* __restrict__ park, int lane)
{
#pragma unroll
    for (int g = 0; g < 40; ++g)
        if (g / COVM_OWN != W)
            park[covm_slot(W, g) * 64 + lane] =
                (f32x4){acc[g >> 2][4 * (g & 3)], acc[g >> 2][4 * (g & 3) + 1], acc[g >> 2][4 * (g & 3) + 2], acc[g >> 2][4 * (g & 3) + 3]};
}

// partial layout written here: [g][lane][4] floats (element e of group g is accumulator
// i = 4 (g % 4) + e of tile g / 4)
template <int W>
__device__ __forceinline__ void covm_fold_store(const f32x16 (&acc)[10], const f32x4* __restrict__ park, int lane,
                                                f32x4* __restrict__ S4)
{
    f32x4 p[4][COVM_OWN];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int k = 0; k < COVM_OWN; ++k) {
            const int g = COVM_OWN * W + k;
            if (w == W) p[w][k] = (f32x4){acc[g >> 2][4 * (g & 3)], acc[g >> 2][4 * (g & 3) + 1], acc[g >> 2][4 * (g & 3) + 2], acc[g >> 2][4 * (g & 3) + 3]};
            else p[w][k] = park[covm_slot(w, g) * 64 + lane];
        }
#pragma unroll
    for (int k = 0; k < COVM_OWN; ++k) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = ((p[0][k][e] + p[1][k][e]) + p[2][k][e]) + p[3][k][e];
        S4[(COVM_OWN * W + k) * 64 + lane] = v;
    }
}

// A sequence of n rows is summed in as few chunks of at most `chunk_tokens` as hold it, dealt evenly to the 4 x `live` waves in blocks of
// `unit` rows; the other work-groups of a unit end at once and leave no partial, and cov_finalize_* counts the same way.  (With full
// chunks from the front and full shares to the waves of each, a last chunk took as long as a full one however short, and an
// empty one 11 us to sum, store and read zeros.)
__device__ __forceinline__ int live_chunks(int n, int chunk_tokens) { return (n + chunk_tokens - 1) / chunk_tokens; }
__device__ __forceinline__ void wave_rows(int n, int live, int unit, int w, int& first, int& last)
{
    const int blocks = (n + unit - 1) / unit, each = blocks / (4 * live), more = blocks - each * 4 * live;
    first = min((w * each + min(w, more)) * unit, n);
    last = min(first + (each + (w < more ? 1 : 0)) * unit, n);
}

template <bool GATHER>
__global__ __launch_bounds__(256) void cov_partial_mfma(RowsDev rows, int Hkv, int n_chunks, int chunk_tokens,
                                                        float* __restrict__ part_S, float* __restrict__ part_sum)
{
    // the chunk number is rotated by head and batch item: with a chunk count that is a multiple of 8 an
    // XCD (work-groups are dealt to the XCDs by linear index) would otherwise own one chunk position of
    // every sequence, and ragged batches have few sequences with the last positions
    const int h = blockIdx.y, b = blockIdx.z;
    const int chunk = (int)((blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x);
    const int u = b * Hkv + h;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: loop control stays scalar
    const int g2 = lane >> 5, m = lane & 31, o = m & 15, par = m >> 4;
    const uint32_t sel = par ? 0x07060302u : 0x05040100u;
    const int n_b = rows_count(rows, b);
    const int live = live_chunks(n_b, chunk_tokens);
    if (chunk >= live) return;
    int tw0, tw1;                                               // this wave's rows: whole turns of the stage ring but for the last wave's
    wave_rows(n_b, live, 16 * COVM_STAGES, 4 * chunk + wave, tw0, tw1);
    tw0 = __builtin_amdgcn_readfirstlane(tw0);
    tw1 = __builtin_amdgcn_readfirstlane(tw1);
    const int nks = tw1 > tw0 ? (tw1 - tw0 + 15) >> 4 : 0;      // 16-token k-steps, the last may be partial
    const int nfull = tw1 > tw0 ? (tw1 - tw0) >> 4 : 0;         // k-steps with all 16 tokens valid
    const bf16_t* base = (const bf16_t*)rows.data;
    const int64_t hb = (int64_t)b * rows.sb + (int64_t)h * rows.sh, rst = rows.st;
    const int32_t* list = GATHER ? rows.tok_idx + rows.tok_off[b] : nullptr;
    // this lane's first row piece: token tw0 + 8 g2, channels 8 o ..+7 (used when there is no token list)
    const bf16_t* lane_ptr = base + hb + (int64_t)(tw0 + 8 * g2) * rst + 8 * o;

    extern __shared__ __attribute__((aligned(16))) float cov_smem[];
    f32x4* bufv = (f32x4*)cov_smem;             // parked accumulator groups: [wave][30][lane]
    float (*ssum)[D] = (float (*)[D])(cov_smem + 4 * 30 * 4 * 64);

    f32x16 acc[10];
#pragma unroll
    for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    float csum[4] = {0.f, 0.f, 0.f, 0.f};

    if (nks > 0) {
        uint4 st[COVM_STAGES][8];
        int ks = 0;
        // Every wave owns a run of rows (often 256 x a power of two bytes at a multiple of that); walking them all from
        // the start would keep the 1024 waves of the grid on the same few HBM channels at any
        // instant.  A full wave therefore starts at a wave/chunk/head dependent
        // k-step and wraps around (the sum is order-independent up to fp32 rounding, and the
        // order is still fixed for a given launch shape).
        const bool wraps = nfull == nks && nks >= 2 * COVM_STAGES && nks % COVM_STAGES == 0;
        const int shift = wraps ? ((wave * 8 + chunk * 5 + u * 11) & ((1 << (31 - __clz(nks))) - 1)) : 0;
        int at = shift;                                             // the k-step that is requested next
        auto next_tok = [&]() {
            const int tok = 16 * at;
            ++at;
            at = wraps && at == nks ? 0 : at;
            return tok;
        };
        if (GATHER && nfull >= 2 * COVM_STAGES) {
            int ix[COVM_STAGES][8];
            const int last = nfull - 1;             // (behind the last full step of a wave that does not wrap it is read again, not used)
            auto next_full = [&]() {
                const int tok = next_tok();
                return wraps ? tok : min(tok, 16 * last);
            };
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) covm_load_idx_full(ix[s], list, tw0 + next_full() + 8 * g2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) {
                covm_load_rows(st[s], base, hb, rst, ix[s], o);
                covm_load_idx_full(ix[s], list, tw0 + next_full() + 8 * g2);
                __builtin_amdgcn_sched_barrier(0);
            }
            for (; ks + 2 * COVM_STAGES <= nfull; ks += COVM_STAGES) {
#pragma unroll
                for (int s = 0; s < COVM_STAGES; ++s) {
                    covm_step(st[s], sel, acc, csum);
                    covm_load_rows(st[s], base, hb, rst, ix[s], o);           // k-step ks + s + STAGES
                    covm_load_idx_full(ix[s], list, tw0 + next_full() + 8 * g2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else if (nfull >= 2 * COVM_STAGES) {
            // Long chunk (the normal case).  The fill and the steady loop use plain loads of
            // full k-steps with no branch anywhere near them, so every wait on them is exact
            // (a conservative wait-count state entering the loop would be paid every iteration).
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) {
                covm_load_full(st[s], lane_ptr + (int64_t)next_tok() * rst, rst);
                __builtin_amdgcn_sched_barrier(0);      // stage 0 must be the OLDEST load on loop entry
            }
            for (; ks + 2 * COVM_STAGES <= nfull; ks += COVM_STAGES) {
#pragma unroll
                for (int s = 0; s < COVM_STAGES; ++s) {
                    covm_step(st[s], sel, acc, csum);
                    covm_load_full(st[s], lane_ptr + (int64_t)next_tok() * rst, rst);
                    // keep "consume stage s, refill stage s" together: without this the scheduler
                    // hoists all four stages' math above all 32 loads and the pipeline collapses
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) covm_load<GATHER>(st[s], base, hb, rst, list, tw0 + 16 * s + 8 * g2, tw1 - 1, o);
        }
        // The stages in flight, and in the last wave of a sequence (or a short one) up to as many k-steps again, the last of them
        // possibly partial: all requested before the first is waited for.
        const int left = nks - ks;
        int ix[COVM_STAGES][8];
        if (GATHER && left > COVM_STAGES) {
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) covm_load_idx(ix[s], list, tw0 + 16 * (ks + s + COVM_STAGES) + 8 * g2, tw1 - 1);
        }
        auto step = [&](int s, int k) {
            if (k >= nks) return;
            if (k == nfull) covm_zero_past(st[s], tw0 + 16 * k + 8 * g2, tw1);
            covm_step(st[s], sel, acc, csum);
        };
#pragma unroll
        for (int s = 0; s < COVM_STAGES; ++s) {
            step(s, ks + s);
            if (s + COVM_STAGES < left) {
                if (GATHER) covm_load_rows(st[s], base, hb, rst, ix[s], o);
                else covm_load<false>(st[s], base, hb, rst, list, tw0 + 16 * (ks + s + COVM_STAGES) + 8 * g2, tw1 - 1, o);
            }
        }
        if (left > COVM_STAGES) {
#pragma unroll
            for (int s = 0; s < COVM_STAGES; ++s) step(s, ks + s + COVM_STAGES);
        }
    }

    // ---- sum the four waves, every element as ((w0 + w1) + w2) + w3 ----------------------
    // The 160 accumulators of a lane form 40 groups of four, g = 4 tile + i / 4.  Wave w owns
    // groups [10 w, 10 w + 10): it parks the 30 groups it does not own, and after ONE barrier
    // adds the three parked copies of its own groups to its registers (all 30 reads issued
    // before the first add) and stores its quarter of the chunk's partial, 16 bytes per lane.
#pragma unroll
    for (int cbk = 0; cbk < 4; ++cbk) {
        float s = csum[cbk] + __shfl_xor(csum[cbk], 32);
        if (g2 == 0) ssum[wave][8 * o + 2 * cbk + par] = s;
    }
    switch (wave) {
    case 0: covm_park<0>(acc, bufv, lane); break;
    case 1: covm_park<1>(acc, bufv, lane); break;
    case 2: covm_park<2>(acc, bufv, lane); break;
    default: covm_park<3>(acc, bufv, lane); break;
    }
    __syncthreads();
    f32x4* S4 = (f32x4*)(part_S + ((size_t)u * n_chunks + chunk) * (D * D));
    switch (wave) {
    case 0: covm_fold_store<0>(acc, bufv, lane, S4); break;
    case 1: covm_fold_store<1>(acc, bufv, lane, S4); break;
    case 2: covm_fold_store<2>(acc, bufv, lane, S4); break;
    default: covm_fold_store<3>(acc, bufv, lane, S4); break;
    }
    if (tid < D)
        part_sum[((size_t)u * n_chunks + chunk) * D + tid] = ((ssum[0][tid] + ssum[1][tid]) + ssum[2][tid]) + ssum[3][tid];
}

// ---------------------------------------------------------------------------
// MFMA covariance partial for fp32 Keys: S = K^T K over a chunk with v_mfma_f32_32x32x2_f32.  A 16-byte load of lane
// (h, m) = (lane / 32, lane % 32) takes channels 4 m ..+3 of token 2 t + h: its four elements are the operands of the four
// channel blocks, block cbk holding channels ch(cbk, m) = 4 m + cbk, so rows go from memory to the matrix cores as
// they are, two whole rows per load instruction.  Each wave accumulates the 10 upper-triangular tiles over a quarter of the chunk;
// the end of the chunk and the partial's layout are those of the bf16 kernel.
// Bound: the fp32 matrix rate (10 MFMA of 64 cycles per two tokens).  Chunks of 128 to 512 tokens, see cov_chunk_tokens
// (2 x 512 tokens: 97 us through the plain kernel, 10 us here).
constexpr int COVF_STAGES = 8;             // two-token steps of loads in flight per wave

template <bool GATHER>
__global__ __launch_bounds__(256) void cov_partial_f32(RowsDev rows, int Hkv, int n_chunks, int chunk_tokens,
                                                       float* __restrict__ part_S, float* __restrict__ part_sum)
{
    const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z, u = b * Hkv + h;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hh = lane >> 5, m = lane & 31;
    const int n_b = rows_count(rows, b);
    const int live = live_chunks(n_b, chunk_tokens);
    if (chunk >= live) return;
    int t0, t1;
    wave_rows(n_b, live, 2 * COVF_STAGES, 4 * chunk + wave, t0, t1);
    const int nst = t1 > t0 ? (t1 - t0 + 1) >> 1 : 0;
    const float* base = (const float*)rows.data + (int64_t)b * rows.sb + (int64_t)h * rows.sh + 4 * m;
    const int32_t* list = GATHER ? rows.tok_idx + rows.tok_off[b] : nullptr;

    extern __shared__ __attribute__((aligned(16))) float cov_smem[];
    f32x4* bufv = (f32x4*)cov_smem;             // parked accumulator groups: [wave][30][lane]
    float (*ssum)[D] = (float (*)[D])(cov_smem + 4 * 30 * 4 * 64);

    f32x16 acc[10];
#pragma unroll
    for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    f32x4 csum = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (nst > 0) {
        f32x4 st[COVF_STAGES];
        // rows past the end are read as the last row and count as zeros
        auto load = [&](int step) {
            const int tok = t0 + 2 * step + hh, tc = min(tok, t1 - 1);
            const f32x4 v = *(const f32x4*)(base + (GATHER ? (int64_t)list[tc] : (int64_t)tc) * rows.st);
            return tok < t1 ? v : (f32x4){0.f, 0.f, 0.f, 0.f};
        };
#pragma unroll
        for (int s = 0; s < COVF_STAGES; ++s) st[s] = load(s);
        for (int k = 0; k < nst; k += COVF_STAGES) {
#pragma unroll
            for (int s = 0; s < COVF_STAGES; ++s) {
                const f32x4 x = st[s];          // (steps past the last are zeros)
                csum += x;
                int t = 0;
#pragma unroll
                for (int bi = 0; bi < 4; ++bi)
#pragma unroll
                    for (int bj = bi; bj < 4; ++bj) {
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[bi], x[bj], acc[t], 0, 0, 0);
                        ++t;
                    }
                st[s] = load(k + s + COVF_STAGES);
            }
        }
    }
#pragma unroll
    for (int cbk = 0; cbk < 4; ++cbk) {
        const float s = csum[cbk] + __shfl_xor(csum[cbk], 32);
        if (hh == 0) ssum[wave][4 * m + cbk] = s;
    }
    switch (wave) {
    case 0: covm_park<0>(acc, bufv, lane); break;
    case 1: covm_park<1>(acc, bufv, lane); break;
    case 2: covm_park<2>(acc, bufv, lane); break;
    default: covm_park<3>(acc, bufv, lane); break;
    }
    __syncthreads();
    f32x4* S4 = (f32x4*)(part_S + ((size_t)u * n_chunks + chunk) * (D * D));
    switch (wave) {
    case 0: covm_fold_store<0>(acc, bufv, lane, S4); break;
    case 1: covm_fold_store<1>(acc, bufv, lane, S4); break;
    case 2: covm_fold_store<2>(acc, bufv, lane, S4); break;
    default: covm_fold_store<3>(acc, bufv, lane, S4); break;
    }
    if (tid < D)
        part_sum[((size_t)u * n_chunks + chunk) * D + tid] = ((ssum[0][tid] + ssum[1][tid]) + ssum[2][tid]) + ssum[3][tid];
}

// ---------------------------------------------------------------------------
// Reduce the chunk partials in fp64 and apply the centering correction
// C = S - n mu mu^T (equal to (K-mu)^T (K-mu)).  grid (8, U): block x covers rows
// [16x, 16x+16).
__global__ __launch_bounds__(256) void cov_finalize(RowsDev rows, int Hkv, int n_chunks, int center,
                                                    const float* __restrict__ part_S,
                                                    const float* __restrict__ part_sum,
                                                    float* __restrict__ cov, float* __restrict__ mu_out)
{
    const int u = blockIdx.y, b = u / Hkv;
    const int tid = threadIdx.x;
    const int n_b = rows_count(rows, b);
    __shared__ double smu[D];
    // sum over chunks in ascending order; loads are issued 8 at a time (independent), adds stay ordered
    auto chunk_sum = [&](const float* __restrict__ p, size_t stride) {
        double s = 0.0;
        int ch = 0;
        for (; ch + 8 <= n_chunks; ch += 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = p[(size_t)(ch + k) * stride];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += (double)v[k];
        }
        for (; ch < n_chunks; ++ch) s += (double)p[(size_t)ch * stride];
        return s;
    };
    if (tid < D) {
        double s = chunk_sum(part_sum + (size_t)u * n_chunks * D + tid, D);
        double m = n_b > 0 ? s / (double)n_b : 0.0;
        smu[tid] = m;
        if (blockIdx.x == 0) mu_out[(size_t)u * D + tid] = (float)m;
    }
    __syncthreads();
    const int j = tid & (D - 1);
    for (int ri = 0; ri < 8; ++ri) {
        int i = blockIdx.x * 16 + ri * 2 + (tid >> 7);
        const int pos = i * D + j;
        double s = chunk_sum(part_S + (size_t)u * n_chunks * (D * D) + pos, (size_t)D * D);
        if (center) s -= (double)n_b * (smu[i] * smu[j]);
        cov[(size_t)u * D * D + i * D + j] = (float)s;
    }
}

// Reduction of tile-format partials (written by cov_partial_mfma, or by cov_partial_f32 with its own channel order) in
// their own order: thread =
// one (tile, i, lane) position, so every load is coalesced across the wave and all chunks of a
// position are in flight together; the element goes to cov[r][c] and, for off-diagonal tiles
// and off-diagonal elements of diagonal tiles, cov[c][r] is written by its own position or
// mirrored here.  Grid (40, U): 10 tiles x 1024 positions per (b, h_kv).
template <bool F32>
__global__ __launch_bounds__(256) void cov_finalize_tiled(RowsDev rows, int Hkv, int slots, int chunk_tokens, int center,
                                                          const float* __restrict__ part_S,
                                                          const float* __restrict__ part_sum,
                                                          float* __restrict__ cov, float* __restrict__ mu_out)
{
    const int u = blockIdx.y, b = u / Hkv;
    const int tid = threadIdx.x;
    const int n_b = rows_count(rows, b);
    const int n_chunks = min(live_chunks(n_b, chunk_tokens), slots), last = max(n_chunks - 1, 0);
    __shared__ double smu[D];
    const int posn = blockIdx.x * 256 + tid;            // [tile][i / 4][lane][i % 4], 0 .. 10239
    const float* pS = part_S + (size_t)u * slots * (D * D) + posn;
    // the first 8 chunks of this position: requested before the mean is formed
    float v0[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v0[k] = pS[(size_t)min(k, last) * (D * D)];
    if (tid < D) {
        // column sums of the chunks, eight loads in flight at a time (one at a time this loop was most of
        // the kernel: eight dependent round trips), added in ascending chunk order
        const float* ps = part_sum + (size_t)u * slots * D + tid;
        double s = 0.0;
        for (int ch = 0; ch < n_chunks; ch += 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = ps[(size_t)min(ch + k, last) * D];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += ch + k < n_chunks ? (double)v[k] : 0.0;
        }
        const double m = n_b > 0 ? s / (double)n_b : 0.0;
        smu[tid] = m;
        if (blockIdx.x == 0) mu_out[(size_t)u * D + tid] = (float)m;
    }
    __syncthreads();
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += k < n_chunks ? (double)v0[k] : 0.0;          // ascending chunk order
    for (int ch = 8; ch < n_chunks; ch += 8) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = pS[(size_t)min(ch + k, last) * (D * D)];
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += ch + k < n_chunks ? (double)v[k] : 0.0;
    }
    // position -> (row channel, column channel): the MFMA output layout and the channel permutation undone
    const int t = posn >> 10, i = 4 * ((posn >> 8) & 3) + (posn & 3), lane = (posn >> 2) & 63;
    int br = 0, rem = t;
    while (rem >= 4 - br) { rem -= 4 - br; ++br; }
    const int bc = br + rem;
    const int mr = 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3), mc = lane & 31;
    const int rch = F32 ? 4 * mr + br : ((mr & 15) << 3) | (br << 1) | (mr >> 4);
    const int cch = F32 ? 4 * mc + bc : ((mc & 15) << 3) | (bc << 1) | (mc >> 4);
    if (center) acc -= (double)n_b * (smu[rch] * smu[cch]);
    float* Cu = cov + (size_t)u * D * D;
    Cu[rch * D + cch] = (float)acc;
    if (br != bc) Cu[cch * D + rch] = (float)acc;       // diagonal tiles hold both (r, c) and (c, r)
}

// The same sums in the same order for many units, one work-group per (b, h_kv) and class of rows: the 32 channels of one
// channel block, whose four tiles (those of the blocks before it transposed) come out through LDS as whole rows of cov.  In
// cov_finalize_tiled every position stores four bytes here and four there, a line's pieces from work-groups on different XCDs, and
// 40 work-groups per unit form the mean.  128 units of 3 chunks 12.8 -> 9.8 us, 512 of one 35.7 -> 17.2.
template <bool F32>
__global__ __launch_bounds__(256) void cov_finalize_rows(RowsDev rows, int Hkv, int slots, int chunk_tokens, int center,
                                                         const float* __restrict__ part_S, const float* __restrict__ part_sum,
                                                         float* __restrict__ cov, float* __restrict__ mu_out)
{
    constexpr int LD = D + 4, NC = 4;
    __shared__ double smu[D];
    __shared__ __attribute__((aligned(16))) float out[32 * LD];
    const int u = blockIdx.y, q = blockIdx.x, b = u / Hkv, tid = threadIdx.x, lane = tid & 63;
    const int n_b = rows_count(rows, b);
    const int n_chunks = min(live_chunks(n_b, chunk_tokens), slots), last = max(n_chunks - 1, 0);
    // four positions of each tile: groups [tile][i / 4][lane][i % 4] of cov_partial_mfma
    const f32x4* pS = (const f32x4*)(part_S + (size_t)u * slots * (D * D)) + tid;
    auto tile = [&](int c) { const int lo = min(q, c), hi = max(q, c); return 4 * lo - lo * (lo - 1) / 2 + hi - lo; };
    f32x4 v[NC][4];
    auto load = [&](int ch) {
#pragma unroll
        for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[k][c] = pS[(size_t)min(ch + k, last) * (D * D / 4) + 256 * tile(c)];
    };
    load(0);                                            // requested before the mean is formed
    if (tid < D) {
        const float* ps = part_sum + (size_t)u * slots * D + tid;
        double s = 0.0;
        for (int ch = 0; ch < n_chunks; ch += 8) {
            float w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = ps[(size_t)min(ch + k, last) * D];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += ch + k < n_chunks ? (double)w[k] : 0.0;
        }
        const double m = n_b > 0 ? s / (double)n_b : 0.0;
        smu[tid] = m;
        if (q == 0) mu_out[(size_t)u * D + tid] = (float)m;
    }
    __syncthreads();
    double acc[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[c][e] = 0.0;
    for (int ch = 0; ch < n_chunks; ch += NC) {
        if (ch) load(ch);
#pragma unroll
        for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][e] += ch + k < n_chunks ? (double)v[k][c][e] : 0.0;
    }
    auto channel = [](int block, int m) { return F32 ? 4 * m + block : ((m & 15) << 3) | (block << 1) | (m >> 4); };
    const int mc = lane & 31;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int mr = 8 * (tid >> 6) + 4 * (lane >> 5) + e;
            const int row = q <= c ? mr : mc, col = channel(c, q <= c ? mc : mr);
            double x = acc[c][e];
            if (center) x -= (double)n_b * (smu[channel(q, row)] * smu[col]);
            out[row * LD + col] = (float)x;
        }
    __syncthreads();
    float* Cu = cov + (size_t)u * D * D;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = (tid >> 5) + 8 * k;
        *(f32x4_any*)(Cu + channel(q, row) * D + 4 * (tid & 31)) = *(const f32x4*)(out + row * LD + 4 * (tid & 31));
    }
}

// ---------------------------------------------------------------------------
// Most chunks under COV_CHUNK tokens that a call makes per (b, h_kv): fp32 only, 512 work-groups in all (the workspace is sized
// by it, without a device to ask).
int cov_short_chunks(int dtype, int64_t units) { return dtype == 0 ? (int)(512 / units) : 0; }
// Work-groups run one per compute unit (registers and LDS): rounds of n_cu.  The chunk length that comes out cheapest:
int cov_chunk_tokens(int dtype, bool mfma, int64_t units, int max_tokens, int n_cu)
{
    if (!mfma) return COV_CHUNK;
    int best = COV_CHUNK;
    double least = 1e30;
    if (dtype == 1) {
        // A full chunk of 2048 tokens takes about 21 us of streaming when all units stream, and a work-group about 5 us beside it
        // (dispatch, end of chunk); a shorter chunk is taken where it is at least 15 % cheaper so priced.  (Rows are dealt evenly to as few
        // chunks as hold them, so a chunk is seldom full; the price is that of the longest one, and the reduction's partials go with the
        // count.)  Covariance, reduction and one subspace round, us, chunks of 512 / 1024 / 2048: 32 heads x 2944 tokens 32.4 / 33.0 / 34.2; 8 x
        // 1024 26.6 / 28.5 / 28.5; 64 x 3000 43.2 / 37.6 / 39.4, ragged 42.8 / 37.7 / 39.5; 128 x 5000 81.9 / 69.0 / 63.4; 128 ragged lists, up to 4128
        // rows, 67.8 / 53.9 / 46.7; 32 x 9000 ragged 42.3 / 43.4 / 37.3.  Of 28 shapes one is off by more than 0.6 us (8 x 16384: 512 tokens, 35.1 / 32.3 / 34.8).
        for (int ct = COVM_CHUNK; ct >= COV_CHUNK; ct /= 2) {
            const double wgs = (double)units * ((max_tokens + ct - 1) / ct), rounds = (double)((int64_t)(wgs + n_cu - 1) / n_cu);
            const double t = rounds * (21.0 * ct / COVM_CHUNK + 5.0);
            if (t < 0.85 * least) { least = t; best = ct; }
        }
        return best;
    }
    // fp32: 5 us of matrix work per 128 tokens and 3 us beside it, then the reduction, which reads eight chunks at a time (1 us of
    // latency each, and their bytes).  Whole fit, 1 x 65536 tokens: 94 us with 512 chunks of 128 tokens, 60 with 128 of 512; 8 x
    // 8192: 50 (128), 42 (256), 48 (512); 8 x 4000: 38, 38, 46; 32 x 3000: 50 with 512.
    const int few = cov_short_chunks(dtype, units);
    for (int ct = COV_CHUNK; ct >= COV_CHUNK_MIN; ct /= 2) {
        const int nc = (max_tokens + ct - 1) / ct;
        if (ct < COV_CHUNK && nc > few) break;
        const double rounds = (double)(((int64_t)units * nc + n_cu - 1) / n_cu);
        const double t = rounds * (5.1 * ct / 128 + 3.0) + ((nc + 7) / 8) * (1.0 + 0.1 * (double)units);
        if (t < least) { least = t; best = ct; }
    }
    return best;
}

hipError_t launch_cov_partial(int dtype, bool mfma, const RowsDev& rows, int B, int Hkv, int n_chunks, int chunk_tokens,
                              float* part_S, float* part_sum, hipStream_t st)
{
    dim3 grid(n_chunks, Hkv, B);
    if (mfma) {
        const auto kernel = dtype == 1 ? (rows.tok_idx ? cov_partial_mfma<true> : cov_partial_mfma<false>)
                                       : (rows.tok_idx ? cov_partial_f32<true> : cov_partial_f32<false>);
        const hipError_t e = allow_dynamic_lds((const void*)kernel, COVM_LDS_BYTES);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, dim3(256), COVM_LDS_BYTES, st, rows, Hkv, n_chunks, chunk_tokens, part_S, part_sum);
        return hipGetLastError();
    }
    if (dtype == 0)
        hipLaunchKernelGGL(cov_partial_generic<float>, grid, dim3(256), 0, st, rows, Hkv, n_chunks, part_S, part_sum);
    else
        hipLaunchKernelGGL(cov_partial_generic<bf16_t>, grid, dim3(256), 0, st, rows, Hkv, n_chunks, part_S, part_sum);
    return hipGetLastError();
}

hipError_t launch_cov_finalize(int dtype, bool mfma, const RowsDev& rows, int B, int Hkv, int n_chunks, int chunk_tokens, bool center,
                               const float* part_S, const float* part_sum, float* cov, float* mu, int n_cu, hipStream_t st)
{
    // (n_chunks: what the host's bound takes; of shorter sequences fewer are live, and both forms read only those.)
    // By rows from two work-groups a compute unit on, and not for long sequences of few units: four chunks are in flight in place of
    // eight, and off-diagonal tiles are read twice.  By rows / by positions: 32 units x 2 chunks 7.4 / 6.2 us; 128 x 2 10.2 / 11.7, x 12 18.7 /
    // 20.2, x 14 21.1 / 20.8, x 16 25.4 / 22.0; 256 x 12 33.5 / 37.2, x 16 45.4 / 42.3; 384 x 14 57 / 61, x 16 65 / 66; 512 x 14 72 / 81; fp32 128 x 6
    // 12.1 / 12.3, x 16 25.6 / 21.5.
    const int U = B * Hkv;
    if (mfma && 2 * U >= n_cu && (n_chunks <= 12 || 2 * U >= 3 * n_cu)) {
        const auto kernel = dtype == 1 ? cov_finalize_rows<false> : cov_finalize_rows<true>;
        hipLaunchKernelGGL(kernel, dim3(4, U), dim3(256), 0, st, rows, Hkv, n_chunks, chunk_tokens, center ? 1 : 0, part_S, part_sum, cov, mu);
    } else if (mfma && dtype == 1)
        hipLaunchKernelGGL(cov_finalize_tiled<false>, dim3(40, U), dim3(256), 0, st, rows, Hkv, n_chunks, chunk_tokens,
                           center ? 1 : 0, part_S, part_sum, cov, mu);
    else if (mfma)
        hipLaunchKernelGGL(cov_finalize_tiled<true>, dim3(40, U), dim3(256), 0, st, rows, Hkv, n_chunks, chunk_tokens,
                           center ? 1 : 0, part_S, part_sum, cov, mu);
    else
        hipLaunchKernelGGL(cov_finalize, dim3(8, U), dim3(256), 0, st, rows, Hkv, n_chunks, center ? 1 : 0,
                           part_S, part_sum, cov, mu);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Alg. 1 step 4: sigma_j = ||(Q_W)_{:,j}||_2 over the window of recent queries, pooled over the G query heads that
// share a KV head.  One work-group per (b, h_kv), of 1024 threads unless there are many: a row of 128 channels is read by 128 / VEC lanes, VEC
// elements (16 bytes where base and strides allow it, else one) each, and the other lanes take other rows, so that a
// window of 7 x 32 rows is four loads per thread, all out together.  (One thread per channel walking the rows two at a
// time: 30-51 us for 32 work-groups of 224 rows, a memory round trip for every pair of rows; now 4.6 us.)
template <typename T, int VEC, int THREADS>
__global__ __launch_bounds__(THREADS) void sigma_window_kernel(const T* __restrict__ qw, int64_t sb, int64_t sh,
                                                                   int64_t sw, int Hq, int Hkv, int W,
                                                                   float* __restrict__ sigma)
{
    constexpr int CG = D / VEC, RG = THREADS / CG, NF = 4;
    __shared__ float part[RG][D + 4];
    const int u = blockIdx.x, b = u / Hkv, hk = u % Hkv, G = Hq / Hkv;
    const int cg = threadIdx.x % CG, rg = threadIdx.x / CG;
    const T* base = qw + (int64_t)b * sb + (int64_t)hk * G * sh + cg * VEC;
    float a[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) a[e] = 0.f;
    // rows rg, rg + RG, ... of the G W rows, as head g and position w: a pointer that steps, no division or product per row
    const int qg = RG / W, qr = RG - qg * W;
    const int64_t step = qg * sh + qr * sw, wrap = sh - W * sw;
    int g = rg / W, w = rg - g * W;
    const T* next = base + g * sh + w * sw;
    while (g < G) {
        alignas(16) T x[NF][VEC];
        bool in[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {               // rows past the end are read as the first and count for nothing
            in[f] = g < G;
            const T* src = in[f] ? next : base;
            if constexpr (VEC == 1) x[f][0] = *src;
            else *(uint4*)x[f] = *(const uint4*)src;
            g += qg;
            w += qr;
            next += step;
            if (w >= W) { w -= W; ++g; next += wrap; }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float v = in[f] ? ld_elem(&x[f][e]) : 0.f;
                a[e] = fmaf(v, v, a[e]);
            }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) part[rg][cg * VEC + e] = a[e];
    __syncthreads();
    // the row groups in ranges, then the ranges, both in ascending order
    constexpr int NR = THREADS / D;
    __shared__ float sums[NR][D];
    {
        const int c = threadIdx.x & (D - 1), k = threadIdx.x >> 7;
        float t = 0.f;
        for (int i = k * RG / NR; i < (k + 1) * RG / NR; ++i) t += part[i][c];
        sums[k][c] = t;
    }
    __syncthreads();
    if (threadIdx.x < D) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < NR; ++k) t += sums[k][threadIdx.x];
        sigma[(size_t)u * D + threadIdx.x] = sqrtf(t);
    }
}

template <int THREADS>
static void launch_sigma_threads(int dtype, bool vec, const void* qw, int64_t sb, int64_t sh, int64_t sw, int U, int Hq, int Hkv,
                                 int W, float* sigma, hipStream_t st)
{
    const dim3 grid(U), block(THREADS);
    if (dtype == 0 && vec)
        hipLaunchKernelGGL((sigma_window_kernel<float, 4, THREADS>), grid, block, 0, st, (const float*)qw, sb, sh, sw, Hq, Hkv, W, sigma);
    else if (dtype == 0)
        hipLaunchKernelGGL((sigma_window_kernel<float, 1, THREADS>), grid, block, 0, st, (const float*)qw, sb, sh, sw, Hq, Hkv, W, sigma);
    else if (vec)
        hipLaunchKernelGGL((sigma_window_kernel<bf16_t, 8, THREADS>), grid, block, 0, st, (const bf16_t*)qw, sb, sh, sw, Hq, Hkv, W, sigma);
    else
        hipLaunchKernelGGL((sigma_window_kernel<bf16_t, 1, THREADS>), grid, block, 0, st, (const bf16_t*)qw, sb, sh, sw, Hq, Hkv, W, sigma);
}

hipError_t launch_sigma_window(int dtype, const void* qw, int64_t sb, int64_t sh, int64_t sw, int B, int Hq,
                               int Hkv, int W, float* sigma, hipStream_t st)
{
    // 16-byte reads need every row on a 16-byte boundary; the entry point takes any base and strides
    const int64_t es = dtype == 0 ? 4 : 2;
    const bool vec = (((int64_t)(uintptr_t)qw | sb * es | sh * es | sw * es) & 15) == 0;
    const int U = B * Hkv;
    const int64_t rows = (int64_t)(Hq / Hkv) * W;
    // Few units: 1024 threads, so that a window is in flight at once.  From 512 on (two such work-groups a compute unit) small ones,
    // of as many threads as the window has loads for (2048 units: 32 rows 10.3 us with 1024 threads, 4.8 with 128; 64 rows 14.7
    // and 5.3; 128 rows 15.5, 11.4 with 256).
    if (U < 512) launch_sigma_threads<1024>(dtype, vec, qw, sb, sh, sw, U, Hq, Hkv, W, sigma, st);
    else if (rows > 64) launch_sigma_threads<256>(dtype, vec, qw, sb, sh, sw, U, Hq, Hkv, W, sigma, st);
    else launch_sigma_threads<128>(dtype, vec, qw, sb, sh, sw, U, Hq, Hkv, W, sigma, st);
    return hipGetLastError();
}

}  // namespace rk
