// Rotate + gather + pack of the Key cache (Alg. 1 step 14: K~ = K R_k, stored in
// place of K, rounded once to the cache dtype), re-tiling of the Values into the
// decode kernel's fragment-major layout, the frozen-R append of new tokens (the
// rotation is fitted once at the end of prefill and reused, Sec. 3.2 Step (1)),
// and the inverse re-tiling used to inspect a cache.
#include "rk_kernels.hpp"
#include <type_traits>

namespace rk {

// ---------------------------------------------------------------------------
// Plain kernel, any dtype and any r: 64 tokens per block, K tile in LDS as fp32,
// thread (t, j) accumulates over the 128 channels in ascending order.
template <typename T>
__global__ __launch_bounds__(256) void compress_generic(RowsDev rows, int Hkv, int cap, int r,
                                                        const float* __restrict__ Rr, T* __restrict__ Kp,
                                                        int32_t* __restrict__ seq_len_out)
{
    const int h = blockIdx.y, b = blockIdx.z, u = b * Hkv + h;
    const int tid = threadIdx.x;
    const int n_b = min(rows_count(rows, b), cap);
    if (blockIdx.x == 0 && h == 0 && tid == 0 && seq_len_out) seq_len_out[b] = n_b;
    const int t0 = blockIdx.x * 64;
    if (t0 >= n_b) return;
    const int nt = min(64, n_b - t0);
    const int rp = keep_padded(r);
    const T* base = (const T*)rows.data;
    __shared__ float tile[64][D];
    for (int idx = tid; idx < nt * D; idx += 256) {
        int t = idx >> 7, c = idx & 127;
        tile[t][c] = ld_elem(base + rows_offset(rows, b, h, t0 + t) + c);
    }
    __syncthreads();
    const float* Ru = Rr + (size_t)u * D * r;
    T* Ku = Kp + (size_t)u * slab_tokens(cap) * rp;
    for (int o = tid; o < nt * rp; o += 256) {
        int t = o / rp, j = o - t * rp;
        float a = 0.f;
        if (j < r)                                  // channels r .. rp - 1 are the layout's zero padding
            for (int c = 0; c < D; ++c) a = fmaf(tile[t][c], Ru[c * r + j], a);
        st_elem(Ku + kidx(t0 + t, j, rp), a);
    }
}

// ---------------------------------------------------------------------------
// Values -> fragment-major V cache: NB blocks of 32 tokens from token t0 on, transposed through LDS; rows past the sequence end
// inside the last block are zero-filled.  All rows are requested before the first is parked (bf16: 32 KB a work-group with NB = 4).
template <typename T>
struct alignas(16) Oct { T v[8]; };
constexpr int RETILE_LD = 17;                    // 16 octets per row + 1 pad

template <typename T, int NB>
__device__ __forceinline__ void retile_blocks(const RowsDev& rows, int b, int h, int n_b, int t0, T* __restrict__ Vu,
                                              Oct<T>* __restrict__ tile)
{
    const int tid = threadIdx.x;
    const T* base = (const T*)rows.data;
    Oct<T> x[2 * NB];
    auto fetch = [&](int t) { return *(const Oct<T>*)(base + rows_offset(rows, b, h, t) + (tid & 15) * 8); };
#pragma unroll
    for (int k = 0; k < 2 * NB; ++k) {           // several blocks: nothing conditional between the loads, the last row in place of those past it
        const int t = t0 + 16 * k + (tid >> 4);
        if (NB > 1 || t < n_b) x[k] = fetch(NB > 1 ? min(t, n_b - 1) : t);
    }
#pragma unroll
    for (int k = 0; k < 2 * NB; ++k) {
        const int row = 16 * k + (tid >> 4);
        if (t0 + row >= n_b) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[k].v[e] = (T)0;
        }
        tile[row * RETILE_LD + (tid & 15)] = x[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2 * NB; ++k) {
        const int tb = t0 + 32 * (k >> 1);
        if (tb >= n_b) break;
        const int o = tid + 256 * (k & 1);       // piece index: [cb][g][n]
        const int cb = o >> 6, g = (o >> 4) & 3, n = o & 15;
        const int c = 16 * cb + n;
        Oct<T> y;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int tl = 32 * (k >> 1) + (jj < 4 ? 4 * g + jj : 16 + 4 * g + (jj - 4));
            y.v[jj] = tile[tl * RETILE_LD + (c >> 3)].v[c & 7];
        }
        T* to = Vu + (size_t)(tb >> 5) * 4096 + (size_t)o * 8;
        if constexpr (sizeof(Oct<T>) == 16) nt_store16(to, __builtin_bit_cast(uint4, y));
        else *(Oct<T>*)to = y;
    }
}

// The Values of the call, by work-groups behind those of the Keys in the same launch (grid.z from `batch` on, `per_head` work-groups a
// head).  They need nothing of the Keys' result, so the launch's ramp and tail are paid once, and the short work-groups
// here fill up the compute units that the rotation leaves early.
template <typename T>
struct ValuesJob {
    static constexpr int NB = sizeof(T) == 2 ? 4 : 1;
    static constexpr size_t LDS_BYTES = (size_t)NB * 32 * RETILE_LD * sizeof(Oct<T>);
    RowsDev rows;
    T* dst;
    int batch, heads, per_head;
};
struct NoValues {};
template <typename T, bool VALUES>
using ValuesArg = std::conditional_t<VALUES, ValuesJob<T>, NoValues>;

template <typename T>
__device__ __forceinline__ void retile_job(const ValuesJob<T>& v, int Hkv, int cap, Oct<T>* tile)
{
    const int id = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * (blockIdx.z - v.batch)), u = id / v.per_head;
    if (u >= v.heads) return;
    // The block number is rotated by the head, as the Keys' is: with as many blocks a head as a multiple of 8, sequences far below the bound would
    // have all their rows on a few XCDs (r = 64, in order / rotated, us: 128 x 1 heads x 100 of 2000 tokens 17.8 / 7.7; 64 x 1 x 1000 of 2000 17.3 / 13.8;
    // 16 x 8 x 1024 ragged 18.9 / 14.7; full sequences alike).  Heads fastest would be better for the shortest and up to 9 % worse for full ones.
    const int b = u / Hkv, t0 = (int)(((unsigned)id + (unsigned)u) % (unsigned)v.per_head) * 32 * ValuesJob<T>::NB;
    const int n_b = min(rows_count(v.rows, b), cap);
    if (t0 < n_b) retile_blocks<T, ValuesJob<T>::NB>(v.rows, b, u - b * Hkv, n_b, t0, v.dst + (size_t)u * slab_tokens(cap) * D, tile);
}

// a launch of its own
template <typename T>
__global__ __launch_bounds__(256) void v_retile(RowsDev rows, int Hkv, int cap, T* __restrict__ dst)
{
    __shared__ Oct<T> tile[32 * RETILE_LD];
    const int h = blockIdx.y, b = blockIdx.z;
    const int n_b = min(rows_count(rows, b), cap), t0 = blockIdx.x * 32;
    if (t0 < n_b) retile_blocks<T, 1>(rows, b, h, n_b, t0, dst + (size_t)(b * Hkv + h) * slab_tokens(cap) * D, tile);
}

// ---------------------------------------------------------------------------
// MFMA kernel (bf16; R = r padded to a multiple of 16, columns r .. R - 1 of R_r read as
// zero, which writes the layout's zero padding).  Per wave: D^T[j, token] = R_r^T . K^T
// with v_mfma_f32_16x16x32_bf16; the B operand (lane (g, n): token n, channels
// 32 i + 8 g ..+7) is a plain 16-byte load of a Key row, so Keys go from HBM
// straight into MFMA registers.  R_r is split into bf16 head + remainder
// (two MFMAs) to keep ~fp32 accuracy of the fp32 rotation.  The rows of the A
// operand are permuted so that after output blocks 2i and 2i+1 lane (g, n) holds
// the 8 output channels 32 i + 8 g ..+7 of token n -- one 16-byte piece of the
// packed layout, and consecutive lanes write consecutive pieces.
template <int R>
struct CompressCfg {
    static constexpr int JB = R / 16;                 // 16-wide output-channel blocks
    static constexpr int NF = R / 32;                 // full 32-channel groups
    static constexpr bool TAIL = (R % 32) != 0;       // one trailing 16-channel block
    static constexpr int TT = 2;                      // 16-token tiles per wave and pass (two passes in flight)
    static constexpr int TOK_PER_PASS = 4 * TT * 16;  // tokens one pass of the 4 waves covers
    static constexpr int PASSES = 4;                  // passes per work-group (amortise the R_r fragment build)
    static constexpr int TOK_PER_BLOCK = PASSES * TOK_PER_PASS;
    static constexpr size_t LDS_BYTES = (size_t)JB * 4 * 2 * 64 * 16;   // A fragments, hi+lo
    // output channel held by A row a of block jb
    __host__ __device__ static constexpr int chan(int jb, int a) {
        return (jb < 2 * NF) ? 32 * (jb >> 1) + 8 * (a >> 2) + 4 * (jb & 1) + (a & 3) : 32 * NF + a;
    }
};

__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
    return (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16);
}

enum { ORDER_FEW, ORDER_MANY, ORDER_PART_LAST };

// VALUES: the launch also lays out the Values (a kernel of its own: with the branch in every launch, 4 x 32 heads through token lists took 23.2
// us instead of 20.9).
template <int R, bool GATHER, bool VALUES>
__global__ __launch_bounds__(256, 2) void compress_mfma(RowsDev rows, int Hkv, int cap, int r, int order,
                                                     const float* __restrict__ Rr, bf16_t* __restrict__ Kp,
                                                     int32_t* __restrict__ seq_len_out, ValuesArg<bf16_t, VALUES> vals)
{
    typedef CompressCfg<R> Cfg;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if constexpr (VALUES) {
        if ((int)blockIdx.z >= vals.batch) {
            retile_job(vals, Hkv, cap, (Oct<bf16_t>*)smem_raw);
            return;
        }
    }
    bf16x8* frag = (bf16x8*)smem_raw;       // [JB][4][2][64]

    // ORDER_PART_LAST: the last block number is a partly filled one.  Its work-groups then start behind all others, where they fill
    // up the compute units that the full ones leave; among them, a compute unit gets two full ones while the next gets two short ones
    // (16 x 16 heads x 600 rows, r = 32: 15.4 -> 11.8 us; 4 x 32 x 2100, r = 128: 43 -> 34.6; 1 x 32 x 16500, r = 64: 45.7 -> 41.6).
    int h = blockIdx.y, b = blockIdx.z, nx = gridDim.x, bx = blockIdx.x;
    bool rotate = true;
    int vals_batch = gridDim.z;
    if constexpr (VALUES) vals_batch = vals.batch;
    if (order == ORDER_PART_LAST) {
        const int id = bx + nx * (h + Hkv * b), full = --nx * (int)gridDim.y * vals_batch;
        rotate = id < full;
        const int w = rotate ? id / nx : id - full;
        bx = __builtin_amdgcn_readfirstlane(rotate ? id - w * nx : nx);
        b = __builtin_amdgcn_readfirstlane(w / Hkv);
        h = __builtin_amdgcn_readfirstlane(w - b * Hkv);
    }
    // Work-groups go to the 8 XCDs round-robin by linear index.  The block number is rotated by head and batch item, so that
    // an XCD does not end up with "block 7 of every sequence" (which only the longest sequences have); an odd count of blocks walks
    // over the XCDs by itself, and rotated like that 9, 17, .. blocks would stand still.  ORDER_FEW: a compute unit for
    // every work-group; always rotated, as the covariance kernel rotates its chunks (whose rows start elsewhere but for lengths that fill
    // them): fit by eigenvectors and rotation, r = 32, us, so / in the other orders: 1 x 8 heads x 1100 tokens 148.3 / 148.7; 1 x 16 x 3000 152.3 / 153.1; 2 x 8,
    // 1700 listed rows, with Values 157.0 / 158.4; 1 x 8, 4500 listed rows, 157.4 / 158.9; 1 x 8, 2410 listed 149.8 / 150.0.
    if (rotate && (order == ORDER_FEW || !(nx & 1))) bx = (int)((unsigned)(bx + h + b) % (unsigned)nx);
    const int u = b * Hkv + h;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, n = lane & 15;
    const int n_b = min(rows_count(rows, b), cap);
    if (bx == 0 && h == 0 && tid == 0 && seq_len_out) seq_len_out[b] = n_b;
    const int blk0 = bx * Cfg::TOK_PER_BLOCK;
    if (blk0 >= n_b) return;

    const bf16_t* base = (const bf16_t*)rows.data;
    const int64_t hb = (int64_t)b * rows.sb + (int64_t)h * rows.sh;
    const int32_t* list = GATHER ? rows.tok_idx + rows.tok_off[b] : nullptr;
    bf16_t* Ku = Kp + (size_t)u * slab_tokens(cap) * R;

    // Row numbers of one pass of this wave (token list entries; the token itself without a list).
    // Rows past the end are clamped to the last row (never stored).
    auto load_rows_idx = [&](int (&idx)[Cfg::TT], int w0) {
#pragma unroll
        for (int tt = 0; tt < Cfg::TT; ++tt) {
            const int tok = min(w0 + tt * 16 + n, n_b - 1);
            idx[tt] = GATHER ? list[tok] : tok;
        }
    };
    // Key rows of one pass, straight into B-operand registers.  Every row is read once: non-temporal.
    auto load_keys_at = [&](bf16x8 (&kb)[Cfg::TT][4], const int (&idx)[Cfg::TT]) {
#pragma unroll
        for (int tt = 0; tt < Cfg::TT; ++tt) {
            const bf16_t* row = base + hb + (int64_t)idx[tt] * rows.st;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                kb[tt][i] = __builtin_bit_cast(bf16x8, __builtin_nontemporal_load((const u32x4*)(row + 32 * i + 8 * g)));
        }
    };
    auto load_keys = [&](bf16x8 (&kb)[Cfg::TT][4], int w0) {
        int idx[Cfg::TT];
        load_rows_idx(idx, w0);
        load_keys_at(kb, idx);
    };
    // rotate one pass and store its packed rows
    auto rotate_store = [&](const bf16x8 (&kb)[Cfg::TT][4], int w0, auto all_valid) {
        f32x4 acc[Cfg::TT][Cfg::JB];
#pragma unroll
        for (int tt = 0; tt < Cfg::TT; ++tt)
#pragma unroll
            for (int jb = 0; jb < Cfg::JB; ++jb) acc[tt][jb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jb = 0; jb < Cfg::JB; ++jb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bf16x8 ah = frag[((jb * 4 + i) * 2 + 0) * 64 + lane];
                bf16x8 al = frag[((jb * 4 + i) * 2 + 1) * 64 + lane];
#pragma unroll
                for (int tt = 0; tt < Cfg::TT; ++tt) {
                    acc[tt][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, kb[tt][i], acc[tt][jb], 0, 0, 0);
                    acc[tt][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, kb[tt][i], acc[tt][jb], 0, 0, 0);
                }
            }
            // the fragment reads of one output block at a time: hoisting all of them costs 128 registers
            if (Cfg::JB > 4 && (jb & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        // lane (g, n): blocks 2i, 2i+1 hold channels 32 i + 8 g + (0..3), (4..7) of token w0 + 16 tt + n
#pragma unroll
        for (int tt = 0; tt < Cfg::TT; ++tt) {
            int tok = w0 + tt * 16 + n;
            if (decltype(all_valid)::value || tok < n_b) {
                bf16_t* blk = Ku + (size_t)((w0 >> 4) + tt) * (16 * R);
#pragma unroll
                for (int i = 0; i < Cfg::NF; ++i) {
                    uint4 pk;
                    pk.x = pack2_bf16(acc[tt][2 * i][0], acc[tt][2 * i][1]);
                    pk.y = pack2_bf16(acc[tt][2 * i][2], acc[tt][2 * i][3]);
                    pk.z = pack2_bf16(acc[tt][2 * i + 1][0], acc[tt][2 * i + 1][1]);
                    pk.w = pack2_bf16(acc[tt][2 * i + 1][2], acc[tt][2 * i + 1][3]);
                    nt_store16(blk + (4 * i) * 128 + lane * 8, pk);
                }
                if (Cfg::TAIL) {
                    uint2 pk;
                    pk.x = pack2_bf16(acc[tt][Cfg::JB - 1][0], acc[tt][Cfg::JB - 1][1]);
                    pk.y = pack2_bf16(acc[tt][Cfg::JB - 1][2], acc[tt][Cfg::JB - 1][3]);
                    nt_store8(blk + (4 * Cfg::NF + (g >> 1)) * 128 + n * 8 + 4 * (g & 1), pk);
                }
            }
        }
    };

    // A fragments: block jb, k-step i, lane (gk, a): row a <-> output channel chan(jb, a);
    // k slots <-> input channels 32 i + 8 gk + jj.  Thread tid builds fragment (jb = it, i = tid / 64,
    // lane = tid % 64) for it = 0 .. JB - 1: R_r elements first (all loads of a thread in flight
    // together), the split into bf16 head + remainder after them.
    const float* Ru = Rr + (size_t)u * D * r;
    const int fi = tid >> 6, fgk = lane >> 4, fa = lane & 15;
    float rx[Cfg::JB][8];
    // EXACT: r is the kernel's own width (the common case), so the row stride of R_r is a compile-time
    // constant; otherwise r < R and the columns r .. R - 1 are the zero padding
    auto fetch_Rr = [&](auto exact) {
        constexpr bool EXACT = decltype(exact)::value;
        const int rs = EXACT ? R : r;
#pragma unroll
        for (int jb = 0; jb < Cfg::JB; ++jb) {
            const int j = Cfg::chan(jb, fa);
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                rx[jb][jj] = Ru[(32 * fi + 8 * fgk + jj) * rs + (EXACT ? j : min(j, r - 1))];
        }
    };
    auto park_fragments = [&]() {
#pragma unroll
        for (int jb = 0; jb < Cfg::JB; ++jb) {
            const bool pad = Cfg::chan(jb, fa) >= r;
            bf16x8 hi, lo;
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                __bf16 xh, xl;
                split_bf16(pad ? 0.f : rx[jb][jj], xh, xl);
                hi[jj] = xh;
                lo[jj] = xl;
            }
            frag[((jb * 4 + fi) * 2 + 0) * 64 + lane] = hi;
            frag[((jb * 4 + fi) * 2 + 1) * 64 + lane] = lo;
        }
    };
    if (r == R) fetch_Rr(std::true_type{});
    else fetch_Rr(std::false_type{});
    __builtin_amdgcn_sched_barrier(0);

    const int w_first = blk0 + wave * (Cfg::TT * 16);
    // Passes in pairs, the Key rows of pass p + 1 requested before pass p is rotated, the first pass
    // before R_r is even split -- R_r's loads are older than the Key loads, so the wait for them does
    // not wait for Keys.  Nothing is loaded conditionally (rows past the end are clamped to the last
    // row and never stored) and the trip count is uniform, so every wait on a load is exact.  A full
    // block makes PASSES passes; the ragged last block of a sequence makes as many as it has rows for,
    // rounded up to a pair.
    static_assert(Cfg::PASSES % 2 == 0 && Cfg::PASSES >= 4, "passes are taken in pairs");
    auto run_block = [&](auto full, int np2) {
        constexpr int TP = Cfg::TOK_PER_PASS;
        bf16x8 ka[Cfg::TT][4], kc[Cfg::TT][4];
        if (!GATHER) {
            load_keys(ka, w_first);
            __builtin_amdgcn_sched_barrier(0);
            park_fragments();
            __syncthreads();
#pragma unroll 1
            for (int p = 0; p < np2 - 2; p += 2) {
                load_keys(kc, w_first + (p + 1) * TP);
                __builtin_amdgcn_sched_barrier(0);
                rotate_store(ka, w_first + p * TP, full);
                load_keys(ka, w_first + (p + 2) * TP);
                __builtin_amdgcn_sched_barrier(0);
                rotate_store(kc, w_first + (p + 1) * TP, full);
            }
            load_keys(kc, w_first + (np2 - 1) * TP);
            __builtin_amdgcn_sched_barrier(0);
            rotate_store(ka, w_first + (np2 - 2) * TP, full);
            rotate_store(kc, w_first + (np2 - 1) * TP, full);
            return;
        }
        // With a token list a row's address comes from a load.  The row numbers of pass p + 2 are
        // requested BEFORE the rows of pass p + 1, so that waiting for them (the oldest loads in flight
        // by then) leaves the rows of the pass in between in flight; requested together with the rows
        // they address, every pass would begin with a full round trip and an empty pipeline.
        int ia[Cfg::TT], ic[Cfg::TT];
        load_rows_idx(ia, w_first);
        load_rows_idx(ic, w_first + TP);
        __builtin_amdgcn_sched_barrier(0);
        load_keys_at(ka, ia);
        __builtin_amdgcn_sched_barrier(0);
        park_fragments();
        __syncthreads();
#pragma unroll 1
        for (int p = 0; p < np2 - 2; p += 2) {
            load_rows_idx(ia, w_first + (p + 2) * TP);
            __builtin_amdgcn_sched_barrier(0);
            load_keys_at(kc, ic);
            __builtin_amdgcn_sched_barrier(0);
            rotate_store(ka, w_first + p * TP, full);
            load_rows_idx(ic, w_first + min(p + 3, np2 - 1) * TP);
            __builtin_amdgcn_sched_barrier(0);
            load_keys_at(ka, ia);
            __builtin_amdgcn_sched_barrier(0);
            rotate_store(kc, w_first + (p + 1) * TP, full);
        }
        load_keys_at(kc, ic);
        __builtin_amdgcn_sched_barrier(0);
        rotate_store(ka, w_first + (np2 - 2) * TP, full);
        rotate_store(kc, w_first + (np2 - 1) * TP, full);
    };
    const int rows_here = min(n_b - blk0, Cfg::TOK_PER_BLOCK);
    run_block(std::false_type{}, (((rows_here + Cfg::TOK_PER_PASS - 1) / Cfg::TOK_PER_PASS) + 1) & ~1);
}

// ---------------------------------------------------------------------------
// MFMA kernel for fp32 caches: D^T[j, token] = R_r^T . K^T with v_mfma_f32_16x16x4_f32, all in fp32.  The contraction
// may run over the channels in any order as long as both operands agree: step (i, e) takes channel 16 i + 4 g + e in lane
// group g, so a lane's four steps of one i are one 16-byte piece of a Key row and one 16-byte LDS read of the
// fragments of R_r ([jb][i][lane]).  Lane (g, n) ends up with output channels 16 jb + 4 g ..+3 of token n: one 16-byte
// piece of the packed layout, consecutive lanes writing consecutive pieces.  128 tokens per work-group, two 16-token
// tiles per wave.  Bound: the fp32 matrix rate (2 R MFMA of 32 cycles per tile), close to the memory time.
// (32 heads x 2944 tokens, r = 64: 154 us through the plain kernel, whose every output is a 128-step loop over R_r
// in memory; 24 us here, 27 on cold Keys.)
template <int R, bool VALUES>
__global__ __launch_bounds__(256) void compress_f32(RowsDev rows, int Hkv, int cap, int r, const float* __restrict__ Rr,
                                                    float* __restrict__ Kp, int32_t* __restrict__ seq_len_out,
                                                    ValuesArg<float, VALUES> vals)
{
    constexpr int JB = R / 16, TT = 2, TOK = 4 * TT * 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if constexpr (VALUES) {
        if ((int)blockIdx.z >= vals.batch) {
            retile_job(vals, Hkv, cap, (Oct<float>*)smem_raw);
            return;
        }
    }
    f32x4* frag = (f32x4*)smem_raw;         // [JB][8][64]
    const int h = blockIdx.y, b = blockIdx.z, u = b * Hkv + h;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, n = lane & 15;
    const int n_b = min(rows_count(rows, b), cap);
    if (blockIdx.x == 0 && h == 0 && tid == 0 && seq_len_out) seq_len_out[b] = n_b;
    const int blk0 = blockIdx.x * TOK;
    if (blk0 >= n_b) return;
    const int w0 = blk0 + wave * (TT * 16);

    f32x4 kb[TT][8];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {       // rows past the end are read as the last row and never stored
        const float* row = (const float*)rows.data + rows_offset(rows, b, h, min(w0 + 16 * tt + n, n_b - 1)) + 4 * g;
#pragma unroll
        for (int i = 0; i < 8; ++i) kb[tt][i] = __builtin_nontemporal_load((const f32x4*)(row + 16 * i));
    }
    const float* Ru = Rr + (size_t)u * D * r;
    for (int f = tid; f < JB * 8 * 64; f += 256) {
        const int fl = f & 63, i = (f >> 6) & 7, j = 16 * (f >> 9) + (fl & 15);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = Ru[(16 * i + 4 * (fl >> 4) + e) * r + min(j, r - 1)];
            v[e] = j < r ? x : 0.f;         // columns r .. R - 1: the layout's zero padding
        }
        frag[f] = v;
    }
    __syncthreads();
    float* Ku = Kp + (size_t)u * slab_tokens(cap) * R;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        f32x4 acc[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[tt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x4 a = frag[(jb * 8 + i) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    acc[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], kb[tt][i][e], acc[tt], 0, 0, 0);
        }
        if (16 * jb + 16 > r) {             // an infinity or NaN in a Key times the zeros there is NaN: the padding stays zero
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[tt][e] = 16 * jb + 4 * g + e < r ? acc[tt][e] : 0.f;
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
            if (w0 + 16 * tt + n < n_b)
                __builtin_nontemporal_store(acc[tt], (f32x4*)(Ku + (size_t)((w0 >> 4) + tt) * (16 * R) +
                                                              (2 * jb + (g >> 1)) * 128 + n * 8 + 4 * (g & 1)));
    }
}

// ---------------------------------------------------------------------------
// Append: block (h, b), 256 threads.  k~_j = sum_c k_new[c] R_r[c][j]: thread (cq, j)
// sums one quarter of the channels (its 32 loads of R_r are independent, one memory
// round trip), the four quarters are added in a fixed order.  The block that
// finishes last for a batch item bumps its length (all blocks of the item read the
// old length before taking a ticket).
template <typename T>
__global__ __launch_bounds__(256) void append_rows(int Hkv, int cap, int r, const T* __restrict__ k_new,
                                                   const T* __restrict__ v_new, const float* __restrict__ Rr,
                                                   T* __restrict__ Kp, T* __restrict__ Vc,
                                                   int32_t* __restrict__ seq_len, int32_t* __restrict__ tickets)
{
    const int h = blockIdx.x, b = blockIdx.y, u = b * Hkv + h;
    const int tid = threadIdx.x;
    const int len = seq_len[b];
    const bool ok = len >= 0 && len < cap;
    __shared__ float kn[D];
    __shared__ float part[4][D];
    if (ok) {
        const int rp = keep_padded(r);
        const float* Ru = Rr + (size_t)u * D * r;
        if (tid < D) kn[tid] = ld_elem(k_new + (size_t)u * D + tid);
        const int npass = (4 * r + 255) / 256;                   // 1 or 2, the same for every thread
        for (int pss = 0; pss < npass; ++pss) {
            const int idx = tid + 256 * pss;
            const bool act = idx < 4 * r;
            const int cq = act ? idx / r : 0, j = act ? idx - cq * r : 0;
            float x[32];
#pragma unroll
            for (int c = 0; c < 32; ++c) x[c] = act ? Ru[(32 * cq + c) * r + j] : 0.f;
            if (pss == 0) __syncthreads();                       // kn staged (uniform branch)
            float a = 0.f;
#pragma unroll
            for (int c = 0; c < 32; ++c) a = fmaf(kn[32 * cq + c], x[c], a);
            if (act) part[cq][j] = a;
        }
        __syncthreads();
        if (tid < rp) st_elem(Kp + (size_t)u * slab_tokens(cap) * rp + kidx(len, tid, rp),        // zeros in the padding
                              tid < r ? (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]) : 0.f);
        if (tid < D) Vc[(size_t)u * slab_tokens(cap) * D + vidx(len, tid)] = v_new[(size_t)u * D + tid];
    }
    __syncthreads();
    if (tid == 0) {
        int old = atomicAdd(&tickets[b], 1);
        if (old == Hkv - 1) {
            tickets[b] = 0;
            if (ok) seq_len[b] = len + 1;
        }
    }
}

// ---------------------------------------------------------------------------
// Inverse re-tiling for inspection: caches -> row-major [B,H_kv,cap,r] / [B,H_kv,cap,d].
template <typename T>
__global__ __launch_bounds__(256) void unpack_cache(int cap, int r, const T* __restrict__ Kp,
                                                    const T* __restrict__ Vc, T* __restrict__ k_rows,
                                                    T* __restrict__ v_rows)
{
    const int u = blockIdx.y;
    const int t0 = blockIdx.x * 32;
    const int rp = keep_padded(r);
    if (k_rows) {
        for (int idx = threadIdx.x; idx < 32 * r; idx += 256) {
            int t = t0 + idx / r, j = idx % r;
            if (t < cap) k_rows[((size_t)u * cap + t) * r + j] = Kp[(size_t)u * slab_tokens(cap) * rp + kidx(t, j, rp)];
        }
    }
    if (v_rows) {
        for (int idx = threadIdx.x; idx < 32 * D; idx += 256) {
            int t = t0 + (idx >> 7), c = idx & 127;
            if (t < cap) v_rows[((size_t)u * cap + t) * D + c] = Vc[(size_t)u * slab_tokens(cap) * D + vidx(t, c)];
        }
    }
}

// ---------------------------------------------------------------------------
template <typename T>
static hipError_t launch_v_retile(const RowsDev& rows, int B, int Hkv, int cap, T* dst, hipStream_t st)
{
    const int nblk = rows.n_tokens > 0 ? (rows.n_tokens + 31) / 32 : 1;
    hipLaunchKernelGGL(v_retile<T>, dim3(nblk, Hkv, B), dim3(256), 0, st, rows, Hkv, cap, dst);
    return hipGetLastError();
}

// The Values' work-groups behind the Keys' (`grid`, one entry of z per batch item), as many more entries of z as hold them.  False: no
// Values (or no rows), or more of their work-groups than `most`, than a grid's third dimension or than an int32 index takes; they then get a launch
// of their own.
template <typename T>
static bool add_values(const RowsDev* values, T* Vc, int B, int Hkv, int64_t most, dim3& grid, ValuesJob<T>& vals)
{
    vals = ValuesJob<T>{RowsDev{}, Vc, B, 0, 1};
    if (!values) return false;
    constexpr int TOK = 32 * ValuesJob<T>::NB;
    const int64_t per_head = ((int64_t)values->n_tokens + TOK - 1) / TOK, heads = (int64_t)B * Hkv;
    const int64_t per_z = (int64_t)grid.x * grid.y, more = (per_head * heads + per_z - 1) / per_z;
    if (per_head == 0 || per_head * heads > most || B + more > 65535 || more * per_z > INT32_MAX) return false;
    vals = ValuesJob<T>{*values, Vc, B, (int)heads, (int)per_head};
    grid.z += (unsigned)more;
    return true;
}

// 512 tokens per work-group.  With 2048 (one R_r fragment build per 2048 rows) the last work-groups decide the time of the launch,
// most where the lengths are on the device (token lists, n_tokens_dev) and the host's bound does not say how many blocks have
// rows, and at some distances of the caches' slabs their concurrent streams meet in the same memory channels.  Call without Values,
// r = 64, 2048 / 512 tokens: 1 x 32 heads x 32768 79 / 75 us; 4 x 32 x 5000 66 / 50; 17 x 16 x 1100 38 / 29; 2 x 32 x 9000 ragged 49 / 29;
// 16 x 16 x 2048 38 / 41.  r = 128, where the fragments are 64 KB: 1 x 32 x 16384 54 / 56; 16 x 16 x 2048 55 / 60; 1 x 64 x 8192 (slabs 8256
// tokens apart) 76 / 59; 1 x 16 x 32768 (33088 apart) 64 / 59.  With 1024: 56, 58, 62, 61, but 16 x 16 x 1536 ragged 41 / 30.
template <int R>
static hipError_t launch_compress_mfma_r(const RowsDev& rows, int B, int Hkv, int cap, int r, const float* Rr, bf16_t* Kp,
                                         int32_t* seq_len_out, const RowsDev* values, bf16_t* Vc, bool join, int n_cu, hipStream_t st)
{
    typedef CompressCfg<R> Cfg;
    int nblk = (rows.n_tokens + Cfg::TOK_PER_BLOCK - 1) / Cfg::TOK_PER_BLOCK;
    if (nblk < 1) nblk = 1;
    const bool part = nblk > 1 && rows.n_tokens % Cfg::TOK_PER_BLOCK != 0 && (int64_t)Hkv * B <= INT32_MAX / nblk;
    const int order = (int64_t)Hkv * B * nblk <= n_cu ? ORDER_FEW : part ? ORDER_PART_LAST : ORDER_MANY;
    dim3 grid(nblk, Hkv, B);
    ValuesJob<bf16_t> vals;
    // In the rotation's registers a compute unit holds two (R = 48, 64; by LDS from 112 on) or three work-groups that re-tile, eight in a launch
    // of their own.  That is enough while the rows are in the last-level cache; beyond, the joined launch is the slower one.  Two launches / one,
    // 32 heads, us: 6100 tokens 32, 35, 37, 41 / 26, 30, 31, 34 (r = 32, 48, 64, 96); 10000 tokens (9.9 work-groups of the Values per compute unit)
    // 49, 53, 55, 61 / 44, 50, 51, 50; 14000: 69, 73, 76, 84 / 70, 82, 85, 82; 16384, r = 80, 96, 112, 128: 92, 95, 100, 105 / 91, 94, 110, 113.
    // 1 x 8 x 1024, r = 32: 9.9 / 7.8; 1 x 4 x 32768, r = 128: 28 / 24.
    const bool joined = add_values(join ? values : nullptr, Vc, B, Hkv, 10 * (int64_t)n_cu, grid, vals);
    const size_t lds = joined && ValuesJob<bf16_t>::LDS_BYTES > Cfg::LDS_BYTES ? ValuesJob<bf16_t>::LDS_BYTES : Cfg::LDS_BYTES;
    if (joined)
        hipLaunchKernelGGL((compress_mfma<R, false, true>), grid, dim3(256), lds, st, rows, Hkv, cap, r, order, Rr, Kp, seq_len_out, vals);
    else
        hipLaunchKernelGGL((rows.tok_idx ? compress_mfma<R, true, false> : compress_mfma<R, false, false>), grid, dim3(256), lds, st, rows, Hkv,
                           cap, r, order, Rr, Kp, seq_len_out, NoValues{});
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && values && !joined ? launch_v_retile(*values, B, Hkv, cap, Vc, st) : e;
}

template <int R>
static hipError_t launch_compress_f32_r(const RowsDev& rows, int B, int Hkv, int cap, int r, const float* Rr, float* Kp,
                                        int32_t* seq_len_out, const RowsDev* values, float* Vc, bool join, hipStream_t st)
{
    constexpr size_t own = (size_t)(R / 16) * 8 * 64 * 16;
    dim3 grid(rows.n_tokens > 0 ? (rows.n_tokens + 127) / 128 : 1, Hkv, B);
    ValuesJob<float> vals;
    // (two launches / one, r = 64: 32 heads x 2944 tokens 46 / 37 us, x 16000 206 / 189)
    const bool joined = add_values(join ? values : nullptr, Vc, B, Hkv, INT64_MAX, grid, vals);
    const size_t lds = joined && ValuesJob<float>::LDS_BYTES > own ? ValuesJob<float>::LDS_BYTES : own;
    hipError_t e = allow_dynamic_lds(joined ? (const void*)compress_f32<R, true> : (const void*)compress_f32<R, false>, lds);
    if (e != hipSuccess) return e;
    if (joined) hipLaunchKernelGGL((compress_f32<R, true>), grid, dim3(256), lds, st, rows, Hkv, cap, r, Rr, Kp, seq_len_out, vals);
    else hipLaunchKernelGGL((compress_f32<R, false>), grid, dim3(256), lds, st, rows, Hkv, cap, r, Rr, Kp, seq_len_out, NoValues{});
    e = hipGetLastError();
    return e == hipSuccess && values && !joined ? launch_v_retile(*values, B, Hkv, cap, Vc, st) : e;
}

hipError_t launch_compress(int dtype, bool mfma, const RowsDev& rows, int B, int Hkv, int cap, int r, const float* Rr, void* Kp,
                           int32_t* seq_len_out, const RowsDev* values, void* Vc, bool join, int n_cu, hipStream_t st)
{
    if (mfma && dtype == 1) {
        bf16_t *kp = (bf16_t*)Kp, *vc = (bf16_t*)Vc;
        switch (keep_padded(r)) {
            case 16: return launch_compress_mfma_r<16>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 32: return launch_compress_mfma_r<32>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 48: return launch_compress_mfma_r<48>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 64: return launch_compress_mfma_r<64>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 80: return launch_compress_mfma_r<80>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 96: return launch_compress_mfma_r<96>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 112: return launch_compress_mfma_r<112>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            case 128: return launch_compress_mfma_r<128>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, n_cu, st);
            default: break;
        }
    }
    if (mfma && dtype == 0) {
        float *kp = (float*)Kp, *vc = (float*)Vc;
        switch (keep_padded(r)) {
            case 16: return launch_compress_f32_r<16>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 32: return launch_compress_f32_r<32>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 48: return launch_compress_f32_r<48>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 64: return launch_compress_f32_r<64>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 80: return launch_compress_f32_r<80>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 96: return launch_compress_f32_r<96>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 112: return launch_compress_f32_r<112>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            case 128: return launch_compress_f32_r<128>(rows, B, Hkv, cap, r, Rr, kp, seq_len_out, values, vc, join, st);
            default: break;
        }
    }
    int nblk = (rows.n_tokens + 63) / 64;
    if (nblk < 1) nblk = 1;
    dim3 grid(nblk, Hkv, B);
    if (dtype == 0)
        hipLaunchKernelGGL(compress_generic<float>, grid, dim3(256), 0, st, rows, Hkv, cap, r, Rr, (float*)Kp,
                           seq_len_out);
    else
        hipLaunchKernelGGL(compress_generic<bf16_t>, grid, dim3(256), 0, st, rows, Hkv, cap, r, Rr, (bf16_t*)Kp,
                           seq_len_out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !values) return e;
    return dtype == 0 ? launch_v_retile(*values, B, Hkv, cap, (float*)Vc, st) : launch_v_retile(*values, B, Hkv, cap, (bf16_t*)Vc, st);
}

hipError_t launch_append(int dtype, int B, int Hkv, int cap, int r, const void* k_new, const void* v_new,
                         const float* Rr, void* Kp, void* Vc, int32_t* seq_len, int32_t* tickets, hipStream_t st)
{
    dim3 grid(Hkv, B);
    if (dtype == 0)
        hipLaunchKernelGGL(append_rows<float>, grid, dim3(256), 0, st, Hkv, cap, r, (const float*)k_new,
                           (const float*)v_new, Rr, (float*)Kp, (float*)Vc, seq_len, tickets);
    else
        hipLaunchKernelGGL(append_rows<bf16_t>, grid, dim3(256), 0, st, Hkv, cap, r, (const bf16_t*)k_new,
                           (const bf16_t*)v_new, Rr, (bf16_t*)Kp, (bf16_t*)Vc, seq_len, tickets);
    return hipGetLastError();
}

hipError_t launch_unpack(int dtype, int U, int cap, int r, const void* Kp, const void* Vc, void* k_rows,
                         void* v_rows, hipStream_t st)
{
    dim3 grid((cap + 31) / 32, U);
    if (dtype == 0)
        hipLaunchKernelGGL(unpack_cache<float>, grid, dim3(256), 0, st, cap, r, (const float*)Kp, (const float*)Vc,
                           (float*)k_rows, (float*)v_rows);
    else
        hipLaunchKernelGGL(unpack_cache<bf16_t>, grid, dim3(256), 0, st, cap, r, (const bf16_t*)Kp,
                           (const bf16_t*)Vc, (bf16_t*)k_rows, (bf16_t*)v_rows);
    return hipGetLastError();
}

}  // namespace rk
