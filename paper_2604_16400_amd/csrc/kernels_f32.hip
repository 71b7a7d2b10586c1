// fp32 kernels of the mixed-batch LoRA linear layer: the same three passes as the bf16 path
// (GEMM with low-rank extension, skinny rank-wide pass, adapter gradients) in 32 bits throughout.
// The fp32 element type exists for exactness on small layers.  What bounds such a pass is the chain of
// dependent steps in one wave (load, multiply, load ..), not bytes or flops: every kernel is cut into many
// short waves, each with its own range of the contraction and many loads in flight (64 K values in the 16-row GEMM, 32 in the
// 32-row one, 128 in the rank-wide pass, 32 rows in the gradients), and the waves of a block add their sums in LDS in wave order.  v_mfma_f32_16x16x4_f32 (fp32 products and sums)
// does the multiplying because its operands come straight from memory: lane l supplies one K value
// (group l / 16) of row or column l % 16, so a lane that loads four consecutive K values feeds four of them.
// Measured on 256 -> 256, 64 tokens, rank 8 (us; before: one thread per output of the narrow passes with a serial sum,
// 64 x 64 LDS tiles): rank-wide passes 22 -> 4.5, gradients 20 -> 4.2, GEMM 35 -> 3.5 on blocks of 16 columns (launch_gemm_f32); the step of a forward
// and a backward call, one among others, 27.9 in six kernels -> 17 in four (dh_dB_f32_kernel, dx_dA_f32_kernel); the shorter chains also halve the
// distance from the 64-bit result (3.3e-7 -> 1.4e-7).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include <algorithm>
#include <cstring>

#include "kernels.h"

namespace collm {

constexpr int kF32Tile = 64;  // rows per row tile of the plan (extension steps are listed per tile)

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kF32Oob = 0x80000000u;  // beyond any buffer (tensors are limited to 2 GiB): reads as zero

__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ floatx4 f32_load4(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ float f32_load1(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <int NC>
__device__ __forceinline__ auto f32_load(__amdgpu_buffer_rsrc_t r, uint32_t off)  // NC consecutive values
{
    typedef float cols_t __attribute__((ext_vector_type(NC)));
    if constexpr (NC == 4) return __builtin_bit_cast(cols_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    else if constexpr (NC == 2) return __builtin_bit_cast(cols_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else return __builtin_bit_cast(cols_t, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// An adapter's table: element(s) from index i on, zero unless `on`.  Through the buffer below 2 GiB (BIG false); larger tables, to
// which 32-bit offsets do not reach, with a 64-bit address.
template <bool BIG, typename I>
__device__ __forceinline__ floatx4 table4(const float *tab, __amdgpu_buffer_rsrc_t rt, bool on, I i)
{
    if constexpr (BIG) return on ? *reinterpret_cast<const floatx4 *>(tab + i) : floatx4{0.f, 0.f, 0.f, 0.f};
    else return f32_load4(rt, on ? i * 4u : kF32Oob);
}
template <bool BIG, typename I>
__device__ __forceinline__ float table1(const float *tab, __amdgpu_buffer_rsrc_t rt, bool on, I i)
{
    if constexpr (BIG) return on ? tab[i] : 0.f;
    else return f32_load1(rt, on ? i * 4u : kF32Oob);
}
template <bool BIG, int NC, typename I>
__device__ __forceinline__ auto table_cols(const float *tab, __amdgpu_buffer_rsrc_t rt, bool on, I i)  // NC of them
{
    typedef float cols_t __attribute__((ext_vector_type(NC)));
    if constexpr (BIG) return on ? *reinterpret_cast<const cols_t *>(tab + i) : cols_t{};
    else return f32_load<NC>(rt, on ? i * 4u : kF32Oob);
}
static bool table_is_big(int rank, int d) { return (int64_t)rank * d * 4 > 0x7fffffff; }

// y[tok(m)][n] = sum_k a[tok(m)][k] b(k, n) + sum_q hs[m][q] table_a(q, n)
//
// One block = 16 RT rows x 16 NC columns; its KW waves split K (and the extension steps) between them.  Column i of
// 16-column block c is n0 + NC i + c: a lane's NC columns are then consecutive both where it loads the second
// operand ([K][N]) and where it stores.
// AHEAD: a wave asks for the operands of its next trip behind the products of this one, and for its first extension step before the first: shorter
// chains where few blocks share a CU.  Else it asks at the start of a trip and multiplies what has come while the rest is on its way, which is
// better with many: forward calls of 32-row blocks, us, ahead / not: 546 rows 1416 -> 3536 87 / 70, 912 rows 3948 -> 2916 [N][K] 328 / 275, 200 drawn
// ones 1.12 (up to 256 blocks of 16 x 64), 1.09 (512), 1.00 (2048), 0.96.
template <int RT, int KW, int NC> constexpr int kF32GemmRed = KW * 16 * RT * (16 * NC + 4);  // floats of LDS
template <bool B_KMAJOR, int RT, int KW, bool BIG, int NC, bool AHEAD>
__device__ __forceinline__ void gemm_f32_block(const GemmArgs &p, int bx, int by, float *red)
{
    using idx_t = std::conditional_t<BIG, uint64_t, uint32_t>;
    constexpr int ROWS = 16 * RT, COLS = 16 * NC, LD = COLS + 4, QUADS = ROWS * COLS / 4;
    typedef float cols_t __attribute__((ext_vector_type(NC)));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int n0 = bx * COLS, m0 = by * ROWS;
    const int tile = m0 / kF32Tile, in_tile = m0 - tile * kF32Tile;
    const int e0 = p.ext_off[tile], e1 = p.ext_off[tile + 1];
    // the tokens this thread stores to in the end
    constexpr int OUTS = QUADS / (KW * 64) > 0 ? QUADS / (KW * 64) : 1;
    int tok_out[OUTS];
#pragma unroll
    for (int i = 0; i < OUTS; ++i) tok_out[i] = tid + i * KW * 64 < QUADS ? p.row_tok[m0 + (tid + i * KW * 64) / (COLS / 4)] : -1;
    const int K = p.K, N = p.N;
    const int n = n0 + NC * l16;  // first of this lane's columns (N is a multiple of 4)
    const __amdgpu_buffer_rsrc_t ra = f32_rsrc(p.a, 0x7fffffffu), rb = f32_rsrc(p.b, 0x7fffffffu);

    uint32_t aoff[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int tok = p.row_tok[m0 + t * 16 + l16];
        aoff[t] = tok >= 0 ? (uint32_t)tok * (uint32_t)p.lda * 4u : kF32Oob;
    }
    floatx4 acc[RT][NC];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[t][c] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int per = (((K + KW - 1) / KW) + 15) & ~15;
    const int k_lo = wave * per, k_hi = (k_lo + per) < K ? (k_lo + per) : K;
    // 16 K values per step (this lane: k + 4 kg .. + 3), U steps of loads in flight
    constexpr int U = RT == 1 ? 4 : 2;
    floatx4 xa[U][RT];
    std::conditional_t<B_KMAJOR, floatx4, cols_t> wb[U][B_KMAJOR ? NC : 4];
    auto load_w = [&](int k0, int u) {
        const int k = k0 + u * 16 + kg * 4;
        // [K][N]: K value k + j, columns n ..; [N][K]: column n + j, K values k .. k + 3
#pragma unroll
        for (int j = 0; j < (B_KMAJOR ? NC : 4); ++j) {
            const bool on = k < k_hi && n + (B_KMAJOR ? j : 0) < N;
            if constexpr (B_KMAJOR) wb[u][j] = f32_load4(rb, on ? ((uint32_t)(n + j) * (uint32_t)p.ldb + (uint32_t)k) * 4u : kF32Oob);
            else wb[u][j] = f32_load<NC>(rb, on ? ((uint32_t)(k + j) * (uint32_t)p.ldb + (uint32_t)n) * 4u : kF32Oob);
        }
    };
    auto load_x = [&](int k0, int u) {
        const int k = k0 + u * 16 + kg * 4;
#pragma unroll
        for (int t = 0; t < RT; ++t) xa[u][t] = f32_load4(ra, k < k_hi && aoff[t] != kF32Oob ? aoff[t] + (uint32_t)k * 4u : kF32Oob);
    };
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            load_x(k0, u);
            load_w(k0, u);
        }
    };
    if constexpr (AHEAD) {
        // (the rows' tokens are on their way while the weight is asked for)
#pragma unroll
        for (int u = 0; u < U; ++u) load_w(k_lo, u);
#pragma unroll
        for (int u = 0; u < U; ++u) load_x(k_lo, u);
    }

    // Low-rank extension: one step = 16 rank indices of one adapter's table against the rows of its run.  A wave's first step is asked for
    // behind its first operands, not behind the contraction: what a small call takes is a chain of trips to memory.
    const float *__restrict__ Hs = reinterpret_cast<const float *>(p.hs);
    struct Step {
        int row_lo, row_hi;
        std::conditional_t<B_KMAJOR, floatx4, cols_t> tb[B_KMAJOR ? NC : 4];
        floatx4 hv[RT];
    };
    auto load_step = [&](int e, Step &s) {
        const ExtStep st = p.ext[e];
        const int koff = (int)(st.koff_rank & 0xffffu), rk = (int)(st.koff_rank >> 16);
        s.row_lo = (int)(st.rows & 0xffffu) - in_tile;
        s.row_hi = (int)(st.rows >> 16) - in_tile;
        if (rk == 0 || s.row_hi <= 0 || s.row_lo >= ROWS) {
            s.row_hi = 0;
            return;
        }
        const uint32_t tab_bytes = (uint32_t)rk * (uint32_t)(B_KMAJOR ? N : p.ext_ld) * 4u;
        const float *tab = reinterpret_cast<const float *>(st.tab);
        const __amdgpu_buffer_rsrc_t rt = f32_rsrc(tab, tab_bytes);
        const int q = koff + kg * 4;
#pragma unroll
        for (int j = 0; j < (B_KMAJOR ? NC : 4); ++j) {
            if constexpr (B_KMAJOR) {
                // table rows are output columns, `rank` long: any rank, so element by element
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    s.tb[j][i] = table1<BIG>(tab, rt, n + j < N && q + i < rk, (idx_t)(n + j) * (idx_t)rk + (idx_t)(q + i));
            } else {
                s.tb[j] = table_cols<BIG, NC>(tab, rt, n < N && q + j < rk, (idx_t)(q + j) * (idx_t)p.ext_ld + (idx_t)n);
            }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            // (zeros lie behind the rank, up to the row's padded length)
            const int r = t * 16 + l16;
            s.hv[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (r >= s.row_lo && r < s.row_hi) s.hv[t] = *reinterpret_cast<const floatx4 *>(Hs + (int64_t)(m0 + r) * p.hs_ld + q);
        }
    };
    Step s;
    s.row_hi = 0;
    if (e0 + wave < e1) load_step(e0 + wave, s);

    for (int k0 = k_lo; k0 < k_hi;) {
        if constexpr (!AHEAD) load(k0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (AHEAD && k0 + 16 * u >= k_hi) break;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        if constexpr (B_KMAJOR) acc[t][c] = mfma_f32(wb[u][c][e], xa[u][t][e], acc[t][c]);
                        else acc[t][c] = mfma_f32(wb[u][e][c], xa[u][t][e], acc[t][c]);
                    }
        }
        k0 += 16 * U;
        if (AHEAD && k0 < k_hi) load(k0);
    }

    // The products of a step are summed apart and added to the rows of the run only, so that a table's infinities
    // and NaNs stay out of other adapters' rows.
    for (int e = e0 + wave; e < e1;) {
        if (s.row_hi > 0) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                floatx4 add[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) add[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        if constexpr (B_KMAJOR) add[c] = mfma_f32(s.tb[c][i], s.hv[t][i], add[c]);
                        else add[c] = mfma_f32(s.tb[i][c], s.hv[t][i], add[c]);
                    }
                const int r = t * 16 + l16;
                if (r >= s.row_lo && r < s.row_hi)
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc[t][c] += add[c];
            }
        }
        e += KW;
        if (e < e1) load_step(e, s);
    }

    // lane holds row l16 and, in register j of block c, column NC (4 kg + j) + c
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            floatx4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[t][(4 * i + e) % NC][(4 * i + e) / NC];
            *reinterpret_cast<floatx4 *>(red + (wave * ROWS + t * 16 + l16) * LD + kg * 4 * NC + i * 4) = v;
        }
    __syncthreads();
    float *__restrict__ Out = reinterpret_cast<float *>(p.out);
#pragma unroll
    for (int i = 0; i < OUTS; ++i) {
        const int idx = tid + i * KW * 64, r = idx / (COLS / 4), c = idx % (COLS / 4) * 4, tok = tok_out[i];
        if (tok < 0 || n0 + c >= N) continue;
        floatx4 sum = *reinterpret_cast<const floatx4 *>(red + r * LD + c);
#pragma unroll
        for (int w = 1; w < KW; ++w) sum += *reinterpret_cast<const floatx4 *>(red + (w * ROWS + r) * LD + c);
        *reinterpret_cast<floatx4 *>(Out + (int64_t)tok * p.ldo + n0 + c) = sum;
    }
}

template <bool B_KMAJOR, int RT, int KW, bool BIG, int NC, bool AHEAD = true>
__global__ void __launch_bounds__(KW * 64) gemm_f32_kernel(GemmArgs p)
{
    __shared__ __align__(16) float red[kF32GemmRed<RT, KW, NC>];
    gemm_f32_block<B_KMAJOR, RT, KW, BIG, NC, AHEAD>(p, blockIdx.x, blockIdx.y, red);
}

// out[m][q] = sum_k in[tok(m)][k] table_a(k, q): one block = one item (up to 16 rows of one adapter) x 16 columns of
// the output row (blockIdx.y; columns beyond the rank are cleared); its eight waves split K.
constexpr int kF32SkinnyWaves = 8;
constexpr int kF32SkinnyRed = kF32SkinnyWaves * 16 * (16 + 4);
template <bool T_KMAJOR, bool BIG>
__device__ __forceinline__ void skinny_f32_block(const SkinnyArgs &p, int item, int by, float *red)
{
    using idx_t = std::conditional_t<BIG, uint64_t, uint32_t>;
    constexpr int KW = kF32SkinnyWaves, LD = 16 + 4;
    const SkinnyItem it = p.items[item];
    const int rank = it.rank, K = p.K;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int q0 = by * 16, q = q0 + l16;
    // the row this thread stores to in the end, and where
    const int m = tid >> 4, qo = q0 + (tid & 15), row = it.row_lo + m;
    float *f32_row = nullptr;
    if (p.f32_out && m < it.n_rows && qo < p.f32_cols) {
        const int tok = p.f32_by_token ? p.row_tok[row] : row;
        if (!p.f32_by_token || p.tok_train[tok]) f32_row = p.f32_out + (int64_t)tok * p.f32_ld;
    }
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    if (q0 < rank) {
        const __amdgpu_buffer_rsrc_t rx = f32_rsrc(p.in, p.in_bytes);
        const float *tab = reinterpret_cast<const float *>(p.tab[it.adapter]);
        const __amdgpu_buffer_rsrc_t rt = f32_rsrc(tab, (uint32_t)rank * (uint32_t)K * 4u);
        const int tok = l16 < it.n_rows ? p.row_tok[it.row_lo + l16] : -1;
        const uint32_t xoff = tok >= 0 ? (uint32_t)tok * (uint32_t)p.ld_in * 4u : kF32Oob;
        const int per = (((K + KW - 1) / KW) + 15) & ~15;
        const int k_lo = wave * per, k_hi = (k_lo + per) < K ? (k_lo + per) : K;
        constexpr int U = 8;  // 128 K values of loads in flight
        for (int k0 = k_lo; k0 < k_hi; k0 += 16 * U) {
            floatx4 xv[U], tv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * 16 + kg * 4;
                const bool on = k < k_hi;
                xv[u] = f32_load4(rx, on && xoff != kF32Oob ? xoff + (uint32_t)k * 4u : kF32Oob);
                if constexpr (T_KMAJOR) {
                    tv[u] = table4<BIG>(tab, rt, on && q < rank, (idx_t)q * (idx_t)K + (idx_t)k);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        tv[u][e] = table1<BIG>(tab, rt, on && q < rank, (idx_t)(k + e) * (idx_t)rank + (idx_t)q);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = mfma_f32(tv[u][e], xv[u][e], acc);
        }
    }
    // lane holds row l16, columns 4 kg ..
    *reinterpret_cast<floatx4 *>(red + (wave * 16 + l16) * LD + kg * 4) = acc;
    __syncthreads();
    if (m >= it.n_rows) return;  // (the second half of the threads: m is 16 and more)
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < KW; ++w) sum += red[(w * 16 + m) * LD + (tid & 15)];
    if (qo >= rank) sum = 0.f;
    if (f32_row) f32_row[qo] = sum * p.f32_mult;
    if (p.bf_out && qo < p.bf_ld) reinterpret_cast<float *>(p.bf_out)[(int64_t)row * p.bf_ld + qo] = sum * p.bf_mult;
}

template <bool T_KMAJOR, bool BIG>
__global__ void __launch_bounds__(kF32SkinnyWaves * 64) skinny_f32_kernel(SkinnyArgs p)
{
    __shared__ __align__(16) float red[kF32SkinnyRed];
    skinny_f32_block<T_KMAJOR, BIG>(p, blockIdx.x, blockIdx.y, red);
}

// out_a(q, n) = sum_t small[t][q] big[tok(t)][n] over the adapter's rows t: one block = one trained adapter x 64 columns
// x 16 rank indices (blockIdx.z); its eight waves split the rows.  Column i of block c is n0 + 4 i + c, as above.
constexpr int kF32GradWaves = 8;
constexpr int kF32GradRed = kF32GradWaves * 16 * (64 + 4);
__device__ __forceinline__ void grad_f32_block(const GradArgs &p, int bx, int by, int bz, float *red)
{
    constexpr int KW = kF32GradWaves, LD = 64 + 4;
    const GradItem it = p.items[by];
    const int N = p.N, rank = it.rank;
    const int q0 = bz * 16;
    if (q0 >= rank) return;
    float *out = reinterpret_cast<float *>(p.out_tab[it.adapter]);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int n0 = bx * 64, n = n0 + 4 * l16, q = q0 + l16;
    const __amdgpu_buffer_rsrc_t rb = f32_rsrc(p.big, p.big_bytes);
    const float *__restrict__ Small = p.small_;
    const int n_rows = it.row_hi - it.row_lo;
    const int per = (((n_rows + KW - 1) / KW) + 3) & ~3;
    const int t_lo = it.row_lo + wave * per, t_hi = (t_lo + per) < it.row_hi ? (t_lo + per) : it.row_hi;
    floatx4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int U = 8;  // 32 rows of loads in flight
    for (int t0 = t_lo; t0 < t_hi; t0 += 4 * U) {
        int tok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * 4 + kg;
            tok[u] = t < t_hi ? p.row_tok[t] : -1;
        }
        floatx4 bv[U];
        float sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * 4 + kg;
            bv[u] = f32_load4(rb, tok[u] >= 0 && n < N ? ((uint32_t)tok[u] * (uint32_t)p.ld_big + (uint32_t)n) * 4u : kF32Oob);
            sv[u] = 0.f;
            if (tok[u] >= 0 && q < rank) sv[u] = Small[(p.small_by_token ? (int64_t)tok[u] : (int64_t)t) * p.ld_small + q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = mfma_f32(bv[u][c], sv[u] * p.small_mult, acc[c]);
    }
    // lane holds rank index l16 and, in register j of block c, column 16 kg + 4 j + c
#pragma unroll
    for (int j = 0; j < 4; ++j)
        *reinterpret_cast<floatx4 *>(red + (wave * 16 + l16) * LD + kg * 16 + j * 4) = floatx4{acc[0][j], acc[1][j], acc[2][j], acc[3][j]};
    __syncthreads();
    const int qn = rank - q0 < 16 ? rank - q0 : 16;
    for (int idx = tid; idx < 64 * qn; idx += KW * 64) {
        // (consecutive threads write consecutive addresses in either layout)
        const int qi = p.out_transposed ? idx % qn : idx >> 6, c = p.out_transposed ? idx / qn : idx & 63;
        if (n0 + c >= N) continue;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < KW; ++w) sum += red[(w * 16 + qi) * LD + c];
        float *dst = p.out_transposed ? out + (int64_t)(n0 + c) * rank + q0 + qi : out + (int64_t)(q0 + qi) * N + n0 + c;
        *dst = p.accumulate ? (*dst + sum) : sum;
    }
}

__global__ void __launch_bounds__(kF32GradWaves * 64) grad_f32_kernel(GradArgs p)
{
    __shared__ __align__(16) float red[kF32GradRed];
    grad_f32_block(p, blockIdx.x, blockIdx.y, blockIdx.z, red);
}

// Two passes of a small backward call that do not depend on each other as one launch (a pass is a chain of a few trips to memory on a part of the
// CUs): dh beside dB, dX beside dA.
__device__ __forceinline__ void grad_f32_blocks(const GradArgs &g, int b, float *red)
{
    const int cols = (g.N + 63) / 64;
    grad_f32_block(g, b % cols, b / cols % g.n_items, b / cols / g.n_items, red);
}
template <bool T_KMAJOR>
__global__ void __launch_bounds__(512) dh_dB_f32_kernel(SkinnyArgs s, GradArgs g)
{
    static_assert(kF32SkinnyWaves == 8 && kF32GradWaves == 8, "one block size");
    __shared__ __align__(16) float red[std::max(kF32SkinnyRed, kF32GradRed)];
    const int b = blockIdx.x, first = s.n_items * ((s.bf_ld + 15) / 16);
    if (b < first) skinny_f32_block<T_KMAJOR, false>(s, b % s.n_items, b / s.n_items, red);
    else grad_f32_blocks(g, b - first, red);
}
template <bool B_KMAJOR, int NC>
__global__ void __launch_bounds__(512) dx_dA_f32_kernel(GemmArgs m, GradArgs g)
{
    __shared__ __align__(16) float red[std::max(kF32GemmRed<1, 8, NC>, kF32GradRed)];
    const int b = blockIdx.x, cols = (m.N + 16 * NC - 1) / (16 * NC), first = cols * ((m.n_rows + 15) / 16);
    if (b < first) gemm_f32_block<B_KMAJOR, 1, 8, false, NC, true>(m, b % cols, b / cols, red);
    else grad_f32_blocks(g, b - first, red);
}

// Plan upload: the host builds the plan in pinned, device-visible memory and this kernel
// copies it into device memory in stream order (a kernel launch costs the host far less than
// an asynchronous memcpy ordered against kernels on the same stream).  The block that
// finishes last publishes the upload's sequence number in a pinned word, which is how the
// host learns that the staging slot may be reused, without any event call.
__global__ void __launch_bounds__(256) plan_copy_kernel(const int4 *__restrict__ src, int4 *__restrict__ dst, int n16,
                                                        int *counter, volatile uint32_t *done_host, uint32_t seq)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += gridDim.x * blockDim.x) dst[i] = src[i];
    __syncthreads();  // every load of this block has returned: its stores have been issued
    if (threadIdx.x == 0) {
        const int old = atomicAdd(counter, 1);
        if (old == (int)gridDim.x - 1) {
            *counter = 0;  // for the next upload (stream order)
            *done_host = seq;
            __threadfence_system();
        }
    }
}

hipError_t launch_plan_copy(const int32_t *src_pinned, int32_t *dst, size_t first_int, size_t n_ints, int *counter,
                            uint32_t *done_host_dev, uint32_t seq, hipStream_t st)
{
    // both ends are rounded outwards to 16 bytes; the plan block is padded accordingly
    const size_t lo = first_int & ~(size_t)3, hi = (first_int + n_ints + 3) & ~(size_t)3;
    const int n16 = (int)((hi - lo) / 4);
    const int blocks = std::max(1, std::min(256, (n16 + 255) / 256));
    COLLM_LAUNCH(plan_copy_kernel, dim3(blocks), dim3(256), 0, st,
                       reinterpret_cast<const int4 *>(src_pinned + lo), reinterpret_cast<int4 *>(dst + lo), n16, counter,
                       done_host_dev, seq);
    return hipGetLastError();
}

// Plan upload without a staging buffer: a chunk of the plan is an argument of the kernel (arguments are copied
// when the launch is enqueued, so the host block may change afterwards), and the kernel stores it.
constexpr int kPlanChunkInts = 896;  // 3.5 KiB of the 4 KiB a kernel's arguments may take
struct PlanChunk {
    int32_t v[kPlanChunkInts];
};
__global__ void __launch_bounds__(256) plan_words_kernel(PlanChunk c, int32_t *__restrict__ dst, int n)
{
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = c.v[i];
}

hipError_t launch_plan_words(const int32_t *src_host, int32_t *dst, size_t n_ints, hipStream_t st)
{
    PlanChunk c;
    for (size_t lo = 0; lo < n_ints; lo += kPlanChunkInts) {
        const int n = (int)std::min<size_t>(kPlanChunkInts, n_ints - lo);
        std::memcpy(c.v, src_host + lo, (size_t)n * sizeof(int32_t));
        COLLM_LAUNCH(plan_words_kernel, dim3(1), dim3(256), 0, st, c, dst + lo, n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

__global__ void __launch_bounds__(64) fill_zero_kernel(int4 *__restrict__ dst, int n16)
{
    for (int i = blockIdx.x * 64 + threadIdx.x; i < n16; i += gridDim.x * 64) dst[i] = make_int4(0, 0, 0, 0);
}

hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t st)
{
    const int n16 = (int)(bytes / 16);
    if (n16 <= 0) return hipSuccess;
    COLLM_LAUNCH(fill_zero_kernel, dim3(std::min(256, (n16 + 63) / 64)), dim3(64), 0, st, reinterpret_cast<int4 *>(dst), n16);
    return hipGetLastError();
}

// Blocks of 16 rows and eight waves: a block's products are the shorter a chain the fewer columns it has, but the rows and the weight are read the more
// often.  16 columns up to 64 blocks of 16 rows x 64 columns, up to 128 on a short contraction, else 32; 64 columns while that is one block per CU; beyond
// a CU has two blocks to run one after the other, and 32 rows with four waves, which read the weight half as often, are better.  Forward calls by
// number of 16 x 64 blocks, the time of the best over that of 16 / 32 / 64 columns / 32 rows, geometric means over 1100 drawn ones of few extension steps:
//   to 64    K <= 512 1.00 / 0.96 / 0.90 / 0.84, longer 1.00 / 0.89 / 0.73 / 0.57
//   to 128   K <= 512 0.99 / 0.98 / 0.93 / 0.84, longer 0.91 / 0.99 / 0.85 / 0.65
//   to 256   K <= 512 0.95 / 0.96 / 0.98 / 0.91, longer 0.86 / 0.90 / 0.98 / 0.78
//   to 512   K <= 512 0.90 / 0.91 / 0.89 / 1.00, longer 0.76 / 0.86 / 0.86 / 0.99;  beyond 0.6 .. 0.8 / 0.7 .. 0.8 / 0.7 .. 0.8 / 1.00
// Extension steps (of a row tile) are trips to memory that the waves share, and a step costs by its columns, most with [N][rank] tables, which
// are read element by element: 16 columns then up to 256 blocks (45 rows 772 -> 1352 of 14 adapters of rank 128 21.5 / 29.2 us with 16 / 32), with [N][rank]
// tables up to 512 (more than six steps and K <= 512 1.00 / 0.92 / 0.85 / 0.85), with the other ones on many steps and a short contraction.
// With dA in the same launch (dX of a backward call; its blocks have 16 rows) 32 columns are best up to 512 blocks of K <= 1024: 0.98, and 0.94 for
// 32 rows and a launch of its own for dA; longer 0.89 and 0.95, more blocks 0.92 and 0.99.
static int64_t blocks_16x64(const GemmArgs &a) { return (int64_t)((a.N + 63) / 64) * ((a.n_rows + 15) / 16); }
static int short_block_cols(const GemmArgs &a, bool b_kmajor, bool with_dA)  // in sixteens; 0: 32 rows
{
    const int64_t blocks = blocks_16x64(a);
    if (a.hs_ld > 0 && table_is_big(a.hs_ld, a.N)) return 0;
    if (blocks <= 64) return 1;
    if (blocks <= 128) return a.K <= 512 || a.tile_steps > (b_kmajor ? 6 : 16) ? 1 : 2;
    if (blocks <= 256) return a.tile_steps > (b_kmajor ? 6 : 40) ? 1 : 4;
    if (blocks > 512) return 0;
    if (with_dA) return a.K <= 1024 ? 2 : 0;
    return (b_kmajor || a.K <= 512) && a.tile_steps > (b_kmajor && a.K <= 512 ? 6 : 16) ? 1 : 0;
}
bool gemm_f32_with_dA(const GemmArgs &a, bool b_kmajor) { return short_block_cols(a, b_kmajor, true) > 0; }

hipError_t launch_gemm_f32(const GemmArgs &a, bool b_kmajor, hipStream_t st)
{
    // (row blocks are the grid's second dimension, which holds 65536: more rows than that go in several launches)
    constexpr int kRows = 65534 * 32;
    static_assert(kRows % kF32Tile == 0, "launches start at a row tile");
    if (a.n_rows > kRows) {
        GemmArgs first = a, rest = a;
        first.n_rows = kRows;
        rest.n_rows = a.n_rows - kRows;
        rest.row_tok = a.row_tok + kRows;
        rest.hs = reinterpret_cast<decltype(a.hs)>(reinterpret_cast<const float *>(a.hs) + (int64_t)kRows * a.hs_ld);
        rest.ext_off = a.ext_off + kRows / kF32Tile;
        const hipError_t e = launch_gemm_f32(first, b_kmajor, st);
        return e == hipSuccess ? launch_gemm_f32(rest, b_kmajor, st) : e;
    }
    const int rows = a.n_rows;  // (the row order is padded to a multiple of 256 rows)
    if (a.N <= 0 || rows <= 0) return hipSuccess;
    auto launch = [&](auto kern, int block_rows, int block_cols, int threads) {
        COLLM_LAUNCH(kern, dim3((a.N + block_cols - 1) / block_cols, (rows + block_rows - 1) / block_rows), dim3(threads), 0, st, a);
    };
    if (a.hs_ld > 0 && table_is_big(a.hs_ld, a.N)) {  // (hs_ld: at least the largest rank)
        if (b_kmajor) launch(gemm_f32_kernel<true, 2, 4, true, 4, false>, 32, 64, 256);
        else launch(gemm_f32_kernel<false, 2, 4, true, 4, false>, 32, 64, 256);
        return hipGetLastError();
    }
    switch (short_block_cols(a, b_kmajor, false)) {
    case 1: b_kmajor ? launch(gemm_f32_kernel<true, 1, 8, false, 1>, 16, 16, 512) : launch(gemm_f32_kernel<false, 1, 8, false, 1>, 16, 16, 512); break;
    case 2: b_kmajor ? launch(gemm_f32_kernel<true, 1, 8, false, 2>, 16, 32, 512) : launch(gemm_f32_kernel<false, 1, 8, false, 2>, 16, 32, 512); break;
    case 4: b_kmajor ? launch(gemm_f32_kernel<true, 1, 8, false, 4>, 16, 64, 512) : launch(gemm_f32_kernel<false, 1, 8, false, 4>, 16, 64, 512); break;
    default:
        if (blocks_16x64(a) <= 1024 || a.K <= 512) b_kmajor ? launch(gemm_f32_kernel<true, 2, 4, false, 4>, 32, 64, 256) : launch(gemm_f32_kernel<false, 2, 4, false, 4>, 32, 64, 256);
        else b_kmajor ? launch(gemm_f32_kernel<true, 2, 4, false, 4, false>, 32, 64, 256) : launch(gemm_f32_kernel<false, 2, 4, false, 4, false>, 32, 64, 256);
    }
    return hipGetLastError();
}

hipError_t launch_skinny_f32(const SkinnyArgs &a, int n_items, bool t_kmajor, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    // 16 columns of the widest output row per block
    const int width = std::max(a.f32_out ? a.f32_cols : 0, a.bf_out ? (int)a.bf_ld : 0);
    const dim3 grid(n_items, (width + 15) / 16);
    if (grid.y == 0) return hipSuccess;
    auto launch = [&](auto kern) { COLLM_LAUNCH(kern, grid, dim3(kF32SkinnyWaves * 64), 0, st, a); };
    if (table_is_big(width, a.K)) launch(t_kmajor ? skinny_f32_kernel<true, true> : skinny_f32_kernel<false, true>);
    else launch(t_kmajor ? skinny_f32_kernel<true, false> : skinny_f32_kernel<false, false>);
    return hipGetLastError();
}

hipError_t launch_grad_f32(const GradArgs &a, int n_grad, int rpad, hipStream_t st)
{
    if (n_grad <= 0 || a.N <= 0) return hipSuccess;
    COLLM_LAUNCH(grad_f32_kernel, dim3((a.N + 63) / 64, n_grad, (rpad + 15) / 16), dim3(kF32GradWaves * 64), 0, st, a);
    return hipGetLastError();
}

// (whoever calls these has looked at gemm_f32_with_dA and pair_f32)
bool pair_f32(int rpad, int d_in, int d_out) { return !table_is_big(rpad, std::max(d_in, d_out)); }
hipError_t launch_dh_dB_f32(const SkinnyArgs &s, const GradArgs &g, int rpad, bool t_kmajor, hipStream_t st)
{
    const int blocks = s.n_items * ((s.bf_ld + 15) / 16) + (g.N + 63) / 64 * g.n_items * ((rpad + 15) / 16);
    if (blocks <= 0) return hipSuccess;
    if (t_kmajor) COLLM_LAUNCH(dh_dB_f32_kernel<true>, dim3(blocks), dim3(512), 0, st, s, g);
    else COLLM_LAUNCH(dh_dB_f32_kernel<false>, dim3(blocks), dim3(512), 0, st, s, g);
    return hipGetLastError();
}
hipError_t launch_dx_dA_f32(const GemmArgs &m, const GradArgs &g, int rpad, bool b_kmajor, hipStream_t st)
{
    const int nc = short_block_cols(m, b_kmajor, true);
    if (nc == 0) return hipErrorInvalidValue;
    const int blocks = (m.N + 16 * nc - 1) / (16 * nc) * ((m.n_rows + 15) / 16) + (g.N + 63) / 64 * g.n_items * ((rpad + 15) / 16);
    if (blocks <= 0) return hipSuccess;
    auto launch = [&](auto kern) { COLLM_LAUNCH(kern, dim3(blocks), dim3(512), 0, st, m, g); };
    switch (nc) {
    case 1: launch(b_kmajor ? dx_dA_f32_kernel<true, 1> : dx_dA_f32_kernel<false, 1>); break;
    case 2: launch(b_kmajor ? dx_dA_f32_kernel<true, 2> : dx_dA_f32_kernel<false, 2>); break;
    default: launch(b_kmajor ? dx_dA_f32_kernel<true, 4> : dx_dA_f32_kernel<false, 4>); break;
    }
    return hipGetLastError();
}

}  // namespace collm
