// Decode-sized inference batches (bf16, up to kDecodeRows rows): the whole call in two kernels.
//
// Such a call is bound by the bytes of the weight and the tables, and by the chain of launches (rank-wide pass, its sums, GEMM, its sums).
// The product with the weight does not need h = x A_a, and y = x W + (s h) B_a is a sum of both, so
//   decode_base    streams the weight (sums of K slices of x W) and, in other blocks of the same grid, the shrink tables (sums of
//                  K slices of x A_a), all in fp32 to the workspace;
//   decode_finish  adds the slices in slice order, multiplies bf16(s h) with B_a and rounds y once.
// A call among others, us, weight and tables in the last-level cache / from memory: eight rows 4096 -> 4096 (33.5 MB) 19.8 / 23.3 in three kernels,
// 12.5 / 16.3 in two (base 8, finish 4); 64 rows of 29 adapters of ranks 8 to 128, 4096 -> 11008 (90 MB of weight, 37 of tables) 44 / 54 in four, 34 / 41 in
// two (27, 12).  A plain read of these weights with the same loads takes 8 and 17 us.
// In the 27 us: the rows of x 3, the sums across waves 2, the MFMAs that one wave per SIMD does not hide 4 (measured without them).
#include "bf16_device.h"

namespace collm {

namespace {

__device__ __forceinline__ uint4 buf16s(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)  // soff: not part of the range check
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Operand of MFMA j of 32 contraction values by 128 columns of a [contraction][column] matrix, out of a lane's eight 16-byte loads: the lane has
// values 8 (l / 16) .. by columns 8 (l % 16) ..  MFMA j takes column j of every lane, its column i is column 8 i + j, and the operand is put
// together in registers: half a dword of each of two loads at a time, 32 v_perm for eight MFMAs.  (No LDS: neither a copy nor a transposing read.)
__device__ __forceinline__ bf16x8 column_operand(const uint4 *v, int j)
{
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        o[q] = __builtin_amdgcn_perm(word(v[2 * q + 1], j >> 1), word(v[2 * q], j >> 1), (j & 1) ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, o);
}

constexpr int kWaves = 4;
constexpr int kRedLd = kDecodeCols + 4;  // floats
constexpr int red_bytes(int row_tiles) { return kWaves * row_tiles * 16 * kRedLd * 4; }

// One strip of 128 columns and one slice of K, all rows (MT tiles of 16).  The waves take rounds of 64 values of the slice in turn; the weight goes
// from memory straight into operand registers, R rounds (16 KB each) per wave in flight: two, and one block per CU (128 KB in flight).
// Tried: eight waves a block with half the rows each (every line of the weight asked for twice: 64 rows 8192 -> 28672 135 us instead of
// 102), one round in flight and two blocks per CU (30 / 26), three rounds (registers spill; 38 / 34 for the call).
// Every XCD (the block id's last three bits) takes one run of the strips of one slice after the other: the lines that two strips share (rows of the
// weight that do not begin at a line) and the slice's share of x are then in one L2.  Calls, weights from memory, strips dealt out to the XCDs /
// this: 12304 -> 6496 41 / 37 us, 9488 -> 21704 91 / 86; 28 of 20 million weights and more 1.05 (0.99 .. 1.15).
template <int MT, int R, bool KM>
__device__ __forceinline__ void base_block(const SkinnyArgs &p, const DecodeArgs &d, int blk, uint8_t *smem)
{
    const int total = d.strips * d.n_slices, per = total >> 3, rem = total & 7, xcd = blk & 7;
    const int pid = xcd * per + (xcd < rem ? xcd : rem) + (blk >> 3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int strip = pid % d.strips, slice = pid / d.strips;
    const int col0 = strip * kDecodeCols;
    const int k_lo = slice * d.k_per_slice, k_hi = k_lo + d.k_per_slice < p.K ? k_lo + d.k_per_slice : p.K;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.in, p.in_bytes), rw = make_rsrc(d.w, d.w_bytes);
    int tok[MT][2];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = 16 * t + pair_row(u, l16);
            tok[t][u] = p.row_tok[row < d.n_rows ? row : d.n_rows - 1];  // (results of rows that do not exist are dropped)
        }
    asm volatile("" ::: "memory");
    const uint32_t ldw = (uint32_t)d.ldw * 2u, ldx = (uint32_t)p.ld_in * 2u;
    uint32_t woff[2];
    if constexpr (KM) {  // (rows beyond the last column lie beyond the weight)
#pragma unroll
        for (int u = 0; u < 2; ++u) woff[u] = (uint32_t)(col0 + pair_row(u, l16)) * ldw + pair_k(u, l16, g) * 2u;
    } else {
        woff[0] = woff[1] = col0 + 8 * l16 < d.N ? (uint32_t)(8 * g) * ldw + (uint32_t)(col0 + 8 * l16) * 2u : kOob;
    }

    // a round: two chunks of 8 KB of the weight and 64 values of every row
    uint4 wreg[R][2][8];
    RowPair xreg[R][MT];
    auto k_of = [&](int r) { return k_lo + (r * kWaves + wave) * 64; };
    auto load_w = [&](int r, int c, int buf) {
        const int k0 = k_of(r);
        if constexpr (KM) {
            // columns 64 c .., 64 values; the loads of a column tile one after the other
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t off = k0 + (int)pair_k(u, l16, g) < k_hi ? woff[u] : kOob;
#pragma unroll
                for (int j = 0; j < 4; ++j) wreg[buf][c][2 * j + u] = buf16s(rw, off + (uint32_t)(64 * c + 16 * j) * ldw, (uint32_t)k0 * 2u);
            }
        } else {
            // values 32 c .., 128 columns
            const uint32_t off = k0 + 32 * c + 8 * g < k_hi ? woff[0] : kOob;
#pragma unroll
            for (int i = 0; i < 8; ++i) wreg[buf][c][i] = buf16s(rw, off, (uint32_t)(k0 + 32 * c + i) * ldw);
        }
    };
    auto load_x = [&](int r, int buf) {
        const int k0 = k_of(r);
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                xreg[buf][t].v[u] = buf16s(rx, k0 + (int)pair_k(u, l16, g) < k_hi ? (uint32_t)tok[t][u] * ldx + pair_k(u, l16, g) * 2u : kOob, (uint32_t)k0 * 2u);
    };
    auto fence = [] { asm volatile("" ::: "memory"); };  // (as in skinny_item: loads of a chunk stay together)

    floatx4 acc[MT][8];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (k_of(0) < k_hi) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            load_w(r, 0, r);
            load_w(r, 1, r);
            fence();
            load_x(r, r);  // (the first round's behind its weight: its row's token is on its way while that is asked for)
            fence();
        }
        for (int rb = 0; k_of(rb) < k_hi; rb += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                bf16x8 x[2][MT];
#pragma unroll
                for (int t = 0; t < MT; ++t) pair_operands(xreg[r][t], l16, x[0][t], x[1][t]);
                fence();
                load_x(rb + r + R, r);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if constexpr (KM) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            bf16x8 w[2];
                            pair_operands(RowPair{{wreg[r][c][2 * j], wreg[r][c][2 * j + 1]}}, l16, w[0], w[1]);
#pragma unroll
                            for (int h = 0; h < 2; ++h)
#pragma unroll
                                for (int t = 0; t < MT; ++t)
                                    acc[t][4 * c + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[h], x[h][t], acc[t][4 * c + j], 0, 0, 0);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const bf16x8 w = column_operand(wreg[r][c], j);
#pragma unroll
                            for (int t = 0; t < MT; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[c][t], acc[t][j], 0, 0, 0);
                        }
                    }
                    fence();
                    load_w(rb + r + R, c, r);
                    fence();
                }
            }
        }
    }

    // lane l holds row l % 16 of every tile; the waves are added in wave order
    float *red = reinterpret_cast<float *>(smem);
    float *out = d.part + (int64_t)slice * d.n_rows * d.N;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        float *mine = red + ((wave * MT + t) * 16 + l16) * kRedLd;
        if constexpr (KM) {
#pragma unroll
            for (int j = 0; j < 8; ++j) *reinterpret_cast<floatx4 *>(mine + 16 * j + 4 * g) = acc[t][j];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                *reinterpret_cast<floatx4 *>(mine + 32 * g + 8 * r) = floatx4{acc[t][0][r], acc[t][1][r], acc[t][2][r], acc[t][3][r]};
                *reinterpret_cast<floatx4 *>(mine + 32 * g + 8 * r + 4) = floatx4{acc[t][4][r], acc[t][5][r], acc[t][6][r], acc[t][7][r]};
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        const int idx = tid + 256 * i, q = (idx & 31) * 4, row = idx >> 5;
        if (row >= d.n_rows || col0 + q >= d.N) continue;
        floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += *reinterpret_cast<const floatx4 *>(red + (w * MT * 16 + row) * kRedLd + q);
        *reinterpret_cast<floatx4 *>(out + (int64_t)row * d.N + col0 + q) = sum;
    }
}

// Blocks: the items' slices of the shrink first (they are the longest chains), then those that put in new table addresses, then strips x slices.
template <int MT, bool KM, int RP, typename Args>
__global__ void __launch_bounds__(kWaves * 64) decode_base_kernel(Args p, DecodeArgs d)
{
    extern __shared__ __align__(16) uint8_t smem[];
    int b = blockIdx.x;
    const int per_cols = p.n_items * d.h_slices, shrink = per_cols * d.h_cols;
    if (b < shrink) {
        const int rest = b % per_cols;
        skinny_item<RP, KM, 1, kWaves, true, true>(p, rest % p.n_items, rest / p.n_items, d.h_slices, smem, b / per_cols * RP);
        return;
    }
    b -= shrink;
    if constexpr (kHasPatch<Args>) {
        if (b < p.patch.blocks) {
            patch_plan(p.patch, b, threadIdx.x, kWaves * 64);
            return;
        }
        b -= p.patch.blocks;
    }
    base_block<MT, 2, KM>(p, d, b, smem);
}

// One item (up to 16 rows of one adapter, or of none) by 512 columns, 128 to a wave.  Bound by the chain item -> table address -> table and by the
// bytes of the tables: the block's threads add the slices, of x W and of h, side by side through LDS while the table is on its way.
constexpr int kFinishCols = kWaves * kDecodeCols;
constexpr int kSumLd = kFinishCols + 4;  // floats
constexpr int finish_low_ld(int rpad) { return ((rpad + 31) & ~31) + 8; }  // bf16
constexpr int finish_lds(int rpad) { return 16 * kSumLd * 4 + 16 * finish_low_ld(rpad) * 2; }
template <bool KM>
__global__ void __launch_bounds__(256, 3) decode_finish_kernel(SkinnyArgs p, DecodeFinishArgs d)
{
    extern __shared__ __align__(16) uint8_t smem[];
    float *sums = reinterpret_cast<float *>(smem);
    uint16_t *lows = reinterpret_cast<uint16_t *>(smem + 16 * kSumLd * 4);
    const int low_ld = finish_low_ld(p.part_ld);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int cw = __builtin_amdgcn_readfirstlane(tid >> 6) * kDecodeCols, cb = blockIdx.x * kFinishCols, col0 = cb + cw;
    int row_lo, n_rows, rank = 0;
    uint64_t tab = 0;
    if ((int)blockIdx.y < p.n_items) {
        const DecodeItem it = d.items[blockIdx.y];
        row_lo = it.rows & 0xffff;
        n_rows = it.rows >> 16;
        rank = it.rank;
        tab = it.tab;
    } else {  // rows on the base weight only come first in the row order
        row_lo = ((int)blockIdx.y - p.n_items) * 16;
        n_rows = d.n_base - row_lo < 16 ? d.n_base - row_lo : 16;
    }
    const int tok = l16 < n_rows ? p.row_tok[row_lo + l16] : -1;

    // table, 32 rank indices at a time, two steps in flight
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(reinterpret_cast<const void *>(tab), (uint32_t)rank * (uint32_t)d.N * 2u);
    const int col = col0 + 8 * l16;
    uint4 breg[2][8];
    auto load_b = [&](int q0, int buf) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (KM) breg[buf][i] = buf16(rb, q0 + 8 * g < rank ? ((uint32_t)(col0 + 16 * i + l16) * (uint32_t)rank + (uint32_t)(q0 + 8 * g)) * 2u : kOob);
            else breg[buf][i] = buf16(rb, col < d.N ? ((uint32_t)(q0 + 8 * g + i) * (uint32_t)d.N + (uint32_t)col) * 2u : kOob);
        }
    };
    if (rank > 0) load_b(0, 0);
    if (rank > 32) load_b(32, 1);
    asm volatile("" ::: "memory");

    const int rp = (rank + 31) & ~31;  // (zeros from the rank on)
    for (int idx = tid; idx < n_rows * (rp >> 2); idx += 256) {
        const int m = idx / (rp >> 2), q = (idx - m * (rp >> 2)) * 4;
        floatx4 h = floatx4{0.f, 0.f, 0.f, 0.f};
        if (q < rank) h = sum_slices(p.part + (int64_t)(row_lo + m) * p.part_ld + q, (int64_t)p.part_rows * p.part_ld, d.h_slices);
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = q + e < rank ? h[e] * d.scale : 0.f;
        *reinterpret_cast<uint2 *>(lows + m * low_ld + q) = make_uint2(pack_bf16(h[0], h[1]), pack_bf16(h[2], h[3]));
    }
    // (a thread's quads lie two rows apart; what counts is the number of trips: eight slices of one of its at most two quads are asked for at a time,
    // or two slices of four; decode_sum_trips)
    if (n_rows <= 4) {
        for (int idx = tid; idx < n_rows * (kFinishCols / 4); idx += 256) {
            const int m = idx / (kFinishCols / 4), q = (idx % (kFinishCols / 4)) * 4;
            if (cb + q < d.N) *reinterpret_cast<floatx4 *>(sums + m * kSumLd + q) = sum_slices(d.part + (int64_t)(row_lo + m) * d.N + cb + q, (int64_t)d.n_rows * d.N, d.n_slices);
        }
    } else {
        const int q = (tid % (kFinishCols / 4)) * 4, m0 = tid / (kFinishCols / 4);
        const int64_t stride = (int64_t)d.n_rows * d.N;
        const float *src = d.part + (int64_t)(row_lo + m0) * d.N + cb + q;
        for (int m = m0; m < n_rows && cb + q < d.N; m += 8, src += 8 * (int64_t)d.N) {
            floatx4 v[4] = {};
            for (int s = 0; s < d.n_slices; s += 2) {
                floatx4 t[2][4] = {};
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (s + u < d.n_slices && m + 2 * i < n_rows) t[u][i] = *reinterpret_cast<const floatx4 *>(src + (s + u) * stride + 2 * i * (int64_t)d.N);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] += t[u][i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (m + 2 * i < n_rows) *reinterpret_cast<floatx4 *>(sums + (m + 2 * i) * kSumLd + q) = v[i];
        }
    }
    __syncthreads();
    if (col0 >= d.N) return;

    // (lanes of rows that do not exist multiply and drop what lies in LDS: a lane's results are of its own row only)
    const int cl = KM ? cw + 4 * g : cw + 32 * g;  // quad i of a lane: columns 4 i further on (KM: 16 i)
    constexpr int QS = KM ? 16 : 4;
    floatx4 acc[8];
    {
        const float *src = sums + l16 * kSumLd + cl;
        floatx4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const floatx4 *>(src + QS * i);
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] = KM ? v[j][r] : v[2 * r + (j >> 2)][j & 3];
    }
    for (int q0 = 0; q0 < rank; q0 += 64) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = q0 + 32 * u;
            if (q >= rank) break;
            const bf16x8 h = *reinterpret_cast<const bf16x8 *>(lows + l16 * low_ld + q + 8 * g);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(KM ? __builtin_bit_cast(bf16x8, breg[u][j]) : column_operand(breg[u], j), h, acc[j], 0, 0, 0);
            if (q + 64 < rank) load_b(q + 64, u);
        }
    }
    if (tok < 0) return;
    uint16_t *y = reinterpret_cast<uint16_t *>(d.y) + (int64_t)tok * d.N + cb + cl;
    if constexpr (KM) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (cb + cl + 16 * j < d.N)
                *reinterpret_cast<uint2 *>(y + 16 * j) = make_uint2(pack_bf16(acc[j][0], acc[j][1]), pack_bf16(acc[j][2], acc[j][3]));
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (cb + cl + 8 * r < d.N)
                *reinterpret_cast<uint4 *>(y + 8 * r) = make_uint4(pack_bf16(acc[0][r], acc[1][r]), pack_bf16(acc[2][r], acc[3][r]),
                                                                   pack_bf16(acc[4][r], acc[5][r]), pack_bf16(acc[6][r], acc[7][r]));
    }
}

template <int MT, bool KM, int RP, typename Args>
hipError_t launch_base(const SkinnyArgs &a, const DecodeArgs &d, hipStream_t st, const PlanPatch *patch)
{
    constexpr int sh = skinny_lds<RP, KM, 1, kWaves, true>(), smem = sh > red_bytes(MT) ? sh : red_bytes(MT);
    constexpr auto kern = decode_base_kernel<MT, KM, RP, Args>;
    const hipError_t e = allow_lds<kern>(smem);
    if (e != hipSuccess) return e;
    Args b;
    static_cast<SkinnyArgs &>(b) = a;
    int extra = 0;
    if constexpr (kHasPatch<Args>) {
        b.patch = *patch;
        extra = patch->blocks;
    }
    COLLM_LAUNCH(kern, dim3(a.n_items * d.h_slices * d.h_cols + extra + d.strips * d.n_slices), dim3(kWaves * 64), smem, st, b, d);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_base(const SkinnyArgs &a, const DecodeArgs &d, int rpad, bool kmajor, hipStream_t st, const PlanPatch *patch)
{
    if (d.n_rows < 1 || d.n_rows > kDecodeRows || d.k_per_slice % 64 != 0 || !a.part || !d.part || rpad > kDecodeRank) return hipErrorInvalidValue;
    auto go = [&](auto mt, auto km, auto rp) -> hipError_t {
        constexpr int MT = decltype(mt)::value, RP = decltype(rp)::value;
        constexpr bool KM = decltype(km)::value;
        return patch ? launch_base<MT, KM, RP, SkinnyPassArgs>(a, d, st, patch) : launch_base<MT, KM, RP, SkinnyArgs>(a, d, st, nullptr);
    };
    auto by_rank = [&](auto mt, auto km) -> hipError_t {
        if (rpad <= 16) return go(mt, km, std::integral_constant<int, 16>());
        return go(mt, km, std::integral_constant<int, kDecodeRankCols>());
    };
    auto by_layout = [&](auto mt) -> hipError_t { return kmajor ? by_rank(mt, std::true_type()) : by_rank(mt, std::false_type()); };
    if (d.n_rows <= 16) return by_layout(std::integral_constant<int, 1>());
    return d.n_rows <= 32 ? by_layout(std::integral_constant<int, 2>()) : by_layout(std::integral_constant<int, 4>());
}

hipError_t launch_decode_finish(const SkinnyArgs &a, const DecodeFinishArgs &d, bool kmajor, hipStream_t st)
{
    const dim3 grid((d.N + kFinishCols - 1) / kFinishCols, a.n_items + (d.n_base + 15) / 16);
    if (grid.y == 0) return hipSuccess;
    if (kmajor) COLLM_LAUNCH(decode_finish_kernel<true>, grid, dim3(256), finish_lds(a.part_ld), st, a, d);
    else COLLM_LAUNCH(decode_finish_kernel<false>, grid, dim3(256), finish_lds(a.part_ld), st, a, d);
    return hipGetLastError();
}

}  // namespace collm
