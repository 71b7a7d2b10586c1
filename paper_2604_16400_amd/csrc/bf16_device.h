// Device code shared by the bf16 kernels: operand types, buffer loads, the plan's new parts that ride on a pass, and the
// rank-wide product of one item.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.h"

namespace collm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    floatx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// ds_read_b64_tr_b16: within each group of 16 lanes, lane s supplies the address of 4
// consecutive 16-bit values (row s / 4, columns 4 (s % 4) ..) of a 4 x 16 block and lane i
// receives column i of that block (checked on the device)
__device__ __forceinline__ bf16x4 lds_tr(const uint8_t *p)
{
    typedef short short4v __attribute__((ext_vector_type(4)));
    const short4v v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (short4v __attribute__((address_space(3))) *)(p));
    return __builtin_bit_cast(bf16x4, v);
}

__device__ __forceinline__ uint4 ldg16(const void *p) { return *reinterpret_cast<const uint4 *>(p); }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kOob = 0x80000000u;  // beyond any buffer (tensors are limited to 2 GiB)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buf16(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Block `blk` of `n_blk` reads its contiguous share of `bytes` bytes at `base` (16-byte aligned), sixteen 16-byte loads
// per thread in flight (the share of a block is mostly one such round: what counts is that everything is asked for
// at once), and drops them.  The values are folded into a word that is stored only if it takes a value the data
// cannot be relied on never to produce and the size is one that never occurs, so that the loads stay.
__device__ __forceinline__ void warm_cache(const void *base, uint64_t bytes, int blk, int n_blk, int tid, int n_thr)
{
    constexpr int U = 16;
    const uint64_t per = ((bytes / 16 + n_blk - 1) / n_blk) * 16;
    const uint64_t lo = (uint64_t)blk * per, hi = lo + per < bytes ? lo + per : bytes;
    const uint8_t *src = reinterpret_cast<const uint8_t *>(base);
    uint32_t fold = 0;
    for (uint64_t off = lo + (uint64_t)tid * 16; off < hi; off += (uint64_t)n_thr * 16 * U) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t o = off + (uint64_t)u * n_thr * 16;
            v[u] = o + 16 <= hi ? ldg16(src + o) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) fold ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    if (fold == 0x9e3779b9u && bytes == 1) *reinterpret_cast<volatile uint32_t *>(const_cast<void *>(base)) = fold;
}

// Block `blk` of patch.blocks copies its share of the plan's new parts; the block that finishes last publishes the
// sequence number, as in plan_copy_kernel.
__device__ __forceinline__ void patch_plan(const PlanPatch &q, int blk, int tid, int n_thr)
{
    const int4 *__restrict__ src = reinterpret_cast<const int4 *>(q.src);
    int4 *__restrict__ dst = reinterpret_cast<int4 *>(q.dst);
#pragma unroll
    for (int part = 0; part < kPatchParts; ++part)
        for (int i = blk * n_thr + tid; i < q.n[part]; i += q.blocks * n_thr) dst[q.lo[part] + i] = src[q.lo[part] + i];
    __syncthreads();  // every load of this block has returned: its stores have been issued
    if (tid == 0) {
        const int old = atomicAdd(q.counter, 1);
        if (old == q.blocks - 1) {
            *q.counter = 0;
            *reinterpret_cast<volatile uint32_t *>(q.done_host) = q.seq;
            __threadfence_system();
        }
    }
}

// Arguments of the passes that carry a patch: kernels of their own, as 1 KiB more of arguments makes every launch dearer
// (three of them in a call of eight decode tokens: 20.0 / 20.3 us).
struct WideArgs : GemmArgs {
    PlanPatch patch;
};
struct SkinnyPassArgs : SkinnyArgs {
    PlanPatch patch;
};
template <typename Args> constexpr bool kHasPatch = std::is_same_v<Args, WideArgs> || std::is_same_v<Args, SkinnyPassArgs>;
// The tiled pass with the 16-row items (of ranks up to RP) in blocks of the same launch, mixed_cols columns of blocks behind its own.
template <int RP, typename Pass>
struct MixedArgs : GemmArgs {
    static constexpr int kRp = RP;
    Pass pass;
    int mixed_split, mixed_cols;
};
template <typename Args> constexpr bool kMixed = false;
template <int RP, typename Pass> constexpr bool kMixed<MixedArgs<RP, Pass>> = true;
template <typename Args>
__device__ __forceinline__ const auto &pass_args(const Args &p)  // what knows the tables and the patch
{
    if constexpr (kMixed<Args>) return p.pass;
    else return p;
}
template <typename Args>
__device__ __forceinline__ int patch_blocks(const Args &p)
{
    if constexpr (kHasPatch<Args>) return p.patch.blocks;
    else return 0;
}
// address of an adapter's table: out of the arguments while the plan's own list is being replaced
template <typename Args>
__device__ __forceinline__ const uint8_t *pass_table(const Args &p, int adapter)
{
    uint64_t v;
    if constexpr (kHasPatch<Args>) v = p.patch.tab[adapter];
    else v = p.tab[adapter];
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);  // (one adapter per block)
}

__device__ __forceinline__ uint32_t word(const uint4 &v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w)); }

// Operands of K-contiguous rows.  An MFMA wants 16 rows x 32 values (lane l: row l % 16, values 8 (l / 16) ..), of which a load would
// touch half of 16 cache lines; two loads of 8 rows x 64 values touch 8 whole lines each: load 0 takes rows 0 .. 7 (lanes l % 16 < 8:
// values 8 (l / 16) .., the others 32 more), load 1 rows 8 .. 15 the other way round.  Then the operand of the first 32 values is in place, half
// of the lanes in each load, and that of the second 32 is the other halves, 8 lanes further in each row of 16.
// (Reading 90 MB of [11008][4096], 344 blocks: 26 us by half lines, 19.7 by whole ones.)
struct RowPair {
    uint4 v[2];
};
__device__ __forceinline__ uint32_t pair_row(int load, int l16) { return (uint32_t)(8 * load + (l16 & 7)); }
__device__ __forceinline__ uint32_t pair_k(int load, int l16, int g) { return (uint32_t)(8 * g + (((l16 >> 3) ^ load) << 5)); }
__device__ __forceinline__ void pair_operands(const RowPair &p, int l16, bf16x8 &first, bf16x8 &second)
{
    u32x4 a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t x = word(p.v[0], i), y = word(p.v[1], i);
        a[i] = l16 < 8 ? x : y;
        b[i] = (uint32_t)__builtin_amdgcn_mov_dpp((int)(l16 < 8 ? y : x), 0x128, 0xf, 0xf, true);  // row_ror:8
    }
    first = __builtin_bit_cast(bf16x8, a);
    second = __builtin_bit_cast(bf16x8, b);
}

// =========================================================================================
// skinny: out[m][q] = sum_k in[tok(m)][k] * table_a(k, q)     (rank-wide output, HBM-bound)
//
// One block = one item (RT = 1 or 2 tiles of 16 rows of one adapter) x one of gridDim.y slices of K.
// Its KW waves split the slice; every wave runs 16x16x32 MFMAs on its own K range for all row
// tiles of the item, so a table fragment is fetched once per item and used RT times.  The
// streamed operand (rows of x or dy) goes from global memory straight into MFMA operand
// registers: lane l holds 8 consecutive K values of row l % 16.  The adapter table is either
// K-major ([rank][K], read the same way) or N-major ([K][rank]): then each wave copies its
// chunk as it lies in memory into a private LDS area and builds the operand with transposing
// reads.  Nothing in the K loop needs a block barrier.  The partial sums of the waves meet in
// LDS in wave order.  With more than one K slice the block writes its sums to a workspace and
// a second, small kernel adds the slices in slice order (fixed order, no float atomics, and no
// fences inside a kernel: on this GPU a device-wide fence writes back and invalidates the L2).
// =========================================================================================
// Where a row's results go: its row of the fp32 copy (token-indexed h_save, training rows only, or row-indexed workspace).  Loads that depend on
// each other: asked for before the sums that they wait for (a row's token, then its flag).
__device__ __forceinline__ float *skinny_f32_row(const SkinnyArgs &p, int row)
{
    if (!p.f32_out) return nullptr;
    if (!p.f32_by_token) return p.f32_out + (int64_t)row * p.f32_ld;
    const int tok = p.row_tok[row];
    return p.tok_train[tok] ? p.f32_out + (int64_t)tok * p.f32_ld : nullptr;
}
// Results of four rank indices q .. q + 3 of a row whose adapter has rank `it_rank`: the fp32 copy and the scaled copy in the element type.
// (The arguments it needs are read once, at its start: read where they are used, they went through scratch memory, a trip for each at the end of a pass.)
__device__ __forceinline__ void skinny_store(const SkinnyArgs &p, float *f32_row, int row, int it_rank, int q, floatx4 sum)
{
    const float f32_mult = p.f32_mult, bf_mult = p.bf_mult;
    const int n_sib = p.n_sib, sib = p.sib, f32_cols = p.f32_cols, bf_ld = p.bf_ld, bf_up = p.bf_up;
    uint16_t *bf_row = p.bf_out ? reinterpret_cast<uint16_t *>(p.bf_out) + (int64_t)row * bf_ld : nullptr;
    asm volatile("" ::: "memory");
    if (n_sib > 1) {
        // one sibling's columns of the row (ranks are multiples of 8 here); the last sibling clears the rest
        const int rank = it_rank / n_sib, co = sib * rank;
        if (q < rank) {
            if (f32_row)
                *reinterpret_cast<floatx4 *>(f32_row + co + q) = sum * f32_mult;
            if (bf_row) {
                uint2 o;
                o.x = pack_bf16(sum[0] * bf_mult, sum[1] * bf_mult);
                o.y = pack_bf16(sum[2] * bf_mult, sum[3] * bf_mult);
                *reinterpret_cast<uint2 *>(bf_row + co + q) = o;
            }
        }
        if (q == 0 && sib == n_sib - 1) {
            if (f32_row)
                for (int z = it_rank; z < f32_cols; ++z) f32_row[z] = 0.f;
            if (bf_row)
                for (int z = it_rank; z < bf_ld; ++z) bf_row[z] = 0;
        }
        return;
    }
    const int rank = it_rank, rp = (rank + 15) & ~15;
    floatx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (q + e < rank) ? sum[e] : 0.f;
    if (f32_row) {
        const floatx4 f = v * f32_mult;
        // zero fill beyond the padded rank (h_save rows are max_rank wide)
        if (((f32_cols | (int)p.f32_ld) & 3) == 0) {
            if (q < f32_cols) *reinterpret_cast<floatx4 *>(f32_row + q) = f;
            if (q + 4 == rp)
                for (int z = rp; z < f32_cols; z += 4) *reinterpret_cast<floatx4 *>(f32_row + z) = floatx4{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (q + e < f32_cols) f32_row[q + e] = f[e];
            if (q + 4 == rp)
                for (int z = rp; z < f32_cols; ++z) f32_row[z] = 0.f;
        }
    }
    if (bf_row) {
        uint2 o;
        o.x = pack_bf16(v[0] * bf_mult, v[1] * bf_mult);
        o.y = pack_bf16(v[2] * bf_mult, v[3] * bf_mult);
        // (bf_up: the second sibling's half of the ranks, a multiple of 16, goes to the second half of the row)
        *reinterpret_cast<uint2 *>(bf_row + (bf_up > 0 && 2 * q >= rank ? q - (rank >> 1) + bf_up : q)) = o;
    }
}

template <int RP>
struct SkinnyCfg {
    static constexpr int CHK = RP <= 64 ? 64 : 32;                    // K values per chunk
    static constexpr int STEPS = CHK / 32;
    static constexpr int KW = RP <= 32 ? 8 : 4;                       // waves per block
    static constexpr int NB = RP / 16;                                // 16-wide rank blocks
    static constexpr int RTMAX = RP <= 128 ? 2 : 1;                   // row tiles per item
    static constexpr int PITCH = RP * 2 + 16;                         // LDS row pitch of an N-major chunk
    static constexpr int STAGE_BYTES = CHK * PITCH;                   // per wave
    static constexpr int RED_LD = RP + 4;                             // floats
};

// Block work of one item and one of n_split slices of K, by KW waves.  SUMS: the sums always go to the workspace, and take
// the place of the waves' stages in LDS.  COLS: columns q_base .. q_base + RP of the table only
// (of more than RP columns where the rank is a multiple of 8).
template <int RP, bool T_KMAJOR, int RT, int KW, bool SUMS>
constexpr int skinny_lds()
{
    using C = SkinnyCfg<RP>;
    constexpr int red = KW * 16 * RT * C::RED_LD * 4, stages = T_KMAJOR ? 0 : KW * C::STAGE_BYTES;
    return SUMS ? (red > stages ? red : stages) : red + stages;
}

template <int RP, bool T_KMAJOR, int RT, int KW, bool SUMS, bool COLS = false, typename Args>
__device__ __forceinline__ void skinny_item(const Args &p, int item, int split, int n_split, uint8_t *smem, int q_base = 0)
{
    using C = SkinnyCfg<RP>;
    constexpr int STEPS = C::STEPS, CHK = C::CHK, NB = C::NB;
    constexpr int ROWS = 16 * RT;
    constexpr int RED_BYTES = KW * ROWS * C::RED_LD * 4;
    float *red = reinterpret_cast<float *>(smem);
    uint8_t *stage = smem + (SUMS ? 0 : RED_BYTES) + (threadIdx.x >> 6) * C::STAGE_BYTES;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (the item is the same for the whole block: kept in scalar registers)
    const SkinnyItem *ip = p.items + item;
    const int adapter = __builtin_amdgcn_readfirstlane(ip->adapter), row_lo = __builtin_amdgcn_readfirstlane(ip->row_lo);
    const int item_rows = __builtin_amdgcn_readfirstlane(ip->n_rows), it_rank = __builtin_amdgcn_readfirstlane(ip->rank);
    const int K = p.K, rank = p.n_sib > 1 ? it_rank / p.n_sib : it_rank;
    if (COLS && q_base >= rank) return;
    const int width = COLS && rank - q_base > RP ? RP : rank - (COLS ? q_base : 0);  // columns of this block
    const int rp = (width + 15) & ~15;
    const int l16 = lane & 15, kg = lane >> 4;
    const int n_rt = (item_rows + 15) >> 4;  // row tiles of this item
    const uint32_t tld = T_KMAJOR && p.tab_ld ? (uint32_t)p.tab_ld : (uint32_t)K, toff = T_KMAJOR ? (uint32_t)p.tab_off : 0u;

    // K range of this wave: the slices of the blocks, cut again into the ranges of their waves
    const int per = (((K + n_split * KW - 1) / (n_split * KW)) + 31) & ~31;
    const int k_lo = (split * KW + wave) * per;
    const int k_hi = (k_lo + per) < K ? (k_lo + per) : K;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.in, p.in_bytes);
    const __amdgpu_buffer_rsrc_t rt = make_rsrc(pass_table(p, adapter),
                                                T_KMAJOR ? (uint32_t)rank * tld * 2u : (uint32_t)rank * (uint32_t)K * 2u);
    // chunks of 64 values by whole cache lines (RowPair)
    constexpr bool PAIR = STEPS == 2;
    uint32_t xoff[RT][STEPS];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int r = t * 16 + (PAIR ? (int)pair_row(s, l16) : l16);
            xoff[t][s] = kOob;
            if (r < item_rows) {
                const int tok = p.row_tok[row_lo + r];
                if (tok >= 0) xoff[t][s] = (uint32_t)tok * (uint32_t)p.ld_in * 2u + (PAIR ? pair_k(s, l16, kg) : kg * 8u) * 2u;
            }
        }
    // first value of the chunk that this lane takes in load s
    auto lane_k = [&](int s) { return PAIR ? (int)pair_k(s, l16, kg) : s * 32 + kg * 8; };

    // D chunks are in flight per wave (a ring of register sets): the pass is bound by memory latency.
    // Four where the registers of a chunk are few enough to keep four waves per SIMD, else two.
    constexpr int D = (RT * STEPS + STEPS * NB <= 8) ? 4 : 2;
    uint4 xreg[D][RT][STEPS];
    auto load_x = [&](int k0, int buf) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) xreg[buf][t][s] = buf16(rx, k0 + lane_k(s) < k_hi ? xoff[t][s] + (uint32_t)k0 * 2u : kOob);
    };

    // K-major table: operand registers straight from memory
    uint4 treg[T_KMAJOR ? D : 1][T_KMAJOR ? STEPS * NB : 1];
    auto load_t_kmajor = [&](int k0, int buf) {
        if constexpr (T_KMAJOR) {
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const int k = k0 + lane_k(s);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int q = (COLS ? q_base : 0) + nb * 16 + (PAIR ? (int)pair_row(s, l16) : l16);
                    treg[buf][s * NB + nb] =
                        buf16(rt, (q < rank && k < k_hi) ? ((uint32_t)q * tld + toff + (uint32_t)k) * 2u : kOob);
                }
            }
        }
    };
    // N-major table: the chunk [CHK][rank] is contiguous; copy it to LDS rows of PITCH bytes
    constexpr int NCP = T_KMAJOR ? 1 : (CHK * RP * 2 / 16 + 63) / 64;  // 16-byte pieces per lane
    uint4 creg[D][NCP];
    // (the chunk starts at a multiple of 32 rows, so its pieces are 16-byte aligned whatever the rank)
    const int n_pieces = (CHK * width) >> 3;
    // piece c holds elements 8 c .. 8 c + 7 of the chunk: first one at row crow, column ccol; the division is done once
    int crow[NCP], ccol[NCP];
    uint32_t coff[NCP];
    if constexpr (!T_KMAJOR) {
#pragma unroll
        for (int i = 0; i < NCP; ++i) {
            const int e = (lane + i * 64) * 8;
            crow[i] = e / width;
            ccol[i] = e - crow[i] * width;
            if constexpr (COLS) coff[i] = rank > RP ? (uint32_t)(crow[i] * rank + q_base + ccol[i]) * 2u : (uint32_t)e * 2u;
        }
    }
    auto load_t_nmajor = [&](int k0, int buf) {
        if constexpr (!T_KMAJOR) {
#pragma unroll
            for (int i = 0; i < NCP; ++i) {
                const int c = lane + i * 64;
                // rows beyond K lie beyond the table and read as zero
                creg[buf][i] = buf16(rt, c < n_pieces ? ((uint32_t)k0 * (uint32_t)rank) * 2u + (COLS ? coff[i] : (uint32_t)c * 16u) : kOob);
            }
        }
    };
    // The loads of a chunk stay together and the chunks stay in order (the compiler may not move memory operations
    // across this): the wait before a chunk's first use then counts exactly the loads of the D - 1 chunks behind it.
    // Left to itself the compiler issues the first chunk's loads last in the prologue, and the loop then waits
    // for all loads at the top of every round.
    auto fence_chunk = [] { asm volatile("" ::: "memory"); };
    // A piece goes to one LDS row where the rank is a multiple of 8; else it may reach into the next row (ranks that are
    // multiples of 4: in halves of 8 bytes) or several (element by element).  901 rows against a [4104][12 .. 64] table:
    // 33.5 us with the table read element by element for ranks 12 and 20, 10.7 us in pieces.
    auto store_t_nmajor = [&](int buf) {
        if constexpr (!T_KMAJOR) {
            // (the addresses of the other ranks' halves and elements are worked out anew for every chunk: hoisted out of the
            // loop they take a hundred registers, and one wave per SIMD instead of two; rank 48, 16384 rows: 124 / 116 us)
            if ((rank & 7) == 0) {
#pragma unroll
                for (int i = 0; i < NCP; ++i)
                    if (lane + i * 64 < n_pieces)
                        *reinterpret_cast<uint4 *>(stage + crow[i] * C::PITCH + ccol[i] * 2) = creg[buf][i];
            } else {
#pragma unroll
                for (int i = 0; i < NCP; ++i) {
                    if (lane + i * 64 >= n_pieces) continue;
                    const uint4 v = creg[buf][i];
                    int row = crow[i], col = ccol[i];
                    asm volatile("" : "+v"(row), "+v"(col));
                    uint8_t *dst = stage + row * C::PITCH;
                    if ((rank & 3) == 0) {
                        *reinterpret_cast<uint2 *>(dst + col * 2) = make_uint2(v.x, v.y);
                        const bool wrap = col + 4 >= rank;
                        *reinterpret_cast<uint2 *>(dst + (wrap ? C::PITCH : (col + 4) * 2)) = make_uint2(v.z, v.w);
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint32_t w = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
                            *reinterpret_cast<uint16_t *>(dst + col * 2) = (uint16_t)(w >> ((e & 1) * 16));
                            if (++col == rank) {
                                col = 0;
                                dst += C::PITCH;
                            }
                        }
                    }
                }
            }
        }
    };

    // (a thread's sums are all of one row)
    static_assert(KW * 64 % ROWS == 0, "a block's threads go over whole columns");
    float *f32_row = nullptr;
    if constexpr (!SUMS) {
        if (n_split == 1 && (int)(tid % ROWS) < item_rows && tid < ROWS * (RP / 4)) f32_row = skinny_f32_row(p, row_lo + tid % ROWS);
    }
    floatx4 acc[RT][NB];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[t][nb] = floatx4{0.f, 0.f, 0.f, 0.f};

    if (k_lo < k_hi) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            load_x(k_lo + d * CHK, d);
            load_t_kmajor(k_lo + d * CHK, d);
            load_t_nmajor(k_lo + d * CHK, d);
            fence_chunk();
        }
        for (int kb = k_lo; kb < k_hi; kb += D * CHK) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int k0 = kb + d * CHK;  // chunks beyond the wave's range were loaded as zeros
                store_t_nmajor(d);
                bf16x8 xf[RT][STEPS];
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    if constexpr (PAIR) pair_operands(RowPair{{xreg[d][t][0], xreg[d][t][1]}}, l16, xf[t][0], xf[t][1]);
                    else xf[t][0] = __builtin_bit_cast(bf16x8, xreg[d][t][0]);
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    if (nb * 16 < rp) {
                        bf16x8 tf[STEPS];
                        if constexpr (T_KMAJOR && PAIR) pair_operands(RowPair{{treg[d][nb], treg[d][NB + nb]}}, l16, tf[0], tf[1]);
                        else if constexpr (T_KMAJOR) tf[0] = __builtin_bit_cast(bf16x8, treg[d][nb]);
#pragma unroll
                        for (int s = 0; s < STEPS; ++s) {
                            if constexpr (!T_KMAJOR) {
                                const uint8_t *src = stage + (s * 32 + kg * 8 + (l16 >> 2)) * C::PITCH + (nb * 16 + (l16 & 3) * 4) * 2;
                                const bf16x4 lo = lds_tr(src), hi = lds_tr(src + 4 * C::PITCH);
                                tf[s] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                            }
#pragma unroll
                            for (int t = 0; t < RT; ++t)
                                if (t < n_rt) acc[t][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tf[s], xf[t][s], acc[t][nb], 0, 0, 0);
                        }
                    }
                }
                // refill this register set with the chunk D further on
                fence_chunk();
                load_x(k0 + D * CHK, d);
                load_t_kmajor(k0 + D * CHK, d);
                load_t_nmajor(k0 + D * CHK, d);
                fence_chunk();
            }
        }
    }

    // lane holds row m = 16 t + lane % 16, columns q = nb*16 + 4*(lane/16) + 0..3
    if constexpr (SUMS) __syncthreads();  // (the sums take the place of the waves' stages)
    {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            float *mine = red + (wave * ROWS + t * 16 + l16) * C::RED_LD;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                *reinterpret_cast<floatx4 *>(mine + nb * 16 + kg * 4) = acc[t][nb];
        }
    }
    __syncthreads();

    // sum over the waves in wave order; with several K slices the sums go to the workspace and a
    // second kernel adds the slices
    const int n_quads = ROWS * (RP / 4);
    for (int idx = tid; idx < n_quads; idx += KW * 64) {
        const int m = idx % ROWS, q = (idx / ROWS) * 4;
        if (m >= item_rows || q >= rp) continue;
        floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < KW; ++w) sum += *reinterpret_cast<const floatx4 *>(red + (w * ROWS + m) * C::RED_LD + q);
        if (SUMS || n_split > 1)
            *reinterpret_cast<floatx4 *>(p.part + ((int64_t)split * p.part_rows + row_lo + m) * p.part_ld + (COLS ? q_base : 0) + q) = sum;
        else
            skinny_store(p, f32_row, row_lo + m, it_rank, q, sum);
    }
}

// Sum of n values that lie `stride` floats apart, added in index order; eight loads are in flight at a time, then four
// (the kernels that add K slices are bound by the latency of these loads, not by their bytes).
template <int COUNT>
__device__ __forceinline__ floatx4 add_slices(floatx4 sum, const float *first, int64_t stride)
{
    floatx4 v[COUNT];
#pragma unroll
    for (int j = 0; j < COUNT; ++j) v[j] = *reinterpret_cast<const floatx4 *>(first + j * stride);
#pragma unroll
    for (int j = 0; j < COUNT; ++j) sum += v[j];
    return sum;
}

__device__ __forceinline__ floatx4 sum_slices(const float *first, int64_t stride, int n)
{
    floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
    int i = 0;
    for (; i + 8 <= n; i += 8) sum = add_slices<8>(sum, first + i * stride, stride);
    if (i + 4 <= n) {
        sum = add_slices<4>(sum, first + i * stride, stride);
        i += 4;
    }
    for (; i < n; ++i) sum += *reinterpret_cast<const floatx4 *>(first + i * stride);
    return sum;
}


// Asks once for the most LDS that launches of KERN take.  (By kernel, not by its type: kernels of one signature differ in LDS.)
template <auto KERN>
static hipError_t allow_lds(int bytes)
{
    static bool done = false;
    if (done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    done = e == hipSuccess;
    return e;
}

}  // namespace collm
