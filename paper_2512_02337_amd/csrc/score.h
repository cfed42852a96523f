// What the kernels that score blocks on the matrix cores share (score_mfma.hip, refresh_tail.hip): see score_mfma.hip.
#pragma once
#include "internal.h"
#include "topk.h"

namespace specpv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kScoreMaxWaves = 16, kScoreMostTiles = 4, kScoreSums = 16;
static inline int score_most_tiles(int waves) { return waves > 4 ? kScoreMostTiles : (waves > 2 ? 2 : 1); }   // of a workgroup, by what LDS holds

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *glb_void_ptr;

// sx, sn: the two score tiles of 32 query rows (q: A operands) against 32 blocks; a: this lane's LDS addresses of the Kmax
// operands, the Kmin operands stand 64 D bytes behind them.  An operand register is read into again behind the matrix
// instruction that was its last reader; "s_nop 11": the twelve wait states between such an instruction and the vector
// ALU's read of its result, which the compiler does not count in here.
__device__ __forceinline__ void score_products(const uint32_t (&a)[8], const bf16x8 (&q)[8], f32x16 &sx, f32x16 &sn)
{
    uint4 b[8];
    asm volatile(
        "ds_read_b128 %[b0], %[a0]\n\t"
        "ds_read_b128 %[b1], %[a1]\n\t"
        "ds_read_b128 %[b2], %[a2]\n\t"
        "ds_read_b128 %[b3], %[a3]\n\t"
        "ds_read_b128 %[b4], %[a4]\n\t"
        "ds_read_b128 %[b5], %[a5]\n\t"
        "ds_read_b128 %[b6], %[a6]\n\t"
        "ds_read_b128 %[b7], %[a7]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q0], %[b0], 0\n\t"
        "ds_read_b128 %[b0], %[a0] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q1], %[b1], %[sx]\n\t"
        "ds_read_b128 %[b1], %[a1] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q2], %[b2], %[sx]\n\t"
        "ds_read_b128 %[b2], %[a2] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q3], %[b3], %[sx]\n\t"
        "ds_read_b128 %[b3], %[a3] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q4], %[b4], %[sx]\n\t"
        "ds_read_b128 %[b4], %[a4] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q5], %[b5], %[sx]\n\t"
        "ds_read_b128 %[b5], %[a5] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q6], %[b6], %[sx]\n\t"
        "ds_read_b128 %[b6], %[a6] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q7], %[b7], %[sx]\n\t"
        "ds_read_b128 %[b7], %[a7] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q0], %[b0], 0\n\t"
        "s_waitcnt lgkmcnt(6)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q1], %[b1], %[sn]\n\t"
        "s_waitcnt lgkmcnt(5)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q2], %[b2], %[sn]\n\t"
        "s_waitcnt lgkmcnt(4)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q3], %[b3], %[sn]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q4], %[b4], %[sn]\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q5], %[b5], %[sn]\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q6], %[b6], %[sn]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q7], %[b7], %[sn]\n\t"
        "s_nop 11\n\t"
        "s_waitcnt lgkmcnt(0)"
        : [sx] "=&v"(sx), [sn] "=&v"(sn), [b0] "=&v"(b[0]), [b1] "=&v"(b[1]), [b2] "=&v"(b[2]), [b3] "=&v"(b[3]), [b4] "=&v"(b[4]), [b5] "=&v"(b[5]), [b6] "=&v"(b[6]), [b7] "=&v"(b[7])
        : [a0] "v"(a[0]), [a1] "v"(a[1]), [a2] "v"(a[2]), [a3] "v"(a[3]), [a4] "v"(a[4]), [a5] "v"(a[5]), [a6] "v"(a[6]), [a7] "v"(a[7]),
          [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [q4] "v"(q[4]), [q5] "v"(q[5]), [q6] "v"(q[6]), [q7] "v"(q[7]), [kn] "n"(8192)
        : "memory");
}
__device__ __forceinline__ void score_products(const uint32_t (&a)[4], const bf16x8 (&q)[4], f32x16 &sx, f32x16 &sn)
{
    uint4 b[4];
    asm volatile(
        "ds_read_b128 %[b0], %[a0]\n\t"
        "ds_read_b128 %[b1], %[a1]\n\t"
        "ds_read_b128 %[b2], %[a2]\n\t"
        "ds_read_b128 %[b3], %[a3]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q0], %[b0], 0\n\t"
        "ds_read_b128 %[b0], %[a0] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q1], %[b1], %[sx]\n\t"
        "ds_read_b128 %[b1], %[a1] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q2], %[b2], %[sx]\n\t"
        "ds_read_b128 %[b2], %[a2] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sx], %[q3], %[b3], %[sx]\n\t"
        "ds_read_b128 %[b3], %[a3] offset:%[kn]\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q0], %[b0], 0\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q1], %[b1], %[sn]\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q2], %[b2], %[sn]\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[sn], %[q3], %[b3], %[sn]\n\t"
        "s_nop 11\n\t"
        "s_waitcnt lgkmcnt(0)"
        : [sx] "=&v"(sx), [sn] "=&v"(sn), [b0] "=&v"(b[0]), [b1] "=&v"(b[1]), [b2] "=&v"(b[2]), [b3] "=&v"(b[3])
        : [a0] "v"(a[0]), [a1] "v"(a[1]), [a2] "v"(a[2]), [a3] "v"(a[3]),
          [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [kn] "n"(4096)
        : "memory");
}

struct ScoreArgs {
    const uint16_t *kmax, *kmin;
    float *scores;
    int reduce, last_node;
    int row0, rows;       // the query rows that count lie in row0 .. rows - 1 (row0: a multiple of 32)
    int waves;            // of a workgroup
    int tiles, groups;    // tiles of a workgroup; workgroups of a (sequence, KV head) (streams: of a KV head)
    int rounds;           // streams: groups of tiles that a workgroup needs to go through at most
    int staged;           // the query rows go through LDS (read_q)
    int sums;             // partial sums per tile and lane: one per block of 32 rows, blocks 16 apart share one
    int by_xcd;           // Hkv % 8 == 0: grid (groups * 8, Hkv / 8, batch), KV head g on XCD g % 8; else (groups, Hkv, batch)
    FastDiv div_G, div_B, div_tiles;
};
// bytes of a tile in LDS (Kmax | Kmin), and of a workgroup: tiles, partial sums and, staged, 32 half rows (64 channels: rows)
// of queries per wavefront
constexpr int score_tile_bytes(int D) { return 128 * D; }
constexpr int kScoreStage = 4096;
static inline size_t score_lds(int D, int tiles, int sums, int staged_waves) { return (size_t)tiles * (score_tile_bytes(D) + sums * 256) + (size_t)staged_waves * kScoreStage; }

// What 32 query rows from r0 on (q: A operands) add to `acc`, for the tile of blocks whose operands stand at `at` (tile: where LDS begins).
template <int D, bool BOUND>
__device__ __forceinline__ float score_rows(const uint32_t (&at)[D / 16], const bf16x8 (&q)[D / 16], char *tile, int r0, int R, int reduce, int last_node, int G, int kg, float acc)
{
    constexpr int KS = D / 16, HALF = 64 * D;
    f32x16 sx, sn;
    if constexpr (BOUND) {
#pragma unroll
        for (int x = 0; x < 16; ++x) sx[x] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // the packed bf16 pairs split by sign: 0xffff in the halves whose sign bit is set
            const uint4 w4 = __builtin_bit_cast(uint4, q[ks]);
            const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
            uint32_t pw[4], nw[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t m = ((w[e] >> 15) & 0x00010001u) * 0xffffu;
                nw[e] = w[e] & m;
                pw[e] = w[e] & ~m;
            }
            const char *p = tile + (at[ks] - (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)tile);
            const bf16x8 bx = __builtin_bit_cast(bf16x8, *(const uint4 *)p), bn = __builtin_bit_cast(bf16x8, *(const uint4 *)(p + HALF));
            sx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, make_uint4(pw[0], pw[1], pw[2], pw[3])), bx, sx, 0, 0, 0);
            sx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, make_uint4(nw[0], nw[1], nw[2], nw[3])), bn, sx, 0, 0, 0);
        }
    } else {
        score_products(at, q, sx, sn);
    }
    // accumulator slot x holds row r0 + (x>>2)*8 + kg*4 + (x&3) of this lane's block
    if (reduce == SPECPV_REDUCE_MAX) {
        // (rows past the end are the last row once more)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc = fmaxf(acc, BOUND ? sx[x] : fmaxf(sx[x], sn[x]));
    } else if (reduce != SPECPV_REDUCE_LAST && r0 + 32 <= R) {
        // all 32 rows count (every wavefront but the one with the ragged end): no per-row tests; the
        // same order of operations as below
#pragma unroll
        for (int x = 0; x < 16; ++x) acc += BOUND ? sx[x] : fmaxf(sx[x], sn[x]);
    } else {
        // (a row that does not count weighs in as nothing: with a branch for each, this wavefront was the last one home.
        // Four at a time: all sixteen conditions at once are more scalar registers than there are.)
        const int lo = reduce == SPECPV_REDUCE_LAST ? last_node * G : 0, hi = reduce == SPECPV_REDUCE_LAST ? lo + G : R;
        const int from = r0 + kg * 4 - lo;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            acc += (uint32_t)(from + (x >> 2) * 8 + (x & 3)) < (uint32_t)(hi - lo) ? (BOUND ? sx[x] : fmaxf(sx[x], sn[x])) : 0.f;
            if ((x & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    return acc;
}

// BOUND: the channel-wise bound instead of eq. 2.  Per channel the larger product is q * Kmax
// where q >= 0 and q * Kmin where q < 0 (Kmax >= Kmin), so the bound is the sum of two inner
// products as well: max(q, 0) . Kmax + min(q, 0) . Kmin, accumulated into one tile.
// ACROSS: the scores are read by another workgroup of this launch: agent-scope stores, which go
// past the caches that are private to a part of the chip.
// group, g, b: which piece of work (the kernel's mapping of blockIdx)
// STAGED: see read_staged.
template <int D, bool BOUND, bool ACROSS, bool STAGED>
__device__ __forceinline__ void score_tiles(const Shape &s, const ScoreArgs &a, const int group, const int g, const int b)
{
    constexpr int KS = D / 16;                  // k-steps
    constexpr int LPR = D / 8, RPO = 64 / LPR;  // lanes per row, rows per 1 KiB DMA operation
    constexpr int OPS = D / 16;                 // DMA operations of one half (Kmax or Kmin) of a tile
    constexpr int HALF = 64 * D, TILE = 2 * HALF;
    // the summary tiles of this workgroup's blocks: row-major, 2 D bytes per block, the
    // 16-byte pieces of row t stored at piece index p ^ (t & 15) (64 channels: p ^ ((t >> 1) & 7)) so that
    // the operand reads (16 lanes per cycle, same piece, different rows) spread over all 64 banks
    extern __shared__ __attribute__((aligned(1024))) char score_smem[];
    char *tile = score_smem;
    float *red = (float *)(score_smem + a.tiles * TILE);   // [a.sums][tile][lane]
    const int lane = threadIdx.x & 63, W = a.waves;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, kg = lane >> 5;
    const int i0 = group * 32 * a.tiles;
    const int R = s.M * s.G;
    // a vector load: a scalar one would hold up whoever waits for an argument.  One sequence: only needed at the very end
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const int L_v = s.ctx_len[b + zero];
    // query rows r0 .. r0 + 31 as A operand: lane = row (a wavefront without a block of rows of its own reads the last row and drops it)
    int r0 = a.row0 + wave * 32;
    bf16x8 q[KS];
    auto read_q = [&]() __attribute__((always_inline)) {
        const int r = min(r0 + n, R - 1);
        const int j = (int)a.div_G.div((uint32_t)r), hh = r - j * s.G;
        const uint16_t *qrow = (const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + kg * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q[ks] = __builtin_bit_cast(bf16x8, *(const uint4 *)(qrow + ks * 16));
    };
    // Operand by operand a read touches 32 rows, 32 bytes of each, and a CU takes such a read in at a third of the rate of whole
    // lines: 2.6 of 11.2 us at 60K in blocks of 16, 1.5 of 6.2 at 16K.  Staged, a read brings 128 bytes of eight rows, and they
    // find their lanes through a corner of LDS that is this wavefront's own (no barrier): 16-byte piece p of row t at
    // p ^ ((t >> 1) & 7).  The later turns of a wavefront read operand by operand: they have no registers for more.
    constexpr int H = D / 64;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 raw[H][4];
    auto load_staged = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = min(r0 + 8 * i + (lane >> 3), R - 1);
            const int j = (int)a.div_G.div_straight((uint32_t)r), hh = r - j * s.G;
            const uint16_t *qrow = (const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + (lane & 7) * 8;
#pragma unroll
            for (int h = 0; h < H; ++h) raw[h][i] = *(const u32x4 *)(qrow + 64 * h);
        }
    };
    auto read_staged = [&]() __attribute__((always_inline)) {
        char *mine = (char *)(red + a.sums * a.tiles * 64) + wave * kScoreStage;
        const int to = (lane >> 3) * 128, from = n * 128;
#pragma unroll
        for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(u32x4 *)(mine + 1024 * i + to + 16 * ((lane & 7) ^ ((4 * i + (lane >> 4)) & 7))) = raw[h][i];
            asm volatile("" ::: "memory");   // (other lanes' values: the compiler keeps the order of LDS operations only if told)
#pragma unroll
            for (int x = 0; x < 4; ++x) q[4 * h + x] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(mine + from + 16 * ((2 * x + kg) ^ ((n >> 1) & 7))));
            asm volatile("" ::: "memory");
        }
    };
    auto blocks = [&]() -> int {
        const int L = __builtin_amdgcn_readfirstlane(L_v);
        const int nb = L > 0 ? (int)a.div_B.div((uint32_t)L + (uint32_t)s.B - 1u) : 0;
        return min(nb, s.max_blocks);
    };
    // in a batch the grid covers the longest sequence: workgroups past the end of a shorter one leave
    // at once (there the wait for the length is cheaper than their reads)
    const int lim = s.batch > 1 ? blocks() : s.max_blocks;
    if (i0 >= lim) return;   // (only out of this function: the workgroup still counts itself in)
    const int n_t = min(a.tiles, (lim - i0 + 31) >> 5);

    if constexpr (STAGED) load_staged();   // (in front of the tiles: reads come back in their order)
    // Summary rows go from memory straight into LDS (DMA operations of 1 KiB shared by the
    // wavefronts; operation d of a tile brings RPO rows of Kmax (d < OPS) or Kmin, LPR lanes per row).  Rows past the end of
    // the arrays repeat the last row; their scores are never stored.
    {
        const int rl = lane / LPR, pos = lane % LPR;
        const int64_t arr_row0 = ((int64_t)b * s.Hkv + g) * s.max_blocks;
        const uintptr_t to_min = (uintptr_t)a.kmin - (uintptr_t)a.kmax;   // (chosen as pointers, they are read from memory on every turn)
        for (int d = wave; d < 2 * OPS * n_t; d += W) {
            const int i = d & (OPS - 1), row = RPO * i + rl, t = d / (2 * OPS);
            const int blk = min(i0 + 32 * t + row, s.max_blocks - 1);
            const int piece = pos ^ (D == 128 ? row & 15 : (row >> 1) & 7);
            const char *src = (const char *)((uintptr_t)a.kmax + ((d & OPS) ? to_min : 0)) + ((arr_row0 + blk) * D) * 2 + 16 * piece;
            __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(tile + (d / OPS) * HALF + i * 1024), 16, 0, 2);   // streaming hint: read once
        }
    }
    if constexpr (STAGED) read_staged();
    else read_q();
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wavefront's DMA operations and query rows are in
    __syncthreads();                      // ... and so are everybody else's
    for (int rb = wave; r0 < a.rows; rb += W) {   // block of 32 rows, from row0 on
        // summary tiles as B operands: lane = block, channels 16*ks + 8*kg .. +8
        const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)tile + (uint32_t)n * (2u * D) +
                              ((16u * (uint32_t)kg) ^ (D == 128 ? 16u * ((uint32_t)n & 15u) : 16u * (((uint32_t)n >> 1) & 7u)));
        for (int t = 0; t < n_t; ++t) {
            uint32_t at[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) at[ks] = (base + (uint32_t)(t * TILE)) ^ (32u * (uint32_t)ks);
            float *mine = red + ((rb & (kScoreSums - 1)) * a.tiles + t) * 64 + lane;
            float acc = rb < kScoreSums ? (a.reduce == SPECPV_REDUCE_MAX ? -INFINITY : 0.f) : *mine;
            acc = score_rows<D, BOUND>(at, q, tile, r0, R, a.reduce, a.last_node, s.G, kg, acc);
            *mine = acc;
        }
        r0 += W * 32;
        if (r0 < a.rows) read_q();
    }
    __syncthreads();
    const int nb = blocks();
    for (int t = wave; t < n_t; t += W) {   // a wavefront per tile
        // (all reads of eight sums in one round trip to LDS; a sum past the last weighs in as nothing)
        const bool by_max = a.reduce == SPECPV_REDUCE_MAX;
        float sum = by_max ? -INFINITY : 0.f;
        for (int w0 = 0; w0 < a.sums; w0 += 8) {
            float o[8];
#pragma unroll
            for (int w = 0; w < 8; ++w) o[w] = red[(min(w0 + w, a.sums - 1) * a.tiles + t) * 64 + lane];
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                if (w0 + w >= a.sums) o[w] = by_max ? -INFINITY : 0.f;
                sum = by_max ? fmaxf(sum, o[w]) : sum + o[w];
            }
        }
        const float other = __shfl_xor(sum, 32);
        float out;
        if (a.reduce == SPECPV_REDUCE_MAX) out = fmaxf(sum, other);
        else if (a.reduce == SPECPV_REDUCE_MEAN) out = (sum + other) / (float)R;
        else out = (sum + other) / (float)s.G;
        const int blk = i0 + 32 * t + n;
        if (kg == 0 && blk < nb) {
            float *dst = a.scores + ((int64_t)b * s.Hkv + g) * s.max_blocks + blk;
            if (ACROSS) __hip_atomic_store((uint32_t *)dst, __float_as_uint(out), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *dst = out;
        }
    }
}

// LDS of score_stream: two halves of tiles and of partial sums.
static inline size_t score_stream_lds(int D, int tiles, int sums) { return 2 * (size_t)tiles * (score_tile_bytes(D) + sums * 256); }

// Which stream a workgroup is: the a.groups workgroups of a KV head are dealt to the sequences by their lengths, so that the longest
// way is as short as they allow: the fewest groups of tiles r that a workgroup has to go through, and to each sequence as many
// workgroups as it has r-groups.  (As many for each sequence, sixteen sequences of 2048 blocks, 8 heads, 60 nodes at G = 5: two workgroups
// went through 22 groups of a long one among short ones, 46.8 us of scores and selection; tiles at once 21.5.)  A lane a sequence.
struct ScoreStream {
    int b, L;             // the sequence and its length
    int group, groups;    // groups of tiles from `group` on, every `groups`-th; groups == 0: none
    __device__ __forceinline__ ScoreStream(const Shape &s, const ScoreArgs &a, int w)
    {
        if (s.batch == 1) {
            b = 0; L = s.ctx_len[0]; group = w; groups = a.groups;
            return;
        }
        const int lane = threadIdx.x & 63;
        const int length = lane < s.batch ? s.ctx_len[lane] : 0;
        const int blocks = min(length > 0 ? (int)a.div_B.div((uint32_t)length + (uint32_t)s.B - 1u) : 0, s.max_blocks);
        const uint32_t n = a.div_tiles.div(((uint32_t)blocks + 31u) / 32u + (uint32_t)a.tiles - 1u);   // groups of tiles
        auto workgroups = [&](uint32_t r) { return (int)((n + r - 1u) / r); };
        int lo = 1, hi = a.rounds;   // (a.rounds are enough for sequences that are all as long as may be)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (__builtin_amdgcn_readlane(wave_inclusive_scan(workgroups((uint32_t)mid)), 63) <= a.groups) hi = mid;
            else lo = mid + 1;
        }
        const int mine = workgroups((uint32_t)lo), upto = wave_inclusive_scan(mine);
        const unsigned long long behind = __ballot(w < upto);
        b = L = group = groups = 0;
        if (!behind) return;
        b = __builtin_ctzll(behind);
        groups = __builtin_amdgcn_readlane(mine, b);
        group = w - (__builtin_amdgcn_readlane(upto, b) - groups);
        L = __builtin_amdgcn_readlane(length, b);
    }
};

// Scores of one stream's groups of a.tiles tiles (eq. 2): where a (sequence, KV head) has many tiles, a workgroup
// keeps the query rows in registers, a block of 32 to a wavefront, and goes through its groups while the next one's rows are on their
// way.  One barrier a group: behind it the group's tiles have landed, everybody is done with the half that the next group goes to, and
// the sums of the group before are there, to be added up and stored.  Reads and writes of LDS are assembly: the compiler would have each
// wait for the tiles that are on their way.
template <int D>
__device__ __forceinline__ void score_stream(const Shape &s, const ScoreArgs &a, const ScoreStream &mine, const int g)
{
    const int b = mine.b, L = mine.L;
    constexpr int KS = D / 16, LPR = D / 8, RPO = 64 / LPR, OPS = D / 16, HALF = 64 * D, TILE = 2 * HALF, H = D / 64;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(1024))) char score_smem[];
    const int lane = threadIdx.x & 63, W = a.waves, T = a.tiles, R = s.M * s.G;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, kg = lane >> 5;
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)score_smem;
    const uint32_t red = ring + 2u * (uint32_t)(T * TILE), red_half = (uint32_t)(a.sums * T * 256);   // [half][sums][tile][lane]
    const int nb = min(L > 0 ? (int)a.div_B.div((uint32_t)L + (uint32_t)s.B - 1u) : 0, s.max_blocks);
    const int step = mine.groups * 32 * T;
    int i0 = mine.group * 32 * T;
    if (step == 0 || i0 >= nb) return;
    const int r0 = a.row0 + wave * 32;
    // the query rows as whole lines, through what will be the second half of the tiles (score_tiles: read_staged)
    u32x4 raw[H][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = min(r0 + 8 * i + (lane >> 3), R - 1);
        const int j = (int)a.div_G.div_straight((uint32_t)r), hh = r - j * s.G;
        const uint16_t *qrow = (const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + (lane & 7) * 8;
#pragma unroll
        for (int h = 0; h < H; ++h) raw[h][i] = *(const u32x4 *)(qrow + 64 * h);
    }
    const int rl = lane / LPR, pos = lane % LPR;
    const int64_t arr_row0 = ((int64_t)b * s.Hkv + g) * s.max_blocks;
    const uintptr_t to_min = (uintptr_t)a.kmin - (uintptr_t)a.kmax;
    auto request = [&](int first, int half) __attribute__((always_inline)) {   // (score_tiles has the layout)
        const int n_t = min(T, (nb - first + 31) >> 5);
        for (int d = wave; d < 2 * OPS * n_t; d += W) {
            const int i = d & (OPS - 1), row = RPO * i + rl, t = d / (2 * OPS);
            const int blk = min(first + 32 * t + row, s.max_blocks - 1);
            const int piece = pos ^ (D == 128 ? row & 15 : (row >> 1) & 7);
            const char *src = (const char *)((uintptr_t)a.kmax + ((d & OPS) ? to_min : 0)) + ((arr_row0 + blk) * D) * 2 + 16 * piece;
            __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(score_smem + half * T * TILE + (d / OPS) * HALF + i * 1024), 16, 0, 2);
        }
    };
    request(i0, 0);
    bf16x8 q[KS];
    {
        char *corner = score_smem + T * TILE + wave * kScoreStage;
        const int to = (lane >> 3) * 128, from = n * 128;
#pragma unroll
        for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(u32x4 *)(corner + 1024 * i + to + 16 * ((lane & 7) ^ ((4 * i + (lane >> 4)) & 7))) = raw[h][i];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int x = 0; x < 4; ++x) q[4 * h + x] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(corner + from + 16 * ((2 * x + kg) ^ ((n >> 1) & 7))));
            asm volatile("" ::: "memory");
        }
    }
    const uint32_t lane_at = (uint32_t)n * (2u * D) + ((16u * (uint32_t)kg) ^ (D == 128 ? 16u * ((uint32_t)n & 15u) : 16u * (((uint32_t)n >> 1) & 7u)));
    const bool by_max = a.reduce == SPECPV_REDUCE_MAX;
    auto add_up = [&](int first, int half) __attribute__((always_inline)) {
        const int n_t = min(T, (nb - first + 31) >> 5);
        for (int t = wave; t < n_t; t += W) {   // a wavefront per tile
            float sum = by_max ? -INFINITY : 0.f;
            for (int w0 = 0; w0 < a.sums; w0 += 8) {
                float o[8];
                uint32_t at[8];
#pragma unroll
                for (int w = 0; w < 8; ++w) at[w] = red + (uint32_t)half * red_half + (uint32_t)(((min(w0 + w, a.sums - 1) * T + t) * 64 + lane) * 4);
                asm volatile(
                    "ds_read_b32 %0, %8\n\t"
                    "ds_read_b32 %1, %9\n\t"
                    "ds_read_b32 %2, %10\n\t"
                    "ds_read_b32 %3, %11\n\t"
                    "ds_read_b32 %4, %12\n\t"
                    "ds_read_b32 %5, %13\n\t"
                    "ds_read_b32 %6, %14\n\t"
                    "ds_read_b32 %7, %15\n\t"
                    "s_waitcnt lgkmcnt(0)"
                    : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7])
                    : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7])
                    : "memory");
#pragma unroll
                for (int w = 0; w < 8; ++w) {
                    if (w0 + w >= a.sums) o[w] = by_max ? -INFINITY : 0.f;
                    sum = by_max ? fmaxf(sum, o[w]) : sum + o[w];
                }
            }
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
            const float lo = __uint_as_float(both[0]), hi = __uint_as_float(both[1]);   // sums of lanes n and n + 32
            float out;
            if (by_max) out = fmaxf(lo, hi);
            else if (a.reduce == SPECPV_REDUCE_MEAN) out = (lo + hi) / (float)R;
            else out = (lo + hi) / (float)s.G;
            const int blk = first + 32 * t + n;
            if (kg == 0 && blk < nb) a.scores[arr_row0 + blk] = out;
        }
    };
    int before = -1;
    for (int half = 0;; half ^= 1) {
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int next = i0 + step;
        if (next < nb) request(next, half ^ 1);
        if (before >= 0) add_up(before, half ^ 1);
        const int n_t = min(T, (nb - i0 + 31) >> 5);
        for (int t = 0; t < n_t; ++t) {
            uint32_t at[KS];
            const uint32_t base = ring + (uint32_t)((half * T + t) * TILE) + lane_at;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) at[ks] = base ^ (32u * (uint32_t)ks);
            const float acc = score_rows<D, false>(at, q, score_smem, r0, R, a.reduce, a.last_node, s.G, kg, by_max ? -INFINITY : 0.f);
            asm volatile("ds_write_b32 %0, %1" ::"v"(red + (uint32_t)half * red_half + (uint32_t)(((wave * T + t) * 64 + lane) * 4)), "v"(acc) : "memory");
        }
        before = i0;
        if (next >= nb) {
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            add_up(before, half);
            return;
        }
        i0 = next;
    }
}

// Tiles, wavefronts and workgroups for a shape (score_mfma.hip).  keep_all: one wavefront per block of 32 query rows, as the
// selection in the same launch needs them.
ScoreArgs score_plan(const Shape &s, const void *kmax, const void *kmin, int reduce, int last_node, float *scores, bool keep_all);

}  // namespace specpv
