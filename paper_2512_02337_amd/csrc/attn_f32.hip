// Context part of the verification attention for fp32 where a KV head has several tiles of query rows: the same products as
// attn_generic.hip, fp32 matrix instructions throughout, with the K and V rows of some tokens at a time in LDS for all of them.
//
// A workgroup owns (sequence, KV head, four tiles of 16 query rows, KV split), a wavefront per tile.  Its wavefronts bring the
// rows of a chunk of 16 tokens (64 channels: 32) as whole lines, each a quarter of them, through registers into one of two halves of
// LDS, two chunks ahead of the arithmetic (their list entries three ahead), and all of them work on the chunk that is there; one barrier
// a chunk.  The barrier waits for LDS only, so that reads from memory stay under way across it.
//   S^T = K . Q^T     lane & 15 = token of the A operand, query row of the B operand; lane / 16 picks the channels
//                     16 i + 4 (lane / 16) .. + 3: 16-byte pieces of a K row, piece p of row t at p ^ (t & 15), so that the sixteen
//                     lanes of an LDS read, same piece of sixteen rows, cover all banks;
//   O^T += V^T . P^T  S^T element x of a lane is token 4 (lane / 16) + x of row lane & 15, which is the B operand of
//                     step x; the A operand takes channels 64 jj + 4 (lane & 15) + j as tile (jj, j): 256 adjacent bytes of a V row.
// What bounds it: the matrix instructions of the wavefronts that share a SIMD (64 % of the time busy at 37 nodes and 16K tokens), rows
// that fill up a workgroup's 64, and for small calls a chunk's trip.  Read straight from memory, as in attn_generic.hip, a K operand
// touches 64 bytes of sixteen rows, which a CU takes in at a third of the rate of whole lines, once per tile.  Refresh, fp32, 37 nodes at
// G = 4, 16K tokens: 8 KV heads of 128 channels 239 -> 150 us, of 64 118 -> 82; six sequences of 1137, 2 heads 59 -> 41 (with their scores by way of
// LDS too).  A partial step over 4K tokens of 8 heads, 128 channels, 60 nodes 81 -> 55, 12 nodes 40 -> 28.  Workgroups
// of five to sixteen wavefronts, which read less, are slower (60 nodes, 16K: 173 with four, 174 with eight, 270 with five).
#include "internal.h"

namespace specpv {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 4;

struct F32Args {
    const int32_t *sel_idx, *sel_count;
    int n_sel, nsplit;
    FastDiv M, B, nsplits;
    float scale_log2;
};

__device__ __forceinline__ float max_over_groups(float x)   // over lanes n, n + 16, n + 32, n + 48
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// LDS operations of this wavefront are done, then the workgroup's barrier (__syncthreads would wait for reads from memory too).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// grid: x = part * splits + split, y = KV head, z = sequence.  J: row sets (1 KiB of K and of V) of a chunk that a wavefront brings at most.
template <int D, int H>
__global__ __launch_bounds__(64 * kF32Waves, D == 128 && H == 2 ? 2 : 4) void attn_ctx_f32_kernel(Shape s, F32Args a, Partials part)
{
    constexpr int KQ = D / 16, VQ = D / 64;
    constexpr int TOKENS = 16 * H, W = kF32Waves;   // of a chunk
    constexpr int LPR = D / 4, RPS = 64 / LPR, J = TOKENS / (RPS * W);   // lanes of a row, rows of a set, sets of a wavefront
    static_assert(J * RPS * W == TOKENS, "every row is brought");
    constexpr int ROW = D * 4, HALF = TOKENS * ROW;
    __shared__ __attribute__((aligned(1024))) char ring[2][2][HALF];      // [half][K, V]
    __shared__ __attribute__((aligned(16))) int counts[2][TOKENS];    // tokens that count
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int g = blockIdx.y, b = blockIdx.z, bg = b * s.Hkv + g;
    const int32_t *sel = a.sel_idx ? a.sel_idx + (int64_t)bg * a.n_sel : nullptr;
    const int L = s.ctx_len[b];
    const int listed = sel ? a.sel_count[bg] : 0;
    const int prt = (int)a.nsplits.div(blockIdx.x), sp = (int)blockIdx.x - prt * a.nsplit, R = s.M * s.G;
    const int r0 = (prt * W + wave) * 16;
    f32x4 q[KQ];
    {
        const int r = min(r0 + n, R - 1);   // rows past the end repeat the last one; never stored
        const int hh = (int)a.M.div((uint32_t)r), j = r - hh * s.M;
        const float *qrow = (const float *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + 4 * kg;
#pragma unroll
        for (int i = 0; i < KQ; ++i) q[i] = *(const f32x4 *)(qrow + 16 * i);
    }
    int nb = L > 0 ? (int)a.B.div((uint32_t)L + (uint32_t)s.B - 1u) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    const int cnt = sel ? max(0, min(listed, a.n_sel)) : nb;
    const int T = nb > 0 ? cnt * s.B : 0, C = (int)(((uint32_t)T + (uint32_t)TOKENS - 1u) / (uint32_t)TOKENS);
    const int base = (int)a.nsplits.div((uint32_t)C), rem = C - base * a.nsplit;
    const int c0 = base * sp + min(rem, sp), c1 = c0 + base + (sp < rem ? 1 : 0);
    const float *kbase = (const float *)s.k + (int64_t)b * s.sb + (int64_t)g * s.sh;
    const float *vbase = (const float *)s.v + (int64_t)b * s.sb + (int64_t)g * s.sh;
    const int rl = lane / LPR, piece = lane % LPR;

    int entry[J];            // list entries of this lane's rows, of the chunk after the next one to be requested
    f32x4 kr[J], vr[J];
    bool there[J];
    auto look_up = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int p = c * TOKENS + (wave + j * W) * RPS + rl;
            const int slot = (int)a.B.div((uint32_t)p);
            entry[j] = -1;
            if (c < c1 && p < T) entry[j] = sel ? sel[slot] : slot;
        }
    };
    auto request = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int p = c * TOKENS + (wave + j * W) * RPS + rl;
            const int slot = (int)a.B.div((uint32_t)p), tok = entry[j] * s.B + (p - slot * s.B);
            there[j] = entry[j] >= 0 && entry[j] < nb && tok < L;
            kr[j] = vr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (there[j]) {
                kr[j] = *(const f32x4 *)(kbase + (int64_t)tok * s.st + 4 * piece);
                vr[j] = *(const f32x4 *)(vbase + (int64_t)tok * s.st + 4 * piece);
            }
        }
    };
    auto put = [&](int half) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int row = (wave + j * W) * RPS + rl;
            *(f32x4 *)(ring[half][0] + row * ROW + 16 * (piece ^ (row & 15))) = kr[j];
            *(f32x4 *)(ring[half][1] + row * ROW + 16 * piece) = vr[j];
            if (piece == 0) counts[half][row] = there[j] ? 1 : 0;
        }
    };

    f32x4 O[4 * VQ];
    float m_ref = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int j = 0; j < 4 * VQ; ++j) O[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto use = [&](int half) __attribute__((always_inline)) {
        f32x4 S[H];
#pragma unroll
        for (int h = 0; h < H; ++h) S[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KQ; ++i) {
            f32x4 k[H];
#pragma unroll
            for (int h = 0; h < H; ++h) k[h] = *(const f32x4 *)(ring[half][0] + (16 * h + n) * ROW + 16 * ((4 * i + kg) ^ n));
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int h = 0; h < H; ++h) S[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[h][e], q[i][e], S[h], 0, 0, 0);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int4 ok = *(const int4 *)&counts[half][16 * h + 4 * kg];
            S[h][0] = ok.x ? S[h][0] * a.scale_log2 : -INFINITY;
            S[h][1] = ok.y ? S[h][1] * a.scale_log2 : -INFINITY;
            S[h][2] = ok.z ? S[h][2] * a.scale_log2 : -INFINITY;
            S[h][3] = ok.w ? S[h][3] * a.scale_log2 : -INFINITY;
            mx = fmaxf(mx, fmaxf(fmaxf(S[h][0], S[h][1]), fmaxf(S[h][2], S[h][3])));
        }
        mx = max_over_groups(mx);
        // the reference maximum moves only when the true one gets more than 2^8 ahead
        if (__any(mx > m_ref + 8.f)) {
            const float m_new = mx > m_ref + 8.f ? mx : m_ref;
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_ref - m_new);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int j = 0; j < 4 * VQ; ++j) O[j] *= alpha;
        }
        const float m_use = m_ref == -INFINITY ? 0.f : m_ref;
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                S[h][x] = __builtin_amdgcn_exp2f(S[h][x] - m_use);
                l_run += S[h][x];
            }
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int jj = 0; jj < VQ; ++jj) {
                    const f32x4 v = *(const f32x4 *)(ring[half][1] + (16 * h + 4 * kg + x) * ROW + 256 * jj + 16 * n);
#pragma unroll
                    for (int j = 0; j < 4; ++j) O[4 * jj + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], S[h][x], O[4 * jj + j], 0, 0, 0);
                }
    };

    // At the top of a turn chunk c lies in half c & 1 and chunk c + 1 is on its way into registers.
    if (c0 < c1) {
        look_up(c0);
        request(c0);
        look_up(c0 + 1);
        put(c0 & 1);
        request(c0 + 1);
        look_up(c0 + 2);
        lds_barrier();
        for (int c = c0; c < c1; ++c) {
            if (c + 1 < c1) {
                put((c + 1) & 1);   // (read last in front of the last barrier)
                request(c + 2);
                look_up(c + 3);
            }
            if (r0 < R) use(c & 1);
            lds_barrier();
        }
    }
    if (r0 + n >= R) return;
    float l = l_run;
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const int64_t prow = ((int64_t)bg * a.nsplit + sp) * R + r0 + n;
    float *po = part.o + prow * D;
    // accumulator element x of tile (jj, j) is channel 64 jj + 16 kg + 4 x + j: written once, read once by the combine
#pragma unroll
    for (int jj = 0; jj < VQ; ++jj)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const f32x4 v = {O[4 * jj][x], O[4 * jj + 1][x], O[4 * jj + 2][x], O[4 * jj + 3][x]};
            __builtin_nontemporal_store(v, (f32x4 *)(po + partial_pos(64 * jj + 16 * kg + 4 * x, D)));
        }
    if (kg == 0) *(float2 *)(part.ml + prow * 2) = make_float2(m_ref, l);
}

hipError_t launch_attn_ctx_f32(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count, int n_sel, Partials p, hipStream_t st)
{
    const int parts = (s.M * s.G + kF32Rows - 1) / kF32Rows;
    const F32Args a{sel_idx, sel_count, n_sel, p.nsplit, make_fastdiv((uint32_t)s.M), make_fastdiv((uint32_t)s.B), make_fastdiv((uint32_t)p.nsplit), kLog2e / sqrtf((float)s.D)};
    // At 128 channels 32 tokens a chunk leave room for two workgroups on a CU; more of them bring 16 each, and cover each other's
    // trips.  Partial step, 16 / 32 tokens: 30 nodes, 8 KV heads, 4K tokens 36.8 / 35.5 us, 16 nodes, 2 heads, 16K 41.4 / 38.5; three
    // workgroups, 37 nodes, 8 heads, 16K 134 / 146.
    const bool few = (int64_t)parts * p.nsplit * s.Hkv * s.batch <= 2 * (int64_t)device_cu_count();
    const dim3 grid(p.nsplit * parts, s.Hkv, s.batch), block(64 * kF32Waves);
#define SPECPV_LAUNCH(DD, HH) hipLaunchKernelGGL((attn_ctx_f32_kernel<DD, HH>), grid, block, 0, st, s, a, p)
    if (s.D == 64) SPECPV_LAUNCH(64, 2); else if (few) SPECPV_LAUNCH(128, 2); else SPECPV_LAUNCH(128, 1);
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

}  // namespace specpv
