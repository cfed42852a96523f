// Context part of the verification attention for any supported dtype and head dim on the fp32 matrix
// instructions (small fp32 calls -- larger ones: attn_f32.hip --, and bf16 caches too large for the 32-bit offsets of the bf16 kernels).  Products and
// sums are fp32, as on the vector ALU, at twice its rate.
//
// A wavefront owns NR tiles of 16 query rows of a KV head (row r = head r / M of the group, node r % M) and one KV
// split, and walks the split's tokens 16 at a time (v_mfma_f32_16x16x4_f32):
//   S^T = K . Q^T     lane & 15 = token of the A operand, query row of the B operand; lane / 16 picks the channels
//                     16 i + 4 (lane / 16) .. + 3, so both come from memory as 16-byte pieces, no LDS in between;
//   O^T += V^T . P^T  S^T element x of a lane is token 4 (lane / 16) + x of row lane & 15, which is the B operand of
//                     step x; the A operand takes channels 64 jj + 4 (lane & 15) + j as tile (jj, j), so that V comes
//                     as 16-byte pieces too.
// The next 16 tokens' rows are requested before the present ones are used, their list entries one step earlier.
// What bounds it: a wavefront's chain per 16 tokens for small calls; for large ones the matrix instructions of the one or
// two wavefronts per SIMD that the registers allow.  Whole calls, fp32, against one wavefront per (head, node, split) on
// the vector ALU: 37-node refresh of 16K tokens, 8 KV heads at G = 4, 128 channels 2283 -> 273 us (39 TFLOP/s), 64
// channels 1605 -> 127 us; 60-node partial step over 2K tokens of it 347 -> 57 us; one KV head of 64 channels, 16
// nodes, 2K 23.6 -> 15.5 us.
#include "internal.h"
#include <type_traits>

namespace specpv {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Four adjacent elements as fp32.
template <typename T> struct Quad;
template <> struct Quad<float> {
    static __device__ __forceinline__ f32x4 load(const float *p) { return *(const f32x4 *)p; }
};
template <> struct Quad<bf16_t> {
    static __device__ __forceinline__ f32x4 load(const bf16_t *p)
    {
        const uint2 u = *(const uint2 *)p;
        return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
    }
};

constexpr int kGenericWaves = 4;   // wavefronts per workgroup: neighbouring row tiles of one split (they share its K / V rows in L1)

// The divisions of a call whose listed tokens can be counted in 31 bits (SHORT; any other: 64-bit divisions on the GPU).
struct GenericArgs {
    FastDiv M, B, nsplit;   // by query nodes, block size, splits
    float scale_log2;
};

// grid: x = row tile * splits + split, y = KV head, z = sequence.
// A small call is a chain of trips to memory, so what the first one brings goes out of the leading arguments, which arrive in
// registers: lengths, counts, the list (up to 256 entries, lane t: entries t, t + 64, ...), query rows; the rows that the
// list names are the second.  One KV head of 64 channels, 16 nodes, 9 blocks of 16 out of 2K tokens: 6.4 -> 5.4 us (kernel trace;
// before, the argument block, the lengths, the list and the rows followed one another, with two 64-bit divisions in between);
// selection and partial step of it 16.6 -> 16.0, of which the host takes 15.
template <typename T, int D, int NR, bool SHORT>
__global__ __launch_bounds__(64 * kGenericWaves) __attribute__((amdgpu_waves_per_eu(D == 128 && NR == 2 ? 1 : 2, D == 128 && NR == 2 ? 1 : 2)))
void attn_ctx_generic_kernel(const int32_t *sel_idx, const int32_t *sel_count, const int32_t *a_ctx_len, const void *a_q, int n_sel, int a_M, int a_Hkv,
                             int nsplit, Shape s, Partials part, GenericArgs a)
{
    s.ctx_len = a_ctx_len; s.q = a_q; s.M = a_M; s.Hkv = a_Hkv;
    constexpr int KQ = D / 16, VQ = D / 64;   // 16-byte pieces per lane: of a K or query row; of a V row
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int g = blockIdx.y, b = blockIdx.z, bg = b * s.Hkv + g;
    const int32_t *sel = sel_idx ? sel_idx + (int64_t)bg * n_sel : nullptr;
    // (vector loads: scalar ones return in any order, so that using one waits for the argument block as well)
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const int L_v = s.ctx_len[b + zero], cnt_v = (sel ? sel_count + bg : s.ctx_len + b)[zero];
    const bool in_regs = sel && n_sel > 0 && n_sel <= 256;
    int id[4];
    {
        const int32_t *list = in_regs ? sel : s.ctx_len + b;
#pragma unroll
        for (int x = 0; x < 4; ++x) id[x] = list[in_regs ? min(lane + 64 * x, n_sel - 1) : 0];
    }
    asm volatile("" :: "s"(s.k), "s"(s.v), "s"(s.sb), "s"(s.sh), "s"(s.st), "s"(s.max_blocks), "s"(s.B), "s"(s.Hq), "s"(s.G), "s"(part.o), "s"(part.ml));
    asm volatile("" :: "s"(a.M.mul), "s"(a.M.shift), "s"(a.M.d), "s"(a.B.mul), "s"(a.B.shift), "s"(a.B.d),
                 "s"(a.nsplit.mul), "s"(a.nsplit.shift), "s"(a.nsplit.d));
    const int tile = (int)a.nsplit.div_straight(blockIdx.x), sp = (int)blockIdx.x - tile * nsplit, R = s.M * s.G;
    const int r0 = (tile * kGenericWaves + wave) * (16 * NR);
    if (r0 >= R) return;
    f32x4 q[NR][KQ];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int r = min(r0 + 16 * t + n, R - 1);   // rows past the end repeat the last one; never stored
        const int hh = (int)a.M.div_straight((uint32_t)r), j = r - hh * s.M;
        const T *qrow = (const T *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + 4 * kg;
#pragma unroll
        for (int i = 0; i < KQ; ++i) q[t][i] = Quad<T>::load(qrow + 16 * i);
    }
    const int L = __builtin_amdgcn_readfirstlane(L_v);
    int nb = L > 0 ? (int)a.B.div_straight((uint32_t)L + (uint32_t)s.B - 1u) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    int cnt = nb;
    if (sel) cnt = max(0, min(__builtin_amdgcn_readfirstlane(cnt_v), n_sel));
    typedef typename std::conditional<SHORT, int, int64_t>::type idx;
    const idx T_virtual = nb > 0 ? (idx)cnt * (idx)s.B : 0;
    const idx C = (T_virtual + 15) / 16;
    auto first_group = [&](int w) -> idx {   // C * w / nsplit
        if constexpr (SHORT) {
            const int base = (int)a.nsplit.div_straight((uint32_t)C), rem = C - base * nsplit;
            return base * w + (int)a.nsplit.div_straight((uint32_t)(rem * w));
        } else {
            return C * w / nsplit;
        }
    };
    const idx c0 = first_group(sp), c1 = first_group(sp + 1);
    const T *kbase = (const T *)s.k + (int64_t)b * s.sb + (int64_t)g * s.sh;
    const T *vbase = (const T *)s.v + (int64_t)b * s.sb + (int64_t)g * s.sh;

    // this lane's token (lane & 15) of 16-token group c, or -1.  first: the list entry comes out of the registers where it is there
    auto token = [&](idx c, bool first) -> int {
        const idx p = c * 16 + n;
        const bool in = c < c1 && p < T_virtual;
        int slot;
        if constexpr (SHORT) slot = (int)a.B.div_straight((uint32_t)(in ? p : 0));
        else slot = !in ? 0 : (p < ((int64_t)1 << 31) ? (int)((uint32_t)p / (uint32_t)s.B) : (int)(p / s.B));
        int blk = slot;
        if (first && in_regs) {
            const int src = slot & 63, part_of = slot >> 6;
            blk = __shfl(id[0], src);
#pragma unroll
            for (int x = 1; x < 4; ++x) {
                const int e = __shfl(id[x], src);
                blk = part_of == x ? e : blk;
            }
        } else if (sel && in) {
            blk = sel[slot];
        }
        if (!in || blk < 0 || blk >= nb) return -1;
        const int tok = blk * s.B + (int)(p - (idx)slot * s.B);
        return tok < L ? tok : -1;
    };
    struct Rows { f32x4 k[KQ], v[4][VQ]; unsigned valid; };
    // (a token that does not count reads row 0, which exists where there is any token, and weighs nothing)
    auto fetch = [&](int tok, Rows &r) {
        r.valid = (unsigned)__ballot(tok >= 0);   // bits 16 .. repeat 0 .. 15
        const int row = max(tok, 0);
        const T *kr = kbase + (int64_t)row * s.st + 4 * kg;
#pragma unroll
        for (int i = 0; i < KQ; ++i) r.k[i] = Quad<T>::load(kr + 16 * i);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const T *vr = vbase + (int64_t)__shfl(row, 4 * kg + x) * s.st + 4 * n;
#pragma unroll
            for (int jj = 0; jj < VQ; ++jj) r.v[x][jj] = Quad<T>::load(vr + 64 * jj);
        }
    };

    f32x4 O[NR][4 * VQ];
    float m_ref[NR], l_run[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        m_ref[t] = -INFINITY;
        l_run[t] = 0.f;
#pragma unroll
        for (int j = 0; j < 4 * VQ; ++j) O[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto use = [&](const Rows &r) {
        f32x4 S[NR];
#pragma unroll
        for (int t = 0; t < NR; ++t) S[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KQ; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < NR; ++t) S[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.k[i][e], q[t][i][e], S[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < NR; ++t) {
#pragma unroll
            for (int x = 0; x < 4; ++x) S[t][x] = ((r.valid >> (4 * kg + x)) & 1u) ? S[t][x] * a.scale_log2 : -INFINITY;
            float mx = fmaxf(fmaxf(S[t][0], S[t][1]), fmaxf(S[t][2], S[t][3]));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // the reference maximum moves only when the true one gets more than 2^8 ahead
            if (__any(mx > m_ref[t] + 8.f)) {
                const float m_new = mx > m_ref[t] + 8.f ? mx : m_ref[t];
                const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_ref[t] - m_new);
                m_ref[t] = m_new;
                l_run[t] *= alpha;
#pragma unroll
                for (int j = 0; j < 4 * VQ; ++j) O[t][j] *= alpha;
            }
            const float m_use = m_ref[t] == -INFINITY ? 0.f : m_ref[t];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                S[t][x] = __builtin_amdgcn_exp2f(S[t][x] - m_use);
                l_run[t] += S[t][x];
            }
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int jj = 0; jj < VQ; ++jj)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < NR; ++t)
                        O[t][4 * jj + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.v[x][jj][j], S[t][x], O[t][4 * jj + j], 0, 0, 0);
    };
    if (c0 < c1) {
        Rows ra, rb;
        int tok = token(c0, true);
        fetch(tok, ra);
        tok = token(c0 + 1, true);
        for (idx c = c0;;) {   // two register sets in turn
            if (c + 1 >= c1) { use(ra); break; }
            fetch(tok, rb);
            tok = token(c + 2, false);
            use(ra);
            if (++c + 1 >= c1) { use(rb); break; }
            fetch(tok, ra);
            tok = token(c + 2, false);
            use(rb);
            ++c;
        }
    }
    const int64_t prow0 = ((int64_t)bg * nsplit + sp) * R + r0 + n;
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        float l = l_run[t];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (r0 + 16 * t + n >= R) continue;
        float *po = part.o + (prow0 + 16 * t) * D;
        // accumulator element x of tile (jj, j) is channel 64 jj + 16 kg + 4 x + j: written once, read once by the combine
#pragma unroll
        for (int jj = 0; jj < VQ; ++jj)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const f32x4 v = {O[t][4 * jj][x], O[t][4 * jj + 1][x], O[t][4 * jj + 2][x], O[t][4 * jj + 3][x]};
                __builtin_nontemporal_store(v, (f32x4 *)(po + partial_pos(64 * jj + 16 * kg + 4 * x, D)));
            }
        if (kg == 0) *(float2 *)(part.ml + (prow0 + 16 * t) * 2) = make_float2(m_ref[t], l);
    }
}

hipError_t launch_attn_ctx_generic(const Shape &s, int dtype, const int32_t *sel_idx,
                                   const int32_t *sel_count, int n_sel, Partials p, hipStream_t st)
{
    const int R = s.M * s.G;
    // 32 rows per wavefront halve the K / V reads; 16 where that would leave SIMDs without a wavefront
    const bool wide = (int64_t)((R + 31) / 32) * s.batch * s.Hkv * p.nsplit >= 4 * (int64_t)device_cu_count();
    const int rows = 16 * kGenericWaves * (wide ? 2 : 1), tiles = (R + rows - 1) / rows;
    // (a list may name more blocks than there are)
    const int64_t listed = (int64_t)(sel_idx ? n_sel : s.max_blocks) * s.B;
    const bool short_ = listed < ((int64_t)1 << 31) - 64;
    const GenericArgs a{make_fastdiv((uint32_t)s.M), make_fastdiv((uint32_t)s.B), make_fastdiv((uint32_t)p.nsplit), kLog2e / sqrtf((float)s.D)};
    const dim3 grid(p.nsplit * tiles, s.Hkv, s.batch), block(64 * kGenericWaves);
#define SPECPV_LAUNCH_K(T, DD, NR, SH)                                                                                            \
    hipLaunchKernelGGL((attn_ctx_generic_kernel<T, DD, NR, SH>), grid, block, 0, st, sel_idx, sel_count, s.ctx_len, s.q, sel_idx ? n_sel : 0, s.M, s.Hkv, p.nsplit, s, p, a)
#define SPECPV_LAUNCH(T, DD)                                                                                                      \
    do {                                                                                                                          \
        if (short_) { if (wide) SPECPV_LAUNCH_K(T, DD, 2, true); else SPECPV_LAUNCH_K(T, DD, 1, true); }                           \
        else { if (wide) SPECPV_LAUNCH_K(T, DD, 2, false); else SPECPV_LAUNCH_K(T, DD, 1, false); }                                \
    } while (0)
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) SPECPV_LAUNCH(bf16_t, 128); else SPECPV_LAUNCH(bf16_t, 64);
    } else {
        if (s.D == 128) SPECPV_LAUNCH(float, 128); else SPECPV_LAUNCH(float, 64);
    }
#undef SPECPV_LAUNCH
#undef SPECPV_LAUNCH_K
    return hipGetLastError();
}

}  // namespace specpv
