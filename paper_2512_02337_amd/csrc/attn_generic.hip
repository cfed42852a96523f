// Context part of the verification attention for any supported dtype and head dim on the fp32 matrix
// instructions (fp32 inputs, and bf16 caches too large for the 32-bit offsets of the bf16 kernels).  Products and
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

template <typename T, int D, int NR>
__global__ __launch_bounds__(64 * kGenericWaves) __attribute__((amdgpu_waves_per_eu(D == 128 && NR == 2 ? 1 : 2, D == 128 && NR == 2 ? 1 : 2)))
void attn_ctx_generic_kernel(Shape s, const int32_t *sel_idx, const int32_t *sel_count,
                                                                              int n_sel, Partials part, float scale_log2)
{
    constexpr int KQ = D / 16, VQ = D / 64;   // 16-byte pieces per lane: of a K or query row; of a V row
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int sp = blockIdx.x, bg = blockIdx.z;
    const int b = bg / s.Hkv, g = bg - b * s.Hkv;
    const int R = s.M * s.G;
    const int r0 = ((int)blockIdx.y * kGenericWaves + wave) * (16 * NR);
    if (r0 >= R) return;
    const int L = s.ctx_len[b];
    const int32_t *sel = sel_idx ? sel_idx + (int64_t)bg * n_sel : nullptr;
    const int cnt_raw = sel ? sel_count[bg] : 0;
    f32x4 q[NR][KQ];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        const int r = min(r0 + 16 * t + n, R - 1);   // rows past the end repeat the last one; never stored
        const int hh = r / s.M, j = r - hh * s.M;
        const T *qrow = (const T *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + 4 * kg;
#pragma unroll
        for (int i = 0; i < KQ; ++i) q[t][i] = Quad<T>::load(qrow + 16 * i);
    }
    int nb = L > 0 ? (L + s.B - 1) / s.B : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    int cnt = nb;
    if (sel) cnt = max(0, min(cnt_raw, n_sel));
    const int64_t T_virtual = nb > 0 ? (int64_t)cnt * s.B : 0;
    const int64_t C = (T_virtual + 15) / 16;
    const int64_t c0 = C * sp / part.nsplit, c1 = C * (sp + 1) / part.nsplit;
    const T *kbase = (const T *)s.k + (int64_t)b * s.sb + (int64_t)g * s.sh;
    const T *vbase = (const T *)s.v + (int64_t)b * s.sb + (int64_t)g * s.sh;

    // this lane's token (lane & 15) of 16-token group c, or -1
    auto token = [&](int64_t c) -> int {
        const int64_t p = c * 16 + n;
        if (c >= c1 || p >= T_virtual) return -1;
        const int slot = p < ((int64_t)1 << 31) ? (int)((uint32_t)p / (uint32_t)s.B) : (int)(p / s.B);
        const int blk = sel ? sel[slot] : slot;
        if (blk < 0 || blk >= nb) return -1;
        const int tok = blk * s.B + (int)(p - (int64_t)slot * s.B);
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
            for (int x = 0; x < 4; ++x) S[t][x] = ((r.valid >> (4 * kg + x)) & 1u) ? S[t][x] * scale_log2 : -INFINITY;
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
        int tok = token(c0);
        fetch(tok, ra);
        tok = token(c0 + 1);
        for (int64_t c = c0;;) {   // two register sets in turn
            if (c + 1 >= c1) { use(ra); break; }
            fetch(tok, rb);
            tok = token(c + 2);
            use(ra);
            if (++c + 1 >= c1) { use(rb); break; }
            fetch(tok, ra);
            tok = token(c + 2);
            use(rb);
            ++c;
        }
    }
    const int64_t prow0 = ((int64_t)bg * part.nsplit + sp) * R + r0 + n;
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
    const float scale_log2 = kLog2e / sqrtf((float)s.D);
    // 32 rows per wavefront halve the K / V reads; 16 where that would leave SIMDs without a wavefront
    const bool wide = (int64_t)((R + 31) / 32) * s.batch * s.Hkv * p.nsplit >= 4 * (int64_t)device_cu_count();
    const int rows = 16 * kGenericWaves * (wide ? 2 : 1);
    const dim3 grid(p.nsplit, (R + rows - 1) / rows, s.batch * s.Hkv), block(64 * kGenericWaves);
#define SPECPV_LAUNCH(T, DD)                                                                                                      \
    do {                                                                                                                          \
        if (wide) hipLaunchKernelGGL((attn_ctx_generic_kernel<T, DD, 2>), grid, block, 0, st, s, sel_idx, sel_count, n_sel, p, scale_log2); \
        else hipLaunchKernelGGL((attn_ctx_generic_kernel<T, DD, 1>), grid, block, 0, st, s, sel_idx, sel_count, n_sel, p, scale_log2);     \
    } while (0)
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) SPECPV_LAUNCH(bf16_t, 128); else SPECPV_LAUNCH(bf16_t, 64);
    } else {
        if (s.D == 128) SPECPV_LAUNCH(float, 128); else SPECPV_LAUNCH(float, 64);
    }
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

}  // namespace specpv
