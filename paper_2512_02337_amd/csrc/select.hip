// Block scoring (Section 3.2, eq. 2 and eq. 3) for fp32, and the per-(sequence, KV head) top-k
// selection of sink + retrieval + local blocks.  The scoring kernel for bf16 lives in score_mfma.hip.
#include "internal.h"
#include "topk.h"

namespace specpv {

// ---------------------------------------------------------------------------
// fp32 scoring on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: fp32 products and sums).  A workgroup owns 16
// blocks; its wavefronts hold their two summary rows as B operand (lane & 15 = block, lane / 16 picks channels
// 16 i + 4 (lane / 16) .. + 3) and take 16 query rows at a time as A operand, all read as 16-byte pieces.  A lane ends
// up with four rows of one block; the reduction over rows runs over a wavefront's tiles, then over the four lane
// groups, then over the wavefronts, in the same order for every block: identical blocks get identical scores wherever
// they sit.
// One round trip to memory and D / 2 matrix instructions per tile of rows; a lane per block with the rows in LDS took
// 44.6 us for 128 blocks and 64 rows of 64 channels, because two wavefronts did it all.  Scoring, selection and partial
// step of that shape: 65.2 -> 26.6 us.
// ---------------------------------------------------------------------------
constexpr int kScoreF32MaxWaves = 16;

// STAGED: the summary rows go through LDS, once per workgroup and as whole lines; operand by operand every wavefront reads 64 bytes of
// sixteen rows at a time, which a CU takes in at a third of the rate.  Selection and partial step, 60 nodes at G = 4, 44 blocks, 64
// channels 27.2 -> 25.1 us; refresh, 37 nodes, 128 channels, 6 x 72 blocks 42.4 -> 39.5.  One tile of query rows has nobody to share
// with (1 node, 512 blocks, 43.3; through LDS 44.3).
template <int D, bool STAGED>
__global__ __launch_bounds__(64 * kScoreF32MaxWaves) void score_f32_kernel(Shape s, const float *__restrict__ kmax, const float *__restrict__ kmin,
                                                                           int reduce, int last_node, int kind, float *__restrict__ scores)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int Q = D / 16;   // 16-byte pieces per lane and row
    constexpr int P = D / 4;    // 16-byte pieces of a row
    __shared__ float red[kScoreF32MaxWaves][16];
    __shared__ __attribute__((aligned(1024))) f32x4 rows[STAGED ? 2 : 1][STAGED ? 16 : 1][P];   // Kmax, Kmin of the blocks: piece p of row r at p ^ r
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
    const int n = lane & 15, kg = lane >> 4;
    const int g = blockIdx.y, b = blockIdx.z;
    const int i = blockIdx.x * 16 + n;
    const int R = s.M * s.G;
    const int L = s.ctx_len[b];
    f32x4 q[Q];
    auto read_q = [&](int r0) __attribute__((always_inline)) {
        const int r = min(r0 + n, R - 1);
        const int j = r / s.G, hh = r - j * s.G;
        const float *qrow = (const float *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + 4 * kg;
#pragma unroll
        for (int x = 0; x < Q; ++x) q[x] = *(const f32x4 *)(qrow + 16 * x);
    };
    // (rows past the end of the arrays repeat the last block; their scores are never stored)
    const int64_t arr_row0 = ((int64_t)b * s.Hkv + g) * s.max_blocks;
    f32x4 kx[Q], kn[Q];
    if constexpr (STAGED) {
        for (int t = threadIdx.x; t < 2 * 16 * P; t += blockDim.x) {
            const int row = (t / P) & 15, piece = t % P;
            const float *src = (t < 16 * P ? kmax : kmin) + (arr_row0 + min((int)blockIdx.x * 16 + row, s.max_blocks - 1)) * D + 4 * piece;
            rows[t / (16 * P)][row][piece ^ row] = *(const f32x4 *)src;
        }
        if (wave * 16 < R) read_q(wave * 16);   // (fewer than four tiles of rows leave wavefronts that only bring summaries)
        __syncthreads();
#pragma unroll
        for (int x = 0; x < Q; ++x) { kx[x] = rows[0][n][(4 * x + kg) ^ n]; kn[x] = rows[1][n][(4 * x + kg) ^ n]; }
    } else {
        const int64_t so = (arr_row0 + min(i, s.max_blocks - 1)) * D + 4 * kg;
#pragma unroll
        for (int x = 0; x < Q; ++x) { kx[x] = *(const f32x4 *)(kmax + so + 16 * x); kn[x] = *(const f32x4 *)(kmin + so + 16 * x); }
        read_q(wave * 16);
    }
    float acc = reduce == SPECPV_REDUCE_MAX ? -INFINITY : 0.f;
    for (int r0 = wave * 16; r0 < R; r0 += W * 16) {
        if (r0 > wave * 16) read_q(r0);
        f32x4 sx = {0.f, 0.f, 0.f, 0.f}, sn = sx;
#pragma unroll
        for (int x = 0; x < Q; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // the channel-wise bound takes the larger product per channel: q * Kmax where q >= 0, q * Kmin where
                // q < 0 (Kmax >= Kmin), i.e. the sum of two inner products
                const float qx = kind == SPECPV_SCORE_CHANNEL_BOUND ? fmaxf(q[x][e], 0.f) : q[x][e];
                const float qn = kind == SPECPV_SCORE_CHANNEL_BOUND ? fminf(q[x][e], 0.f) : q[x][e];
                sx = __builtin_amdgcn_mfma_f32_16x16x4f32(qx, kx[x][e], sx, 0, 0, 0);
                sn = __builtin_amdgcn_mfma_f32_16x16x4f32(qn, kn[x][e], sn, 0, 0, 0);
            }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int row = r0 + 4 * kg + x;
            const float sv = kind == SPECPV_SCORE_CHANNEL_BOUND ? sx[x] + sn[x] : fmaxf(sx[x], sn[x]);
            if (row < R) {
                if (reduce == SPECPV_REDUCE_MAX) acc = fmaxf(acc, sv);
                else if (reduce == SPECPV_REDUCE_MEAN || row / s.G == last_node) acc += sv;
            }
        }
    }
    const float o16 = __shfl_xor(acc, 16);
    acc = reduce == SPECPV_REDUCE_MAX ? fmaxf(acc, o16) : acc + o16;
    const float o32 = __shfl_xor(acc, 32);
    acc = reduce == SPECPV_REDUCE_MAX ? fmaxf(acc, o32) : acc + o32;
    if (kg == 0) red[wave][n] = acc;
    __syncthreads();
    if (threadIdx.x >= 16) return;
    float out = red[0][n];
    for (int w = 1; w < W && w * 16 < R; ++w) out = reduce == SPECPV_REDUCE_MAX ? fmaxf(out, red[w][n]) : out + red[w][n];
    if (reduce == SPECPV_REDUCE_MEAN) out /= (float)R;
    else if (reduce == SPECPV_REDUCE_LAST) out /= (float)s.G;
    int nb = L > 0 ? (L + s.B - 1) / s.B : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    if (i < nb) scores[((int64_t)b * s.Hkv + g) * s.max_blocks + i] = out;
}

static hipError_t launch_scores_f32(const Shape &s, const void *kmax, const void *kmin, int reduce, int last_node, int kind,
                                    float *scores, hipStream_t st)
{
    const int row_tiles = (s.M * s.G + 15) / 16;
    const int waves = row_tiles == 1 ? 1 : row_tiles < 4 ? 4 : (row_tiles < kScoreF32MaxWaves ? row_tiles : kScoreF32MaxWaves);
    dim3 grid((s.max_blocks + 15) / 16, s.Hkv, s.batch), block(64 * waves);
#define SPECPV_LAUNCH(DD, ST) \
    hipLaunchKernelGGL((score_f32_kernel<DD, ST>), grid, block, 0, st, s, (const float *)kmax, (const float *)kmin, reduce, last_node, kind, scores)
    if (row_tiles == 1) { if (s.D == 128) SPECPV_LAUNCH(128, false); else SPECPV_LAUNCH(64, false); }
    else { if (s.D == 128) SPECPV_LAUNCH(128, true); else SPECPV_LAUNCH(64, true); }
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Selection.  One 256-thread workgroup per (sequence, KV head).
// Every candidate block gets the 64-bit key  (orderable(score) << 32) | ~index,
// so "larger key" means "higher fp32 score, then lower index", and keys are
// unique.  The k-th largest key is found by an MSB-first radix select (8 passes
// of 8 bits, LDS histogram); the kept set is then every candidate with key >=
// that threshold plus the sink and local blocks, written in ascending block
// order through a ballot / popcount compaction.
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long select_key(float score, int idx)
{
    if (score == 0.f) score = 0.f;  // -0 and +0 compare equal: give them one key
    uint32_t u = __float_as_uint(score);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)u << 32) | (unsigned long long)(0xffffffffu - (uint32_t)idx);
}

__global__ __launch_bounds__(256) void topk_kernel(const float *scores, const int32_t *ctx_len, int B,
                                                   int max_blocks, int Hkv, int ns, int nr, int k, int n_row,
                                                   int32_t *sel_idx, int32_t *sel_count)
{
    __shared__ uint32_t hist[256];
    __shared__ uint32_t suffix[257];
    __shared__ unsigned long long sh_prefix;
    __shared__ int sh_krem;
    __shared__ int wave_tot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = blockIdx.x, b = blockIdx.y;
    const int n_sel = ns + k + nr;
    const int L = ctx_len[b];
    int nb = L > 0 ? (L + B - 1) / B : 0;
    if (nb > max_blocks) nb = max_blocks;
    const float *sc = scores + ((int64_t)b * Hkv + g) * max_blocks;
    int32_t *out = sel_idx + ((int64_t)b * Hkv + g) * n_row;   // n_row >= n_sel entries per row
    const bool all = nb <= n_sel;
    const int lo = ns, hi = nb - nr;
    unsigned long long thresh = ~0ull;
    bool any_topk = false;
    if (!all && k > 0) {   // here hi - lo > k
        any_topk = true;
        if (tid == 0) { sh_prefix = 0ull; sh_krem = k; }
        __syncthreads();
        for (int pass = 0; pass < 8; ++pass) {
            const int shift = 56 - 8 * pass;
            const unsigned long long prefix = sh_prefix;
            const int krem = sh_krem;
            hist[tid] = 0;
            __syncthreads();
            for (int i = lo + tid; i < hi; i += 256) {
                const unsigned long long key = select_key(sc[i], i);
                if (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))
                    atomicAdd(&hist[(uint32_t)(key >> shift) & 255u], 1u);
            }
            __syncthreads();
            // suffix[d] = number of matching keys whose digit is >= d
            suffix[tid] = hist[tid];
            if (tid == 0) suffix[256] = 0;
            __syncthreads();
            for (int off = 1; off < 256; off <<= 1) {
                const uint32_t add = (tid + off < 256) ? suffix[tid + off] : 0u;
                __syncthreads();
                suffix[tid] += add;
                __syncthreads();
            }
            if (suffix[tid] >= (uint32_t)krem && suffix[tid + 1] < (uint32_t)krem) {
                sh_prefix = prefix | ((unsigned long long)tid << shift);
                sh_krem = krem - (int)suffix[tid + 1];
            }
            __syncthreads();
        }
        thresh = sh_prefix;
    }
    int base = 0;
    for (int i0 = 0; i0 < nb; i0 += 256) {
        const int i = i0 + tid;
        bool keep = false;
        if (i < nb) {
            keep = all || i < lo || i >= hi;
            if (!keep && any_topk) keep = select_key(sc[i], i) >= thresh;
        }
        const unsigned long long bal = __ballot(keep);
        if (lane == 0) wave_tot[wave] = __popcll(bal);
        __syncthreads();
        int pos = base + __popcll(bal & ((1ull << lane) - 1ull));
        int tot = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) pos += wave_tot[w];
            tot += wave_tot[w];
        }
        if (keep && pos < n_sel) out[pos] = i;
        base += tot;
        __syncthreads();
    }
    if (base > n_sel) base = n_sel;
    for (int c = base + tid; c < n_row; c += 256) out[c] = -1;
    if (tid == 0) sel_count[(int64_t)b * Hkv + g] = base;
}

// Faster selection for lists of up to NT * P blocks: see topk.h.
template <int P, int NT>
__global__ __launch_bounds__(NT) void topk_fast_kernel(const float *scores, const int32_t *ctx_len, int B,
                                                        int max_blocks, int Hkv, TopkArgs a)
{
    __shared__ TopkLds lds;
    topk_fast_body<P, NT, false>(lds, scores, ctx_len, B, max_blocks, Hkv, blockIdx.x, blockIdx.y, a);
}

// Lists of all blocks (list_all_blocks): the selection where its caller keeps no scores and no sequence can have more blocks than
// sink, retrieval and local blocks together.  One trip for the length; what it takes is the launch.
__global__ __launch_bounds__(256) void list_all_kernel(const int32_t *ctx_len, FastDiv div_B, int max_blocks, int Hkv, TopkArgs a)
{
    list_all_blocks(ctx_len, div_B, max_blocks, Hkv, blockIdx.x, blockIdx.y, a, threadIdx.x, 256);
}

hipError_t launch_list_all(const Shape &s, const TopkArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(list_all_kernel, dim3(s.Hkv, s.batch), dim3(256), 0, st, s.ctx_len, make_fastdiv((uint32_t)s.B), s.max_blocks, s.Hkv, a);
    return hipGetLastError();
}

bool score_mfma_supported(const Shape &s, int dtype);
hipError_t launch_scores_mfma(const Shape &s, const void *kmax, const void *kmin, int reduce,
                              int last_node, int kind, float *scores, const TopkArgs *sel,
                              unsigned long long *arrive, hipStream_t st);

hipError_t launch_scores(const Shape &s, int dtype, const void *kmax, const void *kmin,
                         int reduce, int last_node, int kind, float *scores, const TopkArgs *sel,
                         unsigned long long *arrive, hipStream_t st)
{
    if (score_mfma_supported(s, dtype))
        return launch_scores_mfma(s, kmax, kmin, reduce, last_node, kind, scores, sel, arrive, st);
    if (sel) return hipErrorInvalidValue;   // the caller asks score_select_supported() first
    return launch_scores_f32(s, kmax, kmin, reduce, last_node, kind, scores, st);
}

hipError_t launch_topk(const Shape &s, const float *scores, int ns, int nr, int k, int n_row,
                       int32_t *sel_idx, int32_t *sel_count, hipStream_t st)
{
    // Four blocks a thread as long as the workgroup can grow: the time is the length of a thread's chain.  Scoring and
    // selection of one sequence, eight KV heads, 60 nodes at G = 4, before (256 threads, radix passes only; above 4096
    // blocks the kernel that re-reads the scores) and now: 1024 blocks 11.3 -> 10.7 us, 2048 15.8 -> 13.5,
    // 3840 25.9 -> 21.0, 8192 85.8 -> 29.3.
    const dim3 grid(s.Hkv, s.batch);
    const TopkArgs a{ns, nr, k, n_row, sel_idx, sel_count};
#define SPECPV_TOPK(P, NT) \
    hipLaunchKernelGGL((topk_fast_kernel<P, NT>), grid, dim3(NT), 0, st, scores, s.ctx_len, s.B, s.max_blocks, s.Hkv, a)
    if (s.max_blocks <= 1024) SPECPV_TOPK(4, 256);
    else if (s.max_blocks <= 2048) SPECPV_TOPK(4, 512);
    else if (s.max_blocks <= 4096) SPECPV_TOPK(4, 1024);
    else if (s.max_blocks <= 8192) SPECPV_TOPK(8, 1024);
    else if (s.max_blocks <= 16384) SPECPV_TOPK(16, 1024);
    else
        hipLaunchKernelGGL(topk_kernel, grid, dim3(256), 0, st, scores, s.ctx_len, s.B, s.max_blocks, s.Hkv, ns, nr, k, n_row,
                           sel_idx, sel_count);
#undef SPECPV_TOPK
    return hipGetLastError();
}

}  // namespace specpv
