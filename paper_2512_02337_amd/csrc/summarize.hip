// Block key summaries (Section 3.2, eq. 1), a kernel of their own.  Pure HBM streaming: 5.4 to 6.1 TB/s from 64K tokens of eight KV
// heads on, whatever the block size.  Small blocks had one load a lane under way at a time before (the loop took sixteen passes or
// one): 128K in blocks of 64 / 32 / 16 46.6 / 62.3 / 70.9 us, now 46.3 / 46.7 / 53.1; 64 channels, two sequences of 30011 in blocks of
// 64 / 32 / 16 14.2 / 16.3 / 22.1, now 10.9 / 12.9 / 15.4.
#include "summarize.h"

namespace specpv {

// N > 0: blocks of N passes (summarize_small).  fp32 takes registers for six wavefronts a SIMD and no more: it has fewer to keep, and small
// blocks need the wavefronts (64 channels, 65536 blocks of 2 tokens 21.4 us with five, 19.2 with six; with seven 128 channels spill).
template <typename T, int D, int N>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 6 : 1)
void summarize_kernel(Shape s, int blk_begin, int blk_end, void *kmax, void *kmin)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = blockIdx.y, b = blockIdx.z;
    const int L = s.ctx_len[b];
    if (L <= 0) return;
    int nb = (L + s.B - 1) / s.B;
    if (nb > s.max_blocks) nb = s.max_blocks;
    const int end = (blk_end < 0 || blk_end > nb) ? nb : blk_end;
    constexpr int per = N ? SPECPV_SUM_UNR / N : 1;   // blocks of a wavefront
    const int i = blk_begin + (blockIdx.x * 4 + wave) * per;
    if (i >= end) return;
    if constexpr (N > 0) summarize_small<T, D, N>(s, b, g, i, end, L, kmax, kmin, lane);
    else summarize_block<T, D>(s, b, g, i, L, kmax, kmin, lane);
}

hipError_t launch_summarize(const Shape &s, int dtype, int blk_begin, int blk_end,
                            void *kmax, void *kmin, hipStream_t st)
{
    const int hi = (blk_end < 0 || blk_end > s.max_blocks) ? s.max_blocks : blk_end;
    if (hi <= blk_begin) return hipSuccess;
    // Blocks of two or four passes go by as many to a wavefront as make sixteen loads a lane, where there are more of them than the
    // chip has places for wavefronts: by itself such a block has few bytes under way.  One block / several to a wavefront: blocks of 16,
    // 128 channels, 16384 blocks 15.9 / 15.1 us, 8192 8.4 / 7.8, 4096 4.9 / 5.3, 2048 3.6 / 4.2; 64 channels, 16384 11.8 / 9.6, 4096 4.1 /
    // 5.7.  Blocks of eight passes have enough: 16384 blocks 12.4 / 13.9.  fp32, 128 channels: blocks of 8, 8192 blocks 7.2 / 5.9, 26000
    // 20.5 / 21.3; of 4, 16384 9.9 / 8.2.
    const int rows = 1024 / (s.D * (dtype == SPECPV_BF16 ? 2 : 4)), passes = s.B % rows ? 0 : s.B / rows;
    const bool many = (int64_t)(hi - blk_begin) * s.Hkv * s.batch >= (int64_t)32 * device_cu_count();
    const int N = many && (passes == 2 || passes == 4) ? passes : 0, per = N ? SPECPV_SUM_UNR / N : 1;
    const int waves = (hi - blk_begin + per - 1) / per;
    dim3 grid((waves + 3) / 4, s.Hkv, s.batch), block(256);
#define SPECPV_LAUNCH_N(T, DD, NN) \
    hipLaunchKernelGGL((summarize_kernel<T, DD, NN>), grid, block, 0, st, s, blk_begin, blk_end, kmax, kmin)
#define SPECPV_LAUNCH(T, DD) \
    do { if (N == 2) SPECPV_LAUNCH_N(T, DD, 2); else if (N == 4) SPECPV_LAUNCH_N(T, DD, 4); else SPECPV_LAUNCH_N(T, DD, 0); } while (0)
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) SPECPV_LAUNCH(bf16_t, 128); else SPECPV_LAUNCH(bf16_t, 64);
    } else {
        if (s.D == 128) SPECPV_LAUNCH(float, 128); else SPECPV_LAUNCH(float, 64);
    }
#undef SPECPV_LAUNCH
#undef SPECPV_LAUNCH_N
    return hipGetLastError();
}

}  // namespace specpv
