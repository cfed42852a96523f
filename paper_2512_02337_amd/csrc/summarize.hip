// Block key summaries (Section 3.2, eq. 1), a kernel of their own.  Pure HBM streaming.
#include "summarize.h"

namespace specpv {

template <typename T, int D>
__global__ __launch_bounds__(256) void summarize_kernel(Shape s, int blk_begin, int blk_end,
                                                        void *kmax, void *kmin)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = blockIdx.y, b = blockIdx.z;
    const int L = s.ctx_len[b];
    if (L <= 0) return;
    int nb = (L + s.B - 1) / s.B;
    if (nb > s.max_blocks) nb = s.max_blocks;
    const int end = (blk_end < 0 || blk_end > nb) ? nb : blk_end;
    const int i = blk_begin + blockIdx.x * 4 + wave;
    if (i < end) summarize_block<T, D>(s, b, g, i, L, kmax, kmin, lane);
}

hipError_t launch_summarize(const Shape &s, int dtype, int blk_begin, int blk_end,
                            void *kmax, void *kmin, hipStream_t st)
{
    const int hi = (blk_end < 0 || blk_end > s.max_blocks) ? s.max_blocks : blk_end;
    if (hi <= blk_begin) return hipSuccess;
    dim3 grid((hi - blk_begin + 3) / 4, s.Hkv, s.batch), block(256);
#define SPECPV_LAUNCH(T, DD) \
    hipLaunchKernelGGL((summarize_kernel<T, DD>), grid, block, 0, st, s, blk_begin, blk_end, kmax, kmin)
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) SPECPV_LAUNCH(bf16_t, 128); else SPECPV_LAUNCH(bf16_t, 64);
    } else {
        if (s.D == 128) SPECPV_LAUNCH(float, 128); else SPECPV_LAUNCH(float, 64);
    }
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

}  // namespace specpv
