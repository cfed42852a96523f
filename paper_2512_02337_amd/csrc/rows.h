// Row arithmetic that needs no GPU to be checked.
#pragma once
#ifdef __HIPCC__
#define SPECPV_ROWS __host__ __device__ __forceinline__
#else
#define SPECPV_ROWS static inline
#endif

namespace specpv {

// The row that a wavefront reads for row t of blocks of B rows, of which `end` is the first that it has no business with, in a sequence
// of L tokens: the length lives on the device and may lie beyond the last block that the cache has.  end >= 1, L >= 1.
SPECPV_ROWS int row_below(int t, int L, int end, int B)
{
    const int rows = end * B;   // (a cache has no more than 2^30)
    const int last = (L < rows ? L : rows) - 1;
    return t < last ? t : last;
}

}  // namespace specpv
