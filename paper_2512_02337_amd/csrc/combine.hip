// Final stage of the verification attention: for each (sequence, node, query
// head) attend over the draft-tree segment (the node itself and its ancestors,
// tree decode of Algorithm 1) on the vector ALU, merge that with the split-KV
// partials of the context part by their log-sum-exp weights, normalise and store.
// Sixteen lanes per output row (a lane owns D / 16 adjacent channels), four query heads of one KV group per wavefront, which
// share the node, its root path and the draft K / V rows; or, PACK, any four rows of the KV head.
// What bounds it is a chain: a trip for the parents, one for the draft rows that they name, and the sums, which a wavefront by
// itself issues at one instruction per eight cycles.  The root path is therefore walked with two instructions a node (a lane
// holds where the path goes on from its node, and that is the node itself where it ends: no test, no branch, no bit set), and
// TWO: two wavefronts per four rows.  One takes the first four nodes of the path, the other the partials and the next four:
// each has its rows under way while it works on what is there, and they meet in one exchange through LDS.  With more than
// sixteen partials those are the longer half, and the first one takes all eight.  Up to 16 partials are requested at once, 16
// bytes per lane each, and a lane works out the weights of its own partials only.  In-kernel stamps at one sequence, 60 nodes,
// 8 KV heads at G = 4, 16 splits, us from entry: path walked 0.5, first half of the tree done 1.6, stored 2.2; with a bit set
// of the path, taken apart again node by node, and the whole tree in one wavefront 1.0, 2.4 and 3.2.  Whole calls in a graph
// of 16 layers 15.37 -> 14.71 us (one card) and 16.69 -> 16.02 (another); fp32, 16 nodes, four launches 18.8 -> 16.3.  A third
// wavefront for the second half took another 0.8 %, and has no place at eight heads a KV head and more.
// (A tree segment on the matrix cores, dense over 32 nodes with a bit mask, was slower: a call 18.6 us with 8 splits.)
#include "combine.h"

namespace specpv {

template <typename T, int D, int NP, bool MULTI, int NB, bool HALF, bool TWO, bool PACK, bool WIDE = false>
__global__ __launch_bounds__(512, MULTI && HALF ? 4 : 1) void combine_kernel(const int32_t *a_parent, const void *a_q, const float *a_po,
                                                    const float *a_pml, int a_M_Mk, int a_Hq, int a_G, int a_nsplit_groups,
                                                    Shape s, Partials part, void *out, float *lse, float scale_log2)
{
    // the leading scalar arguments repeat what the first round of reads needs; they can be preloaded into registers
    s.parent = a_parent; s.q = a_q; s.M = a_M_Mk & 0xff; s.Mk = a_M_Mk >> 8; s.Hq = a_Hq; s.G = a_G;
    part.o = const_cast<float *>(a_po); part.ml = const_cast<float *>(a_pml); part.nsplit = a_nsplit_groups & 0xffff;
    const int groups = a_nsplit_groups >> 16;   // head_groups_code
    __shared__ float4 tree_od[TWO ? 4 * (D / 64) * 64 : 1];
    __shared__ float2 tree_ml[TWO ? 4 * 64 : 1];
    // x = XCD (workgroups go to the XCDs round-robin in linear order), y = node, z = bg / 8: the rows
    // of (sequence, KV head) bg are merged on XCD bg % 8, where the split kernel produced them
    const int bg = (int)blockIdx.z * 8 + (int)blockIdx.x;
    int b;
    if (groups) {   // (nothing here waits for the argument block)
        b = (int)blockIdx.z >> (groups - 1);
        s.Hkv = 4 << groups;
    } else {
        if (bg >= s.batch * s.Hkv) return;
        b = bg / s.Hkv;
    }
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (blockDim.x is read from memory)
    combine_rows<T, D, NP, MULTI, NB, HALF, TWO, PACK, TWO && NB == 8 && !MULTI, WIDE>(s, part, out, lse, scale_log2, bg, b, (int)blockIdx.y, wave, true, tree_od, tree_ml);
}

// Two wavefronts per four rows shorten the chain; one that does both has less to start.  What decides is the partials: with
// more than eight they are the longer half, and two wavefronts are faster however many rows there are; with eight or fewer
// the tree segment is, and two pay only while the chip has room for every workgroup's extra wavefronts at once.  Whole calls
// in graphs as they are planned, one wavefront / two, us, runs of one side within 1 to 3 % (8 KV heads at G = 4 unless stated;
// workgroups = sequences * KV heads * nodes):
//   eight or fewer splits, up to four heads a KV head: 48 workgroups 9.11 / 8.92, 192 10.71 / 10.68 and 12.77 / 12.61, 384 12.36 / 12.42,
//   480 11.13 / 11.23, 960 12.61 / 12.69 and 15.04 / 14.99, 1920 15.75 / 15.73, 3072 22.8 / 23.0, 3840 21.3 / 21.3, 7680 32.9 / 33.3
//   and 48.8 / 49.5: the line at a workgroup per CU;
//   ... more heads, where one workgroup has several fours of rows that share what they read: two KV heads at G = 8, 120 12.4 / 12.1,
//   240 14.5 / 14.0, 480 15.55 / 14.89 and 12.9 / 12.6, 960 15.64 / 15.64, 1920 20.7 / 21.2: two workgroups per CU;
//   packed rows (below), fours of rows: 240 10.30 / 10.23, 600 11.88 / 11.95 and 13.8 / 13.5, 1200 14.53 / 14.50, 1920 22.65 / 22.19, 2400
//   34.5 / 34.8, 3840 23.7 / 24.4, 9600 38.7 / 40.5: eight of them per CU;
//   nine to sixteen: 192 workgroups 12.42 / 12.10 and 16.1 / 15.4, 384 21.5 / 21.3, 480 14.94 / 14.49; G = 5, 192 16.4 / 15.6, 960 33.8 /
//   33.5 (384 15.8 / 16.1); G = 8, 120 14.8 / 14.5, 240 21.8 / 21.4; fp32, 480 and 512 90.8 / 81.6 and 96.1 / 87.1;
//   more, and shares: 32 splits, 96 35.3 / 31.0; full pass in shares, 1920 74 / 61, 7680 205 / 176, at G = 5 184 / 138; fp32, 64
//   splits, 96 69.6 / 62.3; 64 channels, 480 29.9 / 29.5, shares equal.
// Partially verified tokens in front of the tree that the context kernel has left to the tree segment (fp32) make that long
// enough to be worth a wavefront of its own up to one per SIMD: 16 of them, 64 channels, three splits, 480 35.2 / 34.9, two, 512
// 47.9 / 47.9, one, 1024 91.7 / 92.8, 1920 94.6 / 96.7, 3840 100.2 / 104.7; twelve, 128 channels, eight splits, 128 42.9 / 33.7, 480 82.3 /
// 76.6, 1024 197 / 193, 1920 204 / 206.
static bool combine_two_waves(const Shape &s, const Partials &p, bool pack)
{
    if (p.stream || p.nsplit > 8) return true;
    const int64_t rows = (int64_t)s.batch * s.Hkv * s.M, cus = device_cu_count();
    if (pack) return (rows * s.G + 3) / 4 <= 8 * cus;
    const int64_t fours = (s.G + 3) / 4;
    if (s.koff > s.kctx) return rows * fours <= 4 * cus;
    return rows <= (fours > 1 ? 2 : 1) * cus;
}
// PACK: sixteen lanes take whatever row of the KV head is next, node by node, so that a group size that is no multiple of four
// leaves no lanes idle (five heads take 75 workgroups per 60 nodes, not 120 wavefronts of which every second has one row of
// four).  The rows of a wavefront then have paths of their own: the walk goes through the cross-lane unit.  Four layers in a
// graph, fours by node / packed, us: G = 5, 60 nodes, one sequence 61.3 / 56.6 (2K kept) and 78.5 / 73.3 (4K), 16 nodes 45.4 /
// 43.2, four sequences 166.6 / 155.9, sixteen (2K) 281.8 / 252.0; G = 1 with 16 KV heads 56.9 / 50.9; G = 2, four sequences 82.2
// / 76.8; G = 3 55.4 / 51.2.  bf16 only: with fp32 inputs the rows themselves bind.
bool combine_packed(const Shape &s, int dtype) { return dtype == SPECPV_BF16 && s.G % 4 && s.koff <= s.kctx && !draft_rows_wide(s, sizeof(uint16_t)); }

template <typename T, int D>
static void launch_combine_t(const Shape &s, int dtype, Partials p, void *out, float *lse, hipStream_t st)
{
    const bool wide = draft_rows_wide(s, sizeof(T)), pack = combine_packed(s, dtype), two = wide || combine_two_waves(s, p, pack);
    const int groups = head_groups_code(s.Hkv);
    dim3 grid(8, pack ? (s.M * s.G + 3) / 4 : s.M, (s.batch * s.Hkv + 7) / 8), block((two ? 128 : 64) * (pack ? 1 : (s.G + 3) / 4));
    const float scale_log2 = kLog2e / sqrtf((float)s.D);
    // fp16 partials: bf16 at 128 channels; the other element types and head dims have fp32 ones
    constexpr bool kHalf = std::is_same<T, bf16_t>::value && D == 128;
#define SPECPV_LAUNCH(NP, MULTI, NB, HALF, ...)                                                                                  \
        hipLaunchKernelGGL((combine_kernel<T, D, NP, MULTI, NB, HALF, __VA_ARGS__>), grid, block, 0, st, s.parent, s.q, (const float *)p.o, \
                           (const float *)p.ml, s.M | s.Mk << 8, s.Hq, s.G, p.nsplit | groups << 16, s, p, out, lse, scale_log2)
#define SPECPV_LAUNCH_K(NP, MULTI, NB, HALF)                                                                              \
    do {                                                                                                                \
        constexpr bool kPack = std::is_same<T, bf16_t>::value && NB == 8;                                                    \
        constexpr bool kOne = NP <= 8 && !MULTI;   /* (combine_two_waves) */                                               \
        if (kPack && pack) { if (two || !kOne) SPECPV_LAUNCH(NP, MULTI, NB, HALF, true, kPack); else SPECPV_LAUNCH(NP, MULTI, NB, HALF, !kOne, kPack); }  \
        else { if (two || !kOne) SPECPV_LAUNCH(NP, MULTI, NB, HALF, true, false); else SPECPV_LAUNCH(NP, MULTI, NB, HALF, !kOne, false); }  \
    } while (0)
#define SPECPV_LAUNCH_H(NP, MULTI, NB)                                                                                   \
    do {                                                                                                                \
        if (kHalf && p.o_half) SPECPV_LAUNCH_K(NP, MULTI, NB, kHalf); else SPECPV_LAUNCH_K(NP, MULTI, NB, false);        \
    } while (0)
// (the kernels that write fp16 partials have attended the partially verified tokens: kctx == koff)
#define SPECPV_LAUNCH_NP(NP, MULTI)                                                                                      \
    do {                                                                                                                \
        if (s.koff > s.kctx) SPECPV_LAUNCH_K(NP, MULTI, 24, false); else SPECPV_LAUNCH_H(NP, MULTI, 8);                  \
    } while (0)
    if (wide) { if (kHalf && p.o_half) SPECPV_LAUNCH(8, true, 8, kHalf, true, false, true); else SPECPV_LAUNCH(8, true, 8, false, true, false, true); }   // (any count of partials)
    // A pair's shares are few (more wavefronts have room), and where one sequence is long and has most of them there are rows enough to hide
    // their rounds.  Rounds of eight / four, full passes, equal lengths, one long first and last: 16 sequences of 4K, 8 heads 17.5 / 15.2 us
    // (the combine), 16 of 5500, 60 nodes 1 / 0.97, 0.95, 0.97, 64 of 2400, 64 channels 0.93, 0.84, 0.83; few rows, 16 of 2600, one node, 64
    // channels 1.00, 1.07, 1.16, two heads, 64 of 13.6K, 16 nodes 0.99, 1.01, 1.11.
    else if (p.stream && p.stream <= 4 * (int64_t)s.batch * s.Hkv && p.stream <= 64 * (int64_t)s.Hkv && s.M * s.G >= 64) SPECPV_LAUNCH_NP(4, true);
    else if (p.stream) SPECPV_LAUNCH_NP(8, true);
    else if (p.nsplit <= 2) SPECPV_LAUNCH_NP(2, false);
    else if (p.nsplit <= 4) SPECPV_LAUNCH_NP(4, false);
    else if (p.nsplit <= 8) SPECPV_LAUNCH_NP(8, false);
    else if (p.nsplit <= 16) SPECPV_LAUNCH_NP(16, false);
    else SPECPV_LAUNCH_NP(8, true);
#undef SPECPV_LAUNCH_NP
#undef SPECPV_LAUNCH_H
#undef SPECPV_LAUNCH_K
#undef SPECPV_LAUNCH
}

hipError_t launch_combine(const Shape &s, int dtype, Partials p, void *out, float *lse, hipStream_t st)
{
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) launch_combine_t<bf16_t, 128>(s, dtype, p, out, lse, st); else launch_combine_t<bf16_t, 64>(s, dtype, p, out, lse, st);
    } else {
        if (s.D == 128) launch_combine_t<float, 128>(s, dtype, p, out, lse, st); else launch_combine_t<float, 64>(s, dtype, p, out, lse, st);
    }
    return hipGetLastError();
}

}  // namespace specpv
