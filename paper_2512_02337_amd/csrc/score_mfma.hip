// Block scoring (Section 3.2, eq. 2 and eq. 3; optionally the channel-wise bound) on the matrix
// cores for bf16, head dims 128 and 64.
//
// Per KV head the scores are max(Q . Kmax^T, Q . Kmin^T) reduced over the M*G query rows:
// two [rows x D] x [D x blocks] products.  A workgroup owns one or more tiles of 32 blocks, whose summary rows go into
// LDS once, and spreads the query rows over its wavefronts, 32 rows each, held in registers over all its tiles: query rows
// are the A operand (lane = row), the summaries of a tile the B operands (lane = block), so each lane ends up with 16
// rows of ONE block; the element-wise max of the two accumulators and the reduction over rows (mean / max / rows of one
// node) are lane-local.  All reads of a workgroup are issued at once (one round trip); the wavefronts' partial results
// meet in LDS.  The sum order is the same for every block, so identical blocks get bit-identical scores wherever they sit.
//
// What bounds it: the round trip, then 32 matrix instructions per SIMD and tile (1024 cycles at eight wavefronts).  The
// operand reads stand between the matrix instructions of one assembly statement (score_products): left to the compiler,
// at the 128 registers that two workgroups of eight wavefronts on a CU leave, a tile was sixteen reads one after the
// other, each waited for.
//
// The same launch can do the selection as well: every workgroup of a (sequence, KV head)
// counts itself in when its scores are stored, and the one that finds itself last runs the
// top-k over the scores of all of them (no workgroup waits for another).
#include "score.h"
#include "topk.h"

namespace specpv {

// P = 0: scores only.  P = 4, 8, 16: scores, then the selection over lists of up to 256 * P blocks
// by the last workgroup of each (sequence, KV head) to get here (workgroups of at least 256 threads).
// Arrival is counted on two levels, because agent-scope atomics on one address are executed one
// after the other (64 workgroups on one word: + 4.4 us; 8 + 8: + 0.9 us): the workgroups of a
// (sequence, KV head) are dealt to eight groups by their number % 8, the last of a group counts
// the group in on the pair's own word.  Pair p = b * Hkv + g owns the words arrive[(9 p + i) * wstride],
// i = 0 for the pair, 1 + j for group j; all are zero before the launch, and whoever finds a count
// complete sets it back to zero.
template <int D, bool BOUND, int P, bool STAGED>
__global__ __launch_bounds__(64 * kScoreMaxWaves) void score_mfma_kernel(Shape s, ScoreArgs a, TopkArgs ta, unsigned long long *arrive, int wstride)
{
    // every argument in one trip to memory; left to itself the compiler asks for each where it is first used
    asm volatile("" :: "s"(s.M), "s"(s.G), "s"(s.Hq), "s"(s.Hkv), "s"(s.B), "s"(s.batch), "s"(s.max_blocks), "s"(s.q), "s"(s.ctx_len),
                 "s"(a.kmax), "s"(a.kmin), "s"(a.scores), "s"(a.reduce), "s"(a.last_node), "s"(a.row0), "s"(a.rows), "s"(a.sums), "s"(a.tiles));
    asm volatile("" :: "s"(a.waves), "s"(a.groups), "s"(a.by_xcd), "s"(a.div_G.mul), "s"(a.div_G.shift), "s"(a.div_G.d),
                 "s"(a.div_B.mul), "s"(a.div_B.shift), "s"(a.div_B.d));
    if constexpr (P != 0)
        asm volatile("" :: "s"(arrive), "s"(wstride), "s"(ta.ns), "s"(ta.nr), "s"(ta.k), "s"(ta.n_row), "s"(ta.sel_idx), "s"(ta.sel_count));
    const int group = a.by_xcd ? (int)blockIdx.x >> 3 : (int)blockIdx.x;
    const int g = a.by_xcd ? (int)blockIdx.y * 8 + ((int)blockIdx.x & 7) : (int)blockIdx.y, b = blockIdx.z;
    score_tiles<D, BOUND, P != 0, STAGED>(s, a, group, g, b);
    if constexpr (P != 0) {
        __shared__ TopkLds lds;
        __shared__ int is_last;
        // A store is counted as done (vmcnt) when it has been acknowledged at the scope it was issued
        // with; the counters below are only touched after that, and the last workgroup only reads the
        // scores after it has seen the full counts: no further fence is needed.
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wavefront's score stores are out
        __syncthreads();                      // ... and so are everybody else's
        if (threadIdx.x == 0) {
            unsigned long long *pair = arrive + ((int64_t)b * s.Hkv + g) * 9 * wstride;
            const int j = group & 7;
            unsigned long long *word = pair + (int64_t)(1 + j) * wstride;
            const unsigned long long n_j = (unsigned long long)((a.groups - j + 7) >> 3);     // workgroups with number % 8 == j
            const unsigned long long n_groups = a.groups < 8 ? a.groups : 8;
            bool last = false;
            if (__hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1ull == n_j) {
                __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__hip_atomic_fetch_add(pair, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1ull == n_groups) {
                    __hip_atomic_store(pair, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    last = true;
                }
            }
            is_last = last ? 1 : 0;
        }
        __syncthreads();
        if (!is_last) return;
        topk_fast_body<P, 256, true>(lds, a.scores, s.ctx_len, s.B, s.max_blocks, s.Hkv, g, b, ta);
    }
}

template <int D>
__global__ __launch_bounds__(64 * kScoreMaxWaves) void score_stream_kernel(Shape s, ScoreArgs a)
{
    const int w = a.by_xcd ? (int)blockIdx.x >> 3 : (int)blockIdx.x;   // of the KV head's
    const int g = a.by_xcd ? (int)blockIdx.y * 8 + ((int)blockIdx.x & 7) : (int)blockIdx.y;
    score_stream<D>(s, a, ScoreStream(s, a, w), g);
}

bool score_mfma_supported(const Shape &s, int dtype) { return dtype == SPECPV_BF16; }

bool score_select_supported(const Shape &s, int dtype)
{
    // the selection needs 256 threads, lists of at most 4096 blocks and nine arrival words per (sequence, KV head)
    const int row_tiles = (s.M * s.G + 31) / 32;
    return score_mfma_supported(s, dtype) && row_tiles >= 4 && s.max_blocks <= 256 * 16 &&
           (size_t)s.batch * s.Hkv * 9 * sizeof(unsigned long long) <= kArriveBytes;
}

ScoreArgs score_plan(const Shape &s, const void *kmax, const void *kmin, int reduce, int last_node, float *scores, bool keep_all)
{
    // one wavefront per block of 32 query rows.  `last` reads the rows of one node: the wavefronts whose blocks they lie in
    // (the selection in the same launch needs its 256 threads, so there all of them stay)
    const int R = s.M * s.G;
    const bool one_node = reduce == SPECPV_REDUCE_LAST && !keep_all;
    ScoreArgs a = {};
    a.kmax = (const uint16_t *)kmax; a.kmin = (const uint16_t *)kmin; a.scores = scores;
    a.reduce = reduce; a.last_node = last_node;
    a.row0 = one_node ? last_node * s.G / 32 * 32 : 0;
    a.rows = one_node ? (last_node + 1) * s.G : R;
    const int blocks32 = (a.rows - a.row0 + 31) / 32;
    const int64_t tiles1 = (s.max_blocks + 31) / 32, total = tiles1 * s.Hkv * s.batch, cus = device_cu_count();
    // 128 registers leave a CU 16 wavefronts.  More than eight blocks of rows fill it with one workgroup, which then stands
    // still for its round trip; where there are tiles enough, four wavefronts take them in turns and four workgroups share a
    // CU.  Scoring + selection per call at G = 5, 60 nodes, 8 KV heads, in turns of four / of five / ten wavefronts: 32K + 64K +
    // 96K + 128K 24.2 / 22.1 / 24.7 us, 8 x 64K 25.4 / 29.1 / 27.2; eight blocks of rows, 60K in blocks of 16: 21.0 in turns
    // of four, 18.9 with eight wavefronts.
    int waves = blocks32 < kScoreMaxWaves ? blocks32 : kScoreMaxWaves;
    if (blocks32 > 8 && blocks32 <= kScoreSums && total > cus && !keep_all) {
        const int turns = (blocks32 + 3) / 4;
        waves = (blocks32 + turns - 1) / turns;
    }
    // Tiles of a workgroup: as many as give every workgroup a place on the chip at once, up to what LDS holds.  Scoring +
    // selection, one tile everywhere / by this rule / four: 128K 14.6 / 14.6 / 15.8 us, 60K in blocks of 16 22.8 / 18.8 /
    // 19.2, 16 x 32K 33.1 / 23.8 / 23.8; before (reads left to the compiler, one tile up to 8 workgroups a CU): 15.3, 23.7, 27.5.
    const int per_cu = 16 / waves < 8 ? 16 / waves : 8, most = score_most_tiles(waves);
    int64_t T = (total + per_cu * cus - 1) / (per_cu * cus);
    T = T < 1 ? 1 : (T > most ? most : T);
    a.waves = waves;
    a.sums = blocks32 < kScoreSums ? blocks32 : kScoreSums;
    // Query rows through LDS where that costs no workgroup its place on a CU, and for more than four wavefronts (three sequences of
    // 128K, 30 nodes, four wavefronts of two tiles 9.5 / 9.9 us): 60K in blocks of 16 10.9 / 10.1 us, 128K 8.0 / 7.0, 16K 6.1 / 5.4,
    // 45 nodes, six wavefronts, 128K 7.3 / 6.4, 64K at G = 5, ten, 6.9 / 6.0 (scoring alone, kernel trace).
    auto fit = [&](int staged_waves) { const int n = (int)(160 * 1024 / score_lds(s.D, (int)T, a.sums, staged_waves)); return n < per_cu ? n : per_cu; };
    // (Two tiles staged rather than three that leave no room to stage, as at 128 channels and seven or eight wavefronts: 1536 tiles 16.3 us,
    // 13.5 so.  Where three staged ones fit they stay: scoring + selection of 1100 / 1300 / 1536 tiles, cut to two / three, six
    // wavefronts 15.9 / 14.8, 16.2 / 14.9, 17.1 / 15.7; 64 channels, eight 12.6 / 12.3, 13.0 / 12.6, 13.5 / 13.0; five, 2304 tiles 16.2 / 14.6.)
    if (T == 3 && waves > 4 && waves <= 8 && !keep_all && fit(waves) < fit(0)) T = 2;
    a.tiles = (int)T;
    a.groups = (int)((tiles1 + T - 1) / T);
    a.staged = !keep_all && waves > 4 && fit(waves) == fit(0);
    a.by_xcd = s.Hkv % 8 == 0;
    a.div_G = make_fastdiv((uint32_t)s.G);
    a.div_B = make_fastdiv((uint32_t)s.B);
    return a;
}

// Whether the scores go by streams (score_stream), and their tiles and workgroups: where a workgroup for every place on the chip has a
// group of tiles or more.  One block of query rows is a read of the summaries and little else, and is faster with all of them under way
// at once.  Batches that have several groups to a workgroup go by streams where these are dealt without much loss (equal lengths fill 72 %
// of the rounds; 64 channels, whose tiles cost less than what is lost, 85 %) and where workgroups are left to deal: two to a sequence,
// with 64 channels four.  Scores and selection, tiles at once / by streams, us, equal lengths, 1 / n to n / n, one long and the others a
// sixteenth: 8 KV heads, 60 nodes, G = 5, 16 x 2048 blocks 71 / 62, 45 / 43, 23 / 17, 8 x 1024 24 / 23, 20 / 16, 19 / 12, G = 4, 16 x 2048 57
// / 47, 37 / 30, 23 / 15, 4 x 1024, 78 nodes at G = 5 22 / 16, 20 / 14, 19 / 13.  Beyond the lines: 32 x 824, 37 nodes at G = 8 (as many
// workgroups as sequences) 59 / 51, 38 / 44, 19 / 40; 17 x 512, 60 nodes at G = 5 27 / 29, 21 / 22 (equal lengths fill 40 %); 64 channels,
// 37 nodes, 32 x 597 18.9 / 19.5, 14.6 / 16.2, 24 x 114 9.2 / 10.6, 12 x 554 at G = 8 14.0 / 15.1; one node (one block), 4 x 2048 12.9 / 14.0.
// Of 160 random shapes the slowest of those and of one long last is 0.91 of tiles at once in the mean.
static bool score_stream_plan(const Shape &s, ScoreArgs &a)
{
    const int blocks32 = (a.rows - a.row0 + 31) / 32;
    if (blocks32 < 2 || blocks32 > kScoreMaxWaves) return false;
    const int64_t tiles1 = (s.max_blocks + 31) / 32, pairs = (int64_t)s.Hkv * s.batch, cus = device_cu_count();
    const int T = (blocks32 * kScoreStage + score_tile_bytes(s.D) - 1) / score_tile_bytes(s.D);   // room for the query rows' way
    const int64_t fit = (int64_t)(160 * 1024 / score_stream_lds(s.D, T, blocks32)), per_cu = 16 / blocks32 < fit ? 16 / blocks32 : fit;
    if (per_cu < 1) return false;
    const int64_t phases = (tiles1 + T - 1) / T, groups = per_cu * cus / s.Hkv;   // of the longest sequence; workgroups of a KV head
    if (s.batch > 64 || groups < s.batch || phases < groups / s.batch) return false;   // (a lane a sequence: ScoreStream)
    const int64_t rounds = (phases + groups / s.batch - 1) / (groups / s.batch);
    if (s.batch > 1) {
        if (s.D == 64 && groups < 4 * (int64_t)s.batch) return false;
        if (rounds > 1 && (groups < 2 * (int64_t)s.batch || (double)(phases * pairs) < (s.D == 128 ? 0.72 : 0.85) * (double)(rounds * per_cu * cus))) return false;
    }
    a.rounds = (int)rounds;
    a.div_tiles = make_fastdiv((uint32_t)T);
    a.waves = a.sums = blocks32;
    a.tiles = T;
    a.groups = (int)groups;
    a.staged = 0;
    return true;
}

// sel != nullptr: the selection runs in the same launch (score_select_supported(s, dtype) holds and
// arrive points to zeroed words)
hipError_t launch_scores_mfma(const Shape &s, const void *kmax, const void *kmin, int reduce,
                              int last_node, int kind, float *scores, const TopkArgs *sel,
                              unsigned long long *arrive, hipStream_t st)
{
    ScoreArgs a = score_plan(s, kmax, kmin, reduce, last_node, scores, sel != nullptr);
    if (!sel && kind == SPECPV_SCORE_EQ2 && score_stream_plan(s, a)) {
        const dim3 grid(a.by_xcd ? a.groups * 8 : a.groups, a.by_xcd ? s.Hkv / 8 : s.Hkv), block(64 * a.waves);
#define SPECPV_LAUNCH(DD)                                                                                                       \
        do {                                                                                                                    \
            static PerDeviceOnce once;                                                                                          \
            auto kern = score_stream_kernel<DD>;                                                                                \
            const hipError_t e0 = once.run([&] { return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); }); \
            if (e0 != hipSuccess) return e0;                                                                                    \
            hipLaunchKernelGGL(kern, grid, block, score_stream_lds(DD, a.tiles, a.sums), st, s, a);                             \
        } while (0)
        if (s.D == 128) SPECPV_LAUNCH(128); else SPECPV_LAUNCH(64);
#undef SPECPV_LAUNCH
        return hipGetLastError();
    }
    const int waves = a.waves;
    const dim3 grid(a.by_xcd ? a.groups * 8 : a.groups, a.by_xcd ? s.Hkv / 8 : s.Hkv, s.batch), block(64 * waves);
    const size_t lds = score_lds(s.D, a.tiles, a.sums, a.staged ? waves : 0);
    const int P = !sel ? 0 : (s.max_blocks <= 256 * 4 ? 4 : (s.max_blocks <= 256 * 8 ? 8 : 16));
    const TopkArgs ta = sel ? *sel : TopkArgs{0, 0, 0, 0, nullptr, nullptr};
    // every arrival word on a 128-byte line of its own where the region is large enough for that
    const int wstride = (size_t)s.batch * s.Hkv * 9 * 128 <= kArriveBytes ? 16 : 1;
#define SPECPV_LAUNCH(DD, BOUND, PP, ST)                                                                                        \
    do {                                                                                                                    \
        static PerDeviceOnce once;   /* one per kernel instantiation */                                                    \
        auto kern = score_mfma_kernel<DD, BOUND, PP, ST>;                                                                       \
        const hipError_t e0 = once.run([&] { return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)score_lds(DD, kScoreMostTiles, kScoreSums, kScoreMaxWaves)); }); \
        if (e0 != hipSuccess) return e0;                                                                                    \
        hipLaunchKernelGGL(kern, grid, block, lds, st, s, a, ta, arrive, wstride);                                          \
    } while (0)
#define SPECPV_LAUNCH_P(DD, BOUND)                                                                                          \
    do { if (P == 0 && a.staged) SPECPV_LAUNCH(DD, BOUND, 0, true); else if (P == 0) SPECPV_LAUNCH(DD, BOUND, 0, false); else if (P == 4) SPECPV_LAUNCH(DD, BOUND, 4, false);                              \
         else if (P == 8) SPECPV_LAUNCH(DD, BOUND, 8, false); else SPECPV_LAUNCH(DD, BOUND, 16, false); } while (0)
    if (s.D == 128) { if (kind == SPECPV_SCORE_CHANNEL_BOUND) SPECPV_LAUNCH_P(128, true); else SPECPV_LAUNCH_P(128, false); }
    else { if (kind == SPECPV_SCORE_CHANNEL_BOUND) SPECPV_LAUNCH_P(64, true); else SPECPV_LAUNCH_P(64, false); }
#undef SPECPV_LAUNCH_P
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

}  // namespace specpv
