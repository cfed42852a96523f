// What a full verification does behind its context attention, in one launch: the merge of the partials (combine.hip) and the
// scores of the blocks (score_mfma.hip).  Neither needs the other.  The merge is a chain of round trips with few wavefronts a
// CU and no matrix work; the scores are a round trip and then matrix work: side by side the shorter one costs nothing, and
// one launch less is waited for.  The grid goes by eights of (sequence, KV head) pairs: of each the first workgroups score (the
// selection that follows waits for all of them), the others merge, as many rows each as a scoring workgroup has wavefronts for.
// Results are those of the two launches to the bit: the same functions on the same pieces.  (Times: launch_refresh_tail.  What is
// left is bound by the longer of the two, three round trips and the partials' 8 to 20 MB, and by the start of the launch.)
#include "combine.h"
#include "score.h"
#include "topk.h"

namespace specpv {

struct TailArgs {
    int score_rows;   // of the grid's y in each z: workgroups that score (all: and one that lists)
    int n_score;      // scoring workgroups
    int rows, units;  // query rows (PACK: fours of rows) of a KV head; of a workgroup
    int n_bg;
    int all;          // every block is listed, by a workgroup of each KV head in front of the others
    FastDiv div_groups, div_heads, div_hkv;   // by the scoring workgroups of a KV head, by KV heads (by_xcd: by eights of them), by KV heads
};

// SHARED (combine_rows) is not needed for the bits and takes registers that two scoring workgroups on a CU do not leave.
template <int D, int NP, bool MULTI, bool PACK, bool STAGED>
__global__ __launch_bounds__(64 * kScoreMaxWaves) void refresh_tail_kernel(const int32_t *a_parent, const void *a_q, const float *a_po, const float *a_pml,
                                                                           Shape s, Partials part, void *out, float *lse, float scale_log2, ScoreArgs a, TailArgs t, TopkArgs lists)
{
    extern __shared__ __attribute__((aligned(1024))) char tail_smem[];
    s.parent = a_parent; s.q = a_q;
    part.o = const_cast<float *>(a_po); part.ml = const_cast<float *>(a_pml);
    if ((int)blockIdx.y < t.score_rows) {
        if (t.all && blockIdx.y == 0) {
            const int bg = (int)blockIdx.z * 8 + (int)blockIdx.x;
            if (bg >= t.n_bg) return;
            const int b = (int)t.div_hkv.div((uint32_t)bg);
            list_all_blocks(s.ctx_len, a.div_B, s.max_blocks, s.Hkv, bg - b * s.Hkv, b, lists, threadIdx.x, blockDim.x);
            return;
        }
        const int row = (int)blockIdx.z * (t.score_rows - t.all) + (int)blockIdx.y - t.all;
        int group, g, b;
        if (a.by_xcd) {   // KV head g on XCD g % 8
            if (row * 8 >= t.n_score) return;
            const int hb = (int)t.div_groups.div((uint32_t)row);
            group = row - hb * a.groups;
            b = (int)t.div_heads.div((uint32_t)hb);
            g = (hb - b * (s.Hkv >> 3)) * 8 + (int)blockIdx.x;
        } else {
            const int u = row * 8 + (int)blockIdx.x;
            if (u >= t.n_score) return;
            const int hb = (int)t.div_groups.div((uint32_t)u);
            group = u - hb * a.groups;
            b = (int)t.div_heads.div((uint32_t)hb);
            g = hb - b * s.Hkv;
        }
        score_tiles<D, false, false, STAGED>(s, a, group, g, b);
        return;
    }
    const int bg = (int)blockIdx.z * 8 + (int)blockIdx.x;
    if (bg >= t.n_bg) return;
    const int b = (int)t.div_hkv.div((uint32_t)bg);
    const int per_row = PACK ? 1 : (s.G + 3) >> 2;   // fours of heads; two wavefronts each
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int unit = wave, first = 0;
    if (per_row == 1) {
        unit = wave >> 1;
        first = unit * 2;
    } else {
        unit = 0;
        while (first + 2 * per_row <= wave) { first += 2 * per_row; ++unit; }
    }
    if (unit >= t.units) {   // wavefronts left over
        __syncthreads();
        return;
    }
    const int row = ((int)blockIdx.y - t.score_rows) * t.units + unit;
    float4 *tree_od = (float4 *)tail_smem + unit * per_row * (D / 64) * 64;
    float2 *tree_ml = (float2 *)((float4 *)tail_smem + t.units * per_row * (D / 64) * 64) + unit * per_row * 64;
    combine_rows<bf16_t, D, NP, MULTI, 8, D == 128, true, PACK, false>(s, part, out, lse, scale_log2, bg, b, min(row, t.rows - 1), wave - first, row < t.rows, tree_od, tree_ml);
}

bool refresh_tail_supported(const Shape &s, int dtype, const Partials &p, int kind)
{
    // (the grid's y counts a KV head's scoring workgroups and its rows, z eights of KV heads)
    return dtype == SPECPV_BF16 && kind == SPECPV_SCORE_EQ2 && s.koff <= s.kctx && (p.o_half != 0) == (s.D == 128) &&
           s.max_blocks <= 32 * 60000 && (int64_t)s.batch * s.Hkv <= 8 * 65535 && !draft_rows_wide(s, sizeof(uint16_t));
}

// Where the merge alone has so many fours of rows for every CU and there is little to score, the merge's workgroups pay more for the LDS and
// the wavefronts of the scoring ones than a launch costs; how many, follows from how long a four takes.  Whole refreshes of 150 shapes (1 to 32
// sequences) with up to 4096 blocks of 32 query rows times tiles of 32 blocks to score, apart / together, equal lengths, 1 / n to n / n, one long, means
// by fours a CU.  128 channels, splits: 6 to 8 1.01, 1.02, 1.03; 8 to 11 0.98, 0.98, 1.01 (4 of 3480 by quarters, 66 nodes at G = 4 43.8 / 46.6 us);
// 14 to 18 0.93, 0.93, 0.96.  Shares, whose places are found by the lengths: 8 to 14 1.00, 1.00, 1.04; 14 to 18 0.95, 0.95, 0.97; beyond 24 0.91,
// 0.92, 0.93.  64 channels, whose partials are twice the bytes: 14 to 18 1.01, 1.02, 1.02; 18 to 24 0.99, 1.00, 0.99; beyond 0.92, 0.92, 0.89.  With more to
// score, 4480 / 4800 / 5120 / 7680: 0.92 / 0.99, 0.99 / 0.99, 0.96 / 0.99, 1.01 / 1.01; 20480: tail 28.2 / 10.9 + 24.5 us.
bool refresh_tail_pays(const Shape &s, const Partials &p, int reduce, int last_node)
{
    const bool pack = combine_packed(s, SPECPV_BF16);
    const ScoreArgs a = score_plan(s, nullptr, nullptr, reduce, last_node, nullptr, false);
    const int64_t pairs = (int64_t)s.batch * s.Hkv, fours = pairs * (pack ? (s.M * s.G + 3) / 4 : s.M * ((s.G + 3) / 4));
    const int64_t line = s.D == 64 ? 18 : (p.stream ? 14 : 8);
    return fours < line * (int64_t)device_cu_count() || (int64_t)((a.rows - a.row0 + 31) / 32) * ((s.max_blocks + 31) / 32) * pairs > 4096;
}

hipError_t launch_refresh_tail(const Shape &s, Partials p, void *out, float *lse, const void *kmax, const void *kmin, int reduce, int last_node,
                               float *scores, const TopkArgs *all, hipStream_t st)
{
    const bool pack = combine_packed(s, SPECPV_BF16);
    ScoreArgs a = score_plan(s, kmax, kmin, reduce, last_node, scores, false);
    const int per_row = pack ? 1 : (s.G + 3) / 4;
    if (a.waves < 2 * per_row || !scores) a.waves = 2 * per_row;   // (the others find no rows to score)
    TailArgs t = {};
    t.units = a.waves / (2 * per_row);
    t.rows = pack ? (s.M * s.G + 3) / 4 : s.M;
    t.n_bg = s.batch * s.Hkv;
    const int64_t z = (t.n_bg + 7) / 8, merging = 8 * z * ((t.rows + t.units - 1) / t.units);
    // Tiles of a scoring workgroup: as many as leave every workgroup a CU to itself, or all that fit (score_plan fills the chip
    // with scoring workgroups, and the merging ones would wait for them).  Merge, scores and selection of a refresh, us, apart /
    // one, two, four tiles: 8 KV heads at G = 4, 60 nodes, 8K 14.5 / 9.8 / 11.0 / 13.4, 64K 19.5 / 15.8 / 13.9 / 17.3, 128K 22.2 /
    // 19.9 / 17.5 / 17.5; 78 nodes, 64K 26.8 / 23.0 / 18.5 / 18.6 (three); four sequences of 32K in blocks of 32 29.0 / 31.5 / 27.3
    // / 26.5; 32K + 64K + 96K + 128K at G = 5 39.5 / 34.5 / 29.0 (at most two fit there).
    {
        const int64_t tiles1 = (s.max_blocks + 31) / 32, total = tiles1 * t.n_bg, room = device_cu_count() - merging;
        const int64_t most = score_most_tiles(a.waves), T = room > 0 ? (total + room - 1) / room : most;
        a.tiles = (int)(T < 1 ? 1 : (T > most ? most : T));
        a.groups = (int)((tiles1 + a.tiles - 1) / a.tiles);
        // (what a CU has to itself may as well take the LDS for it: 16K 11.1 -> 9.4 us, 64K 14.9 -> 14.3)
        a.staged = a.waves > 4 && room > 0 && (int64_t)a.groups * t.n_bg <= room;
    }
    if (!scores) { a.groups = a.tiles = a.sums = a.staged = 0; }
    const int64_t n_score = (int64_t)a.groups * s.Hkv * s.batch;
    t.n_score = (int)n_score;
    t.all = all ? 1 : 0;
    t.score_rows = (int)(((n_score + 7) / 8 + z - 1) / z) + t.all;
    t.div_groups = make_fastdiv((uint32_t)(a.groups > 0 ? a.groups : 1));
    t.div_heads = make_fastdiv((uint32_t)(a.by_xcd ? s.Hkv / 8 : s.Hkv));
    t.div_hkv = make_fastdiv((uint32_t)s.Hkv);
    const dim3 grid(8, t.score_rows + (t.rows + t.units - 1) / t.units, (unsigned)z), block(64 * a.waves);
    if (n_score > (int64_t)1 << 30 || grid.y > 65535u) return hipErrorInvalidConfiguration;   // (not with refresh_tail_supported)
    const size_t meet = (size_t)t.units * per_row * 64 * (s.D / 64 * sizeof(float4) + sizeof(float2));
    const size_t scoring = score_lds(s.D, a.tiles, a.sums, a.staged ? a.waves : 0), lds = scoring > meet ? scoring : meet;
    const float scale_log2 = kLog2e / sqrtf((float)s.D);
#define SPECPV_LAUNCH_K(DD, NP, MULTI, PACK, ST)                                                                               \
    do {                                                                                                                    \
        static PerDeviceOnce once;   /* one per kernel instantiation */                                                    \
        auto kern = refresh_tail_kernel<DD, NP, MULTI, PACK, ST>;                                                               \
        const hipError_t e0 = once.run([&] { return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)score_lds(DD, kScoreMostTiles, kScoreSums, kScoreMaxWaves)); }); \
        if (e0 != hipSuccess) return e0;                                                                                    \
        hipLaunchKernelGGL(kern, grid, block, lds, st, s.parent, s.q, (const float *)p.o, (const float *)p.ml, s, p, out, lse, scale_log2, a, t, all ? *all : TopkArgs{}); \
    } while (0)
#define SPECPV_LAUNCH(DD, NP, MULTI, PACK)                                                                                  \
    do { if (a.staged) SPECPV_LAUNCH_K(DD, NP, MULTI, PACK, true); else SPECPV_LAUNCH_K(DD, NP, MULTI, PACK, false); } while (0)
#define SPECPV_LAUNCH_NP(DD, PACK)                                                                                          \
    do {                                                                                                                    \
        if (p.stream || p.nsplit > 16) SPECPV_LAUNCH(DD, 8, true, PACK);                                                     \
        else if (p.nsplit <= 2) SPECPV_LAUNCH(DD, 2, false, PACK);                                                           \
        else if (p.nsplit <= 4) SPECPV_LAUNCH(DD, 4, false, PACK);                                                           \
        else if (p.nsplit <= 8) SPECPV_LAUNCH(DD, 8, false, PACK);                                                           \
        else SPECPV_LAUNCH(DD, 16, false, PACK);                                                                             \
    } while (0)
    if (s.D == 128) { if (pack) SPECPV_LAUNCH_NP(128, true); else SPECPV_LAUNCH_NP(128, false); }
    else { if (pack) SPECPV_LAUNCH_NP(64, true); else SPECPV_LAUNCH_NP(64, false); }
#undef SPECPV_LAUNCH_NP
#undef SPECPV_LAUNCH
#undef SPECPV_LAUNCH_K
    return hipGetLastError();
}

}  // namespace specpv
