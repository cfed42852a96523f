// C ABI of libspecpv: argument validation, workspace layout, split planning and
// the launch sequences of the four calls.  No kernels live here.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "internal.h"

namespace specpv {

static thread_local char g_hip_err[256] = "";

static int fail_hip(hipError_t e)
{
    snprintf(g_hip_err, sizeof(g_hip_err), "%s: %s", hipGetErrorName(e), hipGetErrorString(e));
    return SPECPV_EHIP;
}

int device_cu_count()
{
    // per device, filled on first use; a racing first call writes the same value
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    const bool tracked = dev >= 0 && dev < 64;
    if (tracked) {
        const int c = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
        if (c > 0) return c;
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
    if (tracked) __atomic_store_n(&cached[dev], cus, __ATOMIC_RELAXED);
    return cus;
}

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

static int check_kv(const specpv_kv *kv)
{
    if (!kv || !kv->k || !kv->v || !kv->ctx_len) return SPECPV_EINVAL;
    if (kv->dtype != SPECPV_F32 && kv->dtype != SPECPV_BF16) return SPECPV_EINVAL;
    if (kv->head_dim != 64 && kv->head_dim != 128) return SPECPV_EINVAL;
    if (kv->batch < 1 || kv->n_kv_heads < 1 || kv->block_size < 1 || kv->max_blocks < 1) return SPECPV_EINVAL;
    const int64_t vec = kv->dtype == SPECPV_BF16 ? 8 : 4;  // elements per 16 bytes
    if (kv->stride_t < kv->head_dim || kv->stride_t % vec || kv->stride_h % vec || kv->stride_b % vec)
        return SPECPV_EINVAL;
    if (kv->stride_h < 0 || kv->stride_b < 0) return SPECPV_EINVAL;
    if (((uintptr_t)kv->k | (uintptr_t)kv->v) & 15) return SPECPV_EINVAL;
    if ((int64_t)kv->max_blocks * kv->block_size > ((int64_t)1 << 30)) return SPECPV_ELIMIT;
    return SPECPV_OK;
}

static int check_tree(const specpv_kv *kv, const specpv_tree *tree, bool need_draft_kv)
{
    if (!tree || !tree->q) return SPECPV_EINVAL;
    if (tree->M < 1 || tree->n_q_heads < 1) return SPECPV_EINVAL;
    if (tree->n_key_only < 0 || tree->n_key_only >= tree->M) return SPECPV_EINVAL;
    if (tree->n_q_heads % kv->n_kv_heads) return SPECPV_EINVAL;
    if (tree->M > SPECPV_MAX_M || tree->n_q_heads / kv->n_kv_heads > SPECPV_MAX_G) return SPECPV_ELIMIT;
    if ((uintptr_t)tree->q & 15) return SPECPV_EINVAL;
    if (need_draft_kv) {
        if (!tree->kd || !tree->vd || !tree->parent) return SPECPV_EINVAL;
        if (((uintptr_t)tree->kd | (uintptr_t)tree->vd) & 15) return SPECPV_EINVAL;
    }
    return SPECPV_OK;
}

static int check_cfg(const specpv_tree *tree, const specpv_select_cfg *cfg)
{
    if (!cfg) return SPECPV_EINVAL;
    if (cfg->n_sink_blocks < 0 || cfg->n_recent_blocks < 0 || cfg->k_blocks < 0) return SPECPV_EINVAL;
    if (cfg->reduce != SPECPV_REDUCE_MEAN && cfg->reduce != SPECPV_REDUCE_MAX && cfg->reduce != SPECPV_REDUCE_LAST)
        return SPECPV_EINVAL;
    if (cfg->reduce == SPECPV_REDUCE_LAST && (tree->last_node < tree->n_key_only || tree->last_node >= tree->M))
        return SPECPV_EINVAL;
    if (cfg->score != SPECPV_SCORE_EQ2 && cfg->score != SPECPV_SCORE_CHANNEL_BOUND) return SPECPV_EINVAL;
    if (cfg->n_extra_slots < 0) return SPECPV_EINVAL;
    if ((int64_t)cfg->n_sink_blocks + cfg->n_recent_blocks + cfg->k_blocks + cfg->n_extra_slots > ((int64_t)1 << 24))
        return SPECPV_ELIMIT;
    return SPECPV_OK;
}

static Shape make_shape(const specpv_kv *kv, const specpv_tree *tree)
{
    Shape s;
    memset(&s, 0, sizeof(s));
    s.k = kv->k; s.v = kv->v;
    s.sb = kv->stride_b; s.sh = kv->stride_h; s.st = kv->stride_t;
    s.ctx_len = kv->ctx_len;
    s.batch = kv->batch; s.Hkv = kv->n_kv_heads; s.D = kv->head_dim; s.B = kv->block_size;
    s.max_blocks = kv->max_blocks;
    if (tree) {
        s.q = tree->q; s.kd = tree->kd; s.vd = tree->vd; s.parent = tree->parent;
        s.Mk = tree->M; s.koff = tree->n_key_only; s.M = s.Mk - s.koff;
        s.Hq = tree->n_q_heads; s.G = s.Hq / s.Hkv;
    }
    return s;
}

// What a call with bf16 at 128 channels would take, in microseconds, with one of the matrix-core kernels and `ns` splits,
// less what does not depend on that choice.  The constants were fitted to whole calls in graph replays, of kernels that took
// a chunk at a time; against 1578 other timings of today's (130 shapes: 1 to 78 nodes, G = 2, 4, 5 and 8, 2 to 128 (sequence,
// KV head) pairs, 512 to 131072 attended tokens; profiles/plan_timings) the model is 8 % off, root mean square, and the plan
// it chooses 0.9 % (one card) and 1.4 % (another) slower than the fastest measured one in the mean, 13 and 19 % at most.
// Pairs of chunks took up to 12 % of the cycles of some of the loops; the constants per chunk cut by 5 or 10 %, together and
// one by one, choose plans that lose 1.3 to 2.6 % where these lose 1.4.  Taking the fewest partials among plans that the
// model holds within 1, 2, 4 or 6 % of the best: 1.4, 1.5, 1.6, 2.2 %, so the best it is.  A workgroup per CU at a time takes its token range, p
// chunks one after the other, in `rounds`; besides that the K / V bytes have to come out of the L2s (once per tile) and
// of HBM; partials are written and read back.
struct AttnCost {
    const Shape &s;
    int64_t chunks;
    double kv;   // MB of K and V
    AttnCost(const Shape &sh, int64_t ch) : s(sh), chunks(ch), kv((double)sh.batch * sh.Hkv * (double)ch * 16384e-6) {}
    double us(int64_t rounds, int64_t p, double start, double per_chunk, int64_t tiles, int64_t ns) const
    {
        const double chain = (double)rounds * (start + (double)p * per_chunk);
        const double memory = kv * (0.02 * (double)tiles + 0.115);
        const double partials = (double)s.batch * s.Hkv * (double)ns * s.M * s.G * 512e-6;   // MB
        return sqrt(chain * chain + memory * memory) + (ns > 16 ? 0.82 : 0.0) + 0.199 * partials;
    }
    // the tile kernel with tg token groups (attn_tile.hip)
    double tile(int tg, int64_t ns, int64_t cus) const
    {
        const int64_t rows = 256 / tg, tiles = ((int64_t)s.M * s.G + rows - 1) / rows, bg = (int64_t)s.batch * s.Hkv;
        // (pairs that are a multiple of 8 stay on their XCD)
        const int64_t rounds = bg % 8 ? (bg * tiles * ns + cus - 1) / cus : (bg / 8 * tiles * ns + cus / 8 - 1) / (cus / 8);
        const int64_t p = (chunks + ns * tg - 1) / (ns * tg);
        return us(rounds, p, tg == 2 ? 2.03 : (tg == 4 ? 1.59 : 1.67), tile_chunk_us(tg), tiles, ns);
    }
    static double tile_chunk_us(int tg) { return tg == 2 ? 0.97 : (tg == 4 ? 1.50 : 2.13); }
    // the group kernel (attn_mfma.hip)
    double group(int parts, int blocks, int64_t ns, int64_t cus) const
    {
        const int64_t rounds = ((int64_t)s.batch * s.Hkv * parts * ns + cus - 1) / cus, p = (chunks + ns - 1) / ns;
        return us(rounds, p, 3.11, attn_group_chunk_us(blocks), parts, ns);
    }
    // ... in equal shares of all chunks, whose partials are found by the lengths and merged in rounds
    double shares(int parts, int blocks, int64_t wgs) const
    {
        const double pairs = (double)s.batch * s.Hkv, p = pairs * (double)chunks / (double)wgs;
        const double chain = 3.11 + p * attn_group_chunk_us(blocks) * (double)parts * (double)wgs / (double)device_cu_count(), memory = kv * (0.02 * (double)parts + 0.115);
        return sqrt(chain * chain + memory * memory) + 0.199 * ((double)wgs + pairs) * s.M * s.G * 512e-6 + 6.0;
    }
    // Whether ranges of `p` chunks, `chunk_us` each, hold up against `wgs` shares when the lengths differ as much as they may: one
    // sequence with all the chunks, the others with a sixteenth.  A split's chain stays what it was; the shares' chain is cut to the
    // chunks that there are, but then the long sequence has most of the shares, and its combine takes them in rounds, a tenth of a
    // microsecond each.  For 94 shapes (2 to 32 sequences, 1 to 8 KV heads, 1 to 60 nodes, 1 K to 64 K tokens) with the splits that the
    // costs above choose, the chain that splits have more over the shares of the long pair, against the slowest of equal lengths, 1 / n
    // to n / n, one long first and one long last, splits / shares: up to 0.09 us a share (41 shapes) 1.02 at most, 0.82 in the mean;
    // 0.1 to 0.2: 0.9 to 1.38; 0.2 to 0.5: up to 1.44; beyond: up to 1.55.
    // The group kernel's splits gain elsewhere too: up to four sequences have eleven chunks and a half in hand (130 shapes, refreshes, splits / shares: up to
    // there equal lengths 0.77 to 1.0, 0.84 in the mean, 1 / n to n / n 0.75 to 1.0, one long 0.70 to 1.05, long last 0.59 to 1.0; where the lengths happen to divide into whole
    // shares, one long up to 1.2, a few tokens beside them 1.0: four of 3269 / 3200, 37 nodes at G = 5, 28.2 / 24.3, 29.3 / 29.3 us; four of 8192, 22 chunks, 1.23 at any
    // length), and where there are more pairs than shares, most of which then run through several, two partials of a pair beyond them (64 sequences of 1300, 64 nodes 0.81, 0.49, 0.82, 0.90).
    bool splits_hold(double p, double chunk_us, int blocks, int64_t wgs, bool group) const
    {
        const double of_share = (double)s.Hkv * (double)chunks * (1.0 + (double)(s.batch - 1) / 16.0) / (double)wgs, share = of_share < 1.0 ? 1.0 : of_share;
        const double more = p * chunk_us - share * attn_group_chunk_us(blocks), merged = 0.09 * (double)chunks / share;
        const double beyond = (double)s.batch * s.Hkv - (double)wgs, pairs = group && beyond > 0.0 ? beyond * s.M * s.G * 528e-6 : 0.0, hand = group && s.batch <= 4 ? 11.5 * chunk_us : 0.0;
        return more <= (merged > hand ? merged : hand) + pairs;
    }
};

// The fewest splits that specpv_partial_verify_attn_static has to have room for: the count by which a shape was first
// judged to fit its array (as fp32 partials).  Calls that fitted then still do (plan_attention).
static int64_t first_splits(const Shape &s, int64_t chunks, int64_t cus)
{
    auto best_of = [&](int64_t base, int64_t ranges, int64_t most) {
        int64_t ns = 1, best = -1;
        for (int64_t c = 1; c <= most; ++c) {
            const int64_t cost = (base * c + cus - 1) / cus * ((chunks + ranges * c - 1) / (ranges * c) * 8 + 10) + c;
            if (best < 0 || cost < best) { best = cost; ns = c; }
        }
        return ns;
    };
    auto at_most = [](int64_t c) { return c < 1 ? (int64_t)1 : (c < 64 ? c : (int64_t)64); };
    const int64_t ns = best_of((int64_t)s.batch * s.Hq * ((s.M + 63) / 64), 4, at_most(chunks / 4));
    const int64_t row_blocks = (s.G * s.M + 31) / 32, parts = row_blocks == 9 || row_blocks == 10 ? 1 : (row_blocks + 7) / 8;
    return chunks >= 32 * ns ? best_of((int64_t)s.batch * s.Hkv * parts, 1, at_most(chunks / 8)) : ns;
}

// The array of specpv_partial_verify_attn_static.  Larger than the SPECPV_STATIC_SCRATCH_BYTES by which it takes calls, so that no
// plan has to be cut to those: every call runs the plan that the static one would.  Cut to 16 MiB / as it is now: refresh, fp32, 37
// nodes at G = 4, 16K, 8 KV heads, 26 / 32 splits 175 / 146 us; full pass, 64 channels, 15005 and 30011 tokens, 25 / 32 splits 52.7 / 46.6.
constexpr int64_t kStaticArray = 64 << 20;

// Bytes of a partial row: O as fp16 (bf16 at 128 channels) or fp32, and the (m, l) pair.
static bool half_partials(const Shape &s, int kind) { return kind != kAttnGeneric && s.D == 128; }
static size_t part_row_bytes(const Shape &s, int kind)
{
    return (size_t)s.D * (half_partials(s, kind) ? sizeof(uint16_t) : sizeof(float)) + 2 * sizeof(float);
}

// Workspace: [arrival words, kArriveBytes, zero between calls][partial O][(m, l) pairs], `need` bytes for the rows of a
// plan.  `total` is what specpv_workspace_bytes promises: room for nsplit + 1 slots of fp32 (the context splits and the
// draft-tree segment, as the single-kernel route lays them out: O, pairs at fused_ml) and, behind them, the scores.
// Scores that a call keeps in the workspace stand behind the arrival words: they are written when the partials have been
// read.  A refresh that scores beside the merge puts them behind the rows of its plan, where there is room.
struct Workspace {
    unsigned long long *arrive;
    float *part_o, *part_ml, *fused_ml, *scores;
    size_t need, total, scores_need;
};

static Workspace layout_workspace(const Shape &s, const AttnPlan &plan, void *base)
{
    Workspace w;
    const size_t slots = (size_t)plan.nsplit + 1;
    const size_t po = align_up((size_t)s.batch * s.Hq * slots * s.M * s.D * sizeof(float));
    const size_t pm = align_up((size_t)s.batch * s.Hq * slots * s.M * 2 * sizeof(float));
    const size_t sc = align_up((size_t)s.batch * s.Hkv * s.max_blocks * sizeof(float));
    char *p = (char *)base;
    w.arrive = (unsigned long long *)p;
    w.part_o = (float *)(p + kArriveBytes);
    w.fused_ml = (float *)(p + kArriveBytes + po);
    w.scores = (float *)(p + kArriveBytes);
    w.total = kArriveBytes + po + pm + sc;
    w.scores_need = kArriveBytes + sc;
    const size_t R = (size_t)s.M * s.G, pairs = (size_t)s.batch * s.Hkv;
    const size_t rows = (plan.stream ? (size_t)plan.stream + pairs : pairs * plan.nsplit) * R;   // partial rows in use
    const size_t ho = align_up(rows * (part_row_bytes(s, plan.kind) - 2 * sizeof(float)));
    w.part_ml = (float *)(p + kArriveBytes + ho);
    w.need = kArriveBytes + ho + align_up(rows * 2 * sizeof(float));
    return w;
}

// What specpv_partial_verify_attn_static asks of its array.
static size_t static_need(const Shape &s, const AttnPlan &plan)
{
    const Workspace w = layout_workspace(s, plan, nullptr);
    return plan.stream || half_partials(s, plan.kind) ? w.need : w.total;
}

// Which kernel the context part of the attention runs on and how many KV splits it uses when
// it covers n_blocks blocks per (sequence, KV head).  Host-only and deterministic in its
// arguments, so specpv_workspace_bytes and the calls agree.  full: every block of sequences whose
// lengths only the device knows (n_blocks is the most that any of them has).
// bytes: what the caller's workspace has.  A smaller tree may be worth more splits than a larger one, so a workspace that
// was sized for the largest tree of a decode loop need not hold the plan of every smaller one: then the call takes the
// splits that fit (one always does where the larger tree's plan did).
// taking: the plan, cut to SPECPV_STATIC_SCRATCH_BYTES, by which specpv_partial_verify_attn_static decides whether it takes a call.  It
// runs the plan of every other call then, whose partials fit kStaticArray.
static AttnPlan plan_attention(const Shape &s, int dtype, int64_t n_blocks, bool full, size_t bytes, bool taking = false)
{
    const int64_t array = taking ? (int64_t)SPECPV_STATIC_SCRATCH_BYTES : kStaticArray;
    AttnPlan plan{1, !attn_ctx_mfma_supported(s, dtype) ? kAttnGeneric : (s.D == 64 ? kAttnGroup : kAttnSplit), 4, 0};
    if (plan.kind == kAttnGeneric) plan.tg = 0;
    // partial rows that have room (Workspace), and splits
    const size_t row_bytes = part_row_bytes(s, plan.kind), pair_rows = (size_t)s.M * s.G, fixed_bytes = kArriveBytes + 512;
    const int64_t room_rows = bytes > fixed_bytes ? (int64_t)((bytes - fixed_bytes) / row_bytes) : 0;   // (< 2^63: a row has more than one byte)
    const int64_t room_splits = room_rows / ((int64_t)s.batch * s.Hkv * (int64_t)pair_rows);
    auto at_hand = [&](int64_t ns) { return ns <= room_splits ? ns : (room_splits > 1 ? room_splits : (int64_t)1); };
    // splits that give 4096 (row, split) pairs of 64 tokens or more each
    const int64_t rows = (int64_t)s.batch * s.Hq * s.M;
    auto few_splits = [&](int64_t tokens) {
        int64_t ns = (4096 + rows - 1) / rows;
        const int64_t chunks = (tokens + 63) / 64;
        if (ns > chunks) ns = chunks;
        if (ns > 64) ns = 64;
        return ns < 1 ? (int64_t)1 : ns;
    };
    // (a list may have room for more blocks than there are)
    const int64_t tokens = (n_blocks < s.max_blocks ? n_blocks : (int64_t)s.max_blocks) * s.B;
    if (tokens <= 0) return plan;
    // what specpv_partial_verify_attn_static took with the splits of fp32 partials that a call had at first must fit the
    // array with more of them: no more splits than have room, where those few have in SPECPV_STATIC_SCRATCH_BYTES
    const int64_t static_slot = rows * (s.D + 2) * (int64_t)sizeof(float), static_fixed = (int64_t)kArriveBytes + 1024;
    auto static_splits = [&](int64_t bytes) {
        const bool half = half_partials(s, plan.kind);
        return (bytes - static_fixed) / (half ? rows * (2 * s.D + 8) : static_slot) - (half ? 0 : 1);
    };
    auto static_room_of = [&](int64_t bytes, auto few_of, int64_t ns) {
        const int64_t room = static_splits(bytes);
        if (ns <= room || room < 1) return ns;
        const bool few_fit = static_fixed + static_slot * (few_of() + 1) + (int64_t)s.batch * s.Hkv * s.max_blocks * (int64_t)sizeof(float) <= (int64_t)SPECPV_STATIC_SCRATCH_BYTES;
        return few_fit ? room : ns;
    };
    auto static_room = [&](auto few_of, int64_t ns) { return static_room_of(array, few_of, ns); };
    // whether specpv_partial_verify_attn_static takes the call
    auto taken = [&]() { return taking || static_need(s, plan_attention(s, dtype, n_blocks, full, SIZE_MAX, true)) <= (size_t)SPECPV_STATIC_SCRATCH_BYTES; };
    const int64_t cus = device_cu_count();
    if (plan.kind == kAttnGeneric) {
        // two wavefronts of 32 rows per SIMD, 64 tokens or more each (the few splits up to 1024 tokens, and half that many
        // tokens each for the shortest ranges, whose time is one wavefront's chain)
        const int64_t few = few_splits(tokens);
        int64_t ns = few;
        const int64_t pairs = (int64_t)s.batch * s.Hkv, R = (int64_t)s.M * s.G, parts = (R + kF32Rows - 1) / kF32Rows, chunks = (tokens + 31) / 32;
        // K and V rows by way of LDS (attn_f32.hip) for more than one tile of 16 query rows, where there is enough to do.  Best splits of
        // either, by way of LDS / straight from memory, us: 128 channels, 8 KV heads, 60 nodes at G = 4, 16K 172 / 199, 37 nodes 136 /
        // 199, 8 nodes 60 / 69, one KV head, 16 nodes 43 / 54, 2K 15.4 / 16.2, 8 nodes 14.4 / 14.0; 64 channels, 8 KV heads, 37 nodes, 16K
        // 72 / 93, 2K 20.1 / 21.4, 30 nodes 17.5 / 16.7, 4K 24.5 / 25.9; one KV head, 30 nodes, 16K 24.6 / 28.0, 4K 14.2 / 14.3, 1100 11.2 / 10.7.
        const bool staged = !taking && dtype == SPECPV_F32 && R > 16 && tokens > 1024 && n_blocks * s.B < ((int64_t)1 << 31) - 64 &&
                            (s.D == 128 ? R > 48 || tokens > 2048 : tokens > 4096 || pairs * parts * chunks >= 2048);
        if (staged) {
            // Workgroups of a CU share its matrix cores, four at a time its registers; a chunk (32 tokens here) takes one by itself its
            // latency.  Partials are written and read back.  Fitted to 3000 timings of 190 shapes: the splits that this chooses are 1.7 %
            // slower than the fastest in the mean.
            // Up to 32 rows leave two of a workgroup's four wavefronts idle: half of the share, and no more workgroups than have a place (16
            // sequences of 2400, 20 rows, 8 heads, six splits / eight, equal lengths and one long 0.40 / 0.38, 1.18 / 0.9 of straight from
            // memory; 4 of 5900, 32 rows, 23 / 30, 0.68 / 0.63, 1.03 / 0.92).  Batches have two splits or more: with one, sequences of
            // different lengths keep the chip for as long as the longest (24 of 1350, 60 nodes, one / two, equal lengths and one long 384 /
            // 377, 227 / 153 us).
            const bool half = R <= 32;
            const double share = (s.D == 128 ? 1.48 : 0.73) * (half ? 0.5 : 1.0), alone = s.D == 128 ? 4.0 : 2.4, partials = 1.0 * (double)pairs * (double)R * s.D * 4e-6;
            double best = -1.0;
            int64_t most = static_room([&] { return few; }, chunks < 64 ? chunks : 64);
            if (half && most > 4 * cus / pairs) most = 4 * cus / pairs;
            const int64_t least = full && s.batch > 1 && chunks > 1 ? 2 : 1;
            most = at_hand(most > least ? most : least);
            for (int64_t c = least < most ? least : most; c <= most; ++c) {
                const int64_t here = (pairs * parts * c + cus - 1) / cus, p = (chunks + c - 1) / c;
                const double work = share * (double)here > alone ? share * (double)here : alone;
                const double us = (double)p * work + 0.56 * (double)((here + 3) / 4) + partials * (double)c + (c > 16 ? 0.1 : 0.0);
                if (best < 0.0 || us < best) { best = us; ns = c; }
            }
            plan.tg = 1;
        } else if (tokens > 1024) {
            const int64_t waves = (int64_t)((s.G * s.M + 31) / 32) * s.batch * s.Hkv;
            ns = (8 * cus + waves - 1) / waves;
            if (ns > tokens / 64) ns = tokens / 64;
            if (ns > 64) ns = 64;
            if (ns < few) ns = few;
        } else if (tokens <= 512) {
            const int64_t most = (tokens + 31) / 32 < 8 ? (tokens + 31) / 32 : 8;
            const int64_t want = (4096 + rows - 1) / rows;
            ns = want < most ? want : most;
            if (ns < few) ns = few;
        }
        // (straight from memory: partials of no more than 16 MiB, where a few splits have no more.  16 sequences of 1500, 5 nodes at G = 4, 8 heads, 11
        // splits / 16: equal lengths 170 / 162 us, one long 48 / 65)
        plan.nsplit = (int)at_hand(static_room_of(staged ? array : (int64_t)SPECPV_STATIC_SCRATCH_BYTES, [&] { return few; }, ns));
    } else {
        const int64_t chunks = (tokens + 31) / 32;   // 32-token chunks per (sequence, KV head)
        const int parts = attn_group_parts(s);
        const int64_t base = (int64_t)s.batch * s.Hkv * parts;   // group kernel: workgroups per split
        // ... and workgroups of equal shares (below), eight chunks or more each: one a CU, with 64 channels and for few rows, which leave room
        // for it, two (64 channels, 60 nodes, 8 heads at G = 5, 24 of 3000, equal and 1 / n to n / n, one / two 176 / 172, 146 / 108 us).  For
        // few rows of 128 channels only where a pair can get no more than 64 of them: one long sequence of a few heads has most of them merged for itself.  One /
        // two, equal lengths and one long: 8 heads, one node, 4 of 32K 115 / 97, 44 / 41 us; one head, 24 of 22K 62 / 56, 27.5 / 30.4.
        const bool two = s.D == 64 || (!taking && attn_group_blocks(s) <= 2 && 2 * cus <= 64 * (int64_t)s.Hkv);
        const bool can_share = full && s.batch > 1 && s.batch <= 64;
        int64_t shares = cus * (two ? 2 : 1) / parts;
        if (can_share && shares > (int64_t)s.batch * s.Hkv * chunks / 8) shares = (int64_t)s.batch * s.Hkv * chunks / 8;
        if (shares < 1) shares = 1;
        const AttnCost cost(s, chunks);
        const int blocks = attn_group_blocks(s);
        // the slots of the shares, the workspace of as many splits as hold those, and whether their partials take more than 16 MiB
        const int64_t share_bytes = can_share ? (shares + (int64_t)s.batch * s.Hkv) * (int64_t)(pair_rows * row_bytes) + 512 : 0;
        const int64_t split_bytes = can_share ? rows * (4 * s.D + 8) : 1, share_splits = (share_bytes + split_bytes - 1) / split_bytes > 1 ? (share_bytes + split_bytes - 1) / split_bytes - 1 : 1;
        const bool many_partials = (int64_t)kArriveBytes + share_bytes > (int64_t)SPECPV_STATIC_SCRATCH_BYTES;
        int64_t ns = 1, least = 1;
        bool keep_static = false;
        if (s.D == 64) {
            // the group kernel; two workgroups or more have room on a CU, but share what it gives
            const int64_t few = few_splits(tokens);
            int64_t most = chunks / (taking ? 4 : 2) > 1 ? (chunks / (taking ? 4 : 2) < 64 ? chunks / (taking ? 4 : 2) : 64) : 1;
            most = at_hand(static_room([&] { return few; }, most));
            // up to 1024 tokens: the few splits of the vector-ALU kernel are enough
            if (chunks <= 32 && most > few) most = few;
            // the splits that fill two places a CU
            auto filling = [&](int64_t at_most) {
                const int64_t slots = 2 * cus;
                int64_t best = -1, n = 1;
                for (int64_t c = 1; c <= at_most; ++c) {
                    const int64_t cost = (base * c + slots - 1) / slots * ((chunks + c - 1) / c * 8 + 10) + c;
                    if (best < 0 || cost < best) { best = cost; n = c; }
                }
                return n;
            };
            if (taking) {
                ns = filling(most);
            } else {
                // us, fitted to 3700 timings of 249 shapes (1 to 60 nodes, G = 4, 5 and 8, 2 to 80 pairs, 1100 to 30000 tokens): the
                // splits that this chooses are 0.7 % slower than the fastest in the mean, 2.2 % for batches of lengths 1 / n to n / n.
                // (Splits that filled two places a CU: 8.6 % slower than these.  64 channels, 8 KV heads at G = 4, 37 nodes, 8K 21.2 ->
                // 17.8 us, four sequences of 4K 28.7 -> 24.0; one node, 16 of up to 3000 21.6 -> 16.9.)
                const double chunk = 0.243 + 0.092 * attn_group_blocks(s), partials = 0.371 * (double)s.batch * s.Hkv * (double)(s.M * s.G) * 256e-6;
                double best = -1.0;
                for (int64_t c = 1; c <= most; ++c) {
                    const int64_t here = (base * c + cus - 1) / cus, p = (chunks + c - 1) / c;
                    const double share = 0.808 * (double)here > 1.0 ? 0.808 * (double)here : 1.0;
                    const double us = (double)p * chunk * share + (here > 2 ? 0.973 * (double)(here - 2) : 0.0) + 0.285 * (double)here + partials * (double)c +
                                      0.247 * (double)((c + 7) / 8) + (c > 16 ? 0.486 : 0.0);
                    if (best < 0.0 || us < best) { best = us; ns = c; }
                }
                // The fit is of equal lengths.  Where shares have no room and splits stand in for them, not fewer than fill the chip (with
                // partials of 16 MiB or less, if a few have): 3 sequences of 7800, 24 nodes at G = 5, ten splits (the fit's) / nineteen, equal lengths, 1 / n to n / n, one long
                // 1.07 / 1.00, 1.15 / 1.02, 1.27 / 1.01 of what they were; one head, 6 of 24K, 16 nodes, 42 / 63 one long 21.3 / 20.4 us.
                if (chunks > 32 && ((can_share && (many_partials || share_splits > 64)) || (full && s.batch > 64))) {
                    const int64_t quarter = chunks / 4 > 64 ? 64 : chunks / 4;
                    const int64_t n = filling(at_hand(static_room_of(SPECPV_STATIC_SCRATCH_BYTES, [&] { return few; }, quarter > 1 ? quarter : 1)));
                    if (least < n) least = n;
                }
            }
        } else {
            // AttnCost takes every sequence to be as long as the longest.  The group kernel, below, evens out the lengths of
            // a full pass; the tile kernel, which a few nodes may be faster with, does not.  24 nodes at G = 4, 16 sequences
            // of 16K (512 chunks), 8 KV heads, tile kernel against shares: equal lengths 203 / 209 us, 1/16 to 16/16 of it
            // 159 / 124, one long and fifteen short ones 144 / 47; four sequences of 258 chunks: 37 / 43, 34 / 34, 30 / 25.
            // Few pairs take it where its ranges are so short that shares gain nothing (splits_hold): 30000 + 15000 tokens, 2 KV heads, 37
            // nodes at G = 8 37.5 us, the group kernel 43.7, shares 44.8; with 32 pairs, 6K to 25K tokens, 18 nodes at G = 5 71.8 / 58.1 / 60.4.
            const bool uneven = full && s.batch > 1 && chunks > 256, small = !taking && (int64_t)s.batch * s.Hkv <= 8;
            double best = -1.0, best_tile = -1.0;
            int64_t ns_tile = 1;
            auto take = [&](double us, int kind, int tg, int64_t c) {
                if (uneven && kind == kAttnSplit && !(small && cost.splits_hold((double)((chunks + c * tg - 1) / (c * tg)), AttnCost::tile_chunk_us(tg), blocks, shares, false))) {
                    if (best_tile < 0.0 || us < best_tile) { best_tile = us; ns_tile = c; }
                } else if (best < 0.0 || us < best) {
                    best = us; plan.kind = kind; plan.tg = tg; ns = c;
                }
            };
            // split counts that divide evenly, those that the combine kernel takes in one go, and those that fill the chip
            int64_t cand[16] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
            for (int k = 1; k <= 4; ++k) cand[11 + k] = k * cus / base;
            for (int64_t c : cand) {
                if (c < 1 || c > 64 || c > at_hand(c)) continue;
                for (int tg = 2; tg <= 8; tg *= 2)
                    if (c * tg <= 2 * chunks) take(cost.tile(tg, c, cus), kAttnSplit, tg, c);
                if (chunks >= 2 * c) take(cost.group(parts, blocks, c, cus), kAttnGroup, 4, c);
            }
            ns = static_room([&] { return first_splits(s, chunks, cus); }, ns);
            // (where the tile kernel would have been taken and its partials fit the static array, the group kernel's do too)
            keep_static = best_tile >= 0.0 && best_tile < best && static_room([&] { return first_splits(s, chunks, cus); }, ns_tile) <= static_splits(array) && taken();
            if (keep_static && ns > static_splits(array)) ns = static_splits(array);
        }
        plan.nsplit = (int)ns;
        // The sequences of a batch may differ in length, and the lengths live on the device: for a full pass the group
        // kernel's workgroups take equal shares of all chunks.  (Four times as many splits as fill the chip even that out
        // too, at the price of as many partials: full pass over 32K + 64K + 96K + 128K tokens at G = 5, 64 nodes, attention
        // and combine: 563 us with the splits that fill the chip, 462 with four times as many, 453 with the shares.)  Up to
        // 1024 tokens there is nothing to even out, and little where a split has few chunks: its partials have one place each, where a
        // share's are found by the lengths and merged in rounds.  Shares / splits, us, of equal lengths, 1 / n to n / n, one long and the
        // others a sixteenth of it.  Splits: 3 sequences of 7055, 37 nodes, 4 KV heads, 21 of 11 chunks 34 / 28, 31 / 26, 28 / 27; 2 of 57746,
        // 24 nodes at G = 8, 2 heads, 64 of 29 chunks 52 / 43, 46 / 41, 44 / 39.  Shares: 60 nodes, 8 heads, 16 of 3000 at G = 5, two of 47
        // 99 / 83, 92 / 71, 50 / 66; 10 of 4096, three of 43 69 / 58, 54 / 51, 34 / 48; 4 of 8192, eight of 32 60 / 58, 50 / 52, 39 / 46.
        // 64 channels, up to 32 chunks of a split, which have less to do there: where the pairs are few, so that one long sequence has
        // splits enough, or the shares' partials many.  Shares / splits: 8 heads, 2 sequences of 21.7K, one node 31 / 26, 27 / 25, 25 / 22;
        // 5 of 11K, 60 nodes at G = 5 1.00 / 0.88, 1.00 / 0.95, 1.00 / 0.95; 32 of 1300, 60 nodes 85 / 72, 90 / 59, 45 / 49;
        // up to four sequences of many partials 48 chunks (two of 49K, 24 nodes at G = 8 0.78 / 0.73, 0.78 / 0.74, 0.84 / 0.75 of what they were).  Many pairs of
        // few rows keep the shares: 16 of 2650, one node 28 / 26, 24 / 24, 17 / 21; 32 of 4100, 16 nodes at G = 8 one long 1.00 / 1.65.
        const bool short_splits = !taking && (s.D == 64 ? chunks <= (many_partials && s.batch <= 4 ? 48 : 32) * ns && ((int64_t)s.batch * s.Hkv <= 40 || many_partials) : cost.group(parts, blocks, ns, cus) < cost.shares(parts, blocks, shares) &&
                                                                               cost.splits_hold((double)((chunks + ns - 1) / ns), attn_group_chunk_us(blocks), blocks, shares, true));
        if (can_share && plan.kind == kAttnGroup && chunks > 32 && !short_splits && (int64_t)s.batch * s.Hkv * chunks < ((int64_t)1 << 30)) {
            const int64_t pairs = (int64_t)s.batch * s.Hkv, R = (int64_t)s.M * s.G;
            int64_t wgs = shares;
            const int64_t static_slots = (array - static_fixed) / (R * (int64_t)row_bytes) - pairs;
            if (keep_static && wgs > static_slots && static_slots >= wgs / 2) wgs = static_slots;
            // the workspace of as many splits as hold that many slots
            const int64_t bytes = (wgs + pairs) * R * (int64_t)row_bytes + 512;
            const int64_t splits = (bytes + split_bytes - 1) / split_bytes > 1 ? (bytes + split_bytes - 1) / split_bytes - 1 : 1;
            const bool fits = (int64_t)kArriveBytes + bytes <= array;
            const int64_t at_most = room_rows / R - pairs;   // ... that the caller's has room for
            if (at_most >= 1 && splits <= 64 && (fits || (!keep_static && static_room([&] { return s.D == 64 ? few_splits(tokens) : first_splits(s, chunks, cus); }, 64) == 64))) {
                plan.stream = (int)(wgs < at_most ? wgs : at_most);
                plan.nsplit = (int)splits;
            }
        }
        if (!plan.stream && least > ns) plan.nsplit = (int)(ns = least);
        // ... and for more sequences than the shares are worked out for, about eight workgroups per CU, 64 chunks or more
        // each, for the hardware to deal out.  100 sequences of 16K, 4 KV heads, 60 nodes at G = 4, with the model's three
        // splits / with six: equal lengths 968 / 1004 us, 1/100 to 100/100 of it 539 / 550, one long and the others a
        // sixteenth of it 186 / 169; 72 of 32K, one KV head at G = 8, seven / fifteen: 613 / 670, 360 / 369, 147 / 121; 128 of
        // 16K, 2 KV heads, 24 nodes, one split / two (eight would not fit the static array): 408 / 336, 313 / 232, 292 / 166.
        // What equal lengths lose is less than what one long sequence among short ones gains.
        if (full && s.batch > 64 && plan.kind == kAttnGroup) {
            int64_t c = (8 * cus + base - 1) / base;
            if (c > 64) c = 64;
            while (c > ns && (chunks + c - 1) / c < 64) --c;
            // Each round of workgroups starts and ends for itself: where the splits in hand have partials of 16 MiB or less, no more than
            // stay so.  128 of 16K, 2 KV heads, 24 nodes, refreshed, two splits / four / eight: equal lengths 351-360 / 370 / 376 us, 1/128 to
            // 128/128 of it 241 / 235 / 235.
            auto in = [&](int64_t n, size_t room) {
                const AttnPlan x{(int)n, plan.kind, plan.tg, 0};
                return (room == (size_t)SPECPV_STATIC_SCRATCH_BYTES ? static_need(s, x) : layout_workspace(s, x, nullptr).need) <= room;
            };
            if (in(ns, SPECPV_STATIC_SCRATCH_BYTES))
                while (c > ns && !in(c, SPECPV_STATIC_SCRATCH_BYTES)) --c;
            // A call that specpv_partial_verify_attn_static takes has room in its array.  (72 of 16K, one head at G = 8, 60 nodes, which it does
            // not take: one long 94 us with eight splits, 100 with the seven that would have.)
            if (!taking && c > ns && in(ns, (size_t)array) && !in(c, (size_t)array) && taken())
                while (c > ns && !in(c, (size_t)array)) --c;
            c = at_hand(c);
            if (c > ns) plan.nsplit = (int)c;
        }
    }
    return plan;
}

// Where a full pass on the group kernel recomputes many summaries, some of its workgroups do that beside the others, and
// the plan's splits or shares are cut to the CUs that are left: the attention loop runs at the clock that the chip's power
// allows and leaves a third of the memory's rate unused, the summaries are nothing but reads.  A CU takes in 45 bytes per
// nanosecond (16 KiB in flight per wavefront: blocks of 64, twos of 32 or fours of 16; other small blocks have less, and lose), so the two sides end together with a fraction f / (1 + f) of the CUs on the
// summaries; 0.235 was fitted to the fastest counts: stale refresh of 128K, eight row blocks, 0 / 40 / 48 / 56 / 64
// workgroups: 202 / 211 / 195 / 193 / 196 us; of 64K, ten: 130 / 120 / 122 / 123 / 124; of 16K + 32K + 48K + 64K, eight:
// 247 / 264 / 240 / 238 / 239.  Fewer than eight row blocks leave less of the memory's rate.  Small blocks, two launches /
// so: 64K in blocks of 32 113.8 / 102.9, of 16 118.1 / 108.9; 2 x 30000 at G = 5 in blocks of 16 135.0 / 123.6; 8 x 28046 354 / 350.
static SumArgs side_summaries(const Shape &s, int64_t begin, void *kmax, void *kmin, AttnPlan &plan)
{
    const SumArgs none{0, 0, nullptr, nullptr};
    if (plan.kind != kAttnGroup || s.D != 128 || (s.B < 64 && s.B != 32 && s.B != 16) || attn_group_blocks(s) < 8 || begin >= s.max_blocks) return none;
    const int64_t cus = device_cu_count(), parts = attn_group_parts(s), pairs = (int64_t)s.batch * s.Hkv;
    const int64_t chunks = ((int64_t)s.max_blocks * s.B + 31) / 32, stale = chunks - begin * s.B / 32;
    if (parts * (plan.stream ? plan.stream : pairs * plan.nsplit) > cus) return none;   // more than one round of workgroups
    const double f = 0.235 * (double)stale / (attn_group_chunk_us(attn_group_blocks(s)) * (double)(chunks * parts));
    const int64_t row = 8 * parts, rows = (int64_t)((double)cus * f / (1.0 + f) / (double)row + 0.5);   // of the grid
    const int64_t left = (cus - rows * row) / parts;
    if (rows < 1 || left < (plan.stream ? 1 : pairs)) return none;
    if (plan.stream) plan.stream = (int)(plan.stream < left ? plan.stream : left);
    else plan.nsplit = (int)(plan.nsplit < left / pairs ? plan.nsplit : left / pairs);
    return SumArgs{(int)(rows * row), (int)begin, kmax, kmin};
}

// Process-wide choice of how specpv_partial_verify_attn runs shapes that the eight-wavefront kernel
// takes (a testing aid, see specpv_debug_set_route).
static int g_route = 0;
static unsigned long long *g_timeline = nullptr;   // where instrumented builds (-DSPECPV_TIMELINE) put their time stamps

// The scores that a full pass wants beside the merge of its partials, or the lists themselves where they keep every block (all).
// done: they are there (else they are still to be taken).
struct TailScores {
    const void *kmax, *kmin;
    int kind, reduce, last_node;
    float *scores;
    const TopkArgs *all;
    bool done;
};

static int run_attention(const Shape &s_in, const AttnPlan &plan, int dtype, const int32_t *sel_idx, const int32_t *sel_count,
                         int n_sel, void *out, float *lse, void *workspace, size_t workspace_bytes, const SumArgs &sum, hipStream_t st,
                         TailScores *tail = nullptr)
{
    Shape s = s_in;
    // the matrix-core kernels take the partially verified tokens in front of the tree along with the cache
    // tokens (dense: every query row attends all of them); the vector-ALU kernel leaves them to the combine
    s.kctx = plan.kind != kAttnGeneric ? s.koff : 0;
    const int nsplit = plan.nsplit;
    const Workspace w = layout_workspace(s, plan, workspace);
    if (!workspace || workspace_bytes < w.need) return SPECPV_EWORKSPACE;
    const int route = __atomic_load_n(&g_route, __ATOMIC_RELAXED);
    // The single-kernel route is correct but measured slower than two launches (the last workgroup of a
    // tile reads all of the tile's partials through one CU): it runs only on request.
    const bool fused = plan.kind == kAttnSplit && route >= 2 && nsplit <= 64 && workspace_bytes >= w.total &&
                       (size_t)s.batch * s.Hq * 2 * sizeof(unsigned long long) <= kArriveBytes;
    hipError_t e;
    if (fused) {
        Partials p{w.part_o, w.fused_ml, nsplit + 1, 0, 0, nullptr};
        const FusedArgs f{out, lse, w.arrive, route == 3 ? 1 : 0, g_timeline};
        e = launch_attn_ctx_mfma(s, sel_idx, sel_count, n_sel, p, nsplit, plan.kind, f, SumArgs{}, st);
        return e == hipSuccess ? SPECPV_OK : fail_hip(e);
    }
    Partials p{w.part_o, w.part_ml, nsplit, half_partials(s, plan.kind) ? 1 : 0, plan.stream, g_timeline};
    const FusedArgs none{nullptr, nullptr, nullptr, 0, g_timeline};
    if (plan.kind == kAttnSplit) e = launch_attn_ctx_tile(s, sel_idx, sel_count, n_sel, p, plan.tg, g_timeline, st);
    else if (plan.kind != kAttnGeneric) e = launch_attn_ctx_mfma(s, sel_idx, sel_count, n_sel, p, nsplit, plan.kind, none, sum, st);
    else if (plan.tg) e = launch_attn_ctx_f32(s, sel_idx, sel_count, n_sel, p, st);
    else e = launch_attn_ctx_generic(s, dtype, sel_idx, sel_count, n_sel, p, st);
    if (e != hipSuccess) return fail_hip(e);
    if (tail && (tail->scores || tail->all) && refresh_tail_supported(s, dtype, p, tail->kind) && (!tail->scores || refresh_tail_pays(s, p, tail->reduce, tail->last_node))) {
        e = launch_refresh_tail(s, p, out, lse, tail->kmax, tail->kmin, tail->reduce, tail->last_node, tail->scores, tail->all, st);
        tail->done = true;
    } else {
        e = launch_combine(s, dtype, p, out, lse, st);
    }
    if (e != hipSuccess) return fail_hip(e);
    return SPECPV_OK;
}

// Library-owned scratch for callers that cannot pass a workspace (specpv_partial_verify_attn_static).
// One copy per GPU, alive until the process ends.  In host code the array's name is only a handle:
// the device address comes from hipGetSymbolAddress, once per device, and is what the kernels get.
static __device__ __align__(256) unsigned char scratch[kStaticArray];

static hipError_t static_scratch(void **out)
{
    static void *ptr[64] = {};   // per device; a racing first call stores the same address
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < 64;
    void *p = tracked ? __atomic_load_n(&ptr[dev], __ATOMIC_ACQUIRE) : nullptr;
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // the current device's copy
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        if (tracked) __atomic_store_n(&ptr[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return hipSuccess;
}

// Process-wide choice between one and two launches for scoring + selection (a testing aid, see
// specpv_debug_set_select_route).
static int g_select_route = 0;

static TopkArgs list_args(const specpv_select_cfg *cfg, int32_t *sel_idx, int32_t *sel_count)
{
    return TopkArgs{cfg->n_sink_blocks, cfg->n_recent_blocks, cfg->k_blocks, cfg->n_sink_blocks + cfg->k_blocks + cfg->n_recent_blocks + cfg->n_extra_slots, sel_idx, sel_count};
}

// No sequence can have more blocks than a list keeps: every block is listed, whatever its score, and where the caller does not
// ask for the scores there is no use for them.  Selection and partial step, a layer: 884 tokens, 1 node, 16.4 -> 12.3 us; 2869
// tokens, 59 nodes, 21.5 -> 16.4; fp32, 900 tokens, 18.4 -> 12.8.
static bool keeps_every_block(const Shape &s, const TopkArgs &sel) { return s.max_blocks <= (int64_t)sel.ns + sel.k + sel.nr; }

// arrive: the zeroed arrival words at the head of a workspace, or nullptr where the caller gave none
static int run_select(const Shape &s, int dtype, const specpv_tree *tree, const void *kmax, const void *kmin,
                      const specpv_select_cfg *cfg, int32_t *sel_idx, int32_t *sel_count, float *scores, bool scored,
                      unsigned long long *arrive, hipStream_t st)
{
    const TopkArgs sel = list_args(cfg, sel_idx, sel_count);
    // One launch (the last scoring workgroup of a (sequence, KV head) selects) only on request: it is the
    // slower of the two.  Measured per call at one 128K sequence 18.8 against 16.6 us, at 16K 11.0 against
    // 10.9, for a ragged batch of four 41.4 against 34.6: counting 64 workgroups in costs about what a launch
    // costs, and the last workgroup then starts its selection with cold reads like a fresh kernel would.
    const bool one = arrive && __atomic_load_n(&g_select_route, __ATOMIC_RELAXED) == 1 && score_select_supported(s, dtype);
    // the scoring kernels count query rows: node last_node is row last_node - n_key_only
    hipError_t e = scored ? hipSuccess : launch_scores(s, dtype, kmax, kmin, (int)cfg->reduce, tree->last_node - tree->n_key_only,
                                                       (int)cfg->score, scores, one ? &sel : nullptr, one ? arrive : nullptr, st);
    if (e != hipSuccess) return fail_hip(e);
    if (one && !scored) return SPECPV_OK;
    e = launch_topk(s, scores, sel.ns, sel.nr, sel.k, sel.n_row, sel_idx, sel_count, st);
    if (e != hipSuccess) return fail_hip(e);
    return SPECPV_OK;
}

}  // namespace specpv

using namespace specpv;

extern "C" {

size_t specpv_workspace_bytes(const specpv_kv *kv, const specpv_tree *tree, const specpv_select_cfg *cfg)
{
    if (check_kv(kv) != SPECPV_OK) return 0;
    if (!tree) return kArriveBytes + align_up((size_t)kv->batch * sizeof(int32_t));
    if (check_tree(kv, tree, false) != SPECPV_OK) return 0;
    const Shape s = make_shape(kv, tree);
    AttnPlan plan = plan_attention(s, kv->dtype, s.max_blocks, true, SIZE_MAX);
    if (cfg) {
        const int64_t n_sel = (int64_t)cfg->n_sink_blocks + cfg->k_blocks + cfg->n_recent_blocks + cfg->n_extra_slots;
        const AttnPlan partial = plan_attention(s, kv->dtype, n_sel, false, SIZE_MAX);
        if (partial.nsplit > plan.nsplit) plan = partial;
    }
    return layout_workspace(s, plan, nullptr).total;
}

int specpv_block_summarize(const specpv_kv *kv, int32_t blk_begin, int32_t blk_end,
                           void *kmax, void *kmin, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if (!kmax || !kmin || blk_begin < 0) return SPECPV_EINVAL;
    if (((uintptr_t)kmax | (uintptr_t)kmin) & 15) return SPECPV_EINVAL;
    const Shape s = make_shape(kv, nullptr);
    const hipError_t e = launch_summarize(s, kv->dtype, blk_begin, blk_end, kmax, kmin, (hipStream_t)stream);
    return e == hipSuccess ? SPECPV_OK : fail_hip(e);
}

int specpv_select_blocks(const specpv_kv *kv, const specpv_tree *tree, const void *kmax, const void *kmin,
                         const specpv_select_cfg *cfg, int32_t *sel_idx, int32_t *sel_count, float *scores,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if ((rc = check_tree(kv, tree, false)) != SPECPV_OK) return rc;
    if ((rc = check_cfg(tree, cfg)) != SPECPV_OK) return rc;
    if (!kmax || !kmin || !sel_idx || !sel_count) return SPECPV_EINVAL;
    if (((uintptr_t)kmax | (uintptr_t)kmin) & 15) return SPECPV_EINVAL;
    const Shape s = make_shape(kv, tree);
    const bool no_scores = !scores;
    if (!scores) {
        // behind the arrival words
        const size_t need = kArriveBytes + align_up((size_t)s.batch * s.Hkv * s.max_blocks * sizeof(float));
        if (!workspace || workspace_bytes < need) return SPECPV_EWORKSPACE;
        scores = (float *)((char *)workspace + kArriveBytes);
    }
    const TopkArgs sel = list_args(cfg, sel_idx, sel_count);
    if (no_scores && keeps_every_block(s, sel) && __atomic_load_n(&g_select_route, __ATOMIC_RELAXED) == 0) {
        const hipError_t e = launch_list_all(s, sel, (hipStream_t)stream);
        return e == hipSuccess ? SPECPV_OK : fail_hip(e);
    }
    unsigned long long *arrive = workspace && workspace_bytes >= kArriveBytes ? (unsigned long long *)workspace : nullptr;
    return run_select(s, kv->dtype, tree, kmax, kmin, cfg, sel_idx, sel_count, scores, false, arrive, (hipStream_t)stream);
}

int specpv_partial_verify_attn(const specpv_kv *kv, const specpv_tree *tree, const int32_t *sel_idx,
                               const int32_t *sel_count, int32_t n_sel, void *out, float *lse,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if ((rc = check_tree(kv, tree, true)) != SPECPV_OK) return rc;
    if (!out || ((uintptr_t)out & 15)) return SPECPV_EINVAL;
    if (sel_idx && (!sel_count || n_sel < 0)) return SPECPV_EINVAL;
    if (sel_idx && n_sel > (1 << 24)) return SPECPV_ELIMIT;
    const Shape s = make_shape(kv, tree);
    const AttnPlan plan = plan_attention(s, kv->dtype, sel_idx ? n_sel : s.max_blocks, !sel_idx, workspace_bytes);
    return run_attention(s, plan, kv->dtype, sel_idx, sel_count, n_sel, out, lse, workspace, workspace_bytes, SumArgs{}, (hipStream_t)stream);
}

int specpv_partial_verify_attn_static(const specpv_kv *kv, const specpv_tree *tree, const int32_t *sel_idx,
                                      const int32_t *sel_count, int32_t n_sel, void *out, float *lse, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if ((rc = check_tree(kv, tree, true)) != SPECPV_OK) return rc;
    if (!out || ((uintptr_t)out & 15)) return SPECPV_EINVAL;
    if (sel_idx && (!sel_count || n_sel < 0)) return SPECPV_EINVAL;
    if (sel_idx && n_sel > (1 << 24)) return SPECPV_ELIMIT;
    const Shape s = make_shape(kv, tree);
    // what a plan cut to SPECPV_STATIC_SCRATCH_BYTES has room for there is taken ...
    const int64_t blocks = sel_idx ? n_sel : s.max_blocks;
    const size_t need = static_need(s, plan_attention(s, kv->dtype, blocks, !sel_idx, SIZE_MAX, true));
    if (need > (size_t)SPECPV_STATIC_SCRATCH_BYTES) {
        snprintf(g_hip_err, sizeof(g_hip_err), "static scratch: the call needs %zu bytes, the array holds %zu",
                 need, (size_t)SPECPV_STATIC_SCRATCH_BYTES);
        return SPECPV_ELIMIT;
    }
    // ... and run with the plan of specpv_partial_verify_attn, whose partial results fit the array
    const AttnPlan plan = plan_attention(s, kv->dtype, blocks, !sel_idx, SIZE_MAX);
    if (layout_workspace(s, plan, nullptr).need > (size_t)kStaticArray) {
        snprintf(g_hip_err, sizeof(g_hip_err), "static scratch: the plan needs %zu bytes", layout_workspace(s, plan, nullptr).need);
        return SPECPV_ELIMIT;
    }
    void *ws = nullptr;
    const hipError_t e = static_scratch(&ws);
    if (e != hipSuccess) return fail_hip(e);
    return run_attention(s, plan, kv->dtype, sel_idx, sel_count, n_sel, out, lse, ws, (size_t)kStaticArray, SumArgs{}, (hipStream_t)stream);
}

int specpv_full_verify_refresh(const specpv_kv *kv, const specpv_tree *tree, void *kmax, void *kmin,
                               int32_t stale_blk_begin, const specpv_select_cfg *cfg, void *out, float *lse,
                               int32_t *sel_idx, int32_t *sel_count, float *scores,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if ((rc = check_tree(kv, tree, true)) != SPECPV_OK) return rc;
    if ((rc = check_cfg(tree, cfg)) != SPECPV_OK) return rc;
    if (!kmax || !kmin || !out || !sel_idx || !sel_count) return SPECPV_EINVAL;
    if (((uintptr_t)kmax | (uintptr_t)kmin | (uintptr_t)out) & 15) return SPECPV_EINVAL;
    const Shape s = make_shape(kv, tree);
    AttnPlan plan = plan_attention(s, kv->dtype, s.max_blocks, true, workspace_bytes);
    const Workspace w = layout_workspace(s, plan, workspace);
    if (!workspace || workspace_bytes < w.need || (!scores && workspace_bytes < w.scores_need)) return SPECPV_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    SumArgs sum{};
    if (stale_blk_begin >= 0) sum = side_summaries(s, stale_blk_begin, kmax, kmin, plan);
    if (stale_blk_begin >= 0 && sum.wgs == 0) {
        const hipError_t e = launch_summarize(s, kv->dtype, stale_blk_begin, -1, kmax, kmin, st);
        if (e != hipSuccess) return fail_hip(e);
    }
    // Scores and the merge of the partials in one launch, where the scores have a place of their own: the caller's array, or
    // behind the partials.  (In the place of the partials they can only follow the merge.)
    const size_t behind = align_up(w.need);
    float *apart = scores ? scores : (workspace_bytes >= behind + (w.scores_need - kArriveBytes) ? (float *)((char *)workspace + behind) : nullptr);
    const bool beside = __atomic_load_n(&g_select_route, __ATOMIC_RELAXED) == 0;
    if (!beside) apart = nullptr;   // scoring as a launch of its own, or with the selection
    // Lists of every block go out with the merge as well: one launch less, and no scores that nobody asked for.  Refresh, 60 nodes, 900
    // tokens 14.3 -> 10.5 us, 4000 tokens 18.2 -> 14.3, seven sequences of 624 in blocks of 16 22.2 -> 18.6; 64 channels, 538 tokens,
    // 1 node 13.3 -> 8.9.
    const TopkArgs sel = list_args(cfg, sel_idx, sel_count);
    const bool all = beside && keeps_every_block(s, sel), score = scores || !all;
    const bool all_beside = all && (apart || !score);
    TailScores tail{kmax, kmin, score ? (int)cfg->score : (int)SPECPV_SCORE_EQ2, (int)cfg->reduce, tree->last_node - tree->n_key_only,
                    score ? apart : nullptr, all_beside ? &sel : nullptr, false};
    rc = run_attention(s, plan, kv->dtype, nullptr, nullptr, 0, out, lse, workspace, workspace_bytes, sum, st, &tail);
    if (rc != SPECPV_OK) return rc;
    if (tail.done && tail.all) return SPECPV_OK;
    if (all && !score) {
        const hipError_t e = launch_list_all(s, sel, st);
        return e == hipSuccess ? SPECPV_OK : fail_hip(e);
    }
    return run_select(s, kv->dtype, tree, kmax, kmin, cfg, sel_idx, sel_count, scores ? scores : (apart ? apart : w.scores), tail.done, w.arrive, st);
}

int specpv_gather_blocks(const specpv_kv *kv, const int32_t *sel_idx, const int32_t *sel_count, int32_t n_sel,
                         void *out_k, void *out_v, int32_t *out_len, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if (!sel_idx || !sel_count || !out_k || !out_v || n_sel < 1) return SPECPV_EINVAL;
    if (((uintptr_t)out_k | (uintptr_t)out_v) & 15) return SPECPV_EINVAL;
    if (n_sel > (1 << 24) || (int64_t)n_sel * kv->block_size > ((int64_t)1 << 30)) return SPECPV_ELIMIT;
    if (kv->batch > 65535 || kv->n_kv_heads > 65535) return SPECPV_ELIMIT;   // grid limits, before anything is enqueued
    const Shape s = make_shape(kv, nullptr);
    const hipError_t e = launch_gather(s, kv->dtype, sel_idx, sel_count, n_sel, out_k, out_v, out_len, (hipStream_t)stream);
    return e == hipSuccess ? SPECPV_OK : fail_hip(e);
}

int specpv_select_mode(const specpv_policy *policy, int64_t seq_len, int32_t partial_ready, int32_t n_pending)
{
    if (!policy || policy->partial_budget_tokens < 0 || policy->pending_margin_tokens < 0 || seq_len < 0 || n_pending < 0)
        return SPECPV_EINVAL;
    if (seq_len <= policy->partial_budget_tokens) return SPECPV_MODE_FULL;
    if (!partial_ready) return SPECPV_MODE_FULL;
    if (n_pending > policy->pending_margin_tokens) return SPECPV_MODE_REFRESH;
    return SPECPV_MODE_PARTIAL;
}

int specpv_extend_parents(const int32_t *tree_parent, int32_t M_tree, int32_t n_pending, int32_t *out)
{
    if (!tree_parent || !out || M_tree < 1 || n_pending < 0) return SPECPV_EINVAL;
    if ((int64_t)M_tree + n_pending > SPECPV_MAX_M) return SPECPV_ELIMIT;
    for (int32_t i = 0; i < n_pending; ++i) out[i] = i - 1;
    for (int32_t j = 0; j < M_tree; ++j) {
        if (tree_parent[j] >= j) return SPECPV_EINVAL;
        out[n_pending + j] = tree_parent[j] < 0 ? n_pending - 1 : tree_parent[j] + n_pending;
    }
    return SPECPV_OK;
}

int specpv_commit_accepted(const specpv_kv *kv, void *buf_k, void *buf_v, int32_t pending_cap, int32_t M_tree,
                           int32_t *n_pending, const int32_t *accepted, const int32_t *n_accepted,
                           int32_t max_accept, specpv_mode mode, void *kmax, void *kmin,
                           const specpv_lists *lists, int32_t *dropped,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_kv(kv);
    if (rc != SPECPV_OK) return rc;
    if (!buf_k || !buf_v || !n_pending || !accepted || !n_accepted) return SPECPV_EINVAL;
    if (lists && (!lists->sel_idx || !lists->sel_count || lists->n_sel < 1)) return SPECPV_EINVAL;
    if (lists && lists->n_sel > (1 << 24)) return SPECPV_ELIMIT;
    if (pending_cap < 0 || M_tree < 1 || max_accept < 1) return SPECPV_EINVAL;
    if (mode != SPECPV_MODE_FULL && mode != SPECPV_MODE_PARTIAL && mode != SPECPV_MODE_REFRESH) return SPECPV_EINVAL;
    if (((uintptr_t)buf_k | (uintptr_t)buf_v) & 15) return SPECPV_EINVAL;
    if ((kmax || kmin) && (!kmax || !kmin || (((uintptr_t)kmax | (uintptr_t)kmin) & 15))) return SPECPV_EINVAL;
    if ((int64_t)pending_cap + max_accept > 128 || (int64_t)pending_cap + M_tree > SPECPV_MAX_M) return SPECPV_ELIMIT;
    if (!workspace || workspace_bytes < kArriveBytes + (size_t)kv->batch * sizeof(int32_t)) return SPECPV_EWORKSPACE;
    const Shape s = make_shape(kv, nullptr);
    void *k1 = const_cast<void *>(kv->k), *v1 = const_cast<void *>(kv->v);
    const hipError_t e = launch_commit(s, kv->dtype, 1, &k1, &v1, &buf_k, &buf_v, pending_cap, M_tree, n_pending, accepted,
                                       n_accepted, max_accept, mode != SPECPV_MODE_PARTIAL, &kmax, &kmin,
                                       lists, dropped, (uint32_t *)workspace, (hipStream_t)stream);
    return e == hipSuccess ? SPECPV_OK : fail_hip(e);
}

int specpv_commit_accepted_layers(const specpv_kv *const *kv, void *const *buf_k, void *const *buf_v, int32_t n_layers,
                                  int32_t pending_cap, int32_t M_tree, int32_t *n_pending, const int32_t *accepted,
                                  const int32_t *n_accepted, int32_t max_accept, specpv_mode mode,
                                  void *const *kmax, void *const *kmin, const specpv_lists *lists, int32_t *dropped,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (!kv || !buf_k || !buf_v || n_layers < 1 || n_layers > SPECPV_MAX_LAYERS) return SPECPV_EINVAL;
    if (!n_pending || !accepted || !n_accepted) return SPECPV_EINVAL;
    if (pending_cap < 0 || M_tree < 1 || max_accept < 1) return SPECPV_EINVAL;
    if (mode != SPECPV_MODE_FULL && mode != SPECPV_MODE_PARTIAL && mode != SPECPV_MODE_REFRESH) return SPECPV_EINVAL;
    if ((int64_t)pending_cap + max_accept > 128 || (int64_t)pending_cap + M_tree > SPECPV_MAX_M) return SPECPV_ELIMIT;
    if ((kmax == nullptr) != (kmin == nullptr)) return SPECPV_EINVAL;
    void *kp[SPECPV_MAX_LAYERS], *vp[SPECPV_MAX_LAYERS];
    for (int l = 0; l < n_layers; ++l) {
        const specpv_kv *x = kv[l];
        const int rc = check_kv(x);
        if (rc != SPECPV_OK) return rc;
        // one shape, one set of strides, one dtype and the same length counters for all layers
        if (x->batch != kv[0]->batch || x->n_kv_heads != kv[0]->n_kv_heads || x->head_dim != kv[0]->head_dim ||
            x->block_size != kv[0]->block_size || x->max_blocks != kv[0]->max_blocks || x->dtype != kv[0]->dtype ||
            x->stride_b != kv[0]->stride_b || x->stride_h != kv[0]->stride_h || x->stride_t != kv[0]->stride_t ||
            x->ctx_len != kv[0]->ctx_len)
            return SPECPV_EINVAL;
        if (!buf_k[l] || !buf_v[l] || (((uintptr_t)buf_k[l] | (uintptr_t)buf_v[l]) & 15)) return SPECPV_EINVAL;
        if (kmax) {   // summaries for every layer or for none
            const bool want = kmax[0] != nullptr;
            if ((kmax[l] != nullptr) != want || (kmin[l] != nullptr) != want) return SPECPV_EINVAL;
            if (((uintptr_t)kmax[l] | (uintptr_t)kmin[l]) & 15) return SPECPV_EINVAL;
        }
        if (lists) {
            if (!lists[l].sel_idx || !lists[l].sel_count || lists[l].n_sel < 1 || lists[l].n_sel != lists[0].n_sel)
                return SPECPV_EINVAL;
            if (lists[l].n_sel > (1 << 24)) return SPECPV_ELIMIT;
        }
        kp[l] = const_cast<void *>(x->k);
        vp[l] = const_cast<void *>(x->v);
    }
    if (!workspace || workspace_bytes < kArriveBytes + (size_t)kv[0]->batch * sizeof(int32_t)) return SPECPV_EWORKSPACE;
    const Shape s = make_shape(kv[0], nullptr);
    const hipError_t e = launch_commit(s, kv[0]->dtype, n_layers, kp, vp, buf_k, buf_v, pending_cap, M_tree, n_pending,
                                       accepted, n_accepted, max_accept, mode != SPECPV_MODE_PARTIAL, kmax, kmin,
                                       lists, dropped, (uint32_t *)workspace, (hipStream_t)stream);
    return e == hipSuccess ? SPECPV_OK : fail_hip(e);
}

const char *specpv_strerror(int status)
{
    switch (status) {
    case SPECPV_OK: return "ok";
    case SPECPV_EINVAL: return "invalid argument (null pointer, shape, dtype, head dim, stride or alignment)";
    case SPECPV_EWORKSPACE: return "workspace missing or too small (see specpv_workspace_bytes)";
    case SPECPV_ELIMIT: return "size beyond the documented limits";
    case SPECPV_EHIP: return "HIP launch failed (see specpv_last_hip_error)";
    default: return "unknown status";
    }
}

const char *specpv_last_hip_error(void) { return g_hip_err; }

int specpv_debug_set_timeline(void *buf)
{
#ifndef SPECPV_TIMELINE
    if (buf) return SPECPV_EINVAL;   // this build takes no time stamps
#endif
    g_timeline = (unsigned long long *)buf;
    return SPECPV_OK;
}

int specpv_debug_set_route(int route)
{
    if (route < 0 || route > 3) return SPECPV_EINVAL;
    __atomic_store_n(&g_route, route, __ATOMIC_RELAXED);
    return SPECPV_OK;
}

int specpv_debug_set_select_route(int route)
{
    if (route < 0 || route > 2) return SPECPV_EINVAL;
    __atomic_store_n(&g_select_route, route, __ATOMIC_RELAXED);
    return SPECPV_OK;
}

int specpv_version(void) { return 202; }

}  // extern "C"
