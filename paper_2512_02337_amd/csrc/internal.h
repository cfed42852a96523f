// Internal declarations shared by the HIP translation units of libspecpv.
// Each .hip file owns its kernels and exposes one host launcher; api.hip
// validates arguments and calls the launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "specpv.h"

namespace specpv {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Exact n / d for 0 <= n < 2^31 with a host-prepared multiplier (no integer divide
// on the GPU: one takes about forty vector instructions).
struct FastDiv {
    uint32_t mul, shift, d;
    __device__ __forceinline__ uint32_t div(uint32_t n) const { return d == 1 ? n : (__umulhi(n, mul) >> shift); }
    // the same without a branch: its three numbers are then read where it stands, not at the kernel's entry
    __device__ __forceinline__ uint32_t div_straight(uint32_t n) const
    {
        const uint32_t q = __umulhi(n, mul) >> shift;
        return d == 1 ? n : q;
    }
};
static FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    f.d = d;
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;                       // l = ceil(log2 d)
    if (d <= 1) { f.mul = 0; f.shift = 0; return f; }
    f.mul = (uint32_t)(((1ull << (31 + l)) + d - 1) / d);   // ceil(2^(31+l) / d) <= 2^32 - 1 for d >= 2
    f.shift = l - 1;
    return f;
}

// Flat view of one call's tensors, passed by value to the kernels.
struct Shape {
    const void *k, *v;            // context KV, read in place
    int64_t sb, sh, st;           // element strides of k / v: batch, head, token
    const int32_t *ctx_len;       // [batch]
    const void *q;                // [batch, M, Hq, D]
    const void *kd, *vd;          // [batch, Mk, Hkv, D]
    const int32_t *parent;        // [batch, Mk]
    int batch, Hkv, Hq, G, D, B, M, max_blocks;
    // M counts the QUERY nodes (rows of q, out, the partials).  The tree has Mk >= M nodes: its
    // first koff = Mk - M nodes are keys only (partially verified tokens on a partial step);
    // query row r is node koff + r.
    int Mk, koff;
    // Of those, the first kctx (0 or koff) are attended by the context kernels as if they were cache
    // tokens -- they are a chain from which every query node descends, so every row sees all of them --
    // and the draft-tree segment (combine kernel, single-kernel route) stops its root paths there.
    int kctx;
};

// How the kernels of one short call find their piece of work without waiting for their argument block: where a sequence has
// 8, 16, 32, ... KV heads, grid z counts groups of eight of them (KV head g on XCD g % 8, which is blockIdx.x % 8), and a shift
// that arrives in a register with the leading arguments does the rest.  0: no such number; else 1 + log2(Hkv / 8).
static inline int head_groups_code(int Hkv)
{
    for (int sh = 0; sh < 16; ++sh)
        if (Hkv == 8 << sh) return 1 + sh;
    return 0;
}

// Split-KV partial results of the context part, one per (b, g, split, row), row hh * M + j of KV head g being node j of
// its query head hh (the single-kernel route keeps its own order, [batch, Hq, nsplit, M]: it reads them back itself):
//   part_ml [batch, Hkv, nsplit, M * G, 2] fp32   (m, l): m = max_t z_t, l = sum_t 2^(z_t - m),
// with z = q.k * log2(e)/sqrt(D).  A split without any valid token stores m = -inf, l = 0.
//   part_o, one of two forms:
//   o_half == 0:  [batch, Hkv, nsplit, M * G, D] fp32   sum_t 2^(z_t - m) v_t   (not normalised).  Inside a row
//     with D = 128 the channels are stored in the order the combine kernel reads them (a lane of 16 owns
//     channels 8 i .. 8 i + 7 and fetches them as two 16-byte pieces, each piece dense over the 16 lanes):
//     channel c sits at partial_pos(c).  D = 64: in order.  (vector-ALU kernel: fp32 inputs and their 1e-5
//     bar; 64 channels; single-kernel route.)
//   o_half == 1:  [batch, Hkv, nsplit, M * G, D] fp16   the split's own softmax result, sum_t 2^(z_t - m) v_t / l
//     (0 if l = 0), channels in order.  A convex combination of V rows, so within fp16's range as long as
//     |v| <= 65504 (larger magnitudes are clamped); its 11 significant bits are 8 times finer than the
//     bf16 output.  Half the bytes of the fp32 form: the partials are the call's second-largest traffic.
// stream > 0: no fixed number of splits.  The chunks of all (sequence, KV head) pairs in a row are dealt to `stream`
// workgroups in equal, contiguous shares (StreamShare), and the partial of workgroup w for pair u stands in slot w + u --
// pairs and workgroups both advance along the row, so no two (w, u) that meet share a slot, and a pair's slots are
// adjacent.
struct Partials {
    float *o;
    float *ml;
    int nsplit;
    int o_half;
    int stream;
    unsigned long long *timeline;   // instrumented builds (-DSPECPV_TIMELINE): the combine kernel's time stamps go to rows 2048.. of this buffer
};
__host__ __device__ constexpr int partial_pos(int c, int D)
{
    return D == 128 ? ((c >> 2) & 1) * 64 + (c >> 3) * 4 + (c & 3) : c;
}
// ... and the channel that sits at position p (the inverse)
__host__ __device__ constexpr int partial_chan(int p, int D)
{
    return D == 128 ? ((p & 63) >> 2) * 8 + (p >> 6) * 4 + (p & 3) : p;
}
constexpr bool partial_order_is_a_permutation()
{
    for (int D = 64; D <= 128; D += 64)
        for (int p = 0; p < D; ++p) {
            const int c = partial_chan(p, D);
            if (c < 0 || c >= D || partial_pos(c, D) != p) return false;
            // a lane's 16-byte piece holds four consecutive channels, in order
            if ((p & 3) != 0 && c != partial_chan(p - 1, D) + 1) return false;
        }
    return true;
}
static_assert(partial_order_is_a_permutation(), "partial_pos / partial_chan must be inverse permutations of a row");

// The shares of the workgroups where Partials::stream > 0: every wavefront works them out from the sequence lengths (at
// most 64 sequences, one per lane).  A sequence counts its chunks of 32 cache tokens (whole blocks) and of partially
// verified tokens.
struct StreamShare {
    int chunks, upto;     // of sequence `lane`: its chunks, and those of the sequences 0 .. lane (one KV head)
    int total, wgs;       // chunks of all pairs; workgroups with a share
    int share, longer;    // the first `longer` shares have share + 1 chunks, the others share
    __device__ __forceinline__ StreamShare(const Shape &s, int lane, int stream)
    {
        const int L = lane < s.batch ? s.ctx_len[lane] : 0;
        int nb = L > 0 ? (int)(((uint32_t)L + (uint32_t)s.B - 1u) / (uint32_t)s.B) : 0;
        if (nb > s.max_blocks) nb = s.max_blocks;
        chunks = lane < s.batch ? (int)(((uint32_t)nb * (uint32_t)s.B + 31u) >> 5) + ((s.kctx + 31) >> 5) : 0;
        upto = chunks;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int below = __shfl_up(upto, o);
            upto += lane >= o ? below : 0;
        }
        total = __builtin_amdgcn_readlane(upto, 63) * s.Hkv;
        wgs = min(stream, total);
        share = wgs > 0 ? (int)((uint32_t)total / (uint32_t)wgs) : 0;
        longer = total - share * wgs;
    }
    // where the share of workgroup w begins, and the workgroup whose share chunk x lies in
    __device__ __forceinline__ int begin(int w) const { return w * share + min(w, longer); }
    __device__ __forceinline__ int owner(int x) const
    {
        const int head = longer * (share + 1);
        return x < head ? (int)((uint32_t)x / (uint32_t)(share + 1)) : longer + (int)((uint32_t)(x - head) / (uint32_t)share);
    }
};

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kPerVec = 4;  // elements per 16-byte vector
    static __device__ __forceinline__ void unpack(const uint4 &u, float *f) {
        f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y);
        f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
    }
    static __device__ __forceinline__ uint4 pack(const float *f) {
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    }
    static __device__ __forceinline__ float load(const void *p, int64_t i) { return ((const float *)p)[i]; }
    static __device__ __forceinline__ void store(void *p, int64_t i, float x) { ((float *)p)[i] = x; }
    static __device__ __forceinline__ void store_stream(void *p, int64_t i, float x) { __builtin_nontemporal_store(x, (float *)p + i); }
};
struct bf16_t { uint16_t bits; };
__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }
// Two fp32 values as bf16, rounded to nearest, ties to even (NaN stays NaN): v_cvt_pk_bf16_f32, the same bits as integer arithmetic
// for all 2^32 inputs.  That is sixteen instructions a value, with a branch for NaN that keeps the values of a row from
// overlapping; partial verification at 128K, 16 layers, 236.9 us with it in the combine kernel, 233.7 so.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b)
{
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
template <> struct Elem<bf16_t> {
    static constexpr int kPerVec = 8;
    static __device__ __forceinline__ void unpack(const uint4 &u, float *f) {
        f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xffff0000u);
        f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xffff0000u);
        f[4] = __uint_as_float(u.z << 16); f[5] = __uint_as_float(u.z & 0xffff0000u);
        f[6] = __uint_as_float(u.w << 16); f[7] = __uint_as_float(u.w & 0xffff0000u);
    }
    static __device__ __forceinline__ uint4 pack(const float *f) {   // values that are exactly representable
        return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
    }
    static __device__ __forceinline__ float load(const void *p, int64_t i) {
        return bf16_bits_to_float(((const uint16_t *)p)[i]);
    }
    static __device__ __forceinline__ void store(void *p, int64_t i, float x) {
        ((uint16_t *)p)[i] = (uint16_t)pack_bf16x2(x, x);
    }
    static __device__ __forceinline__ void store_stream(void *p, int64_t i, float x) {
        __builtin_nontemporal_store((uint16_t)pack_bf16x2(x, x), (uint16_t *)p + i);
    }
};

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// Sum over the 16 lanes of a DPP row, result in every lane of the row: lane ^ 1, lane ^ 2,
// then the mirrors inside 8 and 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_row(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_sum(float x)
{
    x += dpp_row<0xB1>(x);
    x += dpp_row<0x4E>(x);
    x += dpp_row<0x141>(x);
    x += dpp_row<0x140>(x);
    return x;
}

// The root path of tree node j as a bit set; par0 / par1 hold parent[lane] / parent[lane + 64].  Everything is
// wave-uniform (scalar registers).  Nodes below `stop` (partially verified tokens that the context kernels have attended
// already) end the walk.
__device__ __forceinline__ void root_path(int j, int n_nodes, int stop, int par0, int par1, unsigned long long &lo, unsigned long long &hi)
{
    int at = j;
    for (int guard = 0; at >= stop && guard < n_nodes; ++guard) {
        // (values, not a choice between two variables: the compiler would put those into memory)
        const unsigned long long bit = 1ull << (at & 63);
        lo |= at < 64 ? bit : 0ull;
        hi |= at < 64 ? 0ull : bit;
        const int pa = __builtin_amdgcn_readlane(at < 64 ? par0 : par1, at & 63);
        at = pa < at ? pa : -1;   // a malformed parent[] (not strictly decreasing) ends the walk
    }
}
// lowest node of the set (removed from it), or -1
__device__ __forceinline__ int pop_node(unsigned long long &lo, unsigned long long &hi)
{
    const bool low = lo != 0ull;
    const unsigned long long word = low ? lo : hi;
    const int at = word ? __builtin_ctzll(word) + (low ? 0 : 64) : -1;
    lo &= lo - (low ? 1ull : 0ull);
    hi &= hi - (low || hi == 0ull ? 0ull : 1ull);
    return at;
}

// ---- launchers (each returns the hipError_t of its launches) ----
hipError_t launch_summarize(const Shape &s, int dtype, int blk_begin, int blk_end,
                            void *kmax, void *kmin, hipStream_t st);
// One selection: kept-block lists of n_row entries (>= ns + k + nr; the rest is padding for later
// commits), ascending, -1 behind the count.
struct TopkArgs {
    int ns, nr, k, n_row;
    int32_t *sel_idx, *sel_count;
};
// kind: SPECPV_SCORE_EQ2 or SPECPV_SCORE_CHANNEL_BOUND.  sel != nullptr: the selection runs in the same
// launch; only where score_select_supported() holds, with arrive pointing to the kArriveBytes of zeroed
// arrival words at the head of a workspace (zero again when the launch has finished).
bool score_select_supported(const Shape &s, int dtype);
hipError_t launch_scores(const Shape &s, int dtype, const void *kmax, const void *kmin,
                         int reduce, int last_node, int kind, float *scores, const TopkArgs *sel,
                         unsigned long long *arrive, hipStream_t st);
// n_row: entries per list row (>= ns + k + nr; the rest is padding for later commits)
hipError_t launch_topk(const Shape &s, const float *scores, int ns, int nr, int k, int n_row,
                       int32_t *sel_idx, int32_t *sel_count, hipStream_t st);
// every block into every list: s.max_blocks <= ns + k + nr
hipError_t launch_list_all(const Shape &s, const TopkArgs &a, hipStream_t st);
// fp32 with several tiles of query rows to a KV head (attn_f32.hip), kF32Rows rows to a workgroup
constexpr int kF32Rows = 64;
hipError_t launch_attn_ctx_f32(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count, int n_sel, Partials p, hipStream_t st);
hipError_t launch_attn_ctx_generic(const Shape &s, int dtype, const int32_t *sel_idx,
                                   const int32_t *sel_count, int n_sel, Partials p, hipStream_t st);
bool attn_ctx_mfma_supported(const Shape &s, int dtype);
// Which kernel computes the context part, and with how many KV splits.  kAttnSplit: eight
// wavefronts per (query head, split), for short token ranges; kAttnGroup: the query heads of a KV
// head in one workgroup (two or more for more than eight 32-row blocks), for long ranges;
// kAttnGeneric: any dtype / head dim.
enum AttnKind { kAttnGeneric = 0, kAttnSplit = 1, kAttnGroup = 3 };
struct AttnPlan {
    int nsplit;
    int kind;
    int tg;       // kAttnSplit: token groups per workgroup; kAttnGeneric: 1 where attn_f32.hip does it
    int stream;   // kAttnGroup: workgroups that share the chunks of all pairs (see Partials), or 0
};
// The whole call in the eight-wavefront kernel (kAttnSplit only): the draft-tree segment as one more
// partial (slot nctx of nctx + 1), arrival words, the last workgroup of a tile merges and stores.
// out == nullptr: the kernel only writes partials and launch_combine finishes.
struct FusedArgs {
    void *out;                     // [batch, M, Hq, 128] bf16
    float *lse;                    // optional [batch, M, Hq]
    unsigned long long *arrive;    // [batch, Hq, 2] arrival words, zero between calls
    int force_recompute;           // test hook: the last workgroup of a tile takes the recompute route
    unsigned long long *timeline;  // builds with -DSPECPV_TIMELINE: 16 time stamps per workgroup (else unused)
};
constexpr size_t kArriveBytes = 64 << 10;   // head of every workspace: 8192 arrival words
// The summaries that a full pass recomputes on the side (kAttnGroup): workgroups for it, or 0; the blocks from `begin` on.
struct SumArgs {
    int wgs, begin;
    void *kmax, *kmin;
};
// p.nsplit: slots per (sequence, head) in the partial arrays = nctx, or nctx + 1 when fused
hipError_t launch_attn_ctx_mfma(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count,
                                int n_sel, Partials p, int nctx, int kind, const FusedArgs &f, const SumArgs &sum, hipStream_t st);
// the kAttnSplit kernel (two-kernel route): tg = 2, 4 or 8 token groups and 256 / tg query rows per workgroup
hipError_t launch_attn_ctx_tile(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count, int n_sel, Partials p,
                                int tg, unsigned long long *timeline, hipStream_t st);
// workgroups per (sequence, KV head, split) of the kAttnGroup kernel
int attn_group_parts(const Shape &s);
int attn_group_blocks(const Shape &s);   // row blocks of each
double attn_group_chunk_us(int blocks);
hipError_t launch_combine(const Shape &s, int dtype, Partials p, void *out, float *lse, hipStream_t st);
bool combine_packed(const Shape &s, int dtype);
// the merge and the scores (eq. 2; scores == nullptr: none) in one launch; kind: as for launch_scores.  all != nullptr: and lists of
// every block (launch_list_all)
bool refresh_tail_supported(const Shape &s, int dtype, const Partials &p, int kind);
bool refresh_tail_pays(const Shape &s, const Partials &p, int reduce, int last_node);   // (with scores)
hipError_t launch_refresh_tail(const Shape &s, Partials p, void *out, float *lse, const void *kmax, const void *kmin, int reduce, int last_node,
                               float *scores, const TopkArgs *all, hipStream_t st);
// to_cache != 0: pending + accepted rows go to the cache tail (lengths, summaries updated);
// otherwise the accepted rows join the pending rows of the buffer.  missed_words: the zeroed words at the
// head of a workspace (kArriveBytes; zero again when the launches have finished).
// n_layers layers that share shape, strides and counters are committed together.
// lists (n_layers entries, or nullptr): kept-block lists that take in the blocks a commit to the
// cache touches.  dropped ([batch, 2], or nullptr): tokens not stored, list entries not found.
hipError_t launch_commit(const Shape &s, int dtype, int n_layers, void *const *k, void *const *v,
                         void *const *buf_k, void *const *buf_v, int P, int Mt,
                         int32_t *n_pending, const int32_t *accepted, const int32_t *n_accepted,
                         int max_accept, int to_cache, void *const *kmax, void *const *kmin,
                         const specpv_lists *lists, int32_t *dropped, uint32_t *missed_words,
                         hipStream_t st);

hipError_t launch_gather(const Shape &s, int dtype, const int32_t *sel_idx, const int32_t *sel_count, int n_sel,
                         void *out_k, void *out_v, int32_t *out_len, hipStream_t st);

int device_cu_count();   // of the current device

// One-time set-up per (kernel, device): `fn` runs once for each device it is asked for, also when
// several threads make their first call at the same moment.  Devices beyond 63 run it every time.
struct PerDeviceOnce {
    unsigned long long done = 0;   // bit d: fn has succeeded on device d (accessed atomically)
    template <typename F> hipError_t run(F fn)
    {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const bool tracked = dev >= 0 && dev < 64;
        if (tracked && ((__atomic_load_n(&done, __ATOMIC_ACQUIRE) >> dev) & 1ull)) return hipSuccess;
        e = fn();   // idempotent: two threads that race here both set the same attribute
        if (e == hipSuccess && tracked) __atomic_fetch_or(&done, 1ull << dev, __ATOMIC_RELEASE);
        return e;
    }
};

}  // namespace specpv
