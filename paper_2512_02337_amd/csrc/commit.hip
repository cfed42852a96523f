// KV side of what follows a verify step (Section 3.2: the candidates' K/V wait in the buffer
// until verification has decided which of them survive; Section 3.3: a full verification
// moves the partially verified tokens into the cache).  Pure data
// movement of at most a few dozen rows per (sequence, KV head), then the block summaries
// (eq. 1) of the blocks that received tokens.
#include "internal.h"

namespace specpv {

constexpr int kCommitMaxRows = 128;   // pending + accepted rows one call moves per sequence (host-checked)

// Several layers in one launch: blockIdx.z picks the layer's pointers from a table that travels
// with the kernel arguments.  All layers share one shape, one set of strides and the counters.
constexpr int kCommitLayers = 32;   // layers per launch
struct CommitLayers {
    void *k[kCommitLayers], *v[kCommitLayers], *buf_k[kCommitLayers], *buf_v[kCommitLayers];
    void *kmax[kCommitLayers], *kmin[kCommitLayers];
    int32_t *idx[kCommitLayers], *cnt[kCommitLayers];
};
// The same where every layer's tensors follow the last layer's at one distance, as those do that are slices of one tensor of all
// layers: 128 bytes of arguments instead of 2 KiB, which the host copies for every launch: 32 layers
// with lists and summaries, host 7.8 -> 6.4 us, pass 10.8 -> 10.3 (the GPU's) or 12.2 -> 10.1 (the host's).
struct CommitStacked {
    struct Array {
        char *first;
        int64_t step;
        template <typename T = void> __host__ __device__ __forceinline__ T *at(int l) const { return (T *)(first + l * step); }
        // n pointers (nullptr: of none)
        bool set(void *const *p, int n)
        {
            first = (char *)p[0];
            step = n > 1 ? (int64_t)((uintptr_t)p[1] - (uintptr_t)p[0]) : 0;
            for (int l = 2; l < n; ++l)
                if ((uintptr_t)p[l] != (uintptr_t)first + (uintptr_t)(l * step)) return false;
            return true;
        }
    } k, v, buf_k, buf_v, kmax, kmin, idx, cnt;
    bool set(const CommitLayers &x, int n)
    {
        return k.set(x.k, n) && v.set(x.v, n) && buf_k.set(x.buf_k, n) && buf_v.set(x.buf_v, n) && kmax.set(x.kmax, n) && kmin.set(x.kmin, n) &&
               idx.set((void *const *)x.idx, n) && cnt.set((void *const *)x.cnt, n);
    }
};
// A layer's tensors.
struct CommitLayer {
    void *k, *v, *buf_k, *buf_v, *kmax, *kmin;
    int32_t *idx, *cnt;
};
__device__ __forceinline__ CommitLayer layer_of(const CommitLayers &t, int l) { return {t.k[l], t.v[l], t.buf_k[l], t.buf_v[l], t.kmax[l], t.kmin[l], t.idx[l], t.cnt[l]}; }
__device__ __forceinline__ CommitLayer layer_of(const CommitStacked &t, int l)
{
    return {t.k.at(l), t.v.at(l), t.buf_k.at(l), t.buf_v.at(l), t.kmax.at(l), t.kmin.at(l), t.idx.at<int32_t>(l), t.cnt.at<int32_t>(l)};
}
// Words of a sequence at the head of the workspace, zero before and after the call: list entries that found no room, the
// workgroups that have arrived (see arrive_and_update), and those of each of sixteen groups of them.  Each on a 128-byte line
// of its own where a launch has few enough sequences.
constexpr int kCommitWords = 18;
constexpr int kCommitSeqs = (int)(kArriveBytes / (kCommitWords * sizeof(uint32_t)));   // sequences per launch
struct CommitArrive {
    uint32_t *words;
    int stride;      // of a sequence's words, in words
    int workgroups;  // of a sequence; 0: a launch follows that moves the counters
    int32_t *ctx_len, *n_pending, *dropped;
};

// The counters (lengths, pending tokens) are read by every workgroup and moved once: by the workgroup of a sequence that finds
// itself last to have read them.  Nobody waits, and no launch of a thread a sequence stands behind this one (32 layers: kernels
// 7.6 + 1.4 us and the gap between them, 8.4 so; a pass, which is the host's time, 14.6 -> 11.5 us side by side).  Counting goes
// over sixteen groups: atomics on one address go one after the other, 70 ns each.  One lane calls this, behind the barrier that
// its workgroup's reads of the counters stand in front of; a count of missed entries has to be there before its arrival is.
__device__ __forceinline__ void arrive_and_update(const CommitArrive &ar, int bl, int b, int id, uint32_t missed, bool lists, bool to_cache, int L, int n_plus_a, int total)
{
    uint32_t *const w = ar.words + (int64_t)bl * kCommitWords * ar.stride;
    if (missed) {
        const uint32_t before = __hip_atomic_fetch_max(w, missed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::"v"(before) : "memory");
    }
    if (!ar.workgroups) return;
    auto last_of = [](uint32_t *word, uint32_t n) {
        if (__hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u != n) return false;
        __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    };
    const int N = ar.workgroups, j = id & 15;
    if (N > 16 && !last_of(w + (2 + j) * ar.stride, (uint32_t)((N - j + 15) >> 4))) return;
    if (!last_of(w + ar.stride, (uint32_t)min(N, 16))) return;
    const uint32_t all_missed = lists ? __hip_atomic_exchange(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (to_cache) ar.ctx_len[b] = L + total;
    ar.n_pending[b] = to_cache ? 0 : total;
    if (ar.dropped) {
        ar.dropped[2 * b] = n_plus_a - total;        // tokens that found no room
        ar.dropped[2 * b + 1] = (int32_t)all_missed;   // list entries that found no room
    }
}

// Everything that a commit does for one (KV head, sequence, layer), by one workgroup; a row of D elements is
// D * sizeof(T) / 16 lanes.  What bounds it is the chain of cold reads -- counters, then rows, then the touched
// blocks' older rows, with them -- of a few KiB each, so the whole of it is one launch (copy, lists and summaries as launches of
// their own took 4.9 + 3.3 + 8.4 us for 32 layers, of which this takes 7.0).
//  * Rows that move within the buffer are read into registers, all of them, before anything is written; and so are those of a
//    buffer that lies in the cache (one sequence, token-major: candidates written where the cache goes on, and moved up here).
//  * Lists (Section 3.3: the committed tokens stay part of the partial cache): every block that received a token joins
//    the kept-block list behind the entries it has, unless it is listed already (the ragged last block of the local
//    window).
//  * Summaries (eq. 1) of the blocks that received tokens: a wavefront per block, lanes over 16-byte pieces of a row.
// ROWS: the rows that a workgroup keeps in registers.  Rows that move within one array are all of them; others that go to the cache
// go there so many at a time.
// kInPlace: out of a buffer that lies in the cache; the summaries then read the new rows back.
enum CommitTo { kWithinBuffer, kToCache, kInPlace };
template <typename T, int D, int ROWS, CommitTo TO, typename LAYERS>
__global__ __launch_bounds__(256) void commit_kernel(Shape s, LAYERS layers, int b0, int P, int Mt, const int32_t *n_pending,
                                                     const int32_t *accepted, const int32_t *n_accepted, int max_accept,
                                                     int with_sums, int n_sel, CommitArrive ar)
{
    constexpr bool to_cache = TO != kWithinBuffer, IN_PLACE = TO == kInPlace;
    const CommitLayer lay = layer_of(layers, (int)blockIdx.z);
    T *const buf_k = (T *)lay.buf_k, *const buf_v = (T *)lay.buf_v;
    T *const cache_k = (T *)lay.k, *const cache_v = (T *)lay.v;
    constexpr int E = Elem<T>::kPerVec;
    constexpr int LPR = D / E;                     // lanes per row
    constexpr int RPP = 256 / LPR;                 // rows per pass
    constexpr int PASSES = (ROWS + RPP - 1) / RPP;
    const int g = blockIdx.x, bl = blockIdx.y, b = b0 + bl;
    const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int L = s.ctx_len[b];
    const int n_raw = n_pending[b], a_raw = n_accepted[b];
    // the accepted path, requested with the counters: lane t holds entries t and t + 64 (max_accept <= 128)
    const int32_t *acc = accepted + (int64_t)b * max_accept;
    const int acc0 = lane < max_accept ? acc[lane] : 0, acc1 = lane + 64 < max_accept ? acc[lane + 64] : 0;
    const int n = min(max(n_raw, 0), P);
    const int a = min(max(a_raw, 0), max_accept);
    int total = n + a;
    if (to_cache) total = min(total, max(0, s.max_blocks * s.B - L));   // the cache is full: the rest is dropped
    else total = min(total, P);
    const int64_t buf_rows = (int64_t)P + Mt;
    auto buf_row = [&](T *base, int row) -> uint4 * {
        return (uint4 *)(base + (((int64_t)b * buf_rows + row) * s.Hkv + g) * D) + c;
    };
    const bool sums = to_cache && total > 0 && with_sums;    // uniform
    const int first = L / s.B, last = (L + total - 1) / s.B;        // blocks that received tokens (all below max_blocks)
    // The wavefronts of a call to the cache meet once, here, where each has read the counters (the fourth may move them from
    // here on), and then go their own ways: whatever one needs of the rows it reads itself, all of it in one trip.  (Summaries of
    // rows read back from the cache behind the stores, two more trips in the chain: 32 layers of one sequence in blocks of 64 / of
    // 16 tokens, 16 layers of 16 sequences 7.9 / 7.8 / 15.5 us; 7.0 / 6.1 / 13.1 so.)
    if (to_cache) {
        asm volatile("" :: "v"(L), "v"(n_raw), "v"(a_raw) : "memory");
        __builtin_amdgcn_s_barrier();
    }
    // the list that the fourth wavefront looks after: requested with the rows, entries lane and lane + 64
    const bool with_list = wave == 3 && n_sel && to_cache;   // uniform
    int32_t *const list = with_list ? lay.idx + ((int64_t)b * s.Hkv + g) * n_sel : nullptr;
    int32_t *const cntp = with_list ? lay.cnt + (int64_t)b * s.Hkv + g : nullptr;
    int cnt_raw = 0, list0 = -1, list1 = -1;
    if (with_list) {
        cnt_raw = *cntp;
        if (lane < n_sel) list0 = list[lane];
        if (lane + 64 < n_sel) list1 = list[lane + 64];
    }
    // where row i of those that move comes from
    auto source = [&](int i) -> int {
        const int x = i - n;
        const int e0 = __shfl(acc0, x & 63), e1 = __shfl(acc1, x & 63);
        return i < n ? P - n + i                                    // pending token i (oldest first)
                     : P + min(max(x < 64 ? e0 : e1, 0), Mt - 1);   // accepted candidate
    };
    uint4 kr[PASSES], vr[PASSES];
    auto read_rows = [&](int from) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int i = from + p * RPP + r0, src = source(i);
            kr[p] = vr[p] = make_uint4(0u, 0u, 0u, 0u);
            if (i < total) {
                kr[p] = *buf_row(buf_k, src);
                vr[p] = *buf_row(buf_v, src);
            }
        }
    };
    read_rows(0);
    auto cache_row = [&](int i) -> int64_t { return (int64_t)b * s.sb + (int64_t)g * s.sh + (int64_t)(L + i) * s.st; };
    if (TO != kToCache) {
        __syncthreads();   // every source row is read
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int i = p * RPP + r0;
            if (i >= total) continue;
            uint4 *const to_k = IN_PLACE ? (uint4 *)(cache_k + cache_row(i)) + c : buf_row(buf_k, P - total + i);
            uint4 *const to_v = IN_PLACE ? (uint4 *)(cache_v + cache_row(i)) + c : buf_row(buf_v, P - total + i);
            *to_k = kr[p];
            *to_v = vr[p];
        }
        if (!to_cache) {
            if (wave == 3 && lane == 0) arrive_and_update(ar, bl, b, (int)blockIdx.z * s.Hkv + g, 0u, n_sel > 0, false, L, n + a, total);
            return;
        }
        __syncthreads();   // the new rows are in the cache (stores of this workgroup, read back by it)
    }
    // a wavefront per block: eight passes of rows at a time, the first of the older and of the new ones together
    constexpr int WRP = 64 / LPR, U = 8;   // rows per pass
    const int wr = lane / LPR;
    const T *const base = cache_k + (int64_t)b * s.sb + (int64_t)g * s.sh + c * E;   // (64 is a multiple of LPR: c is lane % LPR)
    uint4 u_old[U], u_new[U];
    auto read_old = [&](int t, int t1) {   // rows t .. t1 - 1, as many of them as there are in U passes
#pragma unroll
        for (int x = 0; x < U; ++x)
            if (t + x * WRP < t1) u_old[x] = *(const uint4 *)(base + (int64_t)min(t + x * WRP + wr, t1 - 1) * s.st);   // (the last row again: no effect)
    };
    auto read_new = [&](int r, int r1) {
#pragma unroll
        for (int x = 0; x < U; ++x)
            if (r + x * WRP < r1) u_new[x] = *buf_row(buf_k, source(min(r + x * WRP + wr, r1 - 1)));
    };
    int blk = first + wave, t0 = 0, t1 = 0, n0 = 0, n1 = 0;   // the block's older rows, and its new ones among those that move
    auto request = [&]() {
        t0 = blk * s.B; t1 = min(t0 + s.B, IN_PLACE ? L + total : L);
        if (!IN_PLACE) { n0 = max(t0 - L, 0); n1 = min(t0 + s.B - L, total); }
        read_old(t0, t1);
        read_new(n0, n1);
    };
    if (sums && blk <= last) request();
    if (wave == 3) {
        int missed = 0;
        if (with_list && total > 0) {
            const int cnt0 = min(max(cnt_raw, 0), n_sel);
            int cnt = cnt0;
            for (int i = first; i <= last; ++i) {
                bool here = (lane < cnt0 && list0 == i) || (lane + 64 < cnt0 && list1 == i);
                for (int x = lane + 128; x < cnt0; x += 64) here |= list[x] == i;
                if (__any(here)) continue;
                if (cnt < n_sel) { if (lane == 0) list[cnt] = i; ++cnt; }
                else ++missed;
            }
            if (lane == 0) *cntp = cnt;
        }
        if (lane == 0) arrive_and_update(ar, bl, b, (int)blockIdx.z * s.Hkv + g, (uint32_t)missed, n_sel > 0, true, L, n + a, total);
    }
    for (int from = 0; !IN_PLACE && from < total; from += ROWS) {
        if (from > 0) read_rows(from);
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int i = from + p * RPP + r0;
            if (i >= total) continue;
            *((uint4 *)(cache_k + cache_row(i)) + c) = kr[p];
            *((uint4 *)(cache_v + cache_row(i)) + c) = vr[p];
        }
    }
    if (!sums) return;
    T *const kmax = (T *)lay.kmax, *const kmin = (T *)lay.kmin;
    for (; blk <= last;) {
        float mx[E], mn[E];
#pragma unroll
        for (int e = 0; e < E; ++e) { mx[e] = -INFINITY; mn[e] = INFINITY; }
        auto fold = [&](const uint4 &u) {
            float f[E];
            Elem<T>::unpack(u, f);
#pragma unroll
            for (int e = 0; e < E; ++e) { mx[e] = fmaxf(mx[e], f[e]); mn[e] = fminf(mn[e], f[e]); }
        };
        for (int t = t0; t < t1;) {
#pragma unroll
            for (int x = 0; x < U; ++x) if (t + x * WRP < t1) fold(u_old[x]);
            t += U * WRP;
            if (t < t1) read_old(t, t1);
        }
        for (int r = n0; r < n1;) {
#pragma unroll
            for (int x = 0; x < U; ++x) if (r + x * WRP < n1) fold(u_new[x]);
            r += U * WRP;
            if (r < n1) read_new(r, n1);
        }
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], off));
                mn[e] = fminf(mn[e], __shfl_xor(mn[e], off));
            }
        }
        if (wr == 0) {
            const int64_t o = (((int64_t)b * s.Hkv + g) * s.max_blocks + blk) * D + c * E;
            *(uint4 *)(kmax + o) = Elem<T>::pack(mx);
            *(uint4 *)(kmin + o) = Elem<T>::pack(mn);
        }
        blk += 4;
        if (blk <= last) request();
    }
}

// Whether a layer's buffers lie in its caches (as far as strides and extents tell).
static bool buffer_in_cache(const Shape &s, size_t elem, const void *k, const void *v, const void *buf_k, const void *buf_v, int rows)
{
    const uintptr_t cache = (uintptr_t)(((s.batch - 1) * s.sb + (s.Hkv - 1) * s.sh + ((int64_t)s.max_blocks * s.B - 1) * s.st + s.D) * (int64_t)elem);
    const uintptr_t buf = (uintptr_t)s.batch * rows * s.Hkv * s.D * elem;
    auto meet = [&](const void *c, const void *p) { return (uintptr_t)p < (uintptr_t)c + cache && (uintptr_t)c < (uintptr_t)p + buf; };
    return meet(k, buf_k) || meet(k, buf_v) || meet(v, buf_k) || meet(v, buf_v);
}

// layers: n_layers entries each of k, v (the caches), buf_k, buf_v (the buffers) and, for a commit to
// the cache, kmax, kmin (or all NULL).  s carries the shape, the strides and ctx_len (shared).
hipError_t launch_commit(const Shape &s, int dtype, int n_layers, void *const *k, void *const *v,
                         void *const *buf_k, void *const *buf_v, int P, int Mt,
                         int32_t *n_pending, const int32_t *accepted, const int32_t *n_accepted,
                         int max_accept, int to_cache, void *const *kmax, void *const *kmin,
                         const specpv_lists *lists, int32_t *dropped, uint32_t *missed_words, hipStream_t st)
{
    if (P + max_accept > kCommitMaxRows) return hipErrorInvalidValue;
    const bool summaries = to_cache && kmax && kmin && kmax[0] && kmin[0];
    const bool with_lists = to_cache && lists;
    for (int b0 = 0; b0 < s.batch; b0 += kCommitSeqs) {
        const int n_seq = s.batch - b0 < kCommitSeqs ? s.batch - b0 : kCommitSeqs;
        // the workgroups of every layer read the counters: those of the last launch move them
        CommitArrive ar{missed_words, (size_t)n_seq * kCommitWords * 128 <= kArriveBytes ? 32 : 1, 0, (int32_t *)s.ctx_len, n_pending, dropped};
        for (int l0 = 0; l0 < n_layers; l0 += kCommitLayers) {
            const int nl = n_layers - l0 < kCommitLayers ? n_layers - l0 : kCommitLayers;
            CommitLayers lay = {};
            bool in_place = false;
            for (int l = 0; l < nl; ++l) {
                if (to_cache) in_place |= buffer_in_cache(s, dtype == SPECPV_BF16 ? 2 : 4, k[l0 + l], v[l0 + l], buf_k[l0 + l], buf_v[l0 + l], P + Mt);
                lay.k[l] = k[l0 + l]; lay.v[l] = v[l0 + l];
                lay.buf_k[l] = buf_k[l0 + l]; lay.buf_v[l] = buf_v[l0 + l];
                if (summaries) { lay.kmax[l] = kmax[l0 + l]; lay.kmin[l] = kmin[l0 + l]; }
                if (with_lists) { lay.idx[l] = lists[l0 + l].sel_idx; lay.cnt[l] = lists[l0 + l].sel_count; }
            }
            CommitStacked stacked;
            const bool in_step = stacked.set(lay, nl);
            const dim3 grid(s.Hkv, n_seq, nl);
            ar.workgroups = l0 + nl == n_layers ? s.Hkv * nl : 0;
            // 32 rows are a quarter of the registers: all that a commit to the cache needs, whatever the buffer's size, and all that moves
            // within a buffer of up to 32 pending rows (what finds no room there is dropped).  With registers for 128 everywhere: one
            // sequence, 32 layers 7.2 us, 6.9 so; four, 28 layers 11.2 / 7.8; eight in fp32, 28 layers 21.9 / 15.6; within the
            // buffer, 28 rows with five to eight accepted, one sequence, 32 layers 5.0 / 4.7; sixteen, 16 layers 10.0-12.0 / 9.1-11.2; eight in
            // fp32, 28 layers 17.5-19.7 / 15.3-17.1 (kernel trace).
#define SPECPV_COMMIT_L(T, DD, ROWS, TO, L, ...)                                                                                  \
    hipLaunchKernelGGL((commit_kernel<T, DD, ROWS, TO, L>), grid, dim3(256), 0, st, s, __VA_ARGS__, b0, P, Mt, n_pending, accepted, n_accepted, max_accept, \
                       summaries ? 1 : 0, with_lists ? lists[0].n_sel : 0, ar)
#define SPECPV_COMMIT(T, DD, ROWS, TO)                                                                                            \
    do { if (in_step) SPECPV_COMMIT_L(T, DD, ROWS, TO, CommitStacked, stacked); else SPECPV_COMMIT_L(T, DD, ROWS, TO, CommitLayers, lay); } while (0)
#define SPECPV_COMMIT_D(T, ROWS, TO) do { if (s.D == 128) SPECPV_COMMIT(T, 128, ROWS, TO); else SPECPV_COMMIT(T, 64, ROWS, TO); } while (0)
#define SPECPV_COMMIT_R(T)                                                                                                        \
    do {                                                                                                                          \
        if (in_place) SPECPV_COMMIT_D(T, kCommitMaxRows, kInPlace);                                                               \
        else if (to_cache) SPECPV_COMMIT_D(T, 32, kToCache);                                                                      \
        else if (P <= 32) SPECPV_COMMIT_D(T, 32, kWithinBuffer);                                                                  \
        else SPECPV_COMMIT_D(T, kCommitMaxRows, kWithinBuffer);                                                                   \
    } while (0)
            if (dtype == SPECPV_BF16) SPECPV_COMMIT_R(bf16_t); else SPECPV_COMMIT_R(float);
#undef SPECPV_COMMIT_R
#undef SPECPV_COMMIT_D
#undef SPECPV_COMMIT
#undef SPECPV_COMMIT_L
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace specpv

namespace specpv {

// Gathered (physically contiguous) partial cache, Section 3.2: the workgroups of a (list slot,
// KV head, sequence) copy one block of K and of V with 16-byte accesses, all of a thread's
// reads issued before its writes.
// 16-byte copies with the streaming hint (every byte is read once and written once)
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load16(const void *p)
{
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_t *)p));
}
__device__ __forceinline__ void stream_store16(void *p, uint4 v)
{
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), (u32x4_t *)p);
}

struct GatherArgs {
    Shape s;
    FastDiv div_B;
    void *k, *v;
    int32_t *len;
};

// A workgroup brings U passes of 4 KiB of K and as many of V: small pieces, because what costs time is the chain of
// length, count, index, rows and stores, which many workgroups overlap.  The first workgroup of a sequence works out the
// sequence's gathered length instead (a launch to clear it and atomics before).  Per call at 64 blocks of 64 tokens and
// eight KV heads 12.8 -> 9.8 us, 33.6 MB read and written (passes of a workgroup: launch_gather).
// List entry, count and length are requested together, out of the leading arguments, which arrive in registers: no trip for the
// arguments in front of it and none for the length, and no division.  A layer in a graph, 8 KV heads of 128 channels, 32 blocks of 64
// 6.10 -> 5.48 us, 100 of 32 7.50 -> 7.08, 64 of 16 5.20 -> 4.70 (those with the length's workgroup as it was); 2 heads, 64 of 64 3.82 -> 3.50.  shift_in_turn: + 32, the length first
// (launch_gather).  What need not arrive in registers is one argument (as one each, fifteen in all, two layers of ten blocks of 64, which the host bounds, 9.2 us, so 8.55).
template <typename T, int D, int U>
__global__ __launch_bounds__(256) void gather_blocks_kernel(const int32_t *sel_idx, const int32_t *sel_count, const int32_t *a_ctx_len, int n_sel, int a_Hkv,
                                                            uint32_t parts_mul, uint32_t parts, int shift_in_turn, GatherArgs a)
{
    Shape s = a.s;
    const FastDiv div_B = a.div_B;
    T *const out_k = (T *)a.k, *const out_v = (T *)a.v;
    int32_t *const out_len = a.len;
    const uint32_t parts_shift = (uint32_t)shift_in_turn & 31u;
    const bool in_turn = shift_in_turn & 32;
    s.ctx_len = a_ctx_len; s.Hkv = a_Hkv;
    constexpr int E = Elem<T>::kPerVec;
    constexpr int LPR = D / E;
    constexpr int RPP = 256 / LPR;
    const int g = blockIdx.y, b = blockIdx.z;
    const int at = max((int)blockIdx.x - 1, 0), slot = (int)FastDiv{parts_mul, parts_shift, parts}.div_straight((uint32_t)at), r0 = (at - slot * (int)parts) * U * RPP;
    // (vector loads: a scalar one would be waited for together with the arguments)
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const int64_t bg = (int64_t)b * s.Hkv + g;
    const int L_v = s.ctx_len[b + zero];
    if (in_turn) asm volatile("" :: "s"(__builtin_amdgcn_readfirstlane(L_v)));
    const int cnt_v = sel_count[bg + zero], entry_v = sel_idx[bg * n_sel + slot + zero];
    // every other argument in one trip to memory; left to itself the compiler asks for each where it is first used
    asm volatile("" :: "s"(s.k), "s"(s.v), "s"(s.sb), "s"(s.sh), "s"(s.st), "s"(s.B), "s"(s.max_blocks), "s"(div_B.mul), "s"(div_B.shift), "s"(div_B.d), "s"(out_k),
                 "s"(out_v));
    const int L = __builtin_amdgcn_readfirstlane(L_v);
    int nb = L > 0 ? (int)div_B.div_straight((uint32_t)L + (uint32_t)s.B - 1u) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    if (blockIdx.x == 0) {
        if (g || !out_len) return;
        // 64 entries of a head at a time, a wavefront every fourth of those, four of them together, counts and entries: head by head and
        // count by count this workgroup was what a small gather waited for: a layer in a graph, 8 KV heads of 128 channels, 13 blocks of 64 3.90 -> 3.28 us,
        // 32 5.48 -> 4.97, 64 of 16 4.71 -> 3.81.  With whole heads dealt to the wavefronts, one head left three of them idle: 161 blocks of 24 3.36 -> 2.92,
        // two sequences of 475 of 16, 64 channels, 4.95 -> 3.19.
        int rows = 0;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int pieces = (n_sel + 63) >> 6;   // of a head's entries
        int h = 0, piece = wave;                // (what the wavefront takes next; the counters go on without a division)
        while (h < s.Hkv) {
            int cnt[4], entry[4], at_slot[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                while (piece >= pieces && h < s.Hkv) { piece -= pieces; ++h; }
                const int64_t row = (int64_t)b * s.Hkv + min(h, s.Hkv - 1);   // (past the last head: nothing)
                at_slot[u] = h < s.Hkv ? 64 * piece + lane : n_sel;
                cnt[u] = sel_count[row + zero];
                entry[u] = sel_idx[row * n_sel + min(at_slot[u], n_sel - 1)];
                piece += 4;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)   // token rows up to and including this block
                if (at_slot[u] < min(cnt[u], n_sel) && entry[u] >= 0 && entry[u] < nb) rows = max(rows, at_slot[u] * s.B + min(s.B, L - entry[u] * s.B));
        }
        __shared__ int most[4];
        for (int off = 32; off; off >>= 1) rows = max(rows, __shfl_xor(rows, off));
        if ((threadIdx.x & 63) == 0) most[threadIdx.x >> 6] = rows;
        __syncthreads();
        if (threadIdx.x == 0) out_len[b] = max(max(most[0], most[1]), max(most[2], most[3]));
        return;
    }
    const int blk = slot < __builtin_amdgcn_readfirstlane(cnt_v) ? __builtin_amdgcn_readfirstlane(entry_v) : -1;
    const bool valid = blk >= 0 && blk < nb;
    const int c = threadIdx.x % LPR, rsub = threadIdx.x / LPR;
    const int64_t src0 = (int64_t)b * s.sb + (int64_t)g * s.sh + c * E;
    const int64_t dst0 = (((int64_t)b * s.Hkv + g) * n_sel + slot) * s.B * D + c * E;
    uint4 kk[U], vv[U];
#pragma unroll
    for (int x = 0; x < U; ++x) {
        const int r = r0 + x * RPP + rsub, t = blk * s.B + r;
        kk[x] = make_uint4(0, 0, 0, 0);
        vv[x] = kk[x];
        if (valid && r < s.B && t < L) {
            kk[x] = stream_load16((const T *)s.k + src0 + (int64_t)t * s.st);
            vv[x] = stream_load16((const T *)s.v + src0 + (int64_t)t * s.st);
        }
    }
#pragma unroll
    for (int x = 0; x < U; ++x) {
        const int r = r0 + x * RPP + rsub;
        if (r < s.B) {
            stream_store16(out_k + dst0 + (int64_t)r * D, kk[x]);
            stream_store16(out_v + dst0 + (int64_t)r * D, vv[x]);
        }
    }
}

hipError_t launch_gather(const Shape &s, int dtype, const int32_t *sel_idx, const int32_t *sel_count, int n_sel,
                         void *out_k, void *out_v, int32_t *out_len, hipStream_t st)
{
    const int pass = 256 * 16 / (s.D * (dtype == SPECPV_BF16 ? 2 : 4));   // rows of a pass
    const int64_t cus = device_cu_count();
    auto workgroups = [&](int u) { return (int64_t)((s.B + u * pass - 1) / (u * pass)) * n_sel * s.Hkv * s.batch; };
    // Four passes where those make one to two workgroups a CU: nothing is left to follow them, and each has twice the reads under way.  8 KV
    // heads, 64 blocks of 64, two / four: 8.36 / 7.65 us (4.3 TB/s); fewer workgroups leave CUs idle (2 heads 3.50 / 4.17), more of them
    // cover each other's trips (two sequences 13.3 / 13.8, eight 47 / 49; fp32 13.3 / 13.9).
    const bool four = workgroups(4) > cus && workgroups(4) <= 2 * cus;
    const int rows = (four ? 4 : 2) * pass;   // of a block, per workgroup
    const int parts = (s.B + rows - 1) / rows;
    if (s.batch > 65535 || s.Hkv > 65535 || (int64_t)n_sel * parts >= (1 << 30)) return hipErrorInvalidConfiguration;   // before anything is enqueued
    // More workgroups than have a place at once hide the length's trip, and with their requests spread out the chip's reads and writes
    // interfere less.  Together / the length first: four sequences of 8 heads, 64 blocks of 64, 24.9 / 24.5 us, sixteen 92.6 / 91.5 (5.9
    // TB/s), in blocks of 16 23.7 / 23.0; two (as many as have a place) 13.3 / 13.5.
    const FastDiv div_parts = make_fastdiv((uint32_t)parts);
    const int shift_in_turn = (int)div_parts.shift | (workgroups(2) > 8 * cus ? 32 : 0);
    const GatherArgs a{s, make_fastdiv((uint32_t)s.B), out_k, out_v, out_len};
    const dim3 grid(1 + n_sel * parts, s.Hkv, s.batch);
#define SPECPV_GATHER_U(T, DD, U) \
    hipLaunchKernelGGL((gather_blocks_kernel<T, DD, U>), grid, dim3(256), 0, st, sel_idx, sel_count, s.ctx_len, n_sel, s.Hkv, div_parts.mul, div_parts.d, shift_in_turn, a)
#define SPECPV_GATHER(T, DD) do { if (four) SPECPV_GATHER_U(T, DD, 4); else SPECPV_GATHER_U(T, DD, 2); } while (0)
    if (dtype == SPECPV_BF16) {
        if (s.D == 128) SPECPV_GATHER(bf16_t, 128); else SPECPV_GATHER(bf16_t, 64);
    } else {
        if (s.D == 128) SPECPV_GATHER(float, 128); else SPECPV_GATHER(float, 64);
    }
#undef SPECPV_GATHER
#undef SPECPV_GATHER_U
    return hipGetLastError();
}

}  // namespace specpv
