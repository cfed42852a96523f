// What the kernels that merge partial results share (combine.hip, refresh_tail.hip): see combine.hip.
#pragma once
#include "internal.h"
#include <type_traits>

namespace specpv {

// The draft's K or V rows as a buffer of the hardware's: a read at kNowhere is outside of it and gives zeros.
typedef __amdgpu_buffer_rsrc_t RowsOf;
constexpr uint32_t kNowhere = 0xffff0000u;
// A sequence's draft rows reach beyond such a buffer (fp32, 128 channels, 128 nodes: from 65536 KV heads).
static inline bool draft_rows_wide(const Shape &s, size_t elem) { return (uint64_t)s.Mk * s.Hkv * s.D * elem > kNowhere; }
__device__ __forceinline__ RowsOf rows_of(const char *p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, (int)bytes, 0x00027000); }

// CPL adjacent channels of one row, 16 bytes per memory instruction (rows are 16-byte aligned).
template <typename T, int CPL> struct Chan;
template <int CPL> struct Chan<float, CPL> {
    typedef float4 Raw[CPL / 4];
    static __device__ __forceinline__ void load(const void *p, int64_t i, Raw &r) {
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) r[x] = *(const float4 *)((const float *)p + i + 4 * x);
    }
    static __device__ __forceinline__ void load(RowsOf p, uint32_t off, Raw &r) {
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) r[x] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(p, (int)off + 16 * x, 0, 0));
    }
    static __device__ __forceinline__ void unpack(const Raw &r, float *f) {
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) { f[4 * x] = r[x].x; f[4 * x + 1] = r[x].y; f[4 * x + 2] = r[x].z; f[4 * x + 3] = r[x].w; }
    }
    static __device__ __forceinline__ float dot(const Raw &a, const Raw &b) {
        float d = 0.f;
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) d = fmaf(a[x].w, b[x].w, fmaf(a[x].z, b[x].z, fmaf(a[x].y, b[x].y, fmaf(a[x].x, b[x].x, d))));
        return d;
    }
    static __device__ __forceinline__ void store_stream(void *p, int64_t i, const float *f) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) {
            f32x4 v = {f[4 * x], f[4 * x + 1], f[4 * x + 2], f[4 * x + 3]};
            __builtin_nontemporal_store(v, (f32x4 *)((float *)p + i + 4 * x));
        }
    }
};
// acc + a.lo * b.lo + a.hi * b.hi for packed bf16 pairs: half the instructions of widening both and two fp32 FMAs, and the
// same error (products of bf16 are exact in fp32).  Log-sum-exp of the draft segment alone against 64 bits, 37 and 60
// nodes, queries of 1 and 4 times unit variance: rms 2.2e-7 and 2.3e-7, at most 2.0e-6, at 64 channels, 2.3e-7 and
// 2.4e-7, at most 2.6e-6, at 128, with either.
__device__ __forceinline__ float dot_bf16x2(uint32_t a, uint32_t b, float acc)
{
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), acc, false);
}
template <> struct Chan<bf16_t, 8> {
    typedef uint4 Raw;
    static __device__ __forceinline__ float dot(const Raw &a, const Raw &b) {
        return dot_bf16x2(a.w, b.w, dot_bf16x2(a.z, b.z, dot_bf16x2(a.y, b.y, dot_bf16x2(a.x, b.x, 0.f))));
    }
    static __device__ __forceinline__ void load(const void *p, int64_t i, Raw &r) { r = *(const uint4 *)((const uint16_t *)p + i); }
    static __device__ __forceinline__ void load(RowsOf p, uint32_t off, Raw &r) { r = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(p, (int)off, 0, 0)); }
    static __device__ __forceinline__ void unpack(const Raw &r, float *f) { Elem<bf16_t>::unpack(r, f); }
    static __device__ __forceinline__ void store_stream(void *p, int64_t i, const float *f) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 v;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = pack_bf16x2(f[2 * x], f[2 * x + 1]);
        __builtin_nontemporal_store(v, (u32x4 *)((uint16_t *)p + i));
    }
};
template <> struct Chan<bf16_t, 4> {
    typedef uint2 Raw;
    static __device__ __forceinline__ float dot(const Raw &a, const Raw &b) { return dot_bf16x2(a.y, b.y, dot_bf16x2(a.x, b.x, 0.f)); }
    static __device__ __forceinline__ void load(const void *p, int64_t i, Raw &r) { r = *(const uint2 *)((const uint16_t *)p + i); }
    static __device__ __forceinline__ void load(RowsOf p, uint32_t off, Raw &r) { r = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(p, (int)off, 0, 0)); }
    static __device__ __forceinline__ void unpack(const Raw &r, float *f) {
        f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
        f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    }
    static __device__ __forceinline__ void store_stream(void *p, int64_t i, const float *f) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        u32x2 v;
#pragma unroll
        for (int x = 0; x < 2; ++x) v[x] = pack_bf16x2(f[2 * x], f[2 * x + 1]);
        __builtin_nontemporal_store(v, (u32x2 *)((uint16_t *)p + i));
    }
};
// The lane's CPL fp32 values of a partial row (p: the row's first element + 4 * (lane & 15)), read
// once: streaming hint.  Rows of 128 are stored so that piece x of all 16 lanes is one dense run
// (partial_pos); the values come out in channel order.
template <int CPL> __device__ __forceinline__ void load_partial(const float *p, float *f)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int x = 0; x < CPL / 4; ++x) {
#ifndef SPECPV_PARTIAL_PLAIN
        const f32x4 v = __builtin_nontemporal_load((const f32x4 *)(p + 64 * x));
#else
        const f32x4 v = *(const f32x4 *)(p + 64 * x);
#endif
        f[4 * x] = v[0]; f[4 * x + 1] = v[1]; f[4 * x + 2] = v[2]; f[4 * x + 3] = v[3];
    }
}

// The lane's channels of one partial as they come from memory, and as fp32 once they are used.
template <int CPL, bool HALF> struct Part {   // fp32 form
    float f[CPL];
    __device__ __forceinline__ void load(const char *p) { load_partial<CPL>((const float *)p, f); }
    __device__ __forceinline__ void value(float *v) const
    {
#pragma unroll
        for (int x = 0; x < CPL; ++x) v[x] = f[x];
    }
};
template <> struct Part<8, true> {   // fp16 form: the lane's eight adjacent channels are one 16-byte piece
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 raw;
    __device__ __forceinline__ void load(const char *p) { raw = __builtin_nontemporal_load((const u32x4 *)p); }
    __device__ __forceinline__ void value(float *v) const
    {
        typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
        const f16x8 h = __builtin_bit_cast(f16x8, raw);
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = (float)h[x];
    }
};

// The value of lane U of a row of 16 lanes, in all of them.
template <int U> __device__ __forceinline__ float row_bcast(float v) { return dpp_row<0x150 + U>(v); }   // row_newbcast
__device__ __forceinline__ float row16_max(float x)
{
    x = fmaxf(x, dpp_row<0xB1>(x));
    x = fmaxf(x, dpp_row<0x4E>(x));
    x = fmaxf(x, dpp_row<0x141>(x));
    return fmaxf(x, dpp_row<0x140>(x));
}

#ifdef SPECPV_TIMELINE
#define SPECPV_CSTAMP(i, W)                                                                                  \
    do {                                                                                                     \
        if (part.timeline && threadIdx.x == 64 * (W) && (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x < 1024u) \
            part.timeline[(2048 + ((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 16 + (i)] = \
                __builtin_amdgcn_s_memrealtime();                                                            \
    } while (0)
#else
#define SPECPV_CSTAMP(i, W) do {} while (0)
#endif

// NP: context partials fetched at once (the smallest of 2, 4, 8, 16 that covers the split count keeps
// the registers, and with them the resident wavefronts of a batch, in proportion).
// MULTI: more splits than 16 (a full verification), or shares: rounds of NP = 8 or 4, each round's
// reads requested before the previous round is merged.
// NB: path nodes whose draft K / V rows are requested in the first go: 8 (a tree of candidates alone), or 24
// when partially verified tokens stand in front of the tree as keys (every candidate's path then starts with
// that whole chain; more registers, so only then).
// HALF: the partials' O rows are fp16 and normalised (see Partials); else fp32 sums.
// part.stream > 0 (MULTI only): the number and the place of a pair's partials follow from the sequence lengths, which the
// partials' wavefront reads first.
// bg = b * Hkv + g; at_row: the query row, or, PACK, the four of rows; wave: of the wavefronts that share it; stores: whether
// there is such a row.  tree_od [fours][D / 64][64], tree_ml [fours][64] (TWO): where those wavefronts meet; all of a workgroup
// come to the one barrier.
// WIDE (draft_rows_wide): a buffer for each row.
template <typename T, int D, int NP, bool MULTI, int NB, bool HALF, bool TWO, bool PACK, bool SHARED, bool WIDE = false>
__device__ __forceinline__ void combine_rows(const Shape &s, const Partials &part, void *out, float *lse, const float scale_log2, const int bg, const int b,
                                             const int at_row, const int wave, const bool stores, float4 *tree_od, float2 *tree_ml)
{
    constexpr int CPL = D / 16;   // channels per lane: d = (lane & 15) * CPL + x
    typedef typename Chan<T, CPL>::Raw Raw;
    const int lane = threadIdx.x & 63;
    const int d0 = (lane & 15) * CPL;
    // wavefronts 0 .. n - 1: the tree segments of four rows each; n .. 2n - 1: their partials.  Lanes without a row (PACK: past
    // the last one; else a group size that is no multiple of four) repeat the last one and store nothing
    const int nq = TWO ? (PACK ? 1 : (s.G + 3) >> 2) : 0;
    const bool tree_role = wave < nq;
    const int quad = TWO && !tree_role ? wave - nq : wave;
    const int g = bg - b * s.Hkv;
    int j = at_row, hc;   // query row and head of the lane's sixteen
    bool live;
    if constexpr (PACK) {
        const int row = j * 4 + (lane >> 4), most = s.M * s.G - 1, r = min(row, most);
        j = (int)(((float)r + 0.5f) * __builtin_amdgcn_rcpf((float)s.G));   // (half a row away from the next whole number: r < 2^16)
        hc = r - j * s.G;
        live = row <= most && stores;
    } else {
        const int hh = quad * 4 + (lane >> 4);
        live = hh < s.G && stores;
        hc = min(hh, s.G - 1);
    }
    const int h = g * s.G + hc;
    const int64_t qrow = (((int64_t)b * s.M + j) * s.Hq + h) * D;
    // Draft rows and partials are read from a base that the wavefront shares and 32 bits a lane (128 draft rows; 65 partials, or
    // as many as there are workgroups, of at most 2048 rows).  In 64 bits a lane the addresses were 130 of the kernel's 1900
    // instructions, in front of the reads: partial verification at 128K, 16 layers, 233.1 us so, 231.9 now.
    constexpr uint32_t SZ = sizeof(T);
    if (wave == 0) SPECPV_CSTAMP(0, 0);   // entry

    // ---- draft-tree segment: the node itself and its ancestors, path slot 0, 1, ... ------------------------------------
    // Of NB = 8 slots the first four and the last four are summed apart and then merged, whichever wavefront has them, so that
    // the results have the same bits: SHARED, the tree's wavefront takes slots 0 .. NA - 1 and whatever comes behind the NB, the
    // partials' the others; else all are the tree's.  Those behind the NB go on from the first four.
    constexpr int NA = SHARED ? 4 : NB;
    static_assert(!SHARED || (TWO && NB == 8), "");
    int par0 = 0, par1 = 0;   // where the path goes on from nodes lane and lane + 64: to the node itself where it ends
    Raw qraw;
    auto tree_first = [&]() __attribute__((always_inline)) {
        // the tree has s.Mk nodes; query row j is node j + s.koff (the nodes in front are keys only)
        const int32_t *par = s.parent + (int64_t)b * s.Mk;
        par0 = par[min(lane, s.Mk - 1)];
        if (s.Mk > 64) par1 = par[min(lane + 64, s.Mk - 1)];
        Chan<T, CPL>::load(s.q, qrow + d0, qraw);
    };
    const int64_t drow0 = ((int64_t)b * s.Mk * s.Hkv + g) * (int64_t)(D * SZ);
    const uint32_t draft_step = (uint32_t)s.Hkv * (D * SZ);
    const uint32_t draft_bytes = (uint32_t)s.Mk * draft_step - (uint32_t)g * (D * SZ);
    const char *kd = nullptr, *vd = nullptr;
    int at = j + s.koff, last = -1;    // next slot's node; the slot's before it (the same: the path has ended)
    // N slots: off[u] is a node's row, bias[u] 0; behind the path's end kNowhere and -inf (rows of zeros: a weight of zero times an
    // infinity in whatever row stood there would be NaN).  What the choice costs is not seen: headline 15.34 / 15.35 us a layer, 16 x 32K
    // 87.7 / 87.8, G = 5 in four 39.7 / 39.5, against the path's last row once more
    auto walk = [&](auto count, uint32_t *off, float *bias) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        auto steps = [&](auto next) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < N; ++u) {
                off[u] = at == last ? kNowhere : (WIDE ? (uint32_t)at : (uint32_t)at * draft_step);
                bias[u] = at == last ? -INFINITY : 0.f;
                last = at;
                at = next(at);
            }
        };
        if (PACK && s.Mk <= 64) steps([&](int x) { return __shfl(par0, x); });
        else if (PACK) steps([&](int x) { const int lo = __shfl(par0, x & 63), hi = __shfl(par1, x & 63); return x < 64 ? lo : hi; });
        else if (s.Mk <= 64) steps([&](int x) { return __builtin_amdgcn_readlane(par0, x); });
        else steps([&](int x) { const int lo = __builtin_amdgcn_readlane(par0, x & 63), hi = __builtin_amdgcn_readlane(par1, x & 63); return x < 64 ? lo : hi; });
    };
    auto any = [](bool x) { return PACK ? __any(x) != 0 : x; };   // (of the sixteens' paths; one path is the wavefront's)
    uint32_t off8[NB];
    float bias[NB];
    Raw kd8[NB], vd8[NB];
    static_assert(!WIDE || !PACK, "a row's buffer is the wavefront's");
    auto rows = [&](auto from, auto count) __attribute__((always_inline)) {
        if constexpr (WIDE) {
#pragma unroll
            for (int u = decltype(from)::value; u < decltype(from)::value + decltype(count)::value; ++u) {
                const uint32_t bytes = off8[u] == kNowhere ? 0u : (uint32_t)(D * SZ);
                const int64_t row = drow0 + (bytes ? (int64_t)off8[u] * draft_step : 0);
                Chan<T, CPL>::load(rows_of(kd + row, bytes), (uint32_t)d0 * SZ, kd8[u]);
                Chan<T, CPL>::load(rows_of(vd + row, bytes), (uint32_t)d0 * SZ, vd8[u]);
            }
            return;
        }
        const RowsOf kd_rows = rows_of(kd + drow0, draft_bytes), vd_rows = rows_of(vd + drow0, draft_bytes);
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(from)::value + decltype(count)::value; ++u) {
            const uint32_t off = off8[u] + (uint32_t)d0 * SZ;
            Chan<T, CPL>::load(kd_rows, off, kd8[u]);
            Chan<T, CPL>::load(vd_rows, off, vd8[u]);
        }
    };
    auto tree_path = [&]() __attribute__((always_inline)) {
        // read now, while the parents are on their way: not where they are first used, and not in front of the parents' request
        kd = (const char *)s.kd; vd = (const char *)s.vd;
        asm volatile("" : "+s"(kd), "+s"(vd));
        // nodes below kctx (partially verified tokens that the context kernels have attended already) end a path, and so does
        // a malformed parent[] (not strictly decreasing)
        par0 = par0 >= s.kctx && par0 < lane ? par0 : lane;
        if (s.Mk > 64) par1 = par1 >= s.kctx && par1 < lane + 64 ? par1 : lane + 64;
        walk(std::integral_constant<int, NB>{}, off8, bias);
    };
    struct Sums { float m, l, od[CPL]; } own, more_sums;
    own.m = more_sums.m = -INFINITY;
    own.l = more_sums.l = 0.f;
#pragma unroll
    for (int x = 0; x < CPL; ++x) own.od[x] = more_sums.od[x] = 0.f;
    // online softmax over four slots
    auto four = [&](const float *bi, const Raw *kdv, const Raw *vdv, auto first, Sums &to) __attribute__((always_inline)) {
        float z[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) z[u] = fmaf(row16_sum(Chan<T, CPL>::dot(qraw, kdv[u])), scale_log2, bi[u]);
        float m_new = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
        if (!decltype(first)::value) m_new = fmaxf(m_new, to.m);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        if (!decltype(first)::value) {
            const float alpha = __builtin_amdgcn_exp2f(to.m - m_use);
            to.l *= alpha;
#pragma unroll
            for (int x = 0; x < CPL; ++x) to.od[x] *= alpha;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float pe = __builtin_amdgcn_exp2f(z[u] - m_use);   // 0 for the unused slots
            to.l += pe;
            float vf[CPL];
            Chan<T, CPL>::unpack(vdv[u], vf);
#pragma unroll
            for (int x = 0; x < CPL; ++x) to.od[x] = fmaf(pe, vf[x], to.od[x]);
        }
        to.m = m_new;
    };
    // the second four into `to`, which has the first (both may be -inf: products that overflow weigh nothing)
    auto merge = [](Sums &to, const Sums &f) __attribute__((always_inline)) {
        const float m = fmaxf(to.m, f.m), m_use = m == -INFINITY ? 0.f : m;
        const float w0 = __builtin_amdgcn_exp2f(f.m - m_use), w1 = __builtin_amdgcn_exp2f(to.m - m_use);
        to.m = m;
        to.l = fmaf(f.l, w0, to.l * w1);
#pragma unroll
        for (int x = 0; x < CPL; ++x) to.od[x] = fmaf(f.od[x], w0, to.od[x] * w1);
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 4> I4;
    typedef std::integral_constant<int, 8> I8;
    // slots 0 .. NA - 1, and those behind the NB
    auto tree_sums = [&]() __attribute__((always_inline)) {
        four(bias, kd8, vd8, std::true_type{}, own);
        const bool second = NA == 8 && any(bias[4] == 0.f);
        if (NB == 8) {
            if (second) four(bias + 4, kd8 + 4, vd8 + 4, std::true_type{}, more_sums);
        } else {
#pragma unroll
            for (int u = 4; u < NA; u += 4)
                if (any(bias[u] == 0.f)) four(bias + u, kd8 + u, vd8 + u, std::false_type{}, own);
        }
        while (any(at != last)) {   // longer paths: 8 per trip
            walk(I8{}, off8, bias);
            rows(I0{}, I8{});
            four(bias, kd8, vd8, std::false_type{}, own);
            if (any(bias[4] == 0.f)) four(bias + 4, kd8 + 4, vd8 + 4, std::false_type{}, own);
        }
        if (second) merge(own, more_sums);
    };
    if (TWO && tree_role) {
        tree_first();
        tree_path();
        if (wave == 0) SPECPV_CSTAMP(1, 0);   // parents in, root path walked
        rows(I0{}, std::integral_constant<int, NA>{});
        tree_sums();
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) tree_od[(quad * (CPL / 4) + x) * 64 + lane] = make_float4(own.od[4 * x], own.od[4 * x + 1], own.od[4 * x + 2], own.od[4 * x + 3]);
        tree_ml[quad * 64 + lane] = make_float2(own.m, own.l);
        if (wave == 0) SPECPV_CSTAMP(3, 0);   // draft K / V rows in, tree segment done
        __syncthreads();
        return;
    }

    // ---- context partials -----------------------------------------------------------------
    const int R = s.M * s.G;   // rows of the KV head, head by head
    int ns = part.nsplit;
    int64_t slot0 = (int64_t)bg * ns;
    if (MULTI && part.stream) {
        const StreamShare sh(s, lane, part.stream);
        const int C_b = __builtin_amdgcn_readlane(sh.chunks, b);
        const int at = (__builtin_amdgcn_readlane(sh.upto, b) - C_b) * s.Hkv + g * C_b;
        const int w0 = C_b > 0 ? sh.owner(at) : 0;
        ns = C_b > 0 ? sh.owner(at + C_b - 1) - w0 + 1 : 0;
        slot0 = w0 + bg;
    }
    constexpr uint32_t ROW = D * (HALF ? 2 : 4);   // bytes of a partial row
    const char *const po_base = (const char *)part.o + slot0 * (int64_t)R * ROW, *const ml_base = (const char *)part.ml + slot0 * (int64_t)R * 8;
    const uint32_t prow = (uint32_t)(hc * s.M + j), po_off = prow * ROW + 16u * (uint32_t)(lane & 15), po_step = (uint32_t)R * ROW;
    // (m, l) of partials u, u + 16, ... in lane u of the row's sixteen: each lane works out the weights of its own
    constexpr int KM = MULTI ? 4 : 1;   // (64 partials at a time; a pair that holds most of a batch may have more)
    const int u16 = lane & 15;
    typedef Part<CPL, HALF> P;
    float m_ctx = -INFINITY, l_ctx = 0.f, o[CPL];
#pragma unroll
    for (int x = 0; x < CPL; ++x) o[x] = 0.f;
    auto fetch = [&](int sp0, P (&r)[NP]) {
#pragma unroll
        for (int u = 0; u < NP; ++u) r[u].load(po_base + (po_off + (uint32_t)max(min(sp0 + u, ns - 1), 0) * po_step));
    };
    auto add = [&](const P &r, float wt) {
        float v[CPL];
        r.value(v);
#pragma unroll
        for (int x = 0; x < CPL; ++x) o[x] = fmaf(wt, v[x], o[x]);
    };
    // partials OFF .. of the sixteen whose weights wk holds (weights past the split count are 0)
    auto add_n = [&](const P *r, float wk, auto off, auto count) __attribute__((always_inline)) {
        constexpr int O = decltype(off)::value, N = decltype(count)::value;
        add(r[0], row_bcast<O>(wk)); add(r[1], row_bcast<O + 1>(wk));
        if constexpr (N >= 4) { add(r[2], row_bcast<O + 2>(wk)); add(r[3], row_bcast<O + 3>(wk)); }
        if constexpr (N >= 8) { add(r[4], row_bcast<O + 4>(wk)); add(r[5], row_bcast<O + 5>(wk)); add(r[6], row_bcast<O + 6>(wk)); add(r[7], row_bcast<O + 7>(wk)); }
    };
    bool more = false;   // two wavefronts: the path goes beyond the other one's slots
    if (!TWO || SHARED) tree_first();   // (in front of the partials: reads are waited for in their order)
    for (int s0 = 0;; s0 += 16 * KM) {   // 16 KM partials at a time (one trip, but for a pair with more than 64)
        float2 ml[KM];
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const int sp = s0 + u16 + 16 * k;
            ml[k] = sp < ns ? *(const float2 *)(ml_base + (prow + (uint32_t)sp * (uint32_t)R) * 8u) : make_float2(-INFINITY, 0.f);
        }
        P ra[NP];
        fetch(s0, ra);
        if (s0 == 0 && (!TWO || SHARED)) {
            tree_path();
            if constexpr (!TWO) {
                rows(I0{}, I4{});
                if (NB > 8) rows(I4{}, std::integral_constant<int, NB - 4>{});
                else if (any(bias[4] == 0.f)) rows(I4{}, I4{});
            } else {
                more = any(bias[NA] == 0.f);
                if (more) rows(std::integral_constant<int, NA>{}, std::integral_constant<int, NB - NA>{});
            }
        }
        float m_new = -INFINITY;
#pragma unroll
        for (int k = 0; k < KM; ++k) m_new = fmaxf(m_new, ml[k].y > 0.f ? ml[k].x : -INFINITY);
        m_new = fmaxf(row16_max(m_new), m_ctx);
        if (MULTI && s0 > 0) {
            const float alpha = m_ctx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ctx - m_new);
            l_ctx *= alpha;
#pragma unroll
            for (int x = 0; x < CPL; ++x) o[x] *= alpha;
        }
        m_ctx = m_new;
        float w[KM], l_new = 0.f;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const float e = ml[k].y > 0.f ? __builtin_amdgcn_exp2f(ml[k].x - m_ctx) : 0.f;
            l_new = fmaf(ml[k].y, e, l_new);
            w[k] = HALF ? e * ml[k].y : e;   // a normalised partial weighs in with its l
        }
        l_ctx += row16_sum(l_new);
        if constexpr (!MULTI) {
            add_n(ra, w[0], I0{}, std::integral_constant<int, NP < 8 ? NP : 8>{});
            if constexpr (NP == 16) add_n(ra + 8, w[0], I8{}, I8{});
            break;
        } else {
            static_assert(!MULTI || NP == 8 || NP == 4, "partials per round");
            P rb[NP];
            typedef std::integral_constant<int, 12> I12;
#pragma unroll
            for (int k = 0; k < KM; ++k) {   // two register sets in turn
                const int at = s0 + 16 * k;
                if (at >= ns) break;
                if constexpr (NP == 8) {
                    if (at + 8 < ns) fetch(at + 8, rb);
                    add_n(ra, w[k], I0{}, I8{});
                    if (at + 8 >= ns) break;
                    if (at + 16 < ns && k + 1 < KM) fetch(at + 16, ra);
                    add_n(rb, w[k], I8{}, I8{});
                } else {
                    if (at + 4 < ns) fetch(at + 4, rb);
                    add_n(ra, w[k], I0{}, I4{});
                    if (at + 4 >= ns) break;
                    if (at + 8 < ns) fetch(at + 8, ra);
                    add_n(rb, w[k], I4{}, I4{});
                    if (at + 8 >= ns) break;
                    if (at + 12 < ns) fetch(at + 12, rb);
                    add_n(ra, w[k], I8{}, I4{});
                    if (at + 12 >= ns) break;
                    if (at + 16 < ns && k + 1 < KM) fetch(at + 16, ra);
                    add_n(rb, w[k], I12{}, I4{});
                }
            }
            if (s0 + 16 * KM >= ns) break;
        }
    }
    if (wave == nq) SPECPV_CSTAMP(2, nq);   // context partials in and merged
    if (TWO) {
        if (SHARED && more) four(bias + 4, kd8 + 4, vd8 + 4, std::true_type{}, more_sums);
        __syncthreads();
        const float2 tml = tree_ml[quad * 64 + lane];
        own.m = tml.x;
        own.l = tml.y;
#pragma unroll
        for (int x = 0; x < CPL / 4; ++x) {
            const float4 v = tree_od[(quad * (CPL / 4) + x) * 64 + lane];
            own.od[4 * x] = v.x; own.od[4 * x + 1] = v.y; own.od[4 * x + 2] = v.z; own.od[4 * x + 3] = v.w;
        }
        if (SHARED && more) merge(own, more_sums);
    } else {
        tree_sums();
    }
    // ---- merge the two and store ---------------------------------------------------------
    const float m_all = fmaxf(own.m, m_ctx);   // (-inf only where every product is: no result then)
    const float wd = __builtin_amdgcn_exp2f(own.m - m_all);
    const float wc = m_ctx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ctx - m_all);
    const float den = fmaf(own.l, wd, l_ctx * wc);   // (written out: left to itself the compiler contracts either product, kernel by kernel)
    const float inv = 1.f / den;
    if (!live) return;
    float res[CPL];
#pragma unroll
    for (int x = 0; x < CPL; ++x) res[x] = fmaf(own.od[x], wd, o[x] * wc) * inv;
    Chan<T, CPL>::store_stream(out, qrow + d0, res);
    if (lse && u16 == 0) lse[((int64_t)b * s.M + j) * s.Hq + h] = (m_all + log2f(den)) * kLn2;
    if (wave == nq) SPECPV_CSTAMP(4, nq);   // stored (issued)
}

}  // namespace specpv
