// Block key summaries (Section 3.2, eq. 1): element-wise max and min of the keys of each block, as a device function: one
// wavefront per (block, KV head), or per several small blocks, 16-byte loads, the lanes that share a channel group are folded across lanes.
// The summary kernel calls it, and so do workgroups of a full pass that recomputes them (attn_mfma.hip).
#pragma once
#include "internal.h"
#include "rows.h"
#include <type_traits>
#ifndef SPECPV_SUM_UNR
#define SPECPV_SUM_UNR 16
#endif

namespace specpv {

// 16-byte read of data that is used once: keep it from displacing what the caches hold
__device__ __forceinline__ uint4 load_stream(const uint4 *p)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

template <bool STREAM> __device__ __forceinline__ uint4 load_keys(const uint4 *p)
{
    if constexpr (STREAM) return load_stream(p);
    else return *p;
}

__device__ __forceinline__ float dpp_ror8(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)); }

// The keys that a wavefront has taken in, folded over the lanes that hold the same channels, and stored: lane c + LPR r holds the
// extremes of channels c E .. c E + E - 1 over its rows.  An exchange of halves brings two channels' values together in one
// instruction (half of the lanes go on with one, half with the other), so eight channels are folded over four lanes by six
// exchanges and six comparisons; through LDS they were sixteen of each.
template <typename T, int D>
__device__ __forceinline__ void store_extremes(float (&mx)[Elem<T>::kPerVec], float (&mn)[Elem<T>::kPerVec], T *kmax_row, T *kmin_row, int lane)
{
    constexpr int E = Elem<T>::kPerVec, LPR = D / E, HALVED = LPR <= 16 ? E / 4 : E / 2;   // channels that a lane stores
    static_assert(LPR == 8 || LPR == 16 || LPR == 32, "lanes of a row");
#pragma unroll
    for (int e = 0; e < E / 2; ++e) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx[e]), __float_as_uint(mx[e + E / 2]), false, false);
        const auto n = __builtin_amdgcn_permlane32_swap(__float_as_uint(mn[e]), __float_as_uint(mn[e + E / 2]), false, false);
        mx[e] = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
        mn[e] = fminf(__uint_as_float(n[0]), __uint_as_float(n[1]));
    }
    if constexpr (LPR <= 16) {
#pragma unroll
        for (int e = 0; e < E / 4; ++e) {
            const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx[e]), __float_as_uint(mx[e + E / 4]), false, false);
            const auto n = __builtin_amdgcn_permlane16_swap(__float_as_uint(mn[e]), __float_as_uint(mn[e + E / 4]), false, false);
            mx[e] = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
            mn[e] = fminf(__uint_as_float(n[0]), __uint_as_float(n[1]));
        }
    }
    if constexpr (LPR == 8) {
#pragma unroll
        for (int e = 0; e < HALVED; ++e) { mx[e] = fmaxf(mx[e], dpp_ror8(mx[e])); mn[e] = fminf(mn[e], dpp_ror8(mn[e])); }
    }
    const int chan = (lane % LPR) * E + (lane >> 5) * (E / 2) + (LPR <= 16 ? ((lane >> 4) & 1) * (E / 4) : 0);
    if (LPR == 8 && (lane & 8)) return;
    if constexpr (sizeof(T) == 2) {
        static_assert(HALVED == 2, "a pair of channels");
        *(uint32_t *)(kmax_row + chan) = pack_bf16x2(mx[0], mx[1]);
        *(uint32_t *)(kmin_row + chan) = pack_bf16x2(mn[0], mn[1]);
    } else if constexpr (HALVED == 2) {
        *(float2 *)((float *)kmax_row + chan) = make_float2(mx[0], mx[1]);
        *(float2 *)((float *)kmin_row + chan) = make_float2(mn[0], mn[1]);
    } else {
        static_assert(HALVED == 1, "a channel");
        ((float *)kmax_row)[chan] = mx[0];
        ((float *)kmin_row)[chan] = mn[0];
    }
}

// block i of (sequence b of length L, KV head g); i lies below the sequence's block count
template <typename T, int D>
__device__ __forceinline__ void summarize_block(const Shape &s, int b, int g, int i, int L, void *kmax, void *kmin, int lane)
{
    constexpr int E = Elem<T>::kPerVec;   // elements per 16-byte load
    constexpr int LPR = D / E;            // lanes that cover one token row
    constexpr int RPP = 64 / LPR;         // token rows per wavefront pass
    static_assert(D % E == 0 && LPR <= 64 && 64 % LPR == 0, "head dim does not tile a wavefront");
    const int t0 = i * s.B;
    const int t1 = min(t0 + s.B, L);
    const int c = lane % LPR, rsub = lane / LPR;
    const T *base = (const T *)s.k + (int64_t)b * s.sb + (int64_t)g * s.sh + c * E;
    float mx[E], mn[E];
#pragma unroll
    for (int e = 0; e < E; ++e) { mx[e] = -INFINITY; mn[e] = INFINITY; }
    // Passes of RPP rows, N independent 16-byte loads per lane in flight: the kernel is bound by the bytes it
    // keeps in flight against the memory latency.  Rows behind the last are the last once more.
    auto passes = [&](auto n, auto stream, int from) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value;
        uint4 u[N];
#pragma unroll
        for (int x = 0; x < N; ++x) u[x] = load_keys<decltype(stream)::value>((const uint4 *)(base + (int64_t)min(from + x * RPP + rsub, t1 - 1) * s.st));
#pragma unroll
        for (int x = 0; x < N; ++x) {
            float f[E];
            Elem<T>::unpack(u[x], f);
#pragma unroll
            for (int e = 0; e < E; ++e) { mx[e] = fmaxf(mx[e], f[e]); mn[e] = fminf(mn[e], f[e]); }
        }
    };
    constexpr int UNR = SPECPV_SUM_UNR;
    int t = t0;
    for (; t + UNR * RPP <= t1; t += UNR * RPP) passes(std::integral_constant<int, UNR>(), std::true_type(), t);
    const int left = (t1 - t + RPP - 1) / RPP;   // fewer than UNR
    auto rest = [&](auto stream) __attribute__((always_inline)) {
        if (left > 12) passes(std::integral_constant<int, UNR>(), stream, t);
        else if (left > 8) passes(std::integral_constant<int, 12>(), stream, t);
        else if (left > 4) passes(std::integral_constant<int, 8>(), stream, t);
        else if (left > 2) passes(std::integral_constant<int, 4>(), stream, t);
        else if (left == 2) passes(std::integral_constant<int, 2>(), stream, t);
        else if (left == 1) passes(std::integral_constant<int, 1>(), stream, t);
    };
    // Blocks that are all rest ask for their keys past the caches as well, which costs those that find them there: fp32, and what is left of
    // a longer block, ask for them as before.  16384 blocks, past the caches / not: bf16, 128 channels, blocks of 32 22.8 / 22.3 us, 65536 95 /
    // 108, 8192 10.9 / 12.6; of 100 67.5 / 60.9; fp32, of 16 25.6 / 24.4, 26000 of them 40.4 / 37.2, 64 channels, of 32 36.7 / 33.2.
    if (sizeof(T) == 2 && t == t0) rest(std::true_type());
    else rest(std::false_type());
    const int64_t o = (((int64_t)b * s.Hkv + g) * s.max_blocks + i) * D;
    store_extremes<T, D>(mx, mn, (T *)kmax + o, (T *)kmin + o, lane);
}

// Blocks of N passes of RPP rows, fewer than UNR: as many blocks as have UNR passes together, i0 and those behind it up to `end`,
// their rows all under way at once.  Rows of blocks that are not there, or behind the last token, are the last row once more.
template <typename T, int D, int N>
__device__ __forceinline__ void summarize_small(const Shape &s, int b, int g, int i0, int end, int L, void *kmax, void *kmin, int lane)
{
    constexpr int E = Elem<T>::kPerVec, LPR = D / E, RPP = 64 / LPR, UNR = SPECPV_SUM_UNR;
    const int c = lane % LPR, rsub = lane / LPR, t0 = i0 * (N * RPP);
    const T *base = (const T *)s.k + (int64_t)b * s.sb + (int64_t)g * s.sh + c * E;
    uint4 u[UNR];
#pragma unroll
    for (int x = 0; x < UNR; ++x) u[x] = load_keys<sizeof(T) == 2>((const uint4 *)(base + (int64_t)row_below(t0 + x * RPP + rsub, L, end, N * RPP) * s.st));
    const int64_t o = (((int64_t)b * s.Hkv + g) * s.max_blocks + i0) * D;
#pragma unroll
    for (int j = 0; j < UNR / N; ++j) {
        if (i0 + j >= end) break;
        float mx[E], mn[E];
#pragma unroll
        for (int e = 0; e < E; ++e) { mx[e] = -INFINITY; mn[e] = INFINITY; }
#pragma unroll
        for (int x = 0; x < N; ++x) {
            float f[E];
            Elem<T>::unpack(u[j * N + x], f);
#pragma unroll
            for (int e = 0; e < E; ++e) { mx[e] = fmaxf(mx[e], f[e]); mn[e] = fminf(mn[e], f[e]); }
        }
        store_extremes<T, D>(mx, mn, (T *)kmax + o + j * D, (T *)kmin + o + j * D, lane);
    }
}

}  // namespace specpv
