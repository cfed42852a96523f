// Context part of the verification attention on the matrix cores, for bf16 with
// head dim 128 (Section 3.2: the draft tree attends over the kept blocks as one KV
// segment; with all blocks kept this is the full verification of Section 3.3).
//
// Work decomposition.  A workgroup (8 wavefronts, two per SIMD) owns one query head,
// one tile of up to 64 tree nodes and one KV split; inside it four pairs of
// wavefronts each own a contiguous range of 32-token chunks, the two wavefronts of
// a pair taking 32 rows of the tile each.  Nothing is gathered: K and V rows go
// from their place in the cache straight into a small per-pair LDS ring by LDS-DMA
// (global_load_lds), two chunks ahead of the arithmetic, and from there into MFMA
// operand registers.  The G query heads of a KV head that read the same split are
// placed on one XCD, next to each other in dispatch order, so that the split's K/V
// bytes come from HBM once and from that XCD's L2 afterwards.
//
// Per chunk (v_mfma_f32_32x32x16_bf16, fp32 accumulate):
//   S^T = K . Q^T     tokens are the M index, query rows the N index, so each
//                     lane holds 16 tokens of ONE query row: max, sum and rescale
//                     are lane-local (one exchange with lane ^ 32);
//   O^T += V^T . P^T  the S^T accumulator, converted to bf16, already has the
//                     B-operand layout; V comes out of LDS transposed (8 tokens
//                     of one channel per lane) through ds_read_b64_tr_b16.
// The contraction index may be permuted freely as long as both operands agree,
// which is what makes the register layouts line up.
//
// The reference maximum of a row is only moved when the true maximum runs more than
// 2^8 ahead of it, so rescaling the accumulators is rare.
//
// Epilogue: the four token groups merge their (O, m, l) through LDS and write one
// split-KV partial per (head, split, node).
//
// attn_ctx_mfma_kernel (above description, with the rest of the call in the same kernel) is the single-kernel route
// of specpv_debug_set_route; attn_ctx_mfma_group_kernel, further down, is used when a wavefront has many chunks to go
// through (full verification of a long context, batches): there a workgroup serves all query heads of a KV head.  Short
// ranges (the partial verification over a 4K-token cache) run attn_tile.hip.
#include "attn_mfma.h"
#include "summarize.h"

namespace specpv {

constexpr int kOPitch = 132;         // floats per staged output row (128 + 4: conflict-free 16-byte writes)
constexpr int kStages = 2;           // ring depth per wavefront pair (eight-wavefront kernel)
constexpr int kRingBytes = 4 * kStages * kStageBytes;
constexpr int kQStageBytes = 2 * 8 * 1024;   // the query rows of a workgroup's two row blocks as MFMA operands (eight-wavefront kernel)

__device__ __forceinline__ float max_xor16(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor16(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// max / sum over the 8 lanes 8 u .. 8 u + 7 (lane ^ 1, lane ^ 2, mirror inside 8)
__device__ __forceinline__ float oct_max(float x)
{
    x = fmaxf(x, dpp_row<0xB1>(x));
    x = fmaxf(x, dpp_row<0x4E>(x));
    x = fmaxf(x, dpp_row<0x141>(x));
    return x;
}
__device__ __forceinline__ float oct_sum(float x)
{
    x += dpp_row<0xB1>(x);
    x += dpp_row<0x4E>(x);
    x += dpp_row<0x141>(x);
    return x;
}
// ---- eight-wavefront kernel: one query head, one tile of up to 64 nodes, one KV split ----------
// grid: x = r * 8 + xcd   (r = query head within the group + G * row tile),
//       y = (bg / 8) * nsplit + split   with bg = b * Hkv + g and xcd = bg % 8.
// Workgroups are handed to the 8 XCDs round-robin in linear order and gridDim.x is a multiple of
// 8, so a (sequence, KV head) stays on XCD bg % 8 with all its splits and query heads: the K/V
// bytes of a split come from HBM once and from that XCD's L2 for the other query heads, and the
// split-KV partials of a head meet in one L2.
//
// Workgroup = 8 wavefronts = 4 token groups x 2 row blocks.  Wavefronts tg and tg + 4
// sit on the same SIMD, work on the same chunks (rows 0..31 and 32..63 of the tile)
// and share one LDS ring; the first of the pair requests the K rows, the second the V
// rows.  Two workgroup barriers per chunk order "DMA landed -> both read" and "both
// read -> stage may be refilled".  Every wavefront runs the same number of iterations
// (the largest chunk count in the workgroup), so the barriers always match up.
//
// The whole call in this one kernel (attn_tile.hip is the context part alone, the first of two kernels):
//  * The draft-tree segment (a node attends itself and its ancestors, tree decode of Algorithm 1)
//    is one more partial per row, in slot `nctx` behind the context splits: the workgroup of
//    split sp computes it for the rows r = sp (mod nctx) of its tile on the vector ALU, one row
//    per wavefront, while its first K/V chunks are on their way.
//  * Partials are stored with ordinary stores (they stay in this XCD's L2), then the workgroup
//    adds itself to the tile's arrival word (one 64-bit atomic add: arrival count in the top byte,
//    7 bits of count per hardware XCC id below).  No workgroup ever waits for another one.
//  * The workgroup whose add completes the count merges the nctx + 1 partials of its tile by their
//    log-sum-exp weights, normalises, stores out / lse and zeroes the word.  It reads the
//    others' partials from L2, which is only right if they were written through the SAME L2: if
//    the XCC ids in the word say that any workgroup of the tile ran elsewhere (never seen; the
//    dispatcher's round-robin is not a documented guarantee), the last workgroup recomputes the
//    tile from scratch instead -- every split and the draft segment, merged in its own registers --
//    so the result never depends on where workgroups run.
constexpr int kXccBits = 7;
#ifdef SPECPV_TIMELINE
#define SPECPV_STAMP(i)                                                                                       \
    do {                                                                                                      \
        if (f.timeline && threadIdx.x == 0 && !REDO && blockIdx.y * gridDim.x + blockIdx.x < 2048u)           \
            f.timeline[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 16 + (i)] = __builtin_amdgcn_s_memrealtime(); \
    } while (0)
#else
#define SPECPV_STAMP(i) do {} while (0)
#endif        // per-XCC arrival count (splits <= 64)

// One pass over the token ranges of split `sp0` of `ns_eff` splits.  REDO = false: the ordinary pass of
// a workgroup (ns_eff = nctx); returns true if this workgroup, the last of its tile, has to take the
// recompute route.  REDO = true: that route -- the pass runs as the only split of one (sp0 = 0, ns_eff = 1).
// Everything, the argument-dependent reads included, is done again in the second pass, so that it keeps
// no register of the first one alive.
template <bool ALIGNED, bool REDO>
__device__ __forceinline__ bool attn_ctx_pass(Shape s, Partials part, MfmaArgs a, FusedArgs f, const int nctx,
                                              const int sp0, const int ns_eff, char *lds_raw)
{
    float *ms = (float *)lds_raw;            // [4 token groups][64 rows]
    float *ls = ms + 4 * 64;                 // [4][64]
    char *ring = lds_raw + 2048;             // [4 pairs][kStages][K 8 KiB | V 8 KiB]
    float *obuf = (float *)(lds_raw + 2048); // [4][64][kOPitch], reuses the ring after the main loop
    constexpr bool redo = REDO;
    const int sp = sp0;
    SPECPV_CLOCKS_BEGIN;
    SPECPV_STAMP(0);   // entry

    // ---- which piece of work is this workgroup -------------------------------------
    const int xcd = blockIdx.x & 7, r = blockIdx.x >> 3;
    const int bgh = (int)a.div_nsplit.div(blockIdx.y);
    const int bg = bgh * 8 + xcd;
    if (bg >= a.n_bg) return false;
    const int b = (int)a.div_hkv.div((uint32_t)bg);
    const int g = bg - b * s.Hkv;
    const int rt = r >= s.G ? 1 : 0;          // at most two row tiles (M <= 128)
    const int hh = r - rt * s.G;
    const int h = g * s.G + hh;
    const int m0 = rt * 64;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tg = wave & 3, rb = wave >> 2;
    const int n = lane & 31, kg = lane >> 5;

    // Everything whose address only depends on the kernel arguments is requested up
    // front, so that the cold-miss latencies of these small reads overlap: context
    // length, list length, the kept-block list (up to 256 entries, lane t: entries t, t + 64, ..),
    // the query rows, and for the draft segment the parents and this wavefront's first row.
    const int32_t *sel = a.sel_idx ? a.sel_idx + (int64_t)bg * a.n_sel : nullptr;
    const uint32_t Bu = (uint32_t)s.B;
    const int L = s.ctx_len[b];
    const int cnt_raw = sel ? a.sel_count[bg] : 0;
    const bool list_in_regs = ALIGNED && sel && a.n_sel <= 256;
    int idv[4] = {-1, -1, -1, -1};
    if (list_in_regs) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (lane + 64 * x < a.n_sel) idv[x] = sel[lane + 64 * x];
    }
    // The query rows of a row block are the same for its four wavefronts (one per token group): each brings
    // a quarter of them (k-steps 2 tg, 2 tg + 1) straight into LDS, laid out as the operands are read
    // (k-step ks of row block rb: 1 KiB, lane l's 16 bytes at 16 l), and all four read the whole from there
    // once the requests have landed -- a quarter of the bytes through the CU's memory path in the phase
    // where the first K / V chunks are requested.
    char *qstage = lds_raw + 2048 + max(kRingBytes, 4 * 64 * kOPitch * (int)sizeof(float));
    {
        const int j = min(m0 + rb * 32 + n, s.M - 1);   // rows past M repeat row M-1; never stored
        const char *qrow = (const char *)((const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + h) * 128 + kg * 8);
        char *dst = qstage + (rb * 8 + 2 * tg) * 1024;
        __builtin_amdgcn_global_load_lds((glb_void_ptr)(qrow + 64 * tg), (lds_void_ptr)dst, 16, 0, 0);   // a k-step is 16 channels: 32 bytes
        __builtin_amdgcn_global_load_lds((glb_void_ptr)(qrow + 64 * tg + 32), (lds_void_ptr)(dst + 1024), 16, 0, 0);
    }
    const int rows_tile = min(64, s.M - m0);            // >= 1
    int par0 = -1, par1 = -1;
    uint4 qd_first = make_uint4(0u, 0u, 0u, 0u);
    {
        const int32_t *par = s.parent + (int64_t)b * s.Mk;
        if (lane < s.Mk) par0 = par[lane];
        if (lane + 64 < s.Mk) par1 = par[lane + 64];
        const int r0 = min(sp0 + ns_eff * wave, rows_tile - 1);
        qd_first = *(const uint4 *)((const uint16_t *)s.q + (((int64_t)b * s.M + m0 + r0) * s.Hq + h) * 128 + (lane & 15) * 8);
    }

    int nb = L > 0 ? (int)a.div_B.div((uint32_t)(L + s.B - 1)) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    int cnt = nb;
    if (sel) cnt = max(0, min(cnt_raw, a.n_sel));
    const uint32_t T = nb > 0 ? (uint32_t)cnt * Bu : 0u;   // host guarantees max_blocks * B <= 2^30
    // chunks of cache tokens, then the chunks of the partially verified tokens (the first kctx draft nodes: a
    // chain that every query node descends from, so all rows attend all of them, like cache tokens)
    const uint32_t C_ctx = (T + 31u) >> 5;
    const int kctx = s.kctx;
    const uint32_t C = C_ctx + (((uint32_t)kctx + 31u) >> 5);
    const char *kdb = (const char *)s.kd + (((int64_t)b * s.Mk) * s.Hkv + g) * 256;
    const char *vdb = (const char *)s.vd + (((int64_t)b * s.Mk) * s.Hkv + g) * 256;
    const uint32_t stp = (uint32_t)s.Hkv * 256u;   // bytes from one draft node's row to the next

    // uniform slab bases; per-lane byte offsets inside a slab fit 32 bits (host-checked)
    const char *kb = (const char *)s.k + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const char *vb = (const char *)s.v + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const uint32_t st2 = (uint32_t)s.st * 2u;   // bytes per token row step

    char *my_ring = ring + tg * (kStages * kStageBytes);
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)my_ring;
    // K tile in LDS: row-major, 256 B per token, the 16-byte pieces of row t stored at
    // piece index (p ^ (t & 15)) so that the operand reads below (16 lanes per cycle, same piece,
    // different rows) spread over all 64 banks.  Operand piece of k-step ks: 2*ks + kg.
    uint32_t kread[4];   // + stage * kStageBytes; k-step ks + 4: the address XOR 128 (rows and stages start 256-byte aligned)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        kread[ks] = ring_addr + (uint32_t)n * 256u + (((uint32_t)(32 * ks + 16 * kg)) ^ (16u * ((uint32_t)n & 15u)));
    const uint32_t vread = ring_addr + 8192u + (uint32_t)(4 * kg + ((lane & 15) >> 2)) * kVPiecePitch +
                           32u * (uint32_t)((lane >> 4) & 1) + 8u * (uint32_t)(lane & 3);   // + stage * kStageBytes

    bf16x8 qf[8];   // Q fragments (B operand of S^T = K . Q^T): row = lane & 31; read from LDS in front of the main loop

    const int r4 = lane >> 4, pos = lane & 15;
    const uint32_t sw0 = 16u * (uint32_t)(pos ^ r4), vsw = 16u * (uint32_t)pos;   // K row 4 i + r4: piece pos ^ ((4 i + r4) & 15) = sw0 ^ 64 (i & 3)
    const uint32_t lane_row_off = (uint32_t)r4 * st2;
    constexpr int RPW = 8;  // rows each wavefront finishes in the epilogue

    const int W = ns_eff * 4, wsid = sp * 4 + tg;
    // chunks of a list that precede the share of token group w; shares differ by at most one
    auto first_chunk = [&](uint32_t chunks, int w) -> int {
        const uint32_t base = redo ? (chunks >> 2) : a.div_W.div(chunks), rem = chunks - base * (uint32_t)W;
        return (int)((uint32_t)w * base + min((uint32_t)w, rem));
    };
    const int c0 = first_chunk(C, wsid), c1 = first_chunk(C, wsid + 1);
    const int nch = c1 - c0;
    const int nch_max = first_chunk(C, sp * 4 + 1) - first_chunk(C, sp * 4);   // token group 0 has the most

    // ---- chunk -> token rows (see ChunkRows) ---------------------------------------------
    // ALIGNED (B % 32 == 0): the first rows of the next 64 chunks of this wavefront sit in a register (lane t: chunk
    // row_base + t) and are picked with readlane.
    const ChunkRows rows_of{sel, a.div_B, s.B, nb, L, T};
    int row_base = 0, row0vec = -1;
    auto fill_rows = [&](int cb) {
        row_base = cb;
        int r = -1;
        if (cb + lane < nch && (uint32_t)(c0 + cb + lane) < C_ctx) r = rows_of.first_row<32>((uint32_t)(c0 + cb + lane));
        row0vec = r;
        // wait for the list entries here, inside the rare branch, so that the common path that
        // joins behind it carries no pending load (and no wait on the DMA prefetch)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    };
    // the first 64 chunks: the list sits in registers (lane t: entries t, t + 64, ...), so this is a
    // cross-lane read and no second trip to memory
    auto fill_rows_first = [&]() {
        if (!list_in_regs) { fill_rows(0); return; }
        const uint32_t p0 = (uint32_t)(c0 + lane) * 32u;
        const uint32_t slot = a.div_B.div(p0);
        const int src = (int)(slot & 63u);
        const int e0 = __shfl(idv[0], src), e1 = __shfl(idv[1], src), e2 = __shfl(idv[2], src), e3 = __shfl(idv[3], src);
        const int q4 = (int)(slot >> 6);
        const int blk = q4 == 0 ? e0 : (q4 == 1 ? e1 : (q4 == 2 ? e2 : e3));
        row0vec = (lane < nch && (uint32_t)(c0 + lane) < C_ctx) ? rows_of.encode<32>(blk, p0, slot) : -1;   // p0 < T there: the slot is < cnt
    };

    uint32_t vmask_st[kStages];   // validity bits of the chunk this wavefront last requested rows for, per stage

    // Request this wavefront's half of chunk ci: 8 DMA operations of 1 KiB (one 256-byte row per
    // 16 lanes).  rb == 0: the K rows, operation i brings rows 4i .. 4i+3, pieces swizzled by
    // row & 7.  rb == 1: the V rows, operation i brings rows i, i+8, i+16, i+24 into piece i.
    // rows given per lane (t = lane & 31: token tk of the chunk, bits vm say which are real)
    auto issue_rows = [&](const char *kbase, const char *vbase, const uint32_t stride, const uint32_t tk, char *dst, char *dstv) {
        if (rb == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t tv = (uint32_t)__shfl((int)tk, 4 * i + r4) * stride;
                dma16(kbase + (tv + (sw0 ^ (64u * (uint32_t)(i & 3)))), dst + i * 1024);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t tv = (uint32_t)__shfl((int)tk, 8 * r4 + i) * stride;
                dma16(vbase + (tv + vsw), dstv + i * kVPiecePitch);
            }
        }
    };
    auto issue = [&](int ci) {
        const int stg = ci & (kStages - 1);
        char *dst = my_ring + stg * kStageBytes;
        char *dstv = dst + 8192;
        int tok;
        if (kctx > 0 && (uint32_t)(c0 + ci) >= C_ctx) {
            // a chunk of partially verified tokens: rows of the draft K / V arrays
            const int pr = (int)((uint32_t)(c0 + ci) - C_ctx) * 32 + n;
            const int ptok = pr < kctx ? pr : -1;
            vmask_st[stg] = (uint32_t)__ballot(ptok >= 0);
            issue_rows(kdb, vdb, stp, (uint32_t)max(ptok, 0), dst, dstv);
            return;
        }
        if (ALIGNED) {
            if (ci - row_base >= 64) fill_rows(ci);
            const int r0 = __builtin_amdgcn_readlane(row0vec, ci - row_base);
            if (r0 >= 0) {
                vmask_st[stg] = 0xffffffffu;
                const size_t row0 = (size_t)((uint32_t)r0 * st2);   // fits 32 bits (host-checked)
                if (st2 == 256u) {
                    // rows are 256 bytes apart (the usual head-major cache): the instruction's
                    // immediate offset, added to the global and to the LDS address, covers the step
                    // between consecutive operations (K: 1 KiB on both sides; V: 256 bytes, with the
                    // LDS base adjusted for the rest of the piece pitch)
                    if (rb == 0) {
                        dma16x4(kb + row0, lane_row_off, sw0, dst);
                        dma16x4(kb + row0 + 4096, lane_row_off, sw0, dst + 4096);
                    } else {
                        const char *vsrc = vb + row0 + ((uint32_t)r4 * 2048u + vsw);
#define SPECPV_VOP(i) __builtin_amdgcn_global_load_lds((glb_void_ptr)vsrc, (lds_void_ptr)(dstv + (i) * (kVPiecePitch - 256)), 16, (i) * 256, kKvAux)
                        SPECPV_VOP(0); SPECPV_VOP(1); SPECPV_VOP(2); SPECPV_VOP(3);
                        SPECPV_VOP(4); SPECPV_VOP(5); SPECPV_VOP(6); SPECPV_VOP(7);
#undef SPECPV_VOP
                    }
                } else if (rb == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        dma16(kb + row0 + (size_t)(4 * i) * st2 + (lane_row_off + (sw0 ^ (64u * (uint32_t)(i & 3)))), dst + i * 1024);
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        dma16(vb + row0 + (size_t)(8 * r4 + i) * st2 + vsw, dstv + i * kVPiecePitch);
                }
                return;
            }
            const int rr = -2 - r0;   // r0 == -1 gives -1
            tok = (rr >= 0 && rr + n < L) ? rr + n : -1;
        } else {
            tok = rows_of.row((uint32_t)(c0 + ci), n);
        }
        const uint32_t vm = (uint32_t)__ballot(tok >= 0);
        const uint32_t tk = tok >= 0 ? (uint32_t)tok : 0u;   // row 0 exists (L > 0); masked later
        vmask_st[stg] = vm;
        issue_rows(kb, vb, st2, tk, dst, dstv);
    };

    if (ALIGNED && nch > 0) fill_rows_first();
    // every load above has been consumed here: from now on the only vector-memory
    // operations of this wavefront in flight are its own DMA groups (8 operations each)
    // (as an instruction the compiler knows, not inline assembly: otherwise it assumes that the
    // loads of the prologue may still be in flight at the loop header and waits for vmcnt(0),
    // i.e. for the prefetch just issued, at the first use of Q in every iteration)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), expcnt and lgkmcnt untouched
    asm volatile("" ::: "memory");
    SPECPV_STAMP(1);   // arguments, lengths, list, query rows, parents are in

    // ---- draft-tree segment of this workgroup's rows --------------------------------
    // Row r of the tile (node koff + m0 + r) is handled by the workgroup with sp = r mod ns_eff, there
    // by wavefront (r / ns_eff) mod 8.  Sixteen lanes per draft node (a lane owns 8 adjacent
    // channels), four nodes of the root path at a time; the result goes to slot nctx of the
    // partial arrays like any other partial.  For a wavefront's first row the first two rounds of
    // K / V rows (8 path nodes) are requested in front of the first context chunks.
    auto draft_row = [&](int row, bool live, bool with_chunks) {
        const int jn = s.koff + m0 + row;
        unsigned long long anc_lo = 0ull, anc_hi = 0ull;
        root_path(jn, s.Mk, kctx, par0, par1, anc_lo, anc_hi);
        const int n0 = pop_node(anc_lo, anc_hi), n1 = pop_node(anc_lo, anc_hi), n2 = pop_node(anc_lo, anc_hi),
                  n3 = pop_node(anc_lo, anc_hi), n4 = pop_node(anc_lo, anc_hi), n5 = pop_node(anc_lo, anc_hi),
                  n6 = pop_node(anc_lo, anc_hi), n7 = pop_node(anc_lo, anc_hi);
        const int na = r4 == 0 ? n0 : (r4 == 1 ? n1 : (r4 == 2 ? n2 : n3));
        const int nb2 = r4 == 0 ? n4 : (r4 == 1 ? n5 : (r4 == 2 ? n6 : n7));
        auto drow = [&](const void *base, int node) -> const uint16_t * {
            return (const uint16_t *)base + (((int64_t)b * s.Mk + max(node, 0)) * s.Hkv + g) * 128 + pos * 8;
        };
        uint4 qd = qd_first;
        if (!with_chunks) qd = *(const uint4 *)((const uint16_t *)s.q + (((int64_t)b * s.M + m0 + row) * s.Hq + h) * 128 + pos * 8);
        // requested in front of the first context chunks; the compiler places the wait (it waits for the
        // chunks as well: in-flight registers that it does not know about are not safe to hold)
        const uint4 ka = *(const uint4 *)drow(s.kd, na), va = *(const uint4 *)drow(s.vd, na);
        const uint4 kb2 = *(const uint4 *)drow(s.kd, nb2), vb2 = *(const uint4 *)drow(s.vd, nb2);
        if (with_chunks) {
            if (nch > 0) issue(0);
            if (nch > 1) issue(1);
        }
        float qv[8];
        Elem<bf16_t>::unpack(qd, qv);
        float md = -INFINITY, ld = 0.f, od[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) od[x] = 0.f;
        auto one = [&](int node, const uint4 &kraw, const uint4 &vraw) {
            float kf[8], vf[8];
            Elem<bf16_t>::unpack(kraw, kf);
            Elem<bf16_t>::unpack(vraw, vf);
            float dot = 0.f;
#pragma unroll
            for (int x = 0; x < 8; ++x) dot = fmaf(qv[x], kf[x], dot);
            const float z = node >= 0 ? row16_sum(dot) * a.scale_log2 : -INFINITY;
            const float m_new = fmaxf(md, z);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(md - m_use);   // 0 while nothing has been seen
            const float pe = __builtin_amdgcn_exp2f(z - m_use);      // 0 for an empty slot
            ld = fmaf(ld, alpha, pe);
#pragma unroll
            for (int x = 0; x < 8; ++x) od[x] = fmaf(od[x], alpha, pe * vf[x]);
            md = m_new;
        };
        one(na, ka, va);
        one(nb2, kb2, vb2);
        while (anc_lo | anc_hi) {   // root paths longer than 8 nodes (these reads queue behind the chunks)
            const int c0n = pop_node(anc_lo, anc_hi), c1n = pop_node(anc_lo, anc_hi), c2n = pop_node(anc_lo, anc_hi),
                      c3n = pop_node(anc_lo, anc_hi);
            const int nc = r4 == 0 ? c0n : (r4 == 1 ? c1n : (r4 == 2 ? c2n : c3n));
            const uint4 kc = *(const uint4 *)drow(s.kd, nc), vc = *(const uint4 *)drow(s.vd, nc);
            one(nc, kc, vc);
        }
        // the four lane groups hold disjoint parts of the path: merge them (lanes ^16, ^32)
        const float m_all = max_xor32(max_xor16(md));          // finite: the node itself is on its path
        const float wgt = __builtin_amdgcn_exp2f(md - m_all);   // 0 for a group without a node
        ld = sum_xor32(sum_xor16(ld * wgt));
#pragma unroll
        for (int x = 0; x < 8; ++x) od[x] = sum_xor32(sum_xor16(od[x] * wgt));
        if (live && r4 == 0) {
            // channels 8 pos .. 8 pos + 7 sit at positions 4 pos .. + 3 and 64 + 4 pos .. + 3 of the stored order
            const int64_t prow = ((int64_t)(b * s.Hq + h) * part.nsplit + nctx) * s.M + m0 + row;
            float *po = part.o + prow * 128;
            *(float4 *)(po + 4 * pos) = make_float4(od[0], od[1], od[2], od[3]);
            *(float4 *)(po + 64 + 4 * pos) = make_float4(od[4], od[5], od[6], od[7]);
            if (pos == 0) *(float2 *)(part.ml + prow * 2) = make_float2(m_all, ld);
        }
    };
    auto draft_rows = [&]() {
        const int rr0 = sp + ns_eff * wave;
        draft_row(min(rr0, rows_tile - 1), rr0 < rows_tile, true);      // requests chunks 0 and 1 on its way
        for (int rr = rr0 + ns_eff * 8; rr < rows_tile; rr += ns_eff * 8) draft_row(rr, true, false);
    };

    f32x16 O[4];
    RowState st;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[j][i] = 0.f;

    // ---- main loop ---------------------------------------------------------------------
    // The query operands: this wavefront's quarter has landed (the wait for everything requested in the prologue,
    // above); the barrier covers the other wavefronts' quarters.
    auto read_q = [&]() {
        const uint32_t q0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)qstage + (uint32_t)(rb * 8192 + lane * 16);
        const uint32_t qa[8] = {q0, q0 + 1024u, q0 + 2048u, q0 + 3072u, q0 + 4096u, q0 + 5120u, q0 + 6144u, q0 + 7168u};
        uint4 qraw[8];
        lds_read_k<0>(qa, qraw);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(qraw[ks]);
    };
    draft_rows();
    SPECPV_STAMP(2);   // first chunks requested, draft rows done
    for (int i = 0; i < nch_max; ++i) {
        const bool active = i < nch;
        const int stg = i & 1;
        if (i < 4) SPECPV_STAMP(12 + i);   // done with chunk i - 1, about to wait for chunk i
        // own half of chunk i has landed (the only younger group is chunk i+1's)
        if (i + 1 < nch) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();          // ... and so has the partner's half
        if (i < 4) SPECPV_STAMP(3 + i);   // chunk i has landed
        if (i == 0) read_q();
        uint4 kf[8];
        uint2 v[16];
        const uint32_t vmask = vmask_st[stg];
        if (active) {
            const uint32_t soff = (uint32_t)stg * kStageBytes;
            const uint32_t k0 = kread[0] + soff, k1 = kread[1] + soff, k2 = kread[2] + soff, k3 = kread[3] + soff;
            const uint32_t ka[8] = {k0, k1, k2, k3, k0 ^ 128u, k1 ^ 128u, k2 ^ 128u, k3 ^ 128u};
            lds_read_k<0>(ka, kf);
            lds_read_v<0>(vread + soff, v);
        }
        __builtin_amdgcn_s_barrier();          // both wavefronts of the pair hold chunk i in registers
        if (i + 2 < nch) issue(i + 2);
        if (!active) continue;

        attend_chunk(kf, v, qf, vmask, kg, a.scale_log2, O, st);
    }
    __syncthreads();   // every wavefront is done with the rings: the epilogue reuses that LDS
    SPECPV_STAMP(7);   // main loop done

    // ---- merge the four token groups ---------------------------------------------------
    {
        const float l_run = sum_xor32(st.l);
        const int row = rb * 32 + n;
        if (kg == 0) {
            ms[tg * 64 + row] = st.ref(l_run);
            ls[tg * 64 + row] = l_run;
        }
        // accumulator element 4q + x of tile j is channel 32j + 8q + 4kg + x of this lane's row
        float *dst = obuf + ((size_t)tg * 64 + row) * kOPitch;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4 *)(dst + 32 * j + 8 * q + 4 * kg) = make_float4(O[j][4 * q], O[j][4 * q + 1], O[j][4 * q + 2], O[j][4 * q + 3]);
    }
    __syncthreads();
    const int64_t prow0 = ((int64_t)(b * s.Hq + h) * part.nsplit + sp) * s.M;
    // weights of the four token groups for the rows this wavefront finishes (lane -> row)
    float wgt[4], m_row = -INFINITY, l_row = 0.f;
    {
        const int row = wave * RPW + (lane & (RPW - 1));
        float mw[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) { mw[w] = ms[w * 64 + row]; m_row = fmaxf(m_row, mw[w]); }
        const float m_use = m_row == -INFINITY ? 0.f : m_row;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            wgt[w] = __builtin_amdgcn_exp2f(mw[w] - m_use);   // 0 for a token group without valid tokens
            l_row = fmaf(ls[w * 64 + row], wgt[w], l_row);
        }
    }
    {
        // positions 2 lane, 2 lane + 1 of the stored order
        const int chan0 = partial_chan(2 * lane, 128);
        float2 acc[RPW];
#pragma unroll
        for (int uu = 0; uu < RPW; ++uu) {
            const int row = wave * RPW + uu;
            acc[uu] = make_float2(0.f, 0.f);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float ww = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt[w]), uu));   // uniform: no LDS shuffle
                const float2 x = *(const float2 *)(obuf + ((size_t)w * 64 + row) * kOPitch + chan0);
                acc[uu].x = fmaf(ww, x.x, acc[uu].x);
                acc[uu].y = fmaf(ww, x.y, acc[uu].y);
            }
        }
#pragma unroll
        for (int uu = 0; uu < RPW; ++uu) {
            const int j = m0 + wave * RPW + uu;
            if (j < s.M) *(float2 *)(part.o + (prow0 + j) * 128 + 2 * lane) = acc[uu];   // stays in this XCD's L2
        }
    }
    if (lane < RPW) {
        const int j = m0 + wave * RPW + lane;
        if (j < s.M) *(float2 *)(part.ml + (prow0 + j) * 2) = make_float2(m_row, l_row);
    }
    SPECPV_STAMP(8);   // partial stores issued
    if (!REDO) SPECPV_CLOCKS_END(f.timeline, 3072 + ((size_t)blockIdx.y * gridDim.x + blockIdx.x), C);

    // ---- arrival; the last workgroup of the tile finishes it ------------------------
    unsigned long long *word = f.arrive + ((int64_t)(b * s.Hq + h) * 2 + rt);
    unsigned long long *sh_word = (unsigned long long *)lds_raw;   // ms / ls are dead
    int nslots, slot_step;
    if (!redo) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // this wavefront's partial stores have reached L2
        __syncthreads();                      // ... and everybody else's
        SPECPV_STAMP(9);   // partial stores acknowledged
        if (threadIdx.x == 0) {
            const unsigned xcc = (unsigned)__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 7u;   // XCC_ID, 4 bits
            const unsigned long long inc = (1ull << 56) | (1ull << (kXccBits * xcc));
            const unsigned long long now = __hip_atomic_fetch_add(word, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + inc;
            // all arrivals through this XCC's L2?
            const bool here = ((now >> (kXccBits * xcc)) & ((1ull << kXccBits) - 1ull)) == (unsigned long long)nctx;
            sh_word[0] = now >> 56;
            sh_word[1] = (here && !f.force_recompute) ? 1ull : 0ull;
        }
        __syncthreads();
        SPECPV_STAMP(10);  // arrival known
        if ((int)sh_word[0] != nctx) return false;      // not the last one: done
        if (sh_word[1] == 0ull) {
            __syncthreads();                  // sh_word has been read by all
            return true;                      // recompute route: everything of this tile once more, here
        }
        nslots = nctx + 1; slot_step = 1;
    } else {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        nslots = 2; slot_step = nctx;        // this pass's partial (slot 0) and its draft segment (slot nctx)
    }
    if (threadIdx.x == 0) __hip_atomic_exchange(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // Merge.  Lane 8 u + x owns the (m, l) pairs of row u of this wavefront's 8 rows for the slots
    // x, x + 8, ...; the weights pass through LDS (a wavefront's own corner: its LDS operations are
    // executed in order, no barrier).  Every lane accumulates positions 2 lane, 2 lane + 1 of the
    // stored order -- two adjacent channels -- over the slots; the rows go in two batches of four,
    // each batch with up to 4 x 16 reads in flight, the first one requested before the weights
    // are worked out.
    {
        constexpr int kMaxSlots = 80;   // 64 splits + the draft segment, rounded up to a multiple of 16
        float *ww = (float *)(lds_raw + 2048) + (size_t)wave * (RPW * kMaxSlots);   // [8 rows][kMaxSlots]
        const int u8 = lane >> 3, x8 = lane & 7;
        const int jrow = m0 + wave * RPW + u8;
        const int64_t pbase = (int64_t)(b * s.Hq + h) * part.nsplit * s.M;
        const int64_t slot_rows = (int64_t)slot_step * s.M;     // rows between consecutive slots
        const int jmax = s.M - 1;
        const int chan = partial_chan(2 * lane, 128);
        auto ml_of = [&](int sl) -> float2 {
            float2 ml = make_float2(-INFINITY, 0.f);
            if (sl < nslots && jrow < s.M) ml = *(const float2 *)(part.ml + (pbase + sl * slot_rows + jrow) * 2);
            return ml;
        };
        // rows u0 .. u0 + 3, slots sl0 .. sl0 + 15 (those below nslots): two adjacent values per lane
        auto fetch = [&](int u0, int sl0, float2 (&x)[4][16]) {
#pragma unroll
            for (int xi = 0; xi < 16; ++xi) {
                if (sl0 + xi < nslots) {   // uniform
#pragma unroll
                    for (int uu = 0; uu < 4; ++uu) {
                        const int j = min(m0 + wave * RPW + u0 + uu, jmax);   // rows past M repeat row M-1; never stored
                        x[uu][xi] = *(const float2 *)(part.o + (pbase + (sl0 + xi) * slot_rows + j) * 128 + 2 * lane);
                    }
                } else {
#pragma unroll
                    for (int uu = 0; uu < 4; ++uu) x[uu][xi] = make_float2(0.f, 0.f);
                }
            }
        };
        auto accumulate = [&](int u0, int sl0, const float2 (&x)[4][16], float2 (&acc)[4]) {
#pragma unroll
            for (int uu = 0; uu < 4; ++uu) {
                const float *wrow = ww + (u0 + uu) * kMaxSlots + sl0;
#pragma unroll
                for (int x4 = 0; x4 < 4; ++x4) {
                    const float4 w4 = *(const float4 *)(wrow + 4 * x4);
                    const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int xi = 0; xi < 4; ++xi) {
                        acc[uu].x = fmaf(wv[xi], x[uu][4 * x4 + xi].x, acc[uu].x);
                        acc[uu].y = fmaf(wv[xi], x[uu][4 * x4 + xi].y, acc[uu].y);
                    }
                }
            }
        };
        const float2 ml0 = ml_of(x8), ml1 = ml_of(x8 + 8);
        float2 xa[4][16];
        fetch(0, 0, xa);
        // weights of the slots and the denominator of each row
        float m_all = fmaxf(ml0.y > 0.f ? ml0.x : -INFINITY, ml1.y > 0.f ? ml1.x : -INFINITY);
        for (int sl = x8 + 16; sl < nslots; sl += 8) {   // more than 16 slots: rare
            const float2 ml = ml_of(sl);
            m_all = fmaxf(m_all, ml.y > 0.f ? ml.x : -INFINITY);
        }
        m_all = oct_max(m_all);
        const float m_use = m_all == -INFINITY ? 0.f : m_all;
        float den = 0.f;
        {
            const float w0 = ml0.y > 0.f ? __builtin_amdgcn_exp2f(ml0.x - m_use) : 0.f;   // 0 for a slot without a valid token
            const float w1 = ml1.y > 0.f ? __builtin_amdgcn_exp2f(ml1.x - m_use) : 0.f;
            den = fmaf(ml0.y, w0, fmaf(ml1.y, w1, 0.f));
            ww[u8 * kMaxSlots + x8] = w0;
            ww[u8 * kMaxSlots + x8 + 8] = w1;
        }
        const int nslots16 = (nslots + 15) & ~15;
        for (int sl = x8 + 16; sl < nslots16; sl += 8) {
            const float2 ml = ml_of(sl);                  // (-inf, 0) past the last slot
            const float w = ml.y > 0.f ? __builtin_amdgcn_exp2f(ml.x - m_use) : 0.f;
            den = fmaf(ml.y, w, den);
            ww[u8 * kMaxSlots + sl] = w;
        }
        den = oct_sum(den);
        const float inv = 1.f / den;   // den > 0: a node attends itself
#pragma unroll 1
        for (int u0 = 0; u0 < RPW; u0 += 4) {
            float2 acc[4];
#pragma unroll
            for (int uu = 0; uu < 4; ++uu) acc[uu] = make_float2(0.f, 0.f);
            if (u0 > 0) fetch(u0, 0, xa);
            accumulate(u0, 0, xa, acc);
#pragma unroll 1
            for (int sl0 = 16; sl0 < nslots; sl0 += 16) {
                fetch(u0, sl0, xa);
                accumulate(u0, sl0, xa, acc);
            }
#pragma unroll
            for (int uu = 0; uu < 4; ++uu) {
                const int j = m0 + wave * RPW + u0 + uu;
                const float iv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv), (u0 + uu) * 8));
                const uint32_t packed = pack_bf16x2(acc[uu].x * iv, acc[uu].y * iv);
                if (j < s.M)
                    __builtin_nontemporal_store(packed, (uint32_t *)((uint16_t *)f.out + (((int64_t)b * s.M + j) * s.Hq + h) * 128 + chan));
            }
        }
        if (f.lse && x8 == 0 && jrow < s.M)
            f.lse[((int64_t)b * s.M + jrow) * s.Hq + h] = (m_all + __builtin_amdgcn_logf(den)) * kLn2;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    SPECPV_STAMP(11);  // merged and stored (last workgroup of a tile only)
    return false;
}

template <bool ALIGNED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_ctx_mfma_kernel(const int32_t *a_sel_idx, const int32_t *a_sel_count, const int32_t *a_ctx_len,
                          const void *a_q, int a_n_sel, int a_M, int a_Hq, int a_nctx,
                          Shape s, Partials part, MfmaArgs a, FusedArgs f)
{
    // the leading scalar arguments repeat what the first round of reads needs: they arrive in registers
    s.ctx_len = a_ctx_len; s.q = a_q; s.M = a_M; s.Hq = a_Hq;
    a.sel_idx = a_sel_idx; a.sel_count = a_sel_count; a.n_sel = a_n_sel;
    extern __shared__ char lds_raw[];
    const int sp0 = (int)blockIdx.y - (int)a.div_nsplit.div(blockIdx.y) * a_nctx;
    if (attn_ctx_pass<ALIGNED, false>(s, part, a, f, a_nctx, sp0, a_nctx, lds_raw))
        attn_ctx_pass<ALIGNED, true>(s, part, a, f, a_nctx, 0, 1, lds_raw);
}

// ---- group variant: the query heads of a KV head in one workgroup --------------------------
// For long token ranges.  The G x ceil(M / 32) blocks of 32 query rows that share a KV head are
// dealt to workgroups of up to 12 wavefronts (G = 4, M <= 64: one workgroup of 8; more row blocks than 10: two or more
// workgroups).  A workgroup owns (sequence, KV head, its row blocks, KV split) and walks the split's chunks once for
// all of them: its W wavefronts share ONE ring of four stages and each brings its share of a chunk's 16 DMA
// operations, so every K / V byte is requested from memory exactly once per workgroup, whatever
// the caches do.
// The ring has two halves of two chunks.  One workgroup barrier per TWO chunks: at the barrier in
// front of chunks i, i + 1 both have landed (requested one period earlier), every wavefront
// is done with the other half, and chunks i + 2, i + 3 are requested into it at once.  Measured, us per pass with
// [chunks per barrier, chunks in flight]: partial step of four sequences at G = 5 (two layers, 16 chunks a workgroup)
// [4, 4] 86.2, [2, 6] 84.9, [2, 4] 84.7, [2, 3] 81.8, [2, 2] 80.8, [1, 4] 92.5, [1, 1] 82.3; full pass over 64K tokens and 78 nodes
// [4, 4] 117.0, [2, 6] 114.0, [2, 2] 112.3, [1, 3] 117.4, [1, 1] 115.3; over the ragged batch at G = 5 474, 480, 465, 505, 496.
// A barrier per chunk puts the wavefronts of a SIMD back in step every chunk, so that they queue for the LDS, the
// matrix cores and the vector ALU together instead of filling each other's gaps; requests further ahead gain nothing
// once a period covers the latency of memory, and the first chunks wait behind them.
// A wavefront keeps its rows to itself over the whole split, so the epilogue has nothing to
// merge: it only turns the accumulators into row-major partials.
// The chunk loop is unrolled over the ring stages: with the stage a compile-time constant,
// stage offsets are immediate fields of the LDS reads and of the requests' LDS addresses, the
// validity words of the stages are scalar registers, and the request of a chunk tests the common
// case (32 valid consecutive rows) first.  What a wavefront executes per chunk besides its
// arithmetic is what this loop pays for: measured in core cycles per chunk and workgroup (128K
// context, 32 splits, eight row blocks), 2590 with a run-time stage and a barrier per chunk, 2295 unrolled, 2085
// with a period of four chunks, 2033 with two; 1400 for the requests and barriers alone (timing probe), 1024 for
// the matrix instructions.
// Where every wavefront has a row block to itself and 256 registers (128 channels, four or eight row blocks), the two
// chunks of a ring half are worked on together (score_pair, attend_pair): 1800 cycles per chunk.
constexpr int kGroupPeriod = 2;                  // chunks between two workgroup barriers
constexpr int kGroupStages = 2 * kGroupPeriod;   // two halves
// One 32-token chunk in LDS.  128 channels: as above (kStageBytes).  64 channels: 4 KiB of K (128-byte rows, 16-byte
// pieces XOR-swizzled by (row >> 1) & 7: two rows make one 256-byte bank row), V in four 1 KiB operations of two pieces
// each (lds_read_v64).
template <int D> struct Tile;
template <> struct Tile<128> {
    static constexpr int kK = 8192, kVOpPitch = kVPiecePitch, kStage = kStageBytes;
    static constexpr int kRowPitch = 272, kRows = 32 * kRowPitch, kHandOver = 64 * 64 * 4 + 512;   // staged rows of a row block; accumulators, m and l of another wavefront
};
template <> struct Tile<64> {
    static constexpr int kK = 4096, kVOpPitch = 1152, kStage = kK + 4 * kVOpPitch;
    static constexpr int kRowPitch = 272, kRows = 32 * kRowPitch, kHandOver = 64 * 32 * 4 + 512;
};
static_assert(Tile<64>::kStage % 256 == 0 && kStageBytes % 256 == 0, "K operand addresses are derived by XOR with multiples of 32 below 256: stages (and the rings) must start 256-byte aligned");

// RB row blocks per workgroup: 2, 4, 6, 8 or 10.  The CU has four SIMDs: up to four, or eight, row blocks have a wavefront
// each; the two that 2, 6 and 10 leave over are shared by two wavefronts each, one of which takes the even chunks and one
// the odd ones, so that every SIMD has the same work (before, a wavefront per row block: full pass over a ragged batch of 320K tokens at
// G = 5, 64 nodes, 525 us, 460 with twelve wavefronts; 64 channels, 37 nodes at G = 4 over 45K tokens, 51 us, 43 with
// eight for its five row blocks; one and two row blocks over 8K to 128K tokens, 20 % less).
// Ten row blocks (nine or ten: G = 5 with up to 64 nodes) are twelve wavefronts, three per SIMD, i.e. at most 168
// registers each: that variant takes its K and V operands in halves.
constexpr int group_waves(int rb) { return rb % 4 ? (rb & ~3) + 4 : rb; }
// LDS: the ring, and in its place at the end the staged rows of all row blocks, and the sums that the odd chunks' wavefronts
// hand over.
template <int D> constexpr int group_lds(int rb)
{
    const int ring = kGroupStages * Tile<D>::kStage, rows = rb * Tile<D>::kRows + (rb % 4 ? 2 * Tile<D>::kHandOver : 0);
    return ring > rows ? ring : rows;
}
static_assert(group_lds<128>(10) <= 160 * 1024 && group_lds<128>(4) <= 80 * 1024 && group_lds<64>(8) <= 80 * 1024, "");
// D = 64: half the LDS and half the operand registers, so two workgroups share a CU (four wavefronts per SIMD, 128
// registers): at 64 channels a chunk has half the matrix work against the same softmax, and what counts is how many
// wavefronts the vector ALU can choose from.  The weights enter the second product as three bf16 terms, all 24 bits of
// fp32, and the partials are fp32 sums: the precision, and the range of V, of the vector-ALU kernel that this replaces.
// Rows whose exact result cancels to 0, error relative to sum |w v|, rms over 300 / 2048 / 16384 tokens: vector ALU
// 2.3e-8 / 1.3e-8 / 6.5e-9, here 1.9e-8 / 1.1e-8 / 4.9e-9, with two terms (16 bits) 3.6e-7 / 1.4e-7 / 5.6e-8.  Full pass
// over 15K + 30K tokens, 37 nodes at G = 4, 8 KV heads, token-major, with scoring and selection: 5845 us on the vector
// ALU, 62.4 us here (55.1 us with two terms; 67.4 us with three whose differences take a widening and a subtraction each).
// SK: shares of the chunks of all (sequence, KV head) pairs instead of splits (Partials::stream): a workgroup goes through
// the one to three pairs that its share touches, one after the other.
template <int D, int SPAN, int RB, bool SK>
__global__ __launch_bounds__(64 * group_waves(RB)) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : (RB > 8 ? 3 : 2), D == 64 ? 4 : (RB > 8 ? 3 : 2))))
void attn_ctx_mfma_group_kernel(Shape s, Partials part, MfmaArgs a)
{
    typedef Tile<D> TL;
    constexpr int W = group_waves(RB), F = RB & ~3;   // wavefronts; those with a row block to themselves
    constexpr bool PAIRED = W != RB;                // the others share one between two
    constexpr bool PAIRS = D == 128 && !PAIRED;     // chunks are taken two at a time
    constexpr int KS = D / 16, NT = D / 32;         // k-steps of S^T, channel tiles of O^T
    constexpr int LPR = D / 8, RPO = 64 / LPR;      // lanes per row, rows per 1 KiB operation
    constexpr int KOPS = D / 16, OPS = 2 * KOPS;    // DMA operations of a chunk: K, then V
    SPECPV_CLOCKS_BEGIN;
    extern __shared__ char lds_raw[];
    char *ring = lds_raw;                  // [kGroupStages][K 8 KiB | V 8 pieces of 1088 B]

    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (D == 128 && SPAN == 32) {
        if ((int)blockIdx.y < a.sum_rows) {
            // a workgroup for the summaries: its wavefronts take every n-th of the stale blocks (or twos, fours of small ones) of all pairs
            const int per = s.B == 16 ? 4 : (s.B == 32 ? 2 : 1);
            const int wgs = a.sum_rows * (int)gridDim.x, n = wgs * W;
            int at = wave * wgs + (int)blockIdx.y * (int)gridDim.x + (int)blockIdx.x;
            for (int b = 0; b < s.batch; ++b) {
                const int L = s.ctx_len[b];
                const int nb = min(L > 0 ? (int)a.div_B.div((uint32_t)L + (uint32_t)s.B - 1u) : 0, s.max_blocks), stale = (max(nb - a.sum_begin, 0) + per - 1) / per;
                for (int g = 0; g < s.Hkv; ++g) {
                    for (; at < stale; at += n) {
                        const int i = a.sum_begin + at * per;
                        if (per == 1) summarize_block<bf16_t, D>(s, b, g, i, L, a.kmax, a.kmin, lane);
                        else if (per == 2) summarize_small<bf16_t, D, 8>(s, b, g, i, nb, L, a.kmax, a.kmin, lane);
                        else summarize_small<bf16_t, D, 4>(s, b, g, i, nb, L, a.kmax, a.kmin, lane);
                    }
                    at -= stale;
                }
            }
            return;
        }
    }
    const int xcd = blockIdx.x & 7, wg_part = blockIdx.x >> 3;
    const int u = ((int)blockIdx.y - (D == 128 && SPAN == 32 ? a.sum_rows : 0)) * 8 + xcd;
    if (u >= a.n_units) return;
    // this wavefront's row block: rows r0w .. r0w + 31 of the KV head's M * G query rows.  A
    // workgroup may have a wavefront too many (row block counts that do not divide): it brings
    // its share of the chunks and keeps the barriers, but computes and stores nothing.
    const int rb = wave < F ? wave : F + ((wave - F) >> 1), odd = wave < F ? 0 : (wave - F) & 1;
    const int rbx = wg_part * RB + rb;
    const bool live = rbx < a.n_row_blocks;
    const int R = s.M * s.G;                  // query rows of the KV head: row r is head r / M of the group, node r % M
    const int r0w = (live ? rbx : a.n_row_blocks - 1) * 32;
    int share_at = 0, share_end = 1;   // SK: this workgroup's chunks in the row of all pairs' chunks
    int seq_chunks = 0, seq_upto = 0;
    if (SK) {
        const StreamShare sh(s, lane, part.stream);
        if (u >= sh.wgs) return;
        share_at = sh.begin(u);
        share_end = sh.begin(u + 1);
        seq_chunks = sh.chunks;
        seq_upto = sh.upto;
    }
    do {
    if (SK) asm volatile("" : "+v"(lane));   // what follows from it is worked out per pair, not held in registers
    const int n = lane & 31, kg = lane >> 5;
    int bg, b, g, c0, nch, sp = 0;
    if (SK) {
        b = __popcll(__ballot(seq_upto * s.Hkv <= share_at));
        const int C_b = __builtin_amdgcn_readlane(seq_chunks, b), before = (__builtin_amdgcn_readlane(seq_upto, b) - C_b) * s.Hkv;
        g = (int)((uint32_t)(share_at - before) / (uint32_t)C_b);
        bg = b * s.Hkv + g;
        c0 = share_at - before - g * C_b;
        nch = min(C_b - c0, share_end - share_at);
        share_at += nch;
    } else {
        bg = (int)a.div_nsplit.div((uint32_t)u);
        sp = u - bg * part.nsplit;
        b = (int)a.div_hkv.div((uint32_t)bg);
        g = bg - b * s.Hkv;
    }

    const int32_t *sel = a.sel_idx ? a.sel_idx + (int64_t)bg * a.n_sel : nullptr;
    const int NS = part.nsplit;               // div_W divides by the number of splits here
    const uint32_t Bu = (uint32_t)s.B;
    const int L = s.ctx_len[b];
    const int cnt_raw = sel ? a.sel_count[bg] : 0;
    auto first_chunk = [&](uint32_t chunks, int w) -> int {
        const uint32_t base = a.div_W.div(chunks), rem = chunks - base * (uint32_t)NS;
        return (int)((uint32_t)w * base + min((uint32_t)w, rem));
    };
    uint4 qraw[KS];
    {
        const int r = min(r0w + n, R - 1);    // rows past the end repeat the last one; never stored
        const int hh = (int)a.div_M.div((uint32_t)r), j = r - hh * s.M;
        const uint16_t *qrow = (const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * D + kg * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qraw[ks] = *(const uint4 *)(qrow + ks * 16);
    }

    int nb = L > 0 ? (int)a.div_B.div((uint32_t)(L + s.B - 1)) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    int cnt = nb;
    if (sel) cnt = max(0, min(cnt_raw, a.n_sel));
    const uint32_t T = nb > 0 ? (uint32_t)cnt * Bu : 0u;
    // chunks of cache tokens, then those of the partially verified tokens (see attn_ctx_mfma_kernel)
    const uint32_t C_ctx = (T + 31u) >> 5;
    const uint32_t C = C_ctx + (((uint32_t)s.kctx + 31u) >> 5);
    const char *kdb = (const char *)s.kd + (((int64_t)b * s.Mk) * s.Hkv + g) * (2 * D);
    const char *vdb = (const char *)s.vd + (((int64_t)b * s.Mk) * s.Hkv + g) * (2 * D);
    const uint32_t stp = (uint32_t)s.Hkv * (2u * D);
    // the number of chunks is the same for all wavefronts: the barriers match up
    if (!SK) {
        c0 = first_chunk(C, sp);
        nch = first_chunk(C, sp + 1) - c0;
    }

    const char *kb = (const char *)s.k + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const char *vb = (const char *)s.v + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const uint32_t st2 = (uint32_t)s.st * 2u;

    const uint32_t ring_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ring;
    // K operand of k-step ks: row n, piece 2 ks + kg, at kread ^ (32 ks) (+ stage): the swizzle is an XOR on the piece and
    // rows start 128- or 256-byte aligned
    const uint32_t kread0 = ring_addr + (uint32_t)n * (2u * D) + (16u * (uint32_t)kg ^ (D == 128 ? 16u * ((uint32_t)n & 15u) : 16u * (((uint32_t)n >> 1) & 7u)));
    const uint32_t vp = (uint32_t)(4 * kg + ((lane & 15) >> 2)), vb0 = 32u * (uint32_t)((lane >> 4) & 1) + 8u * (uint32_t)(lane & 3);
    const uint32_t vread = ring_addr + TL::kK + vb0 + (D == 128 ? vp * kVPiecePitch : (vp >> 1) * Tile<64>::kVOpPitch + (vp & 1u) * 576u);
    const uint32_t vread1 = D == 128 ? 0u : (vp & 1u) ? vread - 64u : vread + 64u;   // 64 channels: tile 1 (see lds_read_v64)

    // ---- chunk -> token rows (see ChunkRows) ---------------------------------------------
    // SPAN: the first rows of the next 64 runs sit in a register (lane t: run t from chunk row_base on) and are
    // picked with readlane; kPendingChunk: a chunk of partially verified tokens.
    constexpr int kPendingChunk = (int)0x80000000;
    constexpr int RUN = SPAN ? SPAN : 32, RPC = 32 / RUN, CPF = 64 / RPC;   // tokens of a run, runs of a chunk, chunks of 64 runs
    const ChunkRows rows_of{sel, a.div_B, s.B, nb, min(L, nb * s.B), T};
    int row_base = 0, row0vec = -1;
    auto fill_rows = [&](int cb) {
        row_base = cb;
        const int c = cb + lane / RPC;
        int r = -1;
        if (c < nch && (uint32_t)(c0 + c) >= C_ctx) r = kPendingChunk;
        if (c < nch && (uint32_t)(c0 + c) < C_ctx) r = rows_of.first_row<RUN>((uint32_t)((c0 + cb) * RPC + lane));
        row0vec = r;
        // wait for the list entries here, inside the rare branch, so that the common path that
        // joins behind it carries no pending load (and no wait on the DMA prefetch)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    };

    // Request this wavefront's operations of chunk ci into stage stg (1 KiB each: LPR lanes per row).  K operation i
    // brings rows RPO i .. RPO i + RPO - 1, pieces swizzled; V operation i at 128 channels rows i, i+8, i+16, i+24
    // (piece i), at 64 channels the pieces 2 i and 2 i + 1.  A wavefront takes operations op0, op0 + W, op0 + 2W, ...
    // Returns the validity bits of the chunk's 32 tokens.
    // Everything that depends on the wavefront is folded into a few registers up front, so that
    // the common path is straight-line code.
    constexpr int NOPS = (OPS + W - 1) / W;
    const int op0 = PAIRED ? (wave < F ? wave + W - F : wave - F) : wave;   // (those with half the arithmetic request more)
    const int n_ops = (OPS - op0 + W - 1) / W;       // NOPS or NOPS - 1
    // the row of the chunk that lane ln fetches for operation o, and the byte offset of its 16-byte piece in the row
    auto op_row = [](int o, int ln) -> int {
        const int i = o & (KOPS - 1), rl = ln / LPR;
        if (o < KOPS) return RPO * i + rl;
        return D == 128 ? 8 * rl + i : 2 * i + (rl >> 2) + 8 * (rl & 3);
    };
    auto op_piece = [&](int o, int ln) -> uint32_t {
        const int pos = ln % LPR, row = op_row(o, ln);
        if (o < KOPS) return 16u * (uint32_t)(pos ^ (D == 128 ? row & 15 : (row >> 1) & 7));
        return 16u * (uint32_t)(D == 128 ? pos : pos ^ (4 * (row & 1)));
    };
    const char *src_base[NOPS];   // per operation: K or V slab (wave-uniform: scalar registers)
    uint32_t src_off[NOPS];       // ... this lane's bytes from the chunk's first row (one register each)
    int dst_off[NOPS];            // ... and where it lands in the stage
#pragma unroll
    for (int t = 0; t < NOPS; ++t) {
        const int o = min(op0 + W * t, OPS - 1), i = o & (KOPS - 1);
        src_base[t] = o < KOPS ? kb : vb;
        src_off[t] = (uint32_t)op_row(o, lane) * st2 + op_piece(o, lane);
        dst_off[t] = o < KOPS ? i * 1024 : TL::kK + i * TL::kVOpPitch;
    }
    auto issue_rows = [&](const char *kbase, const char *vbase, const uint32_t stride, const uint32_t tk, char *dst) {
        // (the swizzles are recomputed here, from a lane id the compiler cannot see through: kept in registers
        // across the loop for this rare path they cost the twelve-wavefront variant its last free registers)
        int lane_o = lane;
        asm volatile("" : "+v"(lane_o));
#pragma unroll
        for (int t = 0; t < NOPS; ++t) {
            if (OPS % W != 0 && t == NOPS - 1 && n_ops != NOPS) continue;
            const int o = op0 + W * t;
            const uint32_t tv = (uint32_t)__shfl((int)tk, op_row(o, lane_o)) * stride;
            dma16((o < KOPS ? kbase : vbase) + (tv + op_piece(o, lane_o)), dst + dst_off[t]);
        }
    };
    // both runs of 16 rows whole: this lane's row of an operation lies in the first or in the second
    auto request_runs = [&](int r0, int r1, char *dst) __attribute__((always_inline)) {
        int lane_o = lane;
        asm volatile("" : "+v"(lane_o));
#pragma unroll
        for (int t = 0; t < NOPS; ++t) {
            if (OPS % W != 0 && t == NOPS - 1 && n_ops != NOPS) continue;
            const int o = op0 + W * t;
            const uint32_t run = (uint32_t)(op_row(o, lane_o) < 16 ? r0 : r1 - 16) * st2;   // (modulo 2^32)
            __builtin_amdgcn_global_load_lds((glb_void_ptr)(src_base[t] + (run + src_off[t])), (lds_void_ptr)(dst + dst_off[t]), 16, 0, kKvAux);
        }
    };
    // Stage stg of the ring is a compile-time constant in the loop below (unrolled over the stages).
    auto issue = [&](int ci, int stg) __attribute__((always_inline)) -> uint32_t {
        char *dst = ring + stg * TL::kStage;
        int tok;
        if (SPAN) {
            if (ci - row_base >= CPF) fill_rows(ci);
            const int r0 = __builtin_amdgcn_readlane(row0vec, RPC * (ci - row_base));
            const int r1 = SPAN == 16 ? __builtin_amdgcn_readlane(row0vec, RPC * (ci - row_base) + 1) : 0;
            if (SPAN == 16 && (r0 | r1) >= 0) {
                request_runs(r0, r1, dst);
                return 0xffffffffu;
            }
            if (SPAN == 32 && r0 >= 0) {
                const uint32_t row_off = (uint32_t)r0 * st2;   // fits 32 bits (host-checked)
#pragma unroll
                for (int t = 0; t < NOPS; ++t)
                    if (OPS % W == 0 || t < NOPS - 1 || n_ops == NOPS) {
                        uint32_t so = src_off[t];
                        // (168 registers: keep the 32-bit offset as it is; the compiler would otherwise carry the 64-bit sum
                        // base + offset of every operation through the loop, in registers that this variant does not have)
                        if (RB > 8) asm volatile("" : "+v"(so));
                        __builtin_amdgcn_global_load_lds((glb_void_ptr)((src_base[t] + row_off) + so), (lds_void_ptr)(dst + dst_off[t]), 16, 0, kKvAux);
                    }
                return 0xffffffffu;
            }
            if (r0 == kPendingChunk) {
                const int pr = (int)((uint32_t)(c0 + ci) - C_ctx) * 32 + n;
                const int ptok = pr < s.kctx ? pr : -1;
                issue_rows(kdb, vdb, stp, (uint32_t)max(ptok, 0), dst);
                return (uint32_t)__ballot(ptok >= 0);
            }
            tok = SPAN == 32 ? rows_of.decode(r0, n) : rows_of.decode(n < 16 ? r0 : r1, n & 15);
        } else {
            if (s.kctx > 0 && (uint32_t)(c0 + ci) >= C_ctx) {
                const int pr = (int)((uint32_t)(c0 + ci) - C_ctx) * 32 + n;
                const int ptok = pr < s.kctx ? pr : -1;
                issue_rows(kdb, vdb, stp, (uint32_t)max(ptok, 0), dst);
                return (uint32_t)__ballot(ptok >= 0);
            }
            tok = rows_of.row((uint32_t)(c0 + ci), n);
        }
        const uint32_t vm = (uint32_t)__ballot(tok >= 0);
        const uint32_t tk = tok >= 0 ? (uint32_t)tok : 0u;   // row 0 exists (L > 0); masked later
        issue_rows(kb, vb, st2, tk, dst);
        return vm;
    };

    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = as_bf16x8(qraw[ks]);
    if (SPAN && nch > 0) fill_rows(0);
    // from here on only this wavefront's DMA groups (n_ops operations each) are in flight (an
    // instruction the compiler knows, see attn_ctx_mfma_kernel)
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");

    f32x16 O[NT];
    RowState st;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[j][i] = 0.f;

    // validity bits of the chunks in the ring, one word per stage (the same in every lane)
    uint32_t vm_stage[kGroupStages] = {0u, 0u, 0u, 0u};
    static_assert(kGroupPeriod == 2, "the first requests and the loop below are written for two halves of two stages");
    if (0 < nch) vm_stage[0] = issue(0, 0);
    if (1 < nch) vm_stage[1] = issue(1, 1);
    uint2 v[4 * NT];
    uint4 pf0 = make_uint4(0u, 0u, 0u, 0u), pf1 = pf0;
    auto pv = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const uint2 lo = v[(ks2 * NT + j) * 2], hi = v[(ks2 * NT + j) * 2 + 1];
                O[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)),
                                                               as_bf16x8(ks2 ? pf1 : pf0), O[j], 0, 0, 0);
            }
    };
    // three wavefronts per SIMD: operands in halves (16 registers at a time instead of 32)
    auto pv_halves = [&](const uint32_t vaddr, auto off) __attribute__((always_inline)) {
        constexpr int OFF = decltype(off)::value;
        uint2 vh[8];
        lds_read_v_half<OFF>(vaddr, vh);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            O[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(vh[2 * j].x, vh[2 * j].y, vh[2 * j + 1].x, vh[2 * j + 1].y)),
                                                           as_bf16x8(pf0), O[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        lds_read_v_half<OFF + 512>(vaddr, vh);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            O[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(vh[2 * j].x, vh[2 * j].y, vh[2 * j + 1].x, vh[2 * j + 1].y)),
                                                           as_bf16x8(pf1), O[j], 0, 0, 0);
    };
    // One chunk; its ring stage U = i % 4 is a compile-time constant (the loop below is unrolled over the
    // stages), so that stage offsets are immediate fields of the LDS reads and of the requests' LDS
    // addresses, and the validity words live in scalar registers.
    // The stage inside its ring half is an immediate field of the LDS reads (16 bits), the half is reached through the
    // address register.  A row block's two wavefronts take the even and the odd chunks.
    const bool live0 = live && (!PAIRED || wave < F || odd == 0), live1 = live && (!PAIRED || wave < F || odd == 1);
    auto chunk = [&](auto stage, const uint32_t vmask) __attribute__((always_inline)) {
        constexpr int U = decltype(stage)::value;
        constexpr int SOFF = (U % kGroupPeriod) * TL::kStage;
        constexpr uint32_t HOFF = (uint32_t)(U / kGroupPeriod) * kGroupPeriod * TL::kStage;
        if (!((U & 1) ? live1 : live0)) return;
        f32x16 S;
        if constexpr (RB > 8) {
            // three wavefronts per SIMD: operands in halves, the V operands read behind the softmax (pv_halves)
            // (k-step ks reads 32 ks bytes further, modulo the swizzle: an XOR, as the row starts are 128-byte aligned)
            const uint32_t ka0 = kread0 + HOFF;
            const uint32_t ka[4] = {ka0, ka0 ^ 32u, ka0 ^ 64u, ka0 ^ 96u};
            uint4 kh[4];
            lds_read_k_half<SOFF>(ka, kh);
#pragma unroll
            for (int x = 0; x < 16; ++x) S[x] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kh[ks]), qf[ks], S, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t kb4[4] = {ka0 ^ 128u, ka0 ^ 160u, ka0 ^ 192u, ka0 ^ 224u};
            lds_read_k_half<SOFF>(kb4, kh);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kh[ks]), qf[4 + ks], S, 0, 0, 0);
        } else {
            const uint32_t k0 = kread0 + HOFF, k1 = k0 ^ 32u, k2 = k0 ^ 64u, k3 = k0 ^ 96u;
            uint4 kf[KS];
            if constexpr (D == 128) {
                const uint32_t ka[8] = {k0, k1, k2, k3, k0 ^ 128u, k1 ^ 128u, k2 ^ 128u, k3 ^ 128u};
                lds_read_k<SOFF>(ka, kf);
                lds_read_v<SOFF>(vread + HOFF, v);
            } else {
                const uint32_t ka[4] = {k0, k1, k2, k3};
                lds_read_k_half<SOFF>(ka, kf);
                lds_read_v64<SOFF>(vread + HOFF, vread1 + HOFF, v);
            }
#pragma unroll
            for (int x = 0; x < 16; ++x) S[x] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), qf[ks], S, 0, 0, 0);
        }

        mask_scores(vmask, kg, S);
        follow_max(tile_max(S), a.scale_log2, st, O);
        uint32_t pk[8];
        if constexpr (D == 128) {
            softmax_weights(S, a.scale_log2, st, pk);
        } else {
            float lsum = 0.f;
#pragma unroll
            for (int x = 0; x < 16; x += 2) {
                S[x] = __builtin_amdgcn_exp2f(fmaf(S[x], a.scale_log2, st.neg_ref));
                S[x + 1] = __builtin_amdgcn_exp2f(fmaf(S[x + 1], a.scale_log2, st.neg_ref));
                pk[x >> 1] = pack_bf16x2(S[x], S[x + 1]);
                lsum += S[x] + S[x + 1];
            }
            st.l += lsum;
        }
        pf0 = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        pf1 = make_uint4(pk[4], pk[5], pk[6], pk[7]);
        if constexpr (RB > 8) pv_halves(vread + HOFF, std::integral_constant<int, SOFF>{});
        else pv();
        if constexpr (D == 64) {
            // what the rounding of the weights left over, twice: each term takes eight bits more (the differences are exact)
            const Bf16Halves halves;
#pragma unroll
            for (int term = 1; term < 3; ++term) {
#pragma unroll
                for (int x = 0; x < 16; x += 2) {
                    S[x] = halves.sub_lo(S[x], pk[x >> 1]);
                    S[x + 1] = halves.sub_hi(S[x + 1], pk[x >> 1]);
                    pk[x >> 1] = pack_bf16x2(S[x], S[x + 1]);
                }
                pf0 = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                pf1 = make_uint4(pk[4], pk[5], pk[6], pk[7]);
                pv();
            }
        }
    };
    // Two chunks between two barriers.  At the barrier in front of chunks i0, i0 + 1 (ring half H) every
    // wavefront's requests have landed -- they were made a whole period ago, so the wait is for all of
    // them -- and every wavefront is done with the other half, into which the next two chunks are
    // requested at once; then come two chunks of arithmetic without a request or a wait in between.
    auto period = [&](const int i0, auto half) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value, S0 = kGroupPeriod * H, N0 = kGroupPeriod * (1 - H);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if (i0 + 2 < nch) vm_stage[N0] = issue(i0 + 2, N0);
        if (i0 + 3 < nch) vm_stage[N0 + 1] = issue(i0 + 3, N0 + 1);
        chunk(std::integral_constant<int, S0>{}, vm_stage[S0]);
        if (i0 + 1 < nch) chunk(std::integral_constant<int, S0 + 1>{}, vm_stage[S0 + 1]);
    };
    if constexpr (PAIRS) {
        // A ring half at once, 64 tokens: scores and V operands into registers (score_pair), then softmax and values.
        uint32_t next0 = vm_stage[0], next1 = vm_stage[1];   // validity of the chunks requested last
        // chunks i, i + 1 (even i) into their ring half: what a wavefront executes here is in front of its arithmetic, so the
        // common case, both there and whole, is one test
        auto request = [&](int i) __attribute__((always_inline)) {
            if (SPAN == 32 && i + 1 < nch && i + 1 - row_base < CPF) {
                const int ra = __builtin_amdgcn_readlane(row0vec, i - row_base), rb2 = __builtin_amdgcn_readlane(row0vec, i + 1 - row_base);
                if ((ra | rb2) >= 0) {
                    char *dst = ring + (i & 2) * TL::kStage;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t row_off = (uint32_t)(h ? rb2 : ra) * st2;
#pragma unroll
                        for (int t = 0; t < NOPS; ++t)
                            if (OPS % W == 0 || t < NOPS - 1 || n_ops == NOPS)
                                __builtin_amdgcn_global_load_lds((glb_void_ptr)((src_base[t] + row_off) + src_off[t]), (lds_void_ptr)(dst + h * TL::kStage + dst_off[t]), 16, 0, kKvAux);
                    }
                    next0 = next1 = 0xffffffffu;
                    return;
                }
            }
#pragma unroll 1
            for (int c = i; c < min(i + 2, nch); ++c) {
                const uint32_t vm = issue(c, c & 3);
                next0 = c & 1 ? next0 : vm;
                next1 = c & 1 ? vm : next1;
            }
        };
        int i0 = 0;
        for (; i0 + 1 < nch; i0 += 2) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // chunks i0, i0 + 1 have landed; the other half is free
            const uint32_t vm0 = next0, vm1 = next1;
            request(i0 + 2);
            const uint32_t off = (uint32_t)(i0 & 2) * TL::kStage;
            const uint32_t k0 = kread0 + off, ka[8] = {k0, k0 ^ 32u, k0 ^ 64u, k0 ^ 96u, k0 ^ 128u, k0 ^ 160u, k0 ^ 192u, k0 ^ 224u};
            f32x16 Sa, Sb;
            uint4 va[8], vb[8];
            if (live) score_pair<0, TL::kStage, 0, TL::kStage>(ka, vread + off, qf, Sa, Sb, va, vb);
            if (live) attend_pair(Sa, Sb, va, vb, vm0, vm1, kg, a.scale_log2, O, st);
        }
        if (i0 < nch) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
        }
        if (i0 < nch) {   // an odd chunk at the end
            if (i0 & 2) chunk(std::integral_constant<int, 2>{}, next0);
            else chunk(std::integral_constant<int, 0>{}, next0);
        }
    } else
    for (int i0 = 0; i0 < nch; i0 += kGroupStages) {
        period(i0, std::integral_constant<int, 0>{});
        if (i0 + kGroupPeriod < nch) period(i0 + kGroupPeriod, std::integral_constant<int, 1>{});
    }
    __syncthreads();   // every wavefront is done with the ring: the epilogue reuses that LDS

    // ---- one partial per (head, split, node): accumulators -> row-major through LDS ------
    if (PAIRED) {
        // the odd chunks' wavefront hands its sums over as they lie in its registers, behind the staged rows
        float *raw = (float *)(ring + RB * TL::kRows + (rb - F) * TL::kHandOver);
        if (wave >= F && odd) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(float4 *)(raw + ((j * 4 + q) * 64 + lane) * 4) = make_float4(O[j][4 * q], O[j][4 * q + 1], O[j][4 * q + 2], O[j][4 * q + 3]);
            *(float2 *)(raw + NT * 1024 + 2 * lane) = make_float2(-st.neg_ref, st.l);
        }
        __syncthreads();
        if (wave >= F && !odd) {
            const float2 ml = *(const float2 *)(raw + NT * 1024 + 2 * lane);
            const float ref = -st.neg_ref, ref_new = fmaxf(ref, ml.x);
            const float a0 = __builtin_amdgcn_exp2f(ref - ref_new), a1 = __builtin_amdgcn_exp2f(ml.x - ref_new);
            st.neg_ref = -ref_new;
            st.l = st.l * a0 + ml.y * a1;
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 x = *(const float4 *)(raw + ((j * 4 + q) * 64 + lane) * 4);
                    O[j][4 * q] = fmaf(x.x, a1, O[j][4 * q] * a0);
                    O[j][4 * q + 1] = fmaf(x.y, a1, O[j][4 * q + 1] * a0);
                    O[j][4 * q + 2] = fmaf(x.z, a1, O[j][4 * q + 2] * a0);
                    O[j][4 * q + 3] = fmaf(x.w, a1, O[j][4 * q + 3] * a0);
                }
        }
    }
    if (live && !odd) {
    const float l_run = sum_xor32(st.l);
    const int64_t prow0 = (SK ? (int64_t)(u + bg) : (int64_t)bg * part.nsplit + sp) * R + r0w;
    const int n_rows = min(32, R - r0w);
    // accumulator element 4q + x of tile j is channel 32j + 8q + 4kg + x of this lane's row.  A wavefront reads back
    // only what it wrote itself: no barrier.  Sixteen bytes per lane, four rows per store; at 128 channels normalised and
    // rounded to fp16 on the way into LDS, so that all row blocks have room there at once (as fp32, ten row blocks took
    // turns and stores were a row each: partial step of four sequences at G = 5, two layers, 92.8 us, 88.1 so).
    char *rows = ring + rb * TL::kRows;
    if constexpr (D == 128) {   // the normalised result as fp16
        const float il = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(uint2 *)(rows + n * TL::kRowPitch + 64 * j + 16 * q + 8 * kg) =
                    make_uint2(half_pair(O[j][4 * q] * il, O[j][4 * q + 1] * il), half_pair(O[j][4 * q + 2] * il, O[j][4 * q + 3] * il));
    } else {                    // the sums as fp32
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4 *)(rows + n * TL::kRowPitch + 128 * j + 32 * q + 16 * kg) = make_float4(O[j][4 * q], O[j][4 * q + 1], O[j][4 * q + 2], O[j][4 * q + 3]);
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int uu = 0; uu < 8; ++uu) {
        const int row = 4 * uu + (lane >> 4);
        const u32x4 x = *(const u32x4 *)(rows + row * TL::kRowPitch + 16 * (lane & 15));
        if (row < n_rows) __builtin_nontemporal_store(x, (u32x4 *)(part.o + (prow0 + row) * 64) + (lane & 15));
    }
    if (kg == 0 && n < n_rows) *(float2 *)(part.ml + (prow0 + n) * 2) = make_float2(st.ref(l_run), l_run);
    if (!SK || share_at >= share_end) SPECPV_CLOCKS_END(part.timeline, (size_t)blockIdx.y * gridDim.x + blockIdx.x, nch);
    }
    if (SK) __syncthreads();   // the next pair's chunks go where the rows were staged
    } while (SK && share_at < share_end);
}

bool attn_ctx_mfma_supported(const Shape &s, int dtype)
{
    // per-lane byte offsets inside one (sequence, KV head) slab are kept in 32 bits
    const int64_t span = ((int64_t)s.max_blocks * s.B + 64) * s.st * 2;
    return dtype == SPECPV_BF16 && s.st % 8 == 0 && span < ((int64_t)1 << 31);
}

// The KV head's M * G query rows in blocks of 32 (packed over the query heads: 78 nodes at G = 4 are 10 blocks, not 12),
// and how the group kernel deals them to workgroups: 2, 4, 6, 8 or 10 each.
struct GroupLayout {
    int n_row_blocks, parts, blocks;
};
static GroupLayout group_layout(const Shape &s)
{
    GroupLayout g{(s.G * s.M + 31) / 32, 0, 0};
    // the fewest microseconds per chunk for all row blocks (attn_group_chunk_us; a part also pulls the chunk
    // through its L2; full pass over 128K tokens, 8 KV heads, the best of 16 and 32 splits: eight row blocks in one workgroup
    // 148 us, in two of four 159; ten in one 177, in two of six 219, in two of eight 245; four in one 105, in two of two 112)
    double best = -1.0;
    for (int blocks = 2; blocks <= (s.D == 128 ? 10 : 8); blocks += 2) {
        const int parts = (g.n_row_blocks + blocks - 1) / blocks;
        const double us = parts * (attn_group_chunk_us(blocks) + 0.05);
        if (best < 0.0 || us < best) { best = us; g.parts = parts; g.blocks = blocks; }
    }
    return g;
}
// What a workgroup takes per 32-token chunk with that many row blocks, 128 channels, every CU busy (fitted, see AttnCost in
// api.hip).
double attn_group_chunk_us(int blocks)
{
    return blocks <= 2 ? 0.395 : (blocks <= 4 ? 0.616 : (blocks <= 6 ? 0.72 : (blocks <= 8 ? 0.87 : 1.133)));
}
int attn_group_parts(const Shape &s) { return group_layout(s).parts; }
int attn_group_blocks(const Shape &s) { return group_layout(s).blocks; }

hipError_t launch_attn_ctx_mfma(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count,
                                int n_sel, Partials p, int nctx, int kind, const FusedArgs &f, const SumArgs &sum, hipStream_t st)
{
    if (kind != kAttnSplit && kind != kAttnGroup) return hipErrorInvalidValue;
    if (kind == kAttnSplit && s.D != 128) return hipErrorInvalidValue;
    const bool fused = f.out != nullptr;
    if (fused != (kind == kAttnSplit) || (fused && nctx > 64) || p.nsplit != nctx + (fused ? 1 : 0)) return hipErrorInvalidValue;
    if (p.stream && (kind != kAttnGroup || s.batch > 64 || sel_idx)) return hipErrorInvalidValue;
    const GroupLayout gl = group_layout(s);
    MfmaArgs a = {};
    a.sel_idx = sel_idx;
    a.sel_count = sel_count;
    a.n_sel = n_sel;
    a.scale_log2 = kLog2e / sqrtf((float)s.D);
    a.row_tiles = (s.M + 63) / 64;
    a.n_row_blocks = gl.n_row_blocks;
    a.n_units = p.stream ? p.stream : s.batch * s.Hkv * nctx;
    a.n_bg = s.batch * s.Hkv;
    a.div_nsplit = make_fastdiv((uint32_t)nctx);
    a.div_hkv = make_fastdiv((uint32_t)s.Hkv);
    a.div_B = make_fastdiv((uint32_t)s.B);
    a.div_M = make_fastdiv((uint32_t)s.M);
    // token ranges per split: four (one per token group of a workgroup), or one in the group kernel
    a.div_W = make_fastdiv((uint32_t)nctx * (kind == kAttnGroup ? 1u : 4u));
    const int GR = kind == kAttnGroup ? gl.parts : s.G * a.row_tiles;
    // group kernel: a unit (sequence, KV head, split) per 8 consecutive x; split kernel: (sequence, KV
    // head) bg on XCD bg % 8 with all its splits and query heads (y = (bg / 8) * nctx + split)
    if (sum.wgs > 0) {
        if (kind != kAttnGroup || sel_idx || s.D != 128) return hipErrorInvalidValue;
        a.sum_rows = (sum.wgs + 8 * GR - 1) / (8 * GR);
        a.sum_begin = sum.begin;
        a.kmax = sum.kmax;
        a.kmin = sum.kmin;
    }
    const dim3 grid(8 * GR, a.sum_rows + (kind == kAttnGroup ? (a.n_units + 7) / 8 : ((a.n_bg + 7) / 8) * nctx));
    if (grid.y > 65535u) return hipErrorInvalidConfiguration;
    const bool aligned = s.B % 32 == 0;
    const int span = aligned || !sel_idx ? 32 : (s.B % 16 == 0 ? 16 : 0);   // see ChunkRows
    const size_t lds_split = 2048 + (size_t)max(kRingBytes, 4 * 64 * kOPitch * (int)sizeof(float)) + kQStageBytes;
#define SPECPV_SET_LDS(KERN, LDS)                                                                      \
        static PerDeviceOnce once;   /* one per kernel instantiation */                               \
        auto kern = KERN;                                                                              \
        const hipError_t e0 = once.run([&] {                                                           \
            return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(LDS)); \
        });                                                                                            \
        if (e0 != hipSuccess) return e0
#define SPECPV_LAUNCH_GROUP_K(DD, SP, RR, SS)                                                          \
    do {                                                                                               \
        SPECPV_SET_LDS((attn_ctx_mfma_group_kernel<DD, SP, RR, SS>), group_lds<DD>(RR));                \
        hipLaunchKernelGGL(kern, grid, dim3(64 * group_waves(RR)), group_lds<DD>(RR), st, s, p, a);     \
    } while (0)
#define SPECPV_LAUNCH_GROUP(DD, WW)                                                                    \
    do {                                                                                               \
        if (p.stream) SPECPV_LAUNCH_GROUP_K(DD, 32, WW, true);   /* (no list) */                       \
        else if (span == 32) SPECPV_LAUNCH_GROUP_K(DD, 32, WW, false);                                 \
        else if (span == 16) SPECPV_LAUNCH_GROUP_K(DD, 16, WW, false);                                 \
        else SPECPV_LAUNCH_GROUP_K(DD, 0, WW, false);                                                  \
    } while (0)
#define SPECPV_LAUNCH_SPLIT(AL)                                                                        \
    do {                                                                                               \
        SPECPV_SET_LDS((attn_ctx_mfma_kernel<AL>), lds_split);                                          \
        hipLaunchKernelGGL(kern, grid, dim3(512), lds_split, st, sel_idx, sel_count, s.ctx_len, s.q,    \
                           n_sel, s.M, s.Hq, nctx, s, p, a, f);                                         \
    } while (0)
    if (kind == kAttnGroup) {
        if (s.D == 64) {
            switch (gl.blocks) {
            case 2: SPECPV_LAUNCH_GROUP(64, 2); break;
            case 4: SPECPV_LAUNCH_GROUP(64, 4); break;
            case 6: SPECPV_LAUNCH_GROUP(64, 6); break;
            default: SPECPV_LAUNCH_GROUP(64, 8); break;
            }
        } else {
            switch (gl.blocks) {
            case 2: SPECPV_LAUNCH_GROUP(128, 2); break;
            case 4: SPECPV_LAUNCH_GROUP(128, 4); break;
            case 6: SPECPV_LAUNCH_GROUP(128, 6); break;
            case 10: SPECPV_LAUNCH_GROUP(128, 10); break;
            default: SPECPV_LAUNCH_GROUP(128, 8); break;
            }
        }
    } else {
        if (aligned) SPECPV_LAUNCH_SPLIT(true); else SPECPV_LAUNCH_SPLIT(false);
    }
#undef SPECPV_LAUNCH_SPLIT
#undef SPECPV_LAUNCH_GROUP
#undef SPECPV_LAUNCH_GROUP_K
#undef SPECPV_SET_LDS
    return hipGetLastError();
}

}  // namespace specpv
