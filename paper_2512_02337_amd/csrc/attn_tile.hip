// Context part of the verification attention for short token ranges (the partial verification over a few thousand
// kept tokens): bf16, head dim 128, matrix cores.
//
// Work decomposition.  The M * G query rows of a KV head are packed over its heads (row r = head r / M, node r % M) and
// cut into tiles of 32 * RB rows.  A workgroup of eight wavefronts owns one tile and one KV split; its wavefronts are
// TG token groups x RB row blocks of 32 rows (TG * RB = 8).  A token group owns a contiguous range of 32-token chunks and
// an LDS ring of RB stages; the RB wavefronts of a group bring a chunk's rows together and all read it.  Nothing is
// gathered: K and V rows go from their place in the cache straight into the ring by LDS-DMA (global_load_lds), and
// from there into MFMA operand registers.
//   TG = 8: tiles of 32 rows, one stage per wavefront.  One chunk per wavefront and the call is over in one round trip.
//   TG = 4: tiles of 64 rows, two stages.
//   TG = 2: tiles of 128 rows, four stages, four chunks requested up front.  Each K / V byte is pulled by half as many
//           workgroups as with TG = 4.
// TG = 4 and 2 take two chunks at a time (score_pair, attend_pair).
// What bounds it at one sequence is latency, not a rate.  Headline step, us from entry (timeline.py): arguments, list and query rows 1.3,
// the requests accepted 3.1 (a CU takes 1 KiB per 27 cycles, so 128 KiB are 1.6 us), the first two chunks landed 4.1 and worked
// on 5.5, the other two landed 6.0 and worked on 7.9, partials stored 9.4 (query rows operand by operand: 1.6 and 10.0; with
// them a chunk at a time: the last worked on 8.8, stored 11.0).  The planner (plan_attention) chooses TG and the splits.  Calls of one sequence, 8 KV
// heads at G = 4, in graphs of 16 layers, against tiles of one head's 64 nodes (TG = 4, 8 splits, whatever the node count),
// side by side on one card: 4096 kept tokens, 60 nodes 17.7 -> 17.2 us (TG = 2, 16 splits; on other cards 17.8 -> 17.6 and
// 17.8 -> 18.1), 1 node 14.9 -> 11.6 us (TG = 8, 16 splits); 8192 tokens, 60 nodes 31.8 -> 22.5 us; 2048 tokens, 60 nodes
// 13.8 -> 14.4 us (called one by one 13.8 -> 13.9).
//
// Per chunk (v_mfma_f32_32x32x16_bf16, fp32 accumulate):
//   S^T = K . Q^T     tokens are the M index, query rows the N index, so each
//                     lane holds 16 tokens of ONE query row: max, sum and rescale
//                     are lane-local (one exchange with lane ^ 32);
//   O^T += V^T . P^T  the S^T accumulator, converted to bf16, already has the
//                     B-operand layout; V comes out of LDS transposed (8 tokens
//                     of one channel per lane) through ds_read_b64_tr_b16.
// The reference maximum of a row is only moved when the true maximum runs more than 2^8 ahead of it.
//
// Epilogue: the TG token groups merge their (O, m, l) through LDS and write one split-KV partial per (split, row);
// combine.hip finishes.
//
// grid: x = tile * 8 + xcd, y = (bg / 8) * nsplit + split   with bg = b * Hkv + g and xcd = bg % 8; with 8, 16, 32, ... KV heads
// y = split, z = bg / 8: the same order without a division, which would wait for the argument block.  Workgroups are
// handed to the 8 XCDs round-robin in linear order and gridDim.x is a multiple of 8, so a (sequence, KV head) stays on
// XCD bg % 8 with all its splits and tiles: the K/V bytes of a split come from HBM once and from that XCD's L2 for the
// other tiles, and the partials of a head are merged on the XCD that wrote them.  Where
// the pairs are no multiple of 8 (two KV heads: two XCDs would do all the work), the (pair, split) units are dealt to the
// XCDs instead, y = unit / 8: the tiles of a unit still share an L2.
#include "attn_mfma.h"

namespace specpv {

#ifdef SPECPV_TIMELINE
#define SPECPV_STAMP(i)                                                                                                      \
    do {                                                                                                                     \
        const unsigned nth = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;                                 \
        if (timeline && threadIdx.x == 0 && nth < 2048u) timeline[(size_t)nth * 16 + (i)] = __builtin_amdgcn_s_memrealtime();\
    } while (0)
#else
#define SPECPV_STAMP(i) do {} while (0)
#endif

constexpr int kTileRing = 8 * kStageBytes;
static_assert(kTileRing >= 8 * 16384, "the merge of the token groups reuses the ring");

// SPAN: the rows of a chunk are one run of 32 consecutive ones, two of 16, or, 0, any (see ChunkRows).
// PEND: partially verified tokens may stand in front of the tree (s.kctx > 0).
template <int SPAN, int TG, bool PEND>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_ctx_tile_kernel(const int32_t *a_sel_idx, const int32_t *a_sel_count, const int32_t *a_ctx_len,
                          const void *a_q, int a_n_sel, int a_M, int a_Hq, int a_nctx_groups,
                          Shape s, Partials part, MfmaArgs a, unsigned long long *timeline)
{
    constexpr int RB = 8 / TG, STG = RB;               // row blocks per workgroup; ring stages per token group
    constexpr int KOPS = RB == 4 ? 4 : 8;              // K (or V) operations of a chunk that one wavefront issues
    constexpr int OPS = RB == 1 ? 16 : KOPS;           // all operations of a chunk that one wavefront issues
    constexpr int RUN = SPAN ? SPAN : 32, RPC = 32 / RUN;   // tokens of a run, runs of a chunk
    constexpr int NID = SPAN == 16 ? 8 : 4;            // registers for the kept list, 64 entries each (smaller blocks, longer lists)
    // the leading scalar arguments repeat what the first round of reads needs: they arrive in registers
    s.ctx_len = a_ctx_len; s.q = a_q; s.M = a_M; s.Hq = a_Hq;
    a.sel_idx = a_sel_idx; a.sel_count = a_sel_count; a.n_sel = a_n_sel;
    const int nctx = a_nctx_groups & 0xffff, groups = a_nctx_groups >> 16;   // splits; head_groups_code
    extern __shared__ char lds_raw[];
    float *ms = (float *)lds_raw;            // [TG][32 RB]
    float *ls = ms + 256;                    // [TG][32 RB]
    char *ring = lds_raw + 2048;             // [TG][STG][K 8 KiB | V]
    char *merge = lds_raw + 2048;            // merge of the token groups: reuses the ring after the main loop
    SPECPV_CLOCKS_BEGIN;
    SPECPV_STAMP(0);   // entry

    // ---- which piece of work is this workgroup -------------------------------------
    const int xcd = blockIdx.x & 7, tile = blockIdx.x >> 3;
    int bg, sp, b, g;
    if (groups) {
        // (nothing here waits for a read: the argument block itself takes a trip to memory)
        b = (int)blockIdx.z >> (groups - 1);
        g = (((int)blockIdx.z - (b << (groups - 1))) << 3) + xcd;
        s.Hkv = 4 << groups;
        s.G = s.Hq >> (groups + 2);
        bg = b * s.Hkv + g;
        sp = (int)blockIdx.y;
    } else {
        // (one division for both orders, without branches: its numbers are then read in here and not at the kernel's entry)
        const bool whole = (a.n_bg & 7) == 0;
        const int u = whole ? (int)blockIdx.y : (int)blockIdx.y * 8 + xcd, q = (int)a.div_nsplit.div_straight((uint32_t)u);
        sp = u - q * nctx;
        bg = whole ? q * 8 + xcd : q;
        b = (int)a.div_hkv.div_straight((uint32_t)bg);
        g = bg - b * s.Hkv;
        if (bg >= a.n_bg) return;
    }
    const int R = s.M * s.G, row0 = tile * (32 * RB);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tg = wave & (TG - 1), rb = wave / TG;
    const int n = lane & 31, kg = lane >> 5;

    // Everything whose address only depends on the kernel arguments is requested up
    // front, so that the cold-miss latencies of these small reads overlap: context
    // length, list length, the kept-block list (up to 256 or 512 entries, lane t: entries t, t + 64, ..)
    // and the query rows.
    const int32_t *sel = a.sel_idx + (int64_t)bg * a.n_sel;   // (an offset from null where there are no lists: n_sel is 0)
    const uint32_t Bu = (uint32_t)s.B;
    // These go out before the argument block has arrived (one trip to memory by itself): they take only what came in
    // registers.  The counts are vector loads because scalar ones return in any order, so that using one waits for the
    // argument block as well.  With the combine kernel's reads done the same way: one layer of 128 k tokens of which 4 k are
    // attended 16.7 -> 16.4 us, a call over 2 k listed tokens 13.2 -> 12.5 us.
    const bool list_in_regs = SPAN && a.sel_idx && (uint32_t)(a.n_sel - 1) < 64u * NID;   // (a list may have no room at all)
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const int L_v = s.ctx_len[b + zero], cnt_v = (sel ? a.sel_count + bg : s.ctx_len + b)[zero];
    int idv[NID];
    {
        const int32_t *list = list_in_regs ? sel : s.ctx_len + b;
        const int last = list_in_regs ? a.n_sel - 1 : 0;
#pragma unroll
        for (int x = 0; x < NID; ++x) idv[x] = list[min(lane + 64 * x, last)];   // (past the end: never asked for, slot < cnt <= n_sel)
    }
    // The query rows of a row block are the same for its TG wavefronts: each brings its share of them straight into LDS, four
    // whole rows per operation, laid out like a K tile, and all read the whole from there once the requests have landed --
    // fewer bytes through the CU's memory path in the phase where the first K / V chunks are requested.  (A k-step per
    // operation, 32 bytes of 32 rows each, takes the memory path three times as long: headline 16.5 -> 15.9 us a layer.  The row's
    // head by a reciprocal: it waits for no argument, and is half a row away from the next whole number, r < 2^12.)
    // TG = 2: four row blocks are more than the ring leaves free, so they stand
    // in the groups' last stages, whose first chunk is requested behind them.
    auto q_stage = [&](int rbq) -> char * {
        return TG == 2 ? ring + ((rbq >> 1) * STG + (STG - 1)) * kStageBytes + (rbq & 1) * 8192 : ring + kTileRing + rbq * 8192;
    };
    {
        char *dst = q_stage(rb);
        const float inv = __builtin_amdgcn_rcpf((float)s.M);
#pragma unroll
        for (int x = 0; x < 8 / TG; ++x) {
            const int i = tg * (8 / TG) + x, row = 4 * i + (lane >> 4);
            const int r = min(row0 + rb * 32 + row, R - 1);
            const int hh = (int)(((float)r + 0.5f) * inv), j = r - hh * s.M;
            const char *qrow = (const char *)((const uint16_t *)s.q + (((int64_t)b * s.M + j) * s.Hq + g * s.G + hh) * 128) + 16 * ((lane & 15) ^ (row & 15));
            __builtin_amdgcn_global_load_lds((glb_void_ptr)qrow, (lds_void_ptr)(dst + 1024 * i), 16, 0, 0);
        }
    }

    // the arguments that the chunks need arrive while the reads above are on their way (left to itself the compiler asks for
    // each where it is first used, one trip to memory after the other)
    asm volatile("" :: "s"(s.k), "s"(s.v), "s"(s.sb), "s"(s.sh), "s"(s.st), "s"(s.max_blocks), "s"(s.B), "s"(a.div_W.mul), "s"(a.div_W.shift),
                 "s"(a.div_W.d), "s"(a.div_B.mul), "s"(a.div_B.shift), "s"(a.div_B.d), "s"(s.kd), "s"(s.vd));
    const int L = __builtin_amdgcn_readfirstlane(L_v);
    int nb = L > 0 ? (int)a.div_B.div((uint32_t)(L + s.B - 1)) : 0;
    if (nb > s.max_blocks) nb = s.max_blocks;
    int cnt = nb;
    if (sel) cnt = max(0, min(__builtin_amdgcn_readfirstlane(cnt_v), a.n_sel));
    const uint32_t T = nb > 0 ? (uint32_t)cnt * Bu : 0u;   // host guarantees max_blocks * B <= 2^30
    // chunks of cache tokens, then the chunks of the partially verified tokens (the first kctx draft nodes: a
    // chain that every query node descends from, so all rows attend all of them, like cache tokens)
    const uint32_t C_ctx = (T + 31u) >> 5;
    const int kctx = PEND ? s.kctx : 0;
    const uint32_t C = C_ctx + (((uint32_t)kctx + 31u) >> 5);
    const char *kdb = (const char *)s.kd + (((int64_t)b * s.Mk) * s.Hkv + g) * 256;
    const char *vdb = (const char *)s.vd + (((int64_t)b * s.Mk) * s.Hkv + g) * 256;
    const uint32_t stp = (uint32_t)s.Hkv * 256u;   // bytes from one draft node's row to the next

    // uniform slab bases; per-lane byte offsets inside a slab fit 32 bits (host-checked)
    const char *kb = (const char *)s.k + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const char *vb = (const char *)s.v + ((int64_t)b * s.sb + (int64_t)g * s.sh) * 2;
    const uint32_t st2 = (uint32_t)s.st * 2u;   // bytes per token row step

    char *my_ring = ring + tg * (STG * kStageBytes);
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)my_ring;
    // K tile in LDS: row-major, 256 B per token, the 16-byte pieces of row t stored at
    // piece index (p ^ (t & 15)) so that the operand reads below (16 lanes per cycle, same piece,
    // different rows) spread over all 64 banks.  Operand piece of k-step ks: 2*ks + kg, i.e. kread ^ 32 ks
    // (rows and stages start 256-byte aligned).
    const uint32_t kread = ring_addr + (uint32_t)n * 256u + ((16u * (uint32_t)kg) ^ (16u * ((uint32_t)n & 15u)));   // + stage * kStageBytes
    const uint32_t vread = ring_addr + 8192u + (uint32_t)(4 * kg + ((lane & 15) >> 2)) * kVPiecePitch +
                           32u * (uint32_t)((lane >> 4) & 1) + 8u * (uint32_t)(lane & 3);   // + stage * kStageBytes

    const bool do_k = RB == 1 || rb < RB / 2, do_v = RB == 1 || rb >= RB / 2;   // which half of a chunk this wavefront brings
    const int op0 = RB == 4 ? 4 * (rb & 1) : 0;                                // ... from which operation on

    const int W = nctx * TG, wsid = sp * TG + tg;
    // chunks of a list that precede the share of token group w; shares differ by at most one
    auto first_chunk = [&](uint32_t chunks, int w) -> int {
        const uint32_t base = a.div_W.div(chunks), rem = chunks - base * (uint32_t)W;
        return (int)((uint32_t)w * base + min((uint32_t)w, rem));
    };
    const int c0 = first_chunk(C, wsid), c1 = first_chunk(C, wsid + 1);
    const int nch = c1 - c0;
    const int nch_max = first_chunk(C, sp * TG + 1) - first_chunk(C, sp * TG);   // token group 0 has the most
    SPECPV_STAMP(9);   // lengths and list length are in: the chunk counts are known

    // ---- chunk -> token rows (see ChunkRows) ---------------------------------------------
    // SPAN: the first rows of the next 64 runs of this wavefront's chunks sit in a register (lane t: run t from chunk
    // row_base on) and are picked with readlane.
    const ChunkRows rows_of{sel, a.div_B, s.B, nb, min(L, nb * s.B), T};
    int row_base = 0, row0vec = -1;
    auto fill_rows = [&](int cb) {
        row_base = cb;
        const int c = cb + lane / RPC;
        int r = -1;
        if (c < nch && (uint32_t)(c0 + c) < C_ctx) r = rows_of.first_row<RUN>((uint32_t)((c0 + cb) * RPC + lane));
        row0vec = r;
        // wait for the list entries here, inside the rare branch, so that the common path that
        // joins behind it carries no pending load (and no wait on the DMA prefetch)
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    };
    // the first 64 runs: the list sits in registers (lane t: entries t, t + 64, ...), so this is a
    // cross-lane read and no second trip to memory
    auto fill_rows_first = [&]() {
        if (!list_in_regs) { fill_rows(0); return; }
        const uint32_t p0 = (uint32_t)(c0 * RPC + lane) * (uint32_t)RUN;
        const uint32_t slot = a.div_B.div(p0);
        const int src = (int)(slot & 63u), part_of = (int)(slot >> 6);
        int blk = __shfl(idv[0], src);
#pragma unroll
        for (int x = 1; x < NID; ++x) {
            const int e = __shfl(idv[x], src);
            blk = part_of == x ? e : blk;
        }
        const int r = rows_of.encode<RUN>(blk, p0, slot);   // (without a branch around it)
        row0vec = (lane / RPC < nch && (uint32_t)(c0 + lane / RPC) < C_ctx && p0 < T) ? r : -1;   // p0 < T: the slot is < cnt
    };

    uint32_t vmv = 0u;   // validity words of the chunks in the ring: lane t holds those of stage t

    // Request this wavefront's share of chunk ci, 1 KiB per operation (one 256-byte row per 16 lanes): K operation i
    // brings rows 4i .. 4i+3, pieces swizzled by row & 15; V operation i brings rows i, i+8, i+16, i+24 into piece i.
    // rows given per lane (t = lane & 31: token tk of the chunk)
    auto issue_rows = [&](const char *kbase, const char *vbase, const uint32_t stride, const uint32_t tk, char *dst, const int r4,
                          const uint32_t sw0, const uint32_t vsw) __attribute__((always_inline)) {
        if (do_k) {
#pragma unroll
            for (int x = 0; x < KOPS; ++x) {
                const int i = op0 + x;
                const uint32_t tv = (uint32_t)__shfl((int)tk, 4 * i + r4) * stride;
                dma16(kbase + (tv + (sw0 ^ (64u * (uint32_t)(i & 3)))), dst + i * 1024);
            }
        }
        if (do_v) {
#pragma unroll
            for (int x = 0; x < KOPS; ++x) {
                const int i = op0 + x;
                const uint32_t tv = (uint32_t)__shfl((int)tk, 8 * r4 + i) * stride;
                dma16(vbase + (tv + vsw), dst + 8192 + i * kVPiecePitch);
            }
        }
    };
    auto issue = [&](int ci) __attribute__((always_inline)) {
        const int stg = ci & (STG - 1);
        char *dst = my_ring + stg * kStageBytes;
        // (the lane's offsets are worked out here, from a lane number that the compiler cannot see through: kept over the
        // loop, with the sums of base and offset that it makes of them, they take registers that the pairs of chunks need)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int r4 = ln >> 4, pos = ln & 15, n = ln & 31;
        const uint32_t sw0 = 16u * (uint32_t)(pos ^ r4), vsw = 16u * (uint32_t)pos;   // K row 4 i + r4: piece pos ^ ((4 i + r4) & 15) = sw0 ^ 64 (i & 3)
        const uint32_t lane_row_off = (uint32_t)r4 * st2;
        int tok;
        if (PEND && kctx > 0 && (uint32_t)(c0 + ci) >= C_ctx) {
            // a chunk of partially verified tokens: rows of the draft K / V arrays
            const int pr = (int)((uint32_t)(c0 + ci) - C_ctx) * 32 + n;
            const int ptok = pr < kctx ? pr : -1;
            const uint32_t vm = (uint32_t)__ballot(ptok >= 0);
            vmv = ln == stg ? vm : vmv;
            issue_rows(kdb, vdb, stp, (uint32_t)max(ptok, 0), dst, r4, sw0, vsw);
            return;
        }
        if (SPAN == 16) {
            if (ci - row_base >= 32) fill_rows(ci);
            const int ra = __builtin_amdgcn_readlane(row0vec, 2 * (ci - row_base)), rb16 = __builtin_amdgcn_readlane(row0vec, 2 * (ci - row_base) + 1);
            if ((ra | rb16) >= 0) {
                // both runs whole: K operations 0 .. 3 lie in the first, 4 .. 7 in the second, a V operation has two rows of each
                vmv = ln == stg ? 0xffffffffu : vmv;
                if (do_k) {
#pragma unroll
                    for (int x = 0; x < KOPS; ++x) {
                        const int i = op0 + x;
                        const size_t first = (size_t)((uint32_t)((i < 4 ? ra : rb16) + 4 * (i & 3)) * st2);   // fits 32 bits (host-checked)
                        dma16(kb + first + (lane_row_off + (sw0 ^ (64u * (uint32_t)(x & 3)))), dst + i * 1024);
                    }
                }
                if (do_v) {
                    const uint32_t voff = (uint32_t)((r4 < 2 ? ra : rb16) + 8 * (r4 & 1)) * st2 + vsw;
#pragma unroll
                    for (int x = 0; x < KOPS; ++x) dma16(vb + (size_t)(uint32_t)(op0 + x) * st2 + voff, dst + 8192 + (op0 + x) * kVPiecePitch);
                }
                return;
            }
            tok = rows_of.decode(n < 16 ? ra : rb16, n & 15);
        } else if (SPAN == 32) {
            if (ci - row_base >= 64) fill_rows(ci);
            const int r0 = __builtin_amdgcn_readlane(row0vec, ci - row_base);
            if (r0 >= 0) {
                vmv = ln == stg ? 0xffffffffu : vmv;
                const size_t first = (size_t)((uint32_t)r0 * st2);   // fits 32 bits (host-checked)
                if (st2 == 256u) {
                    // rows are 256 bytes apart (the usual head-major cache): the instruction's
                    // immediate offset, added to the global and to the LDS address, covers the step
                    // between consecutive operations (K: 1 KiB on both sides; V: 256 bytes, with the
                    // LDS base adjusted for the rest of the piece pitch)
                    if (do_k) {
                        dma16x4(kb + first + op0 * 1024, lane_row_off, sw0, dst + op0 * 1024);
                        if (KOPS == 8) dma16x4(kb + first + 4096, lane_row_off, sw0, dst + 4096);
                    }
                    if (do_v) {
                        const char *vsrc = vb + first + op0 * 256 + ((uint32_t)r4 * 2048u + vsw);
                        char *dstv = dst + 8192 + op0 * kVPiecePitch;
#define SPECPV_VOP(i) __builtin_amdgcn_global_load_lds((glb_void_ptr)vsrc, (lds_void_ptr)(dstv + (i) * (kVPiecePitch - 256)), 16, (i) * 256, kKvAux)
                        SPECPV_VOP(0); SPECPV_VOP(1); SPECPV_VOP(2); SPECPV_VOP(3);
                        if (KOPS == 8) { SPECPV_VOP(4); SPECPV_VOP(5); SPECPV_VOP(6); SPECPV_VOP(7); }
#undef SPECPV_VOP
                    }
                } else {
                    if (do_k) {
#pragma unroll
                        for (int x = 0; x < KOPS; ++x)
                            dma16(kb + first + (size_t)(4 * (op0 + x)) * st2 + (lane_row_off + (sw0 ^ (64u * (uint32_t)(x & 3)))), dst + (op0 + x) * 1024);
                    }
                    if (do_v) {
#pragma unroll
                        for (int x = 0; x < KOPS; ++x)
                            dma16(vb + first + (size_t)(8 * r4 + op0 + x) * st2 + vsw, dst + 8192 + (op0 + x) * kVPiecePitch);
                    }
                }
                return;
            }
            tok = rows_of.decode(r0, n);
        } else {
            tok = rows_of.row((uint32_t)(c0 + ci), n);
        }
        const uint32_t vm = (uint32_t)__ballot(tok >= 0);
        vmv = ln == stg ? vm : vmv;
        issue_rows(kb, vb, st2, tok >= 0 ? (uint32_t)tok : 0u, dst, r4, sw0, vsw);   // row 0 exists (L > 0); masked later
    };

    if (SPAN && nch > 0) fill_rows_first();
    // every load above has been consumed here: from now on the only vector-memory
    // operations of this wavefront in flight are its own DMA groups (OPS operations each)
    // (as an instruction the compiler knows, not inline assembly: otherwise it assumes that the
    // loads of the prologue may still be in flight at the loop header and waits for vmcnt(0),
    // i.e. for the prefetch just issued, at the first use of Q in every iteration)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), expcnt and lgkmcnt untouched
    asm volatile("" ::: "memory");
    SPECPV_STAMP(1);   // arguments, lengths, list, query rows are in

    f32x16 O[4];
    RowState st;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[j][i] = 0.f;

    // ---- main loop ---------------------------------------------------------------------
    bf16x8 qf[8];   // Q fragments (B operand of S^T = K . Q^T): row = lane & 31
    // This wavefront's share of the query rows has landed (the wait above); the barrier in front of the first chunk
    // covers the others' shares.
    auto read_q = [&]() {
        const uint32_t q0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)q_stage(rb) + (uint32_t)n * 256u + ((16u * (uint32_t)kg) ^ (16u * ((uint32_t)n & 15u)));
        const uint32_t qa[8] = {q0, q0 ^ 32u, q0 ^ 64u, q0 ^ 96u, q0 ^ 128u, q0 ^ 160u, q0 ^ 192u, q0 ^ 224u};
        uint4 qraw[8];
        lds_read_k<0>(qa, qraw);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = as_bf16x8(qraw[ks]);
    };
    if (0 < nch) issue(0);
    __builtin_amdgcn_s_barrier();   // the other wavefronts' shares of the query rows have landed, too
    read_q();
    if (TG == 2) __builtin_amdgcn_s_barrier();   // the last stages no longer hold query rows
#pragma unroll
    for (int c = 1; c < STG; ++c)
        if (c < nch) issue(c);
    SPECPV_STAMP(2);   // first chunks requested
    auto operand_addresses = [&](int stg, uint32_t (&ka)[8]) {
        const uint32_t k0 = kread + (uint32_t)stg * kStageBytes;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) ka[ks] = k0 ^ (32u * (uint32_t)ks);
    };
    auto one_chunk = [&](int i) {   // it has landed
        const int stg = i & (STG - 1);
        const uint32_t vmask = (uint32_t)__builtin_amdgcn_readlane((int)vmv, stg);
        uint32_t ka[8];
        uint4 kf[8];
        uint2 v[16];
        operand_addresses(stg, ka);
        lds_read_k<0>(ka, kf);
        lds_read_v<0>(vread + (uint32_t)stg * kStageBytes, v);
        if (RB == 1 && i + 1 < nch) issue(i + 1);   // one stage: free as soon as the chunk is in registers
        attend_chunk(kf, v, qf, vmask, kg, a.scale_log2, O, st);
    };
    if constexpr (RB == 1) {
        for (int i = 0; i < nch; ++i) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (i < 4) SPECPV_STAMP(3 + i);
            one_chunk(i);
        }
    } else {
        // Two chunks at a time: one wait, one barrier (two with two stages), one trip to LDS and one test of the maximum.
        // The token groups' numbers of chunks differ by one at most; nch_max is the workgroup's.
        auto landed = [&](int i) __attribute__((always_inline)) {   // chunks i, i + 1 (an odd last one: chunk i) are in LDS
            if (i < 8) SPECPV_STAMP(12 + i / 2);   // about to wait for them
            // own share; in front of the first two, the two requested behind them may stay in flight
            if (TG == 2 && i == 0 && nch > 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * OPS) : "memory");
            else if (TG == 2 && i == 0 && nch > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(OPS) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();          // ... and the other wavefronts' shares
            if (i < 8) SPECPV_STAMP(3 + i / 2);
        };
        auto request = [&](int i) __attribute__((always_inline)) {
#pragma unroll 1
            for (int c = i; c < min(i + 2, nch); ++c) issue(c);
        };
        for (int i = 0; i + 1 < nch_max; i += 2) {
            const int stg = i & (STG - 1);
            landed(i);
            const uint32_t vm0 = (uint32_t)__builtin_amdgcn_readlane((int)vmv, stg), vm1 = (uint32_t)__builtin_amdgcn_readlane((int)vmv, stg + 1);
            const bool both = i + 1 < nch;
            // four stages: those of the two chunks before are free (the first two pairs were requested up front)
            if (TG == 2 && i > 0) request(i + 2);
            uint32_t ka[8];
            f32x16 S0, S1;
            uint4 v0[8], v1[8];
            operand_addresses(stg, ka);
            if (both) score_pair<0, kStageBytes, 0, kStageBytes>(ka, vread + (uint32_t)stg * kStageBytes, qf, S0, S1, v0, v1);
            if (TG == 4 && i + 2 < nch_max) {
                __builtin_amdgcn_s_barrier();      // two stages: both wavefronts of the group hold the chunks in registers
                request(i + 2);
            }
            if (both) attend_pair(S0, S1, v0, v1, vm0, vm1, kg, a.scale_log2, O, st);
        }
        if (nch_max & 1) landed(nch_max - 1);
        if (nch & 1) one_chunk(nch - 1);   // (landed at one of these barriers)
    }
    __syncthreads();   // every wavefront is done with the rings: the epilogue reuses that LDS
    SPECPV_STAMP(7);   // main loop done

    // ---- merge the token groups --------------------------------------------------------
    // A wavefront finishes 64 / TG of the 64 accumulators of its row block's lanes, i.e. 128 / TG channels of 32 rows: it
    // hands the others over as they lie in its registers, to the token groups that finish them, and takes in the other
    // groups' share of its own.  (Every group's accumulators as rows through LDS, for eight wavefronts to pick up by row:
    // twice the bytes each way; 2.2 us from the end of the loop to the stores at the headline shape, 1.5 so.)
    constexpr int E = 64 / TG, E4 = E / 4;   // accumulators a wavefront finishes; as 16-byte pieces
    auto piece = [&](int e4) -> float4 { return make_float4(O[e4 >> 2][4 * (e4 & 3)], O[e4 >> 2][4 * (e4 & 3) + 1], O[e4 >> 2][4 * (e4 & 3) + 2], O[e4 >> 2][4 * (e4 & 3) + 3]); };
    // [row block][finishing group][group][piece][lane]
    auto slot = [&](int to, int from) -> float4 * { return (float4 *)merge + ((((rb * TG + to) * TG + from) * E4) << 6); };
    {
        const float l_run = sum_xor32(st.l);
        if (kg == 0) {
            ms[tg * (32 * RB) + rb * 32 + n] = st.ref(l_run);
            ls[tg * (32 * RB) + rb * 32 + n] = l_run;
        }
#pragma unroll
        for (int to = 0; to < TG; ++to)
            if (to != tg) {
#pragma unroll
                for (int x = 0; x < E4; ++x) slot(to, tg)[64 * x + lane] = piece(to * E4 + x);
            }
    }
    __syncthreads();
    float acc[E], m_row = -INFINITY, l_row = 0.f;
    {
        const int row = rb * 32 + n;
        float mw[TG];
#pragma unroll
        for (int w = 0; w < TG; ++w) { mw[w] = ms[w * (32 * RB) + row]; m_row = fmaxf(m_row, mw[w]); }
        const float m_use = m_row == -INFINITY ? 0.f : m_row;
        float wgt[TG];
#pragma unroll
        for (int w = 0; w < TG; ++w) {
            wgt[w] = __builtin_amdgcn_exp2f(mw[w] - m_use);   // 0 for a token group without valid tokens
            l_row = fmaf(ls[w * (32 * RB) + row], wgt[w], l_row);
        }
        const float il = l_row > 0.f ? 1.f / l_row : 0.f;
#pragma unroll
        for (int x = 0; x < E; ++x) acc[x] = 0.f;
#pragma unroll
        for (int w = 0; w < TG; ++w) {
            const float ww = wgt[w] * il;
            if (w == tg) {
#pragma unroll
                for (int to = 0; to < TG; ++to)
                    if (to == tg) {
#pragma unroll
                        for (int x = 0; x < E; ++x) acc[x] = fmaf(ww, O[(to * E + x) >> 4][(to * E + x) & 15], acc[x]);
                    }
            } else {
#pragma unroll
                for (int x = 0; x < E4; ++x) {
                    const float4 y = slot(tg, w)[64 * x + lane];
                    acc[4 * x] = fmaf(ww, y.x, acc[4 * x]);
                    acc[4 * x + 1] = fmaf(ww, y.y, acc[4 * x + 1]);
                    acc[4 * x + 2] = fmaf(ww, y.z, acc[4 * x + 2]);
                    acc[4 * x + 3] = fmaf(ww, y.w, acc[4 * x + 3]);
                }
            }
        }
    }
    // as fp16 through this wavefront's own corner (nobody else reads it: no barrier), so that stores are whole pieces of rows
    constexpr int RB256 = 256 / TG, PITCH = RB256 + 16, LPR = 16 / TG, RPP = 64 / LPR;   // bytes of a row here; lanes per row, rows per store
    char *rows = (char *)slot(tg, 0);
#pragma unroll
    for (int x = 0; x < E4; ++x)
        *(uint2 *)(rows + n * PITCH + 16 * x + 8 * kg) = make_uint2(half_pair(acc[4 * x], acc[4 * x + 1]), half_pair(acc[4 * x + 2], acc[4 * x + 3]));
    const int64_t prow0 = ((int64_t)bg * part.nsplit + sp) * R + row0 + rb * 32;
    const int n_rows = min(32, R - row0 - rb * 32);   // may be negative
#pragma unroll
    for (int x = 0; x < 32 / RPP; ++x) {
        const int row = RPP * x + lane / LPR;
        const u32x4 y = *(const u32x4 *)(rows + row * PITCH + 16 * (lane & (LPR - 1)));
        if (row < n_rows) __builtin_nontemporal_store(y, (u32x4 *)((char *)(part.o + (prow0 + row) * 64) + tg * RB256) + (lane & (LPR - 1)));   // 128 halves per row
    }
    if (tg == 0 && kg == 0 && n < n_rows) *(float2 *)(part.ml + (prow0 + n) * 2) = make_float2(m_row, l_row);
    SPECPV_STAMP(8);   // partial stores issued
    SPECPV_CLOCKS_END(timeline, 3072 + ((size_t)(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x), first_chunk(C, sp * TG + TG) - first_chunk(C, sp * TG));
    // The combine kernel that follows reads the tree's parents and, one trip later, its K / V rows: nobody
    // has touched those in this call yet.  Ask for them here, on the way out: they are then in this XCD's L2, where that
    // kernel's workgroups of the same KV head run.  Eight lanes per node (four 64-byte pieces of its K row, four of its V
    // row), so that one instruction of the wavefront covers eight nodes.  The loads are ones that the compiler knows and
    // waits for: a load in flight whose register it takes to be free may land in whatever it puts there next, the address
    // of another load for instance.
    if (wave == 0 && s.kd && s.vd && s.parent) {
        const int nw = (int)(gridDim.x >> 3) * nctx, w = tile * nctx + sp;
        const char *base = ((lane & 4) ? (const char *)s.vd : (const char *)s.kd) + ((int64_t)b * s.Mk * s.Hkv + g) * 256 + (lane & 3) * 64;
        uint32_t seen = 0u;
        if (w == 0 && lane < 8 && lane * 16 < s.Mk) seen = (uint32_t)s.parent[(int64_t)b * s.Mk + lane * 16];
        for (int node = w + nw * (lane >> 3); node < s.Mk; node += 8 * nw) seen |= *(const uint32_t *)(base + (int64_t)node * s.Hkv * 256);
        asm volatile("" ::"v"(seen));
    }
}

hipError_t launch_attn_ctx_tile(const Shape &s, const int32_t *sel_idx, const int32_t *sel_count, int n_sel, Partials p,
                                int tg, unsigned long long *timeline, hipStream_t st)
{
    if (s.D != 128 || (tg != 2 && tg != 4 && tg != 8)) return hipErrorInvalidValue;
    const int rows = 256 / tg, tiles = (s.M * s.G + rows - 1) / rows, nctx = p.nsplit;
    MfmaArgs a = {};
    a.sel_idx = sel_idx;
    a.sel_count = sel_count;
    a.n_sel = n_sel;
    a.scale_log2 = kLog2e / sqrtf(128.f);
    a.n_bg = s.batch * s.Hkv;
    a.div_nsplit = make_fastdiv((uint32_t)nctx);
    a.div_hkv = make_fastdiv((uint32_t)s.Hkv);
    a.div_B = make_fastdiv((uint32_t)s.B);
    a.div_W = make_fastdiv((uint32_t)(nctx * tg));   // token ranges: one per token group of every split
    int groups = head_groups_code(s.Hkv);
    if (a.n_bg / 8 > 65535) groups = 0;
    const dim3 grid(8 * tiles, groups ? nctx : (a.n_bg * nctx + 7) / 8, groups ? a.n_bg / 8 : 1);
    if (grid.y > 65535u) return hipErrorInvalidConfiguration;
    const int span = s.B % 32 == 0 || !sel_idx ? 32 : (s.B % 16 == 0 ? 16 : 0);   // see ChunkRows
    const bool pend = s.kctx > 0;
    const size_t lds = 2048 + kTileRing + (tg == 2 ? 0 : (8 / tg) * 8192);
#define SPECPV_LAUNCH(SP, TGV, PE)                                                                                   \
    do {                                                                                                             \
        static PerDeviceOnce once;   /* one per kernel instantiation */                                             \
        auto kern = attn_ctx_tile_kernel<SP, TGV, PE>;                                                               \
        const hipError_t e0 = once.run([&] {                                                                         \
            return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);    \
        });                                                                                                          \
        if (e0 != hipSuccess) return e0;                                                                             \
        hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, sel_idx, sel_count, s.ctx_len, s.q, sel_idx ? n_sel : 0, s.M, s.Hq, \
                           nctx | groups << 16, s, p, a, timeline);                                                         \
    } while (0)
#define SPECPV_LAUNCH_TG(TGV)                                                                                        \
    do {                                                                                                             \
        if (span == 32) { if (pend) SPECPV_LAUNCH(32, TGV, true); else SPECPV_LAUNCH(32, TGV, false); }               \
        else if (span == 16) { if (pend) SPECPV_LAUNCH(16, TGV, true); else SPECPV_LAUNCH(16, TGV, false); }          \
        else { if (pend) SPECPV_LAUNCH(0, TGV, true); else SPECPV_LAUNCH(0, TGV, false); }                            \
    } while (0)
    if (tg == 2) SPECPV_LAUNCH_TG(2);
    else if (tg == 4) SPECPV_LAUNCH_TG(4);
    else SPECPV_LAUNCH_TG(8);
#undef SPECPV_LAUNCH_TG
#undef SPECPV_LAUNCH
    return hipGetLastError();
}

}  // namespace specpv
