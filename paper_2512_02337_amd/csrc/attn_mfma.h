// What the matrix-core attention kernels share: operand types, the layout of a 32-token chunk in LDS, LDS-DMA and the
// hand-written LDS reads, and the form in which partial results are stored.
#pragma once
#include "internal.h"
#include <type_traits>

namespace specpv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *glb_void_ptr;

// One 32-token chunk in LDS: 8 KiB of K (row-major, 16-byte pieces XOR-swizzled by row & 15: the LDS has 64
// banks, so the 16 lanes that a 16-byte read serves per cycle must cover all 16 pieces of a 256-byte bank row;
// with row & 7 the operand reads ran at half the rate) and
// the V rows in 8 pieces of 4 rows (tokens i, i+8, i+16, i+24 in piece i), 1088 bytes apart, for
// the transposing LDS reads (see lds_read_v).
constexpr int kVPiecePitch = 1088;
constexpr int kStageBytes = 8192 + 8 * kVPiecePitch;
// Cache policy of the K / V requests: 2 = the streaming hint (nt).  K / V rows are used once per
// workgroup; with the hint the requests are served faster, and the sharing of a KV head's rows
// between its query heads' workgroups through L2 is unaffected (same fetch counters).
constexpr int kKvAux = 2;
constexpr float kRescaleSlack = 8.f; // the reference max may lag the true max by 2^8

struct MfmaArgs {
    const int32_t *sel_idx, *sel_count;
    int n_sel;
    float scale_log2;
    int n_units, row_tiles, n_bg;
    int n_row_blocks;   // group kernel: 32-row blocks of a KV head's M * G query rows
    FastDiv div_nsplit, div_hkv, div_B, div_W, div_M;
    // group kernel: the first sum_rows rows of the grid recompute the summaries of the blocks from sum_begin on
    int sum_rows, sum_begin;
    void *kmax, *kmin;
};

// Which cache rows the 32-token chunks of one (sequence, KV head) cover: chunk c holds tokens 32 c .. 32 c + 31 of the kept
// blocks, in the order of the list (sel == nullptr: of all blocks).
struct ChunkRows {
    const int32_t *sel;
    FastDiv div_B;
    int B, nb, L;    // block size, blocks and tokens of the sequence (no more tokens than its blocks hold)
    uint32_t T;      // 32 * chunks, or less: tokens of the kept blocks
    // The rows of a chunk come in runs of SPAN consecutive ones: 32 where B % 32 == 0 or all blocks are attended (then they
    // follow each other, whatever the block size), two of 16 where B % 16 == 0.  r >= 0: all rows r .. r + SPAN - 1 of the run
    // are valid tokens (the common case, handled without any further test); -1: no valid token; -2 - r: rows from r on, cut
    // off by the context length.  blk: the list entry of slot, the block that token p0 of the list lies in.
    // Any other block size looks up the row of every token in the list in front of every chunk, and waiting for that read
    // waits for every chunk requested before it.  Blocks of 16, before (looked up) and now: selection and partial step at
    // 60K, 4K kept, four layers 160.0 -> 154.3 us; 16 sequences of 32K 101.9 -> 87.4; refresh at 64K 106.8 -> 89.0.
    template <int SPAN> __device__ __forceinline__ int encode(int blk, uint32_t p0, uint32_t slot) const
    {
        if (blk < 0 || blk >= nb) return -1;
        const int r = blk * B + (int)(p0 - slot * (uint32_t)B);
        return r >= L ? -1 : (r + SPAN > L ? -2 - r : r);
    }
    template <int SPAN> __device__ __forceinline__ int first_row(uint32_t run) const
    {
        const uint32_t p0 = run * (uint32_t)SPAN;
        if (SPAN < 32 && p0 >= T) return -1;   // (32: a chunk of the list starts in it)
        const uint32_t slot = div_B.div(p0);   // < count
        return encode<SPAN>(sel ? sel[slot] : (int)slot, p0, slot);
    }
    // the row of token k of a run, or -1
    __device__ __forceinline__ int decode(int run, int k) const
    {
        const int r = run >= 0 ? run : -2 - run;   // -1 gives -1
        return r >= 0 && r + k < L ? r + k : -1;
    }
    // any block size: the row of token n of chunk c, or -1
    __device__ __forceinline__ int row(uint32_t c, int n) const
    {
        const uint32_t p = c * 32u + (uint32_t)n;
        if (p >= T) return -1;
        const uint32_t slot = div_B.div(p);
        const int blk = sel ? sel[slot] : (int)slot;
        if (blk < 0 || blk >= nb) return -1;
        const int tok = blk * B + (int)(p - slot * (uint32_t)B);
        return tok < L ? tok : -1;
    }
};

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4 &u) { return __builtin_bit_cast(bf16x8, u); }

// acc + lo(p) + hi(p) for a packed bf16 pair
__device__ __forceinline__ float add_bf16x2(uint32_t p, float acc)
{
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), ones, acc, false);
}
// x less the low / the high half of a packed bf16 pair that holds x rounded (the difference is exact): one instruction,
// where widening the half and subtracting it are two.  The constants go through registers: as an immediate, (-1, 0) is
// written as the inline constant -1.0, of which the instruction takes the other half.
struct Bf16Halves {
    uint32_t lo = 0x0000bf80u, hi = 0xbf800000u;   // (-1, 0), (0, -1)
    __device__ __forceinline__ Bf16Halves() { asm("" : "+s"(lo), "+s"(hi)); }
    __device__ __forceinline__ float sub_lo(float x, uint32_t p) const { return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), __builtin_bit_cast(bf16x2, lo), x, false); }
    __device__ __forceinline__ float sub_hi(float x, uint32_t p) const { return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), __builtin_bit_cast(bf16x2, hi), x, false); }
};

// 16 bytes per lane from global memory straight into LDS (no registers involved):
// lane l of the wavefront lands at lds_dst + 16*l.
__device__ __forceinline__ void dma16(const char *gsrc, char *lds_dst)
{
    __builtin_amdgcn_global_load_lds((glb_void_ptr)gsrc, (lds_void_ptr)lds_dst, 16, 0, kKvAux);
}

// Four such operations 1 KiB apart on both sides (K rows 4 i .. 4 i + 3 for i = 0 .. 3, or 4 .. 7): gbase is
// wavefront-uniform, row_off the lane's row (lane / 16) in bytes, sw0 its piece 16 * ((lane & 15) ^ (lane / 16));
// operation i fetches the piece that the swizzle by row & 15 puts at the lane's place, sw0 ^ 64 i.  The
// immediate offset of the instruction is added to the global and to the LDS address.
__device__ __forceinline__ void dma16x4(const char *gbase, uint32_t row_off, uint32_t sw0, char *lds_dst)
{
    __builtin_amdgcn_global_load_lds((glb_void_ptr)(gbase + (row_off + sw0)), (lds_void_ptr)lds_dst, 16, 0, kKvAux);
    __builtin_amdgcn_global_load_lds((glb_void_ptr)(gbase + (row_off + (sw0 ^ 64u))), (lds_void_ptr)lds_dst, 16, 1024, kKvAux);
    __builtin_amdgcn_global_load_lds((glb_void_ptr)(gbase + (row_off + (sw0 ^ 128u))), (lds_void_ptr)lds_dst, 16, 2048, kKvAux);
    __builtin_amdgcn_global_load_lds((glb_void_ptr)(gbase + (row_off + (sw0 ^ 192u))), (lds_void_ptr)lds_dst, 16, 3072, kKvAux);
}

// The LDS reads of staged K / V are written in assembly so that the compiler does not
// put a full vector-memory wait in front of them (it cannot tell which in-flight
// LDS-DMA a read depends on); the waits are placed by hand instead.
template <int OFF>
__device__ __forceinline__ void lds_read_k(const uint32_t (&a)[8], uint4 (&k)[8])
{
    asm volatile(
        "ds_read_b128 %0, %8 offset:%16\n\t"
        "ds_read_b128 %1, %9 offset:%16\n\t"
        "ds_read_b128 %2, %10 offset:%16\n\t"
        "ds_read_b128 %3, %11 offset:%16\n\t"
        "ds_read_b128 %4, %12 offset:%16\n\t"
        "ds_read_b128 %5, %13 offset:%16\n\t"
        "ds_read_b128 %6, %14 offset:%16\n\t"
        "ds_read_b128 %7, %15 offset:%16\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]), "=&v"(k[4]), "=&v"(k[5]), "=&v"(k[6]), "=&v"(k[7])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "n"(OFF)
        : "memory");
}

// Four k-steps (half of a chunk's K operands).
template <int OFF> __device__ __forceinline__ void lds_read_k_half(const uint32_t (&a)[4], uint4 (&k)[4])
{
    asm volatile(
        "ds_read_b128 %0, %4 offset:%8\n\t"
        "ds_read_b128 %1, %5 offset:%8\n\t"
        "ds_read_b128 %2, %6 offset:%8\n\t"
        "ds_read_b128 %3, %7 offset:%8\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3])
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(OFF)
        : "memory");
}

// V operands (A operand of O^T += V^T . P^T: per lane 8 tokens of ONE channel) through the
// transposing LDS read ds_read_b64_tr_b16.  Inside a group of 16 lanes, lane s reads 8 bytes
// (4 channels) and receives, as lane 4a + c, element c of what lanes a, a+4, a+8, a+12 read.
// With lane s reading token (s >> 2) of a token quad and channels 4 * (s & 3) .. +3 of a
// 16-channel group, every lane ends up with the four tokens of the quad for channel
// (lane & 15) of the group: lane m = lane & 31 holds channel 32j + m of tile j, its k-group the
// tokens 16*ks2 + 8*hf + 4*kg + 0..3.  The four rows of a quad sit in four different V pieces,
// 1088 bytes apart, i.e. 64 bytes apart modulo the bank cycle: no bank conflicts.
// v[(ks2 * 4 + j) * 2 + hf]; addr = piece (4*kg + (s >> 2)), byte 32 * (group & 1) + 8 * (s & 3).
// OFF: a constant byte offset (a ring stage), added by the instructions themselves.
template <int OFF = 0>
__device__ __forceinline__ void lds_read_v(uint32_t addr, uint2 (&v)[16])
{
    static_assert(OFF >= 0 && OFF + 960 < 65536, "the offset field has 16 bits");
    asm volatile(
        "ds_read_b64_tr_b16 %0, %16 offset:%17\n\t"
        "ds_read_b64_tr_b16 %1, %16 offset:%17+256\n\t"
        "ds_read_b64_tr_b16 %2, %16 offset:%17+64\n\t"
        "ds_read_b64_tr_b16 %3, %16 offset:%17+320\n\t"
        "ds_read_b64_tr_b16 %4, %16 offset:%17+128\n\t"
        "ds_read_b64_tr_b16 %5, %16 offset:%17+384\n\t"
        "ds_read_b64_tr_b16 %6, %16 offset:%17+192\n\t"
        "ds_read_b64_tr_b16 %7, %16 offset:%17+448\n\t"
        "ds_read_b64_tr_b16 %8, %16 offset:%17+512\n\t"
        "ds_read_b64_tr_b16 %9, %16 offset:%17+768\n\t"
        "ds_read_b64_tr_b16 %10, %16 offset:%17+576\n\t"
        "ds_read_b64_tr_b16 %11, %16 offset:%17+832\n\t"
        "ds_read_b64_tr_b16 %12, %16 offset:%17+640\n\t"
        "ds_read_b64_tr_b16 %13, %16 offset:%17+896\n\t"
        "ds_read_b64_tr_b16 %14, %16 offset:%17+704\n\t"
        "ds_read_b64_tr_b16 %15, %16 offset:%17+960\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]),
          "=&v"(v[8]), "=&v"(v[9]), "=&v"(v[10]), "=&v"(v[11]), "=&v"(v[12]), "=&v"(v[13]), "=&v"(v[14]), "=&v"(v[15])
        : "v"(addr), "n"(OFF)
        : "memory");
}

// Two chunks' worth of operands and both score tiles in one statement (128 channels): K operands of chunks 0 and 1 (byte
// offsets K0, K1 from a[]), S^T = K . Q^T of each, and behind the products the V operands of both (offsets V0, V1 from va;
// the layout of lds_read_v) in the registers that held K.  A wavefront's LDS reads then run under its own matrix
// instructions, and 64 tokens cost one round trip to LDS instead of four.  At most 15 reads are in flight (the counter has
// four bits); a register is read into again only behind the matrix instruction that was its last reader; "s_nop 11": the
// twelve wait states between a 32x32x16 product and the vector ALU's read of it, which the compiler does not count in here.
// With the single test of the maximum for both (attend_pair), core cycles per chunk of the full pass over 128K tokens, eight
// row blocks: 2033 -> 1800.  The chip runs that loop at the clock its power allows (1.4 to 1.9 GHz), so a workgroup's 128
// chunks went from 138 - 150 us to 126 - 139, not in proportion.  Tried as well: the two wavefronts of a SIMD passing the
// barrier at different points of this (2110), one of them requesting behind its scores (1890), wave priorities (no change).
template <int K0, int K1, int V0, int V1>
__device__ __forceinline__ void score_pair(const uint32_t (&a)[8], uint32_t va, const bf16x8 (&q)[8], f32x16 &S0, f32x16 &S1,
                                           uint4 (&v0)[8], uint4 (&v1)[8])
{
    static_assert(K0 >= 0 && K1 >= 0 && V0 >= 0 && V1 >= 0 && K0 < 65536 && K1 < 65536 && V0 + 960 < 65536 && V1 + 960 < 65536, "the offset field has 16 bits");
    asm volatile(
        "ds_read_b128 v[192:195], %[a0] offset:%[k0]\n\t"
        "ds_read_b128 v[196:199], %[a1] offset:%[k0]\n\t"
        "ds_read_b128 v[200:203], %[a2] offset:%[k0]\n\t"
        "ds_read_b128 v[204:207], %[a3] offset:%[k0]\n\t"
        "ds_read_b128 v[208:211], %[a4] offset:%[k0]\n\t"
        "ds_read_b128 v[212:215], %[a5] offset:%[k0]\n\t"
        "ds_read_b128 v[216:219], %[a6] offset:%[k0]\n\t"
        "ds_read_b128 v[220:223], %[a7] offset:%[k0]\n\t"
        "s_waitcnt lgkmcnt(7)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[192:195], %[q0], 0\n\t"
        "ds_read_b128 v[224:227], %[a0] offset:%[k1]\n\t"
        "ds_read_b128 v[228:231], %[a1] offset:%[k1]\n\t"
        "s_waitcnt lgkmcnt(8)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[196:199], %[q1], %[s0]\n\t"
        "ds_read_b128 v[232:235], %[a2] offset:%[k1]\n\t"
        "ds_read_b128 v[236:239], %[a3] offset:%[k1]\n\t"
        "s_waitcnt lgkmcnt(9)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[200:203], %[q2], %[s0]\n\t"
        "ds_read_b128 v[240:243], %[a4] offset:%[k1]\n\t"
        "ds_read_b128 v[244:247], %[a5] offset:%[k1]\n\t"
        "s_waitcnt lgkmcnt(10)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[204:207], %[q3], %[s0]\n\t"
        "ds_read_b128 v[248:251], %[a6] offset:%[k1]\n\t"
        "ds_read_b128 v[252:255], %[a7] offset:%[k1]\n\t"
        "s_waitcnt lgkmcnt(11)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[208:211], %[q4], %[s0]\n\t"
        "ds_read_b64_tr_b16 v[192:193], %[va] offset:%[v0]+0\n\t"
        "ds_read_b64_tr_b16 v[194:195], %[va] offset:%[v0]+256\n\t"
        "s_waitcnt lgkmcnt(12)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[212:215], %[q5], %[s0]\n\t"
        "ds_read_b64_tr_b16 v[196:197], %[va] offset:%[v0]+64\n\t"
        "ds_read_b64_tr_b16 v[198:199], %[va] offset:%[v0]+320\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[216:219], %[q6], %[s0]\n\t"
        "ds_read_b64_tr_b16 v[200:201], %[va] offset:%[v0]+128\n\t"
        "ds_read_b64_tr_b16 v[202:203], %[va] offset:%[v0]+384\n\t"
        "s_waitcnt lgkmcnt(14)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s0], v[220:223], %[q7], %[s0]\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "ds_read_b64_tr_b16 v[204:205], %[va] offset:%[v0]+192\n\t"
        "ds_read_b64_tr_b16 v[206:207], %[va] offset:%[v0]+448\n\t"
        "s_waitcnt lgkmcnt(8)\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[224:227], %[q0], 0\n\t"
        "ds_read_b64_tr_b16 v[208:209], %[va] offset:%[v0]+512\n\t"
        "ds_read_b64_tr_b16 v[210:211], %[va] offset:%[v0]+768\n\t"
        "ds_read_b64_tr_b16 v[224:225], %[va] offset:%[v1]+0\n\t"
        "ds_read_b64_tr_b16 v[226:227], %[va] offset:%[v1]+256\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[228:231], %[q1], %[s1]\n\t"
        "s_waitcnt lgkmcnt(11)\n\t"
        "ds_read_b64_tr_b16 v[212:213], %[va] offset:%[v0]+576\n\t"
        "ds_read_b64_tr_b16 v[214:215], %[va] offset:%[v0]+832\n\t"
        "ds_read_b64_tr_b16 v[228:229], %[va] offset:%[v1]+64\n\t"
        "ds_read_b64_tr_b16 v[230:231], %[va] offset:%[v1]+320\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[232:235], %[q2], %[s1]\n\t"
        "s_waitcnt lgkmcnt(11)\n\t"
        "ds_read_b64_tr_b16 v[216:217], %[va] offset:%[v0]+640\n\t"
        "ds_read_b64_tr_b16 v[218:219], %[va] offset:%[v0]+896\n\t"
        "ds_read_b64_tr_b16 v[232:233], %[va] offset:%[v1]+128\n\t"
        "ds_read_b64_tr_b16 v[234:235], %[va] offset:%[v1]+384\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[236:239], %[q3], %[s1]\n\t"
        "s_waitcnt lgkmcnt(11)\n\t"
        "ds_read_b64_tr_b16 v[220:221], %[va] offset:%[v0]+704\n\t"
        "ds_read_b64_tr_b16 v[222:223], %[va] offset:%[v0]+960\n\t"
        "ds_read_b64_tr_b16 v[236:237], %[va] offset:%[v1]+192\n\t"
        "ds_read_b64_tr_b16 v[238:239], %[va] offset:%[v1]+448\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[240:243], %[q4], %[s1]\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "ds_read_b64_tr_b16 v[240:241], %[va] offset:%[v1]+512\n\t"
        "ds_read_b64_tr_b16 v[242:243], %[va] offset:%[v1]+768\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[244:247], %[q5], %[s1]\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "ds_read_b64_tr_b16 v[244:245], %[va] offset:%[v1]+576\n\t"
        "ds_read_b64_tr_b16 v[246:247], %[va] offset:%[v1]+832\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[248:251], %[q6], %[s1]\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "ds_read_b64_tr_b16 v[248:249], %[va] offset:%[v1]+640\n\t"
        "ds_read_b64_tr_b16 v[250:251], %[va] offset:%[v1]+896\n\t"
        "v_mfma_f32_32x32x16_bf16 %[s1], v[252:255], %[q7], %[s1]\n\t"
        "s_waitcnt lgkmcnt(13)\n\t"
        "ds_read_b64_tr_b16 v[252:253], %[va] offset:%[v1]+704\n\t"
        "ds_read_b64_tr_b16 v[254:255], %[va] offset:%[v1]+960\n\t"
        "s_nop 11\n\t"
        "s_waitcnt lgkmcnt(0)"
        : [s0] "=&v"(S0), [s1] "=&v"(S1),
          "=&{v[192:195]}"(v0[0]), "=&{v[196:199]}"(v0[1]), "=&{v[200:203]}"(v0[2]), "=&{v[204:207]}"(v0[3]),
          "=&{v[208:211]}"(v0[4]), "=&{v[212:215]}"(v0[5]), "=&{v[216:219]}"(v0[6]), "=&{v[220:223]}"(v0[7]),
          "=&{v[224:227]}"(v1[0]), "=&{v[228:231]}"(v1[1]), "=&{v[232:235]}"(v1[2]), "=&{v[236:239]}"(v1[3]),
          "=&{v[240:243]}"(v1[4]), "=&{v[244:247]}"(v1[5]), "=&{v[248:251]}"(v1[6]), "=&{v[252:255]}"(v1[7])
        : [a0] "v"(a[0]), [a1] "v"(a[1]), [a2] "v"(a[2]), [a3] "v"(a[3]), [a4] "v"(a[4]), [a5] "v"(a[5]), [a6] "v"(a[6]), [a7] "v"(a[7]), [va] "v"(va),
          [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [q4] "v"(q[4]), [q5] "v"(q[5]), [q6] "v"(q[6]), [q7] "v"(q[7]),
          [k0] "n"(K0), [k1] "n"(K1), [v0] "n"(V0), [v1] "n"(V1)
        : "memory");
}

// Half of that: the operands of token half ks2 (OFF = 512 ks2), v[j * 2 + hf].
template <int OFF> __device__ __forceinline__ void lds_read_v_half(uint32_t addr, uint2 (&v)[8])
{
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%9\n\t"
        "ds_read_b64_tr_b16 %1, %8 offset:%10\n\t"
        "ds_read_b64_tr_b16 %2, %8 offset:%11\n\t"
        "ds_read_b64_tr_b16 %3, %8 offset:%12\n\t"
        "ds_read_b64_tr_b16 %4, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %5, %8 offset:%14\n\t"
        "ds_read_b64_tr_b16 %6, %8 offset:%15\n\t"
        "ds_read_b64_tr_b16 %7, %8 offset:%16\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
        : "v"(addr), "n"(OFF), "n"(OFF + 256), "n"(OFF + 64), "n"(OFF + 320), "n"(OFF + 128), "n"(OFF + 384), "n"(OFF + 192),
          "n"(OFF + 448)
        : "memory");
}

// 64 channels: the V operands of a chunk, v[(ks2 * 2 + j) * 2 + hf].  A row is 128 bytes; piece p (tokens p, p + 8,
// p + 16, p + 24) sits at 1152 (p >> 1) + 512 (p & 1), and the two 64-byte halves of an odd piece's rows are exchanged:
// the four pieces that a quad's lanes read then cover all 64 banks.  a0, a1: this lane's address of channel tile 0, 1.
template <int OFF>
__device__ __forceinline__ void lds_read_v64(uint32_t a0, uint32_t a1, uint2 (&v)[8])
{
    static_assert(OFF >= 0 && OFF + 384 < 65536, "the offset field has 16 bits");
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%10\n\t"
        "ds_read_b64_tr_b16 %1, %8 offset:%10+128\n\t"
        "ds_read_b64_tr_b16 %2, %9 offset:%10\n\t"
        "ds_read_b64_tr_b16 %3, %9 offset:%10+128\n\t"
        "ds_read_b64_tr_b16 %4, %8 offset:%10+256\n\t"
        "ds_read_b64_tr_b16 %5, %8 offset:%10+384\n\t"
        "ds_read_b64_tr_b16 %6, %9 offset:%10+256\n\t"
        "ds_read_b64_tr_b16 %7, %9 offset:%10+384\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
        : "v"(a0), "v"(a1), "n"(OFF)
        : "memory");
}

// The split-KV partials are written once here and read once by the combine kernel, which runs on
// other CUs (and mostly other XCDs): stored with the streaming hint they do not linger in this
// XCD's L2 as dirty lines that the end of the kernel has to write back (measured: 3.6 % of the
// partial-verify step).
// Two values of a split's normalised result as fp16, clamped to fp16's range.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t half_pair(float a, float b)
{
    const f16x2 hv = {(_Float16)__builtin_amdgcn_fmed3f(a, -65504.f, 65504.f), (_Float16)__builtin_amdgcn_fmed3f(b, -65504.f, 65504.f)};
    return __builtin_bit_cast(uint32_t, hv);
}

// max / sum over the two half-wavefronts (lane and lane ^ 32)
__device__ __forceinline__ float max_xor32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Running state of a query row (lane & 31; each lane's sum runs over its half of the tokens).  The reference maximum only
// moves when the true maximum runs more than 2^8 ahead of it: the common chunk tests that and does nothing else.  Before the first valid token the reference stands at -3e38, where exp2(fma(S, scale, 3e38)) is 0 for a
// masked score (-inf) as anywhere else, so that no test for "nothing seen yet" is needed.
struct RowState {
    float neg_ref = 3e38f;     // minus the reference maximum, in log2 units
    float l = 0.f;
    // reference maximum of a row with sum l_row; -inf for a row without valid tokens
    __device__ __forceinline__ float ref(float l_row) const { return l_row > 0.f ? -neg_ref : -INFINITY; }
};

__device__ __forceinline__ float tile_max(const f32x16 &S)
{
    float mx = fmaxf(fmaxf(S[0], S[1]), S[2]);
#pragma unroll
    for (int x = 3; x < 15; x += 2) mx = fmaxf(fmaxf(mx, S[x]), S[x + 1]);
    return fmaxf(mx, S[15]);
}

// mx: largest raw score of this lane's tokens in the chunk.
template <int NT> __device__ __forceinline__ void follow_max(float mx, float scale_log2, RowState &st, f32x16 (&O)[NT])
{
    if (!__any(fmaf(mx, scale_log2, st.neg_ref) > kRescaleSlack)) return;
    const float top = max_xor32(mx) * scale_log2;   // the row's tokens in both lane halves
    const float ref = -st.neg_ref, ref_new = top > ref + kRescaleSlack ? top : ref;
    const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);
    const bool rescale = __any(alpha != 1.f && st.l != 0.f);   // nothing to rescale while O is still zero
    st.neg_ref = -ref_new;
    st.l *= alpha;
    if (rescale) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) O[j][x] *= alpha;
    }
}

// vmask: which of the chunk's 32 tokens count
__device__ __forceinline__ void mask_scores(uint32_t vmask, int kg, f32x16 &S)
{
    if (vmask == 0xffffffffu) return;
    int kg_o = kg;   // (rare: nothing of it is kept in registers across the caller's loop)
    asm volatile("" : "+v"(kg_o));
    const uint32_t mine = vmask >> (kg_o * 4);
#pragma unroll
    for (int x = 0; x < 16; ++x)
        if (!((mine >> ((x >> 2) * 8 + (x & 3))) & 1u)) S[x] = -INFINITY;
}

// Weights of a chunk as bf16 pairs (the B operands of the second product); the sum runs over the rounded weights that the
// matrix instructions see.
__device__ __forceinline__ void softmax_weights(const f32x16 &S, float scale_log2, RowState &st, uint32_t (&pk)[8])
{
    float lsum = 0.f;
#pragma unroll
    for (int x = 0; x < 16; x += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(S[x], scale_log2, st.neg_ref));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(S[x + 1], scale_log2, st.neg_ref));
        pk[x >> 1] = pack_bf16x2(p0, p1);
        lsum = add_bf16x2(pk[x >> 1], lsum);
    }
    st.l += lsum;
}

// O^T += V^T . P^T of one chunk; v: one 16-byte operand per (token half, channel tile)
__device__ __forceinline__ void add_values(const uint4 (&v)[8], const uint32_t (&pk)[8], f32x16 (&O)[4])
{
    const uint4 pf[2] = {make_uint4(pk[0], pk[1], pk[2], pk[3]), make_uint4(pk[4], pk[5], pk[6], pk[7])};
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            O[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(v[ks2 * 4 + j]), as_bf16x8(pf[ks2]), O[j], 0, 0, 0);
}

// Two chunks whose scores and V operands score_pair has left in registers: one maximum and one test of it for 64 tokens.
__device__ __forceinline__ void attend_pair(f32x16 &S0, f32x16 &S1, const uint4 (&v0)[8], const uint4 (&v1)[8], uint32_t vm0, uint32_t vm1,
                                            int kg, float scale_log2, f32x16 (&O)[4], RowState &st)
{
    if ((vm0 & vm1) != 0xffffffffu) {
        mask_scores(vm0, kg, S0);
        mask_scores(vm1, kg, S1);
    }
    follow_max(fmaxf(tile_max(S0), tile_max(S1)), scale_log2, st, O);
    uint32_t pk[8];
    softmax_weights(S0, scale_log2, st, pk);
    add_values(v0, pk, O);
    softmax_weights(S1, scale_log2, st, pk);
    add_values(v1, pk, O);
}

// One 32-token chunk against a row block of 32 query rows, operands in registers: S^T = K . Q^T, the running maximum and
// sum of each row, O^T += V^T . P^T.  kf: K operands of the eight k-steps; v: V operands (lds_read_v); qf: the query rows.
__device__ __forceinline__ void attend_chunk(const uint4 (&kf)[8], const uint2 (&v)[16], const bf16x8 (&qf)[8], uint32_t vmask, int kg,
                                             float scale_log2, f32x16 (&O)[4], RowState &st)
{
    f32x16 S;
#pragma unroll
    for (int x = 0; x < 16; ++x) S[x] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), qf[ks], S, 0, 0, 0);
    mask_scores(vmask, kg, S);
    follow_max(tile_max(S), scale_log2, st, O);
    uint32_t pk[8];
    softmax_weights(S, scale_log2, st, pk);
    uint4 vv[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) vv[x] = make_uint4(v[2 * x].x, v[2 * x].y, v[2 * x + 1].x, v[2 * x + 1].y);
    add_values(vv, pk, O);
}

// Instrumented builds (-DSPECPV_TIMELINE): core clock against real time over a workgroup's life.  Cycles, 10 ns ticks and
// the number of chunks go to words 0 .. 2 of row ROW of the stamp buffer (the real-time counter runs at 100 MHz
// whatever the chip does, s_memtime counts core cycles).
#ifdef SPECPV_TIMELINE
#define SPECPV_CLOCKS_BEGIN const unsigned long long clk0_ = clock64(), rt0_ = __builtin_amdgcn_s_memrealtime()
#define SPECPV_CLOCKS_END(TL, ROW, NCH)                                                                       \
    do {                                                                                                      \
        if ((TL) && threadIdx.x == 0 && (size_t)(ROW) < 4096) {                                               \
            unsigned long long *t_ = (TL) + (size_t)(ROW) * 16;                                               \
            t_[0] = clock64() - clk0_;                                                                        \
            t_[1] = __builtin_amdgcn_s_memrealtime() - rt0_;                                                  \
            t_[2] = (unsigned long long)(NCH);                                                                \
        }                                                                                                     \
    } while (0)
#else
#define SPECPV_CLOCKS_BEGIN do {} while (0)
#define SPECPV_CLOCKS_END(TL, ROW, NCH) do {} while (0)
#endif

}  // namespace specpv
