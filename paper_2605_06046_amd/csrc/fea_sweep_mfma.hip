// KV sweep on the matrix cores: bf16 caches, head_dim 128, 64 or 256, query groups of
// up to 64 heads per KV head (32 at head_dim 256; any ratio: 7 as in 28/4, 5 as in 40/8, ...).  What
// follows describes head_dim 128.  Head_dim 64 is the same kernel with 2 KB blocks (two
// loads each, 128-byte token rows of eight chunks, swizzled by the row modulo 8), two
// k-steps in the first product and four output products per 16 rows.  Head_dim 256: 8 KB
// blocks (eight loads, 512-byte rows whose halves are swizzled like 256-byte rows),
// eight k-steps, sixteen output products per 16 rows, work items of at most 32 rows (O
// for 32 rows fills half the accumulation registers), and two waves per workgroup, whose
// two 32 KB stages each fill the LDS.
//
// One wave per SIMD (workgroups of four waves, one workgroup per compute unit); the planner has
// cut the stream of 32-token tiles into equal shares, and wave w sweeps the consecutive work
// items of share w.
// An item is a set of up to 64 query rows (one request's query group,
// or a row tile of a prefix group: members x group heads stacked) x one KV head x
// a range of table columns; the wave sweeps the range with an online softmax and
// writes one partial (m, l, acc[128]) per query row.
//
// Per 32-token tile (two 16-token blocks) the wave computes, transposed,
//     S^T = K Q^T           (tokens x rows;  v_mfma_f32_16x16x32_bf16, k = head_dim)
//     O^T += V^T P^T        (dims x rows;    same instruction,        k = tokens)
// The transposed forms are chosen so that (a) one lane owns one query row: the
// row maximum, the running sum and the rescale of O stay in-lane (only the 4
// lane groups are combined, with two cross-lane maxima), and (b) the
// exponentiated scores in the S^T accumulator layout are already the B operand
// of the second product, no data movement in between.
//
// Memory side.  Every 16-token block of one KV head is 4 KB contiguous.  A tile
// (K and V of two blocks, 16 KB) is fetched with sixteen wave-wide 16-byte-per-
// lane loads that write straight into LDS (global_load_lds_dwordx4), so data in
// flight costs no registers: two 16 KB stages per wave, and the fetch of tile
// t+2 is issued as soon as tile t has been read out of its stage, which keeps
// two tiles in flight while a tile is being computed - across item boundaries too:
// the block ids of the next item's first columns are fetched while the current
// item runs, so its last tiles overlap with the first fetches of the next.  Each
// load covers four
// whole 256-byte token rows; inside a row the sixteen 16-byte chunks are placed
// XOR-swizzled by the row number, which makes the "lane = token" reads of the K
// operand bank-conflict free without padding (the DMA path cannot pad).  V needs
// "lane = head dim, 8 tokens per lane", which is how the transposing LDS read hands it
// over (ds_read_b64_tr_b16: the 16 lanes of a group read four token rows, 16 dims of
// each, and lane n is left with dim n of the four).
//
// A wave alone on its SIMD issues an instruction in four cycles and fetches 8 bytes of them in
// 4.7 to 7.2 (by compute unit), so with few query rows on a tile its time is the number of its instructions: 420 a tile at
// head_dim 64 when the waits were a tree over all 50 counts, V was transposed by permutes and selects, every load set M0 and
// the sums were copied back.  Without those, all else as it was then: 48 requests of head_dim 256 on 3000 tokens 53.9 -> 45.8 us a
// call (27 registers were spilled there as well), a layer of nested prefixes, 40/8/128, 37.3 -> 35.7, 128 requests of head_dim 64 in 8
// groups 55.3 -> 53.9, 64 on one prefix of 4096, 32/8/128, 54.7 both.
//
// The LDS writes of those loads are invisible to the compiler, so the waits are
// explicit: vmcnt before a stage is read, lgkmcnt before it is overwritten.
//
// What is computed is the same (m, l, acc) triple per query row as in the generic
// sweep: the pieces of softmax(q K^T / sqrt(d)) V (Section 2.1), scores in the
// base-2 domain.  Products are bf16 x bf16 accumulated in float32; the softmax
// weights are rounded to bf16 for the second product, the sums stay float32.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstdlib>
#include <type_traits>

#include "fea_plan.h"
#include "fea_tile.h"

namespace fea {

constexpr int kD = 128;                 // head dim of the team sequence (the sweep itself is instantiated per head dim)
constexpr int kTileTok = 32;            // tokens per tile (two blocks)
constexpr int kBlkBytes = kBlock * kD * 2;      // one (block, KV head) at that head dim: 4096 bytes
constexpr int kStageBytes = 4 * kBlkBytes;      // a tile stage at that head dim: K b0 | K b1 | V b0 | V b1
constexpr int kStages = 2;
constexpr int kDescWindow = 8;           // item descriptors fetched into LDS at a time
constexpr float kSlack = 24.f;           // log2 of the largest softmax weight tolerated before the reference is raised

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Wave-uniform values that must sit in scalar registers (folded away by the compiler
// where it already knows them to be uniform).
// (The builtin returns a signed int: the halves go through uint32_t so that the low
// word is zero-extended, not sign-extended, when the pointer is put back together.)
__device__ __forceinline__ uint32_t sgpr(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ const char* sgpr(const void* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint64_t lo = sgpr((uint32_t)v), hi = sgpr((uint32_t)(v >> 32));
    return reinterpret_cast<const char*>(lo | (hi << 32));
}

// Four wave-wide loads of 64 x 16 bytes from global memory straight into LDS: load
// i reads base + off_i (per lane) and lane l's bytes land at lds_i + 16 l.  The LDS
// addresses are wave-uniform and go through M0.  The scalar operands may have been
// produced by a vector instruction (v_readfirstlane) just before; the hardware
// wants five wait states between such a write and a memory instruction that reads
// the register, and the compiler cannot see into this block, hence the s_nop (and
// one wait state between each write of M0 and the load that uses it).
__device__ __forceinline__ void dma16x4(const char* base, uint32_t off0, uint32_t off1, uint32_t off2, uint32_t off3,
                                        uint32_t lds0, uint32_t lds1, uint32_t lds2, uint32_t lds3) {
    asm volatile(
        "s_nop 4\n\t"
        "s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %4\n\t"
        "s_mov_b32 m0, %6\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\t"
        "s_mov_b32 m0, %7\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4\n\t"
        "s_mov_b32 m0, %8\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %4"
        :: "v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(base), "s"(lds0), "s"(lds1), "s"(lds2), "s"(lds3)
        : "memory", "m0");
}
// Two such loads (query rows of head_dim 64).
__device__ __forceinline__ void dma16x2(const char* base, uint32_t off0, uint32_t off1, uint32_t lds0, uint32_t lds1) {
    asm volatile(
        "s_nop 4\n\t"
        "s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\t"
        "s_mov_b32 m0, %4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
        :: "v"(off0), "v"(off1), "s"(base), "s"(lds0), "s"(lds1)
        : "memory", "m0");
}
// A tile: the loads of its four blocks, into LDS one behind the other from lds on.  The immediate offset of such a load moves
// both its addresses, so M0 is set once for 4 KB (head_dim 64: 2 KB) instead of for every load.  ONCE: nobody else reads these
// bytes (kOnce), they need not stay in the caches, and kept there they only cost: a scattered read of 2 GB so 6.4 -> 6.9 TB/s, 256
// requests in 8 groups on 4096 (32/8/128) 166 -> 147 us, 64 on one, three sets of caches in turn, 51.3 -> 48.8, five groups of 16 on
// 10240, two sets, 112 -> 100.  49 drawn shapes with more in turn than the memory-side cache holds (800 MB): 0.99 of the time where a
// call reads up to 32 MB, 0.97 up to 64, 0.93 up to 128, 0.91 up to 240.  Where that cache would hold all of it, one batch over and
// over or few layers of it: 1.03, 1.05, 1.01 and 1.01 (0.96 to 1.12), so a call that reads less than 32 MB, eight layers of which
// would stay there, is left to the caches: 0.97 of the time then where all of it is held (39 calls, 0.90 to 1.03), 1.02 where it is not
// (21, 0.99 to 1.06), none slower than before there were such loads.  Columns that others read too are left to the caches: 48
// requests on a system prompt in 6 groups, four layers 148 us, 155 with all of them passing by.
template <int D, bool ONCE>
__device__ __forceinline__ void dma_tile(const char* k0, const char* k1, const char* v0, const char* v1, const uint32_t (&off)[8], uint32_t lds) {
#define FEA_DMA2(A, BASE, AT) "global_load_lds_dwordx4 " A ", " BASE AT "\n\tglobal_load_lds_dwordx4 " A ", " BASE " offset:1024" AT "\n\t"
#define FEA_DMA4(A, B, C, E, BASE, AT) "global_load_lds_dwordx4 " A ", " BASE AT "\n\tglobal_load_lds_dwordx4 " B ", " BASE " offset:1024" AT "\n\t" \
        "global_load_lds_dwordx4 " C ", " BASE " offset:2048" AT "\n\tglobal_load_lds_dwordx4 " E ", " BASE " offset:3072" AT "\n\t"
#define FEA_DMA8(BASE, AT) FEA_DMA4("%0", "%1", "%2", "%3", BASE, AT) FEA_M0_ON FEA_DMA4("%4", "%5", "%6", "%7", BASE, AT)
#define FEA_M0_ON "s_addk_i32 m0, 0x1000\n\ts_nop 0\n\t"
#define FEA_M0_ON2 "s_addk_i32 m0, 0x800\n\ts_nop 0\n\t"
#define FEA_TILE64(AT) asm volatile("s_nop 4\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\t" \
        FEA_DMA2("%0", "%1", AT) FEA_M0_ON2 FEA_DMA2("%0", "%2", AT) FEA_M0_ON2 FEA_DMA2("%0", "%3", AT) FEA_M0_ON2 FEA_DMA2("%0", "%4", AT) \
        :: "v"(off[0]), "s"(k0), "s"(k1), "s"(v0), "s"(v1), "s"(lds) : "memory", "m0", "scc")
#define FEA_TILE128(AT) asm volatile("s_nop 4\n\ts_mov_b32 m0, %8\n\ts_nop 0\n\t" \
        FEA_DMA4("%0", "%1", "%2", "%3", "%4", AT) FEA_M0_ON FEA_DMA4("%0", "%1", "%2", "%3", "%5", AT) FEA_M0_ON \
        FEA_DMA4("%0", "%1", "%2", "%3", "%6", AT) FEA_M0_ON FEA_DMA4("%0", "%1", "%2", "%3", "%7", AT) \
        :: "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(k0), "s"(k1), "s"(v0), "s"(v1), "s"(lds) : "memory", "m0", "scc")
#define FEA_TILE256(AT) asm volatile("s_nop 4\n\ts_mov_b32 m0, %12\n\ts_nop 0\n\t" \
        FEA_DMA8("%8", AT) FEA_M0_ON FEA_DMA8("%9", AT) FEA_M0_ON FEA_DMA8("%10", AT) FEA_M0_ON FEA_DMA8("%11", AT) \
        :: "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), \
           "s"(k0), "s"(k1), "s"(v0), "s"(v1), "s"(lds) : "memory", "m0", "scc")
    if constexpr (D == 64) {
        if constexpr (ONCE) FEA_TILE64(" nt");
        else FEA_TILE64("");
    } else if constexpr (D == 128) {
        if constexpr (ONCE) FEA_TILE128(" nt");
        else FEA_TILE128("");
    } else {
        if constexpr (ONCE) FEA_TILE256(" nt");
        else FEA_TILE256("");
    }
#undef FEA_DMA2
#undef FEA_DMA4
#undef FEA_DMA8
#undef FEA_M0_ON
#undef FEA_M0_ON2
#undef FEA_TILE64
#undef FEA_TILE128
#undef FEA_TILE256
}
// One load of 4 bytes per lane (block ids of 64 table columns), same conventions.
__device__ __forceinline__ void dma4(const void* base, uint32_t lane_off, uint32_t lds_addr) {
    asm volatile("s_nop 4\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(lane_off), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// acc *= f for an accumulator tuple that lives in the accumulation registers.  Done
// by hand so that the register allocator keeps the big O accumulators there (a
// plain C++ multiply would pull all of them into the vector register file and
// make every tile pay for copies).  Only the rare "raise the reference" path runs
// this; the leading s_nop covers the matrix-core write -> read distance even if a
// product into the same tuple were the immediately preceding instruction.
__device__ __forceinline__ void scale_acc(f32x4& acc, float f) {
    float a0 = acc[0], a1 = acc[1], a2 = acc[2], a3 = acc[3];
    float t0, t1;
    asm volatile(
        "s_nop 15\n\ts_nop 3\n\t"
        "v_accvgpr_read_b32 %4, %0\n\tv_accvgpr_read_b32 %5, %1\n\t"
        "v_mul_f32 %4, %4, %6\n\tv_mul_f32 %5, %5, %6\n\t"
        "v_accvgpr_write_b32 %0, %4\n\tv_accvgpr_write_b32 %1, %5\n\t"
        "v_accvgpr_read_b32 %4, %2\n\tv_accvgpr_read_b32 %5, %3\n\t"
        "v_mul_f32 %4, %4, %6\n\tv_mul_f32 %5, %5, %6\n\t"
        "v_accvgpr_write_b32 %2, %4\n\tv_accvgpr_write_b32 %3, %5"
        : "+a"(a0), "+a"(a1), "+a"(a2), "+a"(a3), "=&v"(t0), "=&v"(t1)
        : "v"(f));
    acc[0] = a0; acc[1] = a1; acc[2] = a2; acc[3] = a3;
}
// o[i] += v[i] p in place, and l += ones p with the first four: as the builtin the sums came out in other registers than they went
// in, and every tile copied them back (20 moves for 16 query rows of head_dim 64).  What the vector unit has written into an operand
// wants two wait states before a product reads it.  The compiler sees no products here, and puts a statement, and a copy of one of its
// operands, wherever the data allow: so each statement waits for itself.  (Hidden behind the product before it; as a statement for
// each product, and the wait in the first alone, other schedules than the default one put the weights right before a product.)
template <int AT = 0, int N> __device__ __forceinline__ void add_products(f32x4& l, f32x4 (&o)[N], bf16x8 ones, const bf16x8 (&v)[N], bf16x8 p) {
    if constexpr (AT == 0)
        asm("s_nop 1\n\t"
            "v_mfma_f32_16x16x32_bf16 %0, %5, %6, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %7, %6, %1\n\tv_mfma_f32_16x16x32_bf16 %2, %8, %6, %2\n\t"
            "v_mfma_f32_16x16x32_bf16 %3, %9, %6, %3\n\tv_mfma_f32_16x16x32_bf16 %4, %10, %6, %4"
            : "+a"(l), "+a"(o[0]), "+a"(o[1]), "+a"(o[2]), "+a"(o[3]) : "v"(ones), "v"(p), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
    else
        asm("s_nop 1\n\t"
            "v_mfma_f32_16x16x32_bf16 %0, %5, %4, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %6, %4, %1\n\t"
            "v_mfma_f32_16x16x32_bf16 %2, %7, %4, %2\n\tv_mfma_f32_16x16x32_bf16 %3, %8, %4, %3"
            : "+a"(o[AT]), "+a"(o[AT + 1]), "+a"(o[AT + 2]), "+a"(o[AT + 3]) : "v"(p), "v"(v[AT]), "v"(v[AT + 1]), "v"(v[AT + 2]), "v"(v[AT + 3]));
    if constexpr (AT + 4 < N) add_products<AT + 4>(l, o, ones, v, p);
}
// Sums that the compiler's instructions have just written or are about to read: it does not see the products' side.  The last
// products' results want up to 19 wait states before they are read (one statement for all of an item's sums: each of them is behind
// its products and before its reads); what is written here is there well before the first product.
#define FEA_SUMS4(I) "+a"(o[I]), "+a"(o[I + 1]), "+a"(o[I + 2]), "+a"(o[I + 3])
template <bool READ, int N> __device__ __forceinline__ void settle(f32x4& l, f32x4 (&o)[N]) {
    static_assert(N == 4 || N == 8 || N == 16, "head_dim 64, 128, 256");
    if constexpr (!READ) asm volatile("" : "+a"(l));
    if constexpr (N == 4) {
        if constexpr (READ) asm volatile("s_nop 15\n\ts_nop 3" : "+a"(l), FEA_SUMS4(0));
        else asm volatile("" : FEA_SUMS4(0));
    } else if constexpr (N == 8) {
        if constexpr (READ) asm volatile("s_nop 15\n\ts_nop 3" : "+a"(l), FEA_SUMS4(0), FEA_SUMS4(4));
        else asm volatile("" : FEA_SUMS4(0), FEA_SUMS4(4));
    } else {
        if constexpr (READ) asm volatile("s_nop 15\n\ts_nop 3" : "+a"(l), FEA_SUMS4(0), FEA_SUMS4(4), FEA_SUMS4(8), FEA_SUMS4(12));
        else asm volatile("" : FEA_SUMS4(0), FEA_SUMS4(4), FEA_SUMS4(8), FEA_SUMS4(12));
    }
}
#undef FEA_SUMS4
// Stores issued by hand so that the wave can count them (see Stream): wave-uniform
// base address in scalar registers, 32-bit byte offset per lane.  The hardware reads
// the data registers of a wide store a little after issue and does not interlock
// against a vector instruction overwriting them meanwhile; the compiler pads its own
// stores for that but cannot see these, hence the trailing s_nop.
template <int AT> __device__ __forceinline__ void store_f32x4(const char* base, uint32_t off, f32x4 v) {
    asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 offset:%3\n\ts_nop 1" :: "v"(off), "v"(v), "s"(base), "n"(AT) : "memory");
}
// ... and the 16-byte pieces of one row, 64 bytes apart.
template <int I = 0, int N> __device__ __forceinline__ void store_row(const char* base, uint32_t off, const f32x4 (&v)[N]) {
    if constexpr (I < N) {
        store_f32x4<64 * I>(base, off, v[I]);
        store_row<I + 1>(base, off, v);
    }
}
__device__ __forceinline__ void store_f32x2(const char* base, uint32_t off, float x, float y) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {x, y};
    asm volatile("s_nop 4\n\tglobal_store_dwordx2 %0, %1, %2\n\ts_nop 1" :: "v"(off), "v"(v), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

struct Piece : Item { int once; };   // g: the KV head alone; once: its kOnce

struct Lanes {
    int n;                 // lane % 16: query row of a 16-row tile / token of a block / 16-byte chunk
    int kg;                // lane / 16: k-slot group of the MFMA operands
    uint32_t dma_off[8];   // global byte offset of load i (rows 4i + kg of a block, swizzled chunk), without the load's immediate one
    uint32_t k_off[8];     // LDS byte offset inside a K block of the A operand for k-step ks
    uint32_t v_off;        // LDS byte offset inside a V block of token row 4 kg + n / 4, its dims 4 (n % 4) ..; dims 16 i on: with 32 i exclusive-or'ed in
};

// Fetch blocks b0, b1 of KV head g into the stage at LDS address `stage` (16 loads).
template <int D>
__device__ __forceinline__ void fetch_tile(const SweepArgs& a, int g, int once, int b0, int b1, uint32_t stage, const Lanes& L) {
    constexpr int BLK = kBlock * D * 2;
    const size_t o0 = (size_t)((uint32_t)b0 * (uint32_t)a.Hkv + (uint32_t)g) * BLK;   // (blocks times KV heads: below 2^32, a block has 2 KB or more)
    const size_t o1 = (size_t)((uint32_t)b1 * (uint32_t)a.Hkv + (uint32_t)g) * BLK;
    const char* k0 = sgpr(static_cast<const char*>(a.k_cache) + o0);
    const char* k1 = sgpr(static_cast<const char*>(a.k_cache) + o1);
    const char* v0 = sgpr(static_cast<const char*>(a.v_cache) + o0);
    const char* v1 = sgpr(static_cast<const char*>(a.v_cache) + o1);
    if (once) dma_tile<D, true>(k0, k1, v0, v1, L.dma_off, sgpr(stage));
    else dma_tile<D, false>(k0, k1, v0, v1, L.dma_off, sgpr(stage));
}

// Tile stream of one wave.  `phase` is the stage the current item's tile 0 uses,
// `iss` counts the tiles issued so far, numbered from the current item's tile 0
// (so it can already be 1 or 2 when the item starts: its predecessor fetched them).
//
// Everything the wave loads while it streams goes global -> LDS by hand-issued loads
// the compiler does not see, and the hardware retires a wave's vector-memory
// operations in issue order.  So the wave numbers them itself: `seq` counts the
// loads issued, every consumer remembers the count right after "its" loads (a
// mark), and waiting for a mark means letting at most seq - mark younger
// operations stay outstanding; the stores of the partial rows are issued by hand
// and counted as well.  An operation the compiler issues on its own and that is
// not counted only makes a wait stricter.
struct Stream {
    int phase;
    int iss;
    // Block ids travel through three 64-column windows in LDS: even and odd windows of
    // the current item, and the first window of the next item (which becomes the even
    // window when the items switch).
    int cb0, cb1, cbn;
    bool cols_ready;   // the current item's first window was requested while its predecessor ran
    bool q_ready;      // its query rows were requested (into the LDS query buffer): by its predecessor, or ahead of a share's first tile
    uint32_t seq;      // hand-issued loads so far
    uint32_t done;     // loads [0, done) are known to have landed
    uint32_t tmark0, tmark1;          // mark of the tile in stage 0 / 1
    uint32_t cmark0, cmark1, cmark2;  // marks of the three column windows
    uint32_t qmark;                   // mark of the query buffer
};

__device__ __forceinline__ uint32_t pick3(int i, uint32_t a, uint32_t b, uint32_t c) { return i == 0 ? a : (i == 1 ? b : c); }

// Wait until the load with this mark (and with it every older one) has landed.  The wait takes its count as an immediate: the
// one that a tile mostly needs (a tile's T loads are younger) comes first, then a few, rounded down.  (All 50 as a switch were
// a tree of 250 instructions wherever it stood, and a dozen jumps each time.)
template <int T> __device__ __forceinline__ void wait_for(Stream& sm, uint32_t mark) {
    if ((int32_t)(mark - sm.done) <= 0) return;
    uint32_t n = sm.seq - mark;   // younger loads: they may stay in flight
    auto leave = [&](auto count) { wait_vmcnt<decltype(count)::value>(); n = decltype(count)::value; };
    using std::integral_constant;
    constexpr int kMost = 2 * T + 4 < 50 ? 2 * T + 4 : 50;
    if (__builtin_expect(n == T, 1)) leave(integral_constant<int, T>{});
    else if (n >= kMost) leave(integral_constant<int, kMost>{});
    else if (n >= T + 8) leave(integral_constant<int, T + 8>{});
    else if (n >= T + 4) leave(integral_constant<int, T + 4>{});
    else if (n >= T) leave(integral_constant<int, T>{});
    else if (n >= 4) leave(integral_constant<int, 4>{});
    else if (n >= 1) leave(integral_constant<int, 1>{});
    else leave(integral_constant<int, 0>{});
    sm.done = sm.seq - n;
}
__device__ __forceinline__ void wait_all(Stream& sm) {
    wait_vmcnt<0>();
    sm.done = sm.seq;
}

// Brings an item's query rows into the wave's query buffer, laid out like a K block: one contiguous run of at most 16 rows.
__device__ __forceinline__ bool rows_in_line(const Item& item) { return item.nrows <= 16 && item.mlist_off < 0; }
template <int D>
__device__ __forceinline__ void fetch_rows(const SweepArgs& a, const Item& item, uint32_t q_base, int lane, Stream& sm) {
    const int n = lane & 15, kg = lane >> 4;
    const char* qn = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.q) + ((size_t)item.who * a.Hq + item.g * a.G) * D);
    const uint32_t qb = sgpr(q_base);
    if constexpr (D == 128) {
        uint32_t off[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 4 * j + kg;                          // row of the buffer this lane fills in load j
            off[j] = (uint32_t)min(row, item.nrows - 1) * 256u + (uint32_t)((n ^ row) & 15) * 16u;   // rows past the end repeat the last one
        }
        dma16x4(sgpr(qn), off[0], off[1], off[2], off[3], qb, qb + 1024, qb + 2048, qb + 3072);
        sm.seq += 4;
    } else if constexpr (D == 64) {
        uint32_t off[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 8 * j + (lane >> 3), pos = lane & 7;   // 128-byte rows: eight per load
            off[j] = (uint32_t)min(row, item.nrows - 1) * 128u + (uint32_t)((pos ^ row) & 7) * 16u;
        }
        dma16x2(sgpr(qn), off[0], off[1], qb, qb + 1024);
        sm.seq += 2;
    } else {
        uint32_t off[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = 2 * j + (lane >> 5), pos = lane & 31;  // 512-byte rows: two per load
            off[j] = (uint32_t)min(row, item.nrows - 1) * 512u + (uint32_t)((pos & 16) | ((pos ^ row) & 15)) * 16u;
        }
        dma16x4(sgpr(qn), off[0], off[1], off[2], off[3], qb, qb + 1024, qb + 2048, qb + 3072);
        dma16x4(sgpr(qn), off[4], off[5], off[6], off[7], qb + 4096, qb + 5120, qb + 6144, qb + 7168);
        sm.seq += 8;
    }
    sm.qmark = sm.seq;
}

template <int NT, int D>
__device__ __forceinline__ void sweep_item(const SweepArgs& a, const Piece& item, const Piece& next, bool has_next,
                                           int g_rcp, char* s_stage, const int* s_cols, const char* s_q, uint32_t lds_base,
                                           uint32_t cols_base, uint32_t q_base, const Lanes& L, int lane, Stream& sm) {
    constexpr int BLK = kBlock * D * 2;      // bytes of one (block, KV head)
    constexpr int STG = 4 * BLK;             // K b0 | K b1 | V b0 | V b1
    constexpr int KS = D / 32;               // k-steps of S^T = K Q^T
    constexpr int NI = D / 16;               // products of O^T += V^T P^T per 16 query rows
    const int n = L.n, kg = L.kg;
    const uint16_t* Q = static_cast<const uint16_t*>(a.q);
    const int* mlist = reinterpret_cast<const int*>(a.ws + a.lay.members) + item.mlist_off;
    const int ntiles = (item.c1 - item.c0 + 1) >> 1;
    const int next_pre = has_next ? min(2, (next.c1 - next.c0 + 1) >> 1) : 0;   // tiles of the next item we may fetch

    // Block ids of the item's columns travel through LDS as well, 64 columns per
    // window: the compiler then sees no pending vector-memory load inside the tile
    // loop (it would drain the whole prefetch queue for it).
    const int32_t* trow = a.bt + (size_t)item.who * a.stride;
    const int32_t* nrow = a.bt + (size_t)next.who * a.stride;
    auto fetch_cols = [&](const int32_t* row, int c0, int c1, int win, int buf) {   // clamped: never reads a dead entry
        dma4(sgpr(row), (uint32_t)min(c0 + 64 * win + lane, c1 - 1) * 4u, sgpr(cols_base + buf * 256));
        sm.seq += 1;
        sm.cmark0 = buf == 0 ? sm.seq : sm.cmark0;   // (value selects: the struct must stay in registers)
        sm.cmark1 = buf == 1 ? sm.seq : sm.cmark1;
        sm.cmark2 = buf == 2 ? sm.seq : sm.cmark2;
    };
    auto buf_of = [&](int win) { return (win & 1) ? sm.cb1 : sm.cb0; };
    // Issue stream tile `idx` (own tile idx, or tile idx - ntiles of the next item) if it
    // is the next one due and exists; own tiles must be asked for in increasing order.
    auto issue = [&](int idx) {
        if (idx != sm.iss) return;
        int buf, at;
        int g = item.g, once = item.once;
        if (idx < ntiles) {
            const int w = idx & 31, win = idx >> 5;
            if (w == 0 && idx > 0) fetch_cols(trow, item.c0, item.c1, win + 1, buf_of(win + 1));   // `win` came 32 tiles ago
            buf = buf_of(win);
            at = 2 * w;
        } else {
            const int j = idx - ntiles;
            if (j >= next_pre) return;
            buf = sm.cbn;
            at = 2 * j;
            g = next.g;
            once = next.once;
        }
        wait_for<D / 8>(sm, pick3(buf, sm.cmark0, sm.cmark1, sm.cmark2));   // the window's block ids must have landed
        const int* sc = s_cols + buf * 64 + at;
        // (a table entry of -1 inside a request's length is the caller's error; it must not become a
        // read before the cache)
        const int b0 = max(__builtin_amdgcn_readfirstlane(sc[0]), 0);
        const int b1 = max(__builtin_amdgcn_readfirstlane(sc[1]), 0);
        const int stg = (sm.phase + idx) & 1;
        fetch_tile<D>(a, g, once, b0, b1, lds_base + stg * STG, L);
        sm.seq += D / 8;
        sm.tmark0 = stg == 0 ? sm.seq : sm.tmark0;
        sm.tmark1 = stg == 1 ? sm.seq : sm.tmark1;
        sm.iss = idx + 1;
    };
    if (!sm.cols_ready) fetch_cols(trow, item.c0, item.c1, 0, sm.cb0);
    fetch_cols(trow, item.c0, item.c1, 1, sm.cb1);
    if (has_next) fetch_cols(nrow, next.c0, next.c1, 0, sm.cbn);
    // Own tiles only at this point (no-ops when the predecessor has asked for them):
    // the next item's column window has only just been requested.
    issue(0);
    if (ntiles > 1) issue(1);

    // B operand of the first product: Q^T, lane (n, kg) holds q[row n][32 ks + 8 kg .. +8].
    // The rows of a single request's query group are contiguous in q; the predecessor
    // - or, for the first item of a share at head_dim 64 and 256, the kernel ahead of the
    // item's tiles - has then already brought them into the LDS query buffer (laid out
    // like a K block: 16 rows, chunks swizzled by the row), and nothing has to be waited
    // for that is younger than that.  Otherwise (first item of a share at head_dim 128,
    // rows gathered through a member list, more than 16 rows) they are loaded here and
    // everything in flight is drained once.
    bf16x8 qB[NT][KS];
    bool q_from_lds = false;
    if constexpr (NT == 1) q_from_lds = sm.q_ready;
    if (q_from_lds) {
        wait_for<D / 8>(sm, sm.qmark);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qB[0][ks] = as_bf16x8(ld16(s_q + L.k_off[ks]));
    } else {
        int of = n;                     // (worked out again for each item: kept for the kernel's life these would be spilled)
        asm volatile("" : "+v"(of));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int row = nt * 16 + of;
            const bool ok = row < item.nrows;
            const int mem = (row * g_rcp) >> 16, hh = row - mem * a.G;   // row / G and row % G (rows < 64, G <= 64)
            const int req = ok ? (item.mlist_off < 0 ? item.who : mlist[mem]) : 0;
            const uint16_t* qp = Q + ((size_t)req * a.Hq + item.g * a.G + hh) * D + kg * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                u32x4 v = {0u, 0u, 0u, 0u};
                if (ok) v = ld16(qp + ks * 32);
                qB[nt][ks] = as_bf16x8(v);
            }
        }
        // Everything in flight is consumed here, before the tile loop, so that the
        // compiler has no load of its own pending inside it.
        wait_all(sm);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qB[nt][ks]));
    }
    // Bring in the next item's query rows if they are one contiguous run of at most 16.
    const bool q_next = has_next && rows_in_line(next);
    if (q_next) {
        wait_lgkmcnt0();   // the buffer has been read out
        fetch_rows<D>(a, next, q_base, lane, sm);
    }

    // The softmax denominator is accumulated by the matrix core as well: a V^T row
    // of ones turns the second product into sum_t p_t, taken over the same bf16-
    // rounded weights as the numerator (so numerator and denominator stay consistent).
    u32x4 ones_bits = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    const bf16x8 ones = as_bf16x8(ones_bits);
    f32x4 oacc[NT][NI];
    f32x4 lacc[NT];
    float m_run[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_run[nt] = -INFINITY;
        lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NI; ++i) oacc[nt][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        settle<false>(lacc[nt], oacc[nt]);
    }

    // One tile in two halves.  front(t): wait for the tile, read it out of its stage
    // (handing the stage back for the refill), S^T = K Q^T, and the
    // scaled scores with their per-lane maximum.  back(): weights, denominators and
    // O^T += V^T P^T.  Between the two the reference exponents may have to be raised.
    f32x4 sacc[NT][2]; // S^T of the tile: this lane's 8 tokens (two blocks of 4) per row tile
    float tmax[NT];    // scaled maximum of those, positions past the end left out
    int tile_pos = 0;  // position of the tile's first token
    bool ragged = false;   // the tile reaches past the item's last token (wave-uniform)
    bf16x8 vA[NI];     // vA[i]: head dim 16 i + n, k-slots = the lane group's 8 tokens (4 of each block)
    auto scores = [&](int nt, float (&r)[8]) {   // this lane's 8 scores of row tile nt; -inf past the end
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) r[mt * 4 + jj] = sacc[nt][mt][jj];
        if (__builtin_expect(ragged, 0)) {
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int pos = tile_pos + (x >> 2) * 16 + kg * 4 + (x & 3);
                if (pos >= item.tok_end) r[x] = -INFINITY;
            }
        }
    };
    auto front = [&](int t, auto first) {
        const int stg = (sm.phase + t) & 1;
        const char* st = s_stage + stg * STG;
        wait_for<D / 8>(sm, stg == 0 ? sm.tmark0 : sm.tmark1);   // tile t has landed
        // Read the tile out of its stage and hand the stage back.  With 16 or 32 query
        // rows everything is read up front so that the refill starts at once; with 64
        // rows registers are short, so V is read after the first product (that
        // instantiation computes long enough per tile for the later refill not to matter).
        // V comes out of LDS transposed: the 16 lanes of a group read the group's four token rows, 16 dims of each, and
        // lane n is left with dim n of the four.
        constexpr bool kLate = NT == 4 || D == 256;   // registers are short: K of the second block and V are read after the first product
        bf16x8 kA[kLate ? 1 : 2][KS];
        auto read_v = [&]() {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                typedef short s16x4 __attribute__((ext_vector_type(4)));
                typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
                const uint32_t at = lds_base + stg * STG + 2 * BLK + (L.v_off ^ ((i & 7) * 32)) + (i >> 3) * 256;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)at), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(at + BLK));
                vA[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        auto ask = [&]() {     // (the tile after this one is due only where the look-ahead stopped short of an item of one tile)
            if constexpr (decltype(first)::value)
                if (ntiles == 1) issue(t + 1);
            issue(t + 2);
        };
#pragma unroll
        for (int mt = 0; mt < (kLate ? 1 : 2); ++mt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kA[mt][ks] = as_bf16x8(ld16(st + mt * BLK + L.k_off[ks]));
        if constexpr (!kLate) {
            read_v();
            wait_lgkmcnt0();   // the stage is read out: refill it with stream tile t+2
            ask();
        }

        tile_pos = (item.c0 + 2 * t) * kBlock;
        ragged = tile_pos + kTileTok > item.tok_end;

        // ---- S^T = K Q^T
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sacc[nt][0] = sacc[nt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            if constexpr (kLate) {
                if (mt == 1) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) kA[0][ks] = as_bf16x8(ld16(st + BLK + L.k_off[ks]));
                }
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    sacc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kA[kLate ? 0 : mt][ks], qB[nt][ks], sacc[nt][mt], 0, 0, 0);
        }
        if constexpr (kLate) {
            read_v();
            wait_lgkmcnt0();
            ask();
        }

        // ---- V: zero tokens past the end (they may hold anything)
        if (__builtin_expect(ragged, 0)) {
            u32x4 live;        // the halves of a fragment's registers whose token counts
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int pos = tile_pos + (w >> 1) * 16 + kg * 4 + 2 * (w & 1);
                live[w] = (pos < item.tok_end ? 0xFFFFu : 0u) | (pos + 1 < item.tok_end ? 0xFFFF0000u : 0u);
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) vA[i] = as_bf16x8(__builtin_bit_cast(u32x4, vA[i]) & live);
        }

        // ---- row maxima, one query row per lane (per row tile); the scores themselves stay
        // in the accumulation registers until back() turns them into weights
        bool raise = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float r[8];
            scores(nt, r);
            tmax[nt] = a.scale_log2 *
                fmaxf(fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3])), fmaxf(fmaxf(r[4], r[5]), fmaxf(r[6], r[7])));
            raise = raise || tmax[nt] > m_run[nt] + kSlack;
        }
        return __any(raise);
    };
    // Online softmax.  The running "maximum" is a reference exponent m_ref per row:
    // weights are 2^(s - m_ref).  It is raised to the true row maximum (and l, O
    // rescaled) only when some score exceeds it by more than kSlack, which float32
    // sums absorb without loss; the first tile sets it.  Softmax is shift-invariant, so the result is the same, and the common
    // case costs no cross-lane traffic and no rescale of O.
    auto raise_refs = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (__any(tmax[nt] > m_run[nt] + kSlack)) {
                float rmax = fmaxf(tmax[nt], __shfl_xor(tmax[nt], 16));
                rmax = fmaxf(rmax, __shfl_xor(rmax, 32));
                const float m_new = fmaxf(m_run[nt], rmax);
                const float alpha = exp2_fast(m_run[nt] - m_new);
                scale_acc(lacc[nt], alpha);
#pragma unroll
                for (int i = 0; i < NI; ++i) scale_acc(oacc[nt][i], alpha);
                m_run[nt] = m_new;
            }
        }
    };
    auto back = [&]() {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float neg_m = -m_run[nt];
            float r[8];
            scores(nt, r);
            bf16x8 pB;
#pragma unroll
            for (int x = 0; x < 8; ++x) pB[x] = (__bf16)exp2_fast(fmaf(r[x], a.scale_log2, neg_m));
            add_products(lacc[nt], oacc[nt], ones, vA, pB);
        }
    };
    // First tile: the reference is its row maximum, nothing to rescale yet.
    front(0, std::true_type{});
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float rmax = fmaxf(tmax[nt], __shfl_xor(tmax[nt], 16));
        m_run[nt] = fmaxf(fmaxf(rmax, __shfl_xor(rmax, 32)), kLowest);
    }
    back();
    for (int t = 1; t < ntiles; ++t) {
        if (__builtin_expect(front(t, std::false_type{}), 0)) raise_refs();
        back();
    }

    // ---- partial rows: lane (n, kg) holds, for row 16 nt + n, dims 16 i + 4 kg .. of product i
    const char* ml = sgpr(a.ws + a.lay.ml + (size_t)item.pbase * sizeof(float2));          // the item's first partial row
    const char* pacc = sgpr(a.ws + a.lay.acc + (size_t)item.pbase * (D * sizeof(float)));
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        settle<true>(lacc[nt], oacc[nt]);
        const float l = lacc[nt][0];   // every element of the column holds the row's sum
        const int row = nt * 16 + n;
        if (nt * 16 < item.nrows) {    // wave-uniform: lane 0 has a row here, so all its stores are issued
            if (row < item.nrows) {
                store_row(pacc, (uint32_t)row * (D * 4u) + (uint32_t)kg * 16u, oacc[nt]);
                if (kg == 0) store_f32x2(ml, (uint32_t)row * 8u, m_run[nt], l);
            }
            sm.seq += D / 16 + 1;
        }
    }
    sm.phase = (sm.phase + ntiles) & 1;
    sm.iss -= ntiles;
    const int old0 = sm.cb0;
    sm.cb0 = sm.cbn;   // the next item's first window is already there
    sm.cbn = sm.cb1;
    sm.cb1 = old0;
    sm.cols_ready = has_next;
    sm.q_ready = q_next;
}

// A piece of a shared run swept by a team of 2 or 4 waves of this workgroup, one row tile of up to 64
// query rows per wave, every tile of the piece fetched once for the whole team: the hand-scheduled
// sequences of fea_sweep_core.inc (see gen_sweep_core.py for what they do and why they are written
// out by hand).  Same partial rows as sweep_item.  A sequence uses most of the wave's registers under
// fixed names; the caller ends the wave right after it, so that nothing of the rest of the kernel
// has to live across it.  `team_base`: LDS address of the team's ring (2 x team tiles of K, then of V).
#include "fea_sweep_core.inc"
constexpr int kTeamCols = 1024;   // columns of a piece a team can sweep: their block ids fill the wave's query buffer (4 KB)
__device__ __forceinline__ void sweep_team_core(const SweepArgs& a, const Piece& item, int team, int rank, int g_rcp,
                                                uint32_t team_base, uint32_t tab_base, int lane) {
    // The per-lane inputs are worked out again from a copy of the lane number the compiler cannot
    // see through: they must sit in the few registers the sequence leaves alone, and tying them to
    // the values the rest of the kernel keeps for its whole life would push those into scratch.
    asm volatile("" : "+v"(lane));
    const int n = lane & 15, kg = lane >> 4;
    const uint32_t k_off0 = (uint32_t)(n * 256 + ((kg ^ n) & 15) * 16);             // token row n, chunk kg (k-step 0)
    const int vrow = 4 * kg + (n >> 2);
    const uint32_t v_off0 = (uint32_t)(vrow * 256 + ((((n & 3) >> 1) ^ vrow) & 15) * 16 + (n & 1) * 8);   // token row 4 kg + n / 4, its dims 4 (n % 4) .. (product 0)
    const uint32_t d_off0 = (uint32_t)(kg * 256 + ((n ^ kg) & 15) * 16);            // load 0 of a block: row kg
    const int ntiles = (item.c1 - item.c0) >> 1;
    const int* mlist = reinterpret_cast<const int*>(a.ws + a.lay.members) + item.mlist_off;
    const int32_t* trow = a.bt + (size_t)item.who * a.stride;
    // block ids of all the piece's columns (at most kTeamCols), 64 per load, into this wave's query buffer
    // (not needed here: the sequence keeps the query rows in registers)
    for (int w = 0; w * 64 < item.c1 - item.c0; ++w)
        dma4(sgpr(trow), (uint32_t)min(item.c0 + 64 * w + lane, item.c1 - 1) * 4u, sgpr(tab_base + 256u * (uint32_t)w));
    // byte offset of this lane's part of query row 16 nt + n (rows past the end: the first row again)
    uint32_t qoff[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        int row = nt * 16 + n;
        row = row < item.nrows ? row : 0;
        const int mem = (row * g_rcp) >> 16, hh = row - mem * a.G;
        const int req = item.mlist_off < 0 ? item.who : mlist[mem];
        qoff[nt] = (uint32_t)(((req * a.Hq + item.g * a.G + hh) * kD + kg * 8) * 2);
    }
    wait_vmcnt<0>();
    // this wave's part of every tile: ranks of the lower half fetch K, of the upper half V; in a team of 4 one block each
    const bool loads_v = rank >= team / 2;
    const uint64_t own = reinterpret_cast<uint64_t>(loads_v ? a.v_cache : a.k_cache);
    const uint32_t odd = team == 4 ? (uint32_t)(rank & 1) : 0u;
    const uint32_t own_ring = sgpr((loads_v ? (uint32_t)(2 * team) * (2u * kBlkBytes) : 0u) + odd * kBlkBytes);
    const uint32_t tabsel = sgpr(odd * 4u);
    const uint64_t qbase = reinterpret_cast<uint64_t>(sgpr(a.q));
    const uint64_t accbase = reinterpret_cast<uint64_t>(sgpr(a.ws + a.lay.acc + (size_t)item.pbase * (kD * sizeof(float))));
    const uint64_t mlbase = reinterpret_cast<uint64_t>(sgpr(a.ws + a.lay.ml + (size_t)item.pbase * sizeof(float2)));
    const uint32_t own_lo = sgpr((uint32_t)own), own_hi = sgpr((uint32_t)(own >> 32));
    const uint32_t lane4 = (uint32_t)lane * 4u, dst0 = (uint32_t)n * (kD * 4u) + (uint32_t)kg * 16u;
#define FEA_TEAM_CORE_OPERANDS                                                                                                  \
    : [koff0] "v"(k_off0), [voff0] "v"(v_off0), [doff0] "v"(d_off0), [q0] "v"(qoff[0]), [q1] "v"(qoff[1]), [q2] "v"(qoff[2]),   \
      [q3] "v"(qoff[3]), [lane4] "v"(lane4), [dst0] "v"(dst0), [nrow] "v"(n), [qbase] "s"(qbase), [accbase] "s"(accbase),       \
      [mlbase] "s"(mlbase), [own_lo] "s"(own_lo), [own_hi] "s"(own_hi), [hkv] "s"(sgpr((uint32_t)a.Hkv)),                        \
      [g] "s"(sgpr((uint32_t)item.g)), [ntiles] "s"(sgpr((uint32_t)ntiles)), [nrows] "s"(sgpr((uint32_t)item.nrows)),             \
      [scale] "s"(__builtin_bit_cast(float, sgpr(__builtin_bit_cast(uint32_t, a.scale_log2)))), [team] "s"(sgpr(team_base)),     \
      [tab] "s"(sgpr(tab_base)), [own_ring] "s"(own_ring), [tabsel] "s"(tabsel)                                                   \
    : FEA_TEAM_CORE_CLOBBERS
    if (team == 4) asm volatile(FEA_TEAM4_CORE_ASM : FEA_TEAM_CORE_OPERANDS);
    else asm volatile(FEA_TEAM2_CORE_ASM : FEA_TEAM_CORE_OPERANDS);
#undef FEA_TEAM_CORE_OPERANDS
}

constexpr int kWavesPerGroup = 4;   // one wave per SIMD of a compute unit: a workgroup fills the unit

// Waves per workgroup: four (one per SIMD) - at head_dim 256 two, whose tile stages (2 x 32 KB each) fill the LDS.
template <int D> constexpr int waves_per_group() { return D == 256 ? 2 : kWavesPerGroup; }

// A batch that shares nothing: workgroups take whole histories of a (request, KV head), in the planner's order, and write the
// output.  Wave w of W takes every W-th tile of 32 tokens, two of them in its registers (fea_tile.h): one is worked on while
// the other arrives, and a tile is asked for as soon as the one two before it has been read.  The next history is claimed
// while this one is read.  (A weight enters the second product as two bfloat16 numbers here, the denominator unrounded: 0.7 of
// the shares' error against float64, 0.00166 against 0.00233 for 512 requests of 512 to 4096 tokens, 64/8/128.)
// Every byte is read once, and passes by the caches: 512 requests of 512 to 4096 tokens, 64/8/128, 829 -> 744 us (6.7 TB/s; V
// alone 756), 256 of 512 to 1024, 32/8/128, 148 -> 138 (136).
constexpr int kHistoryRows = 16;
template <int D, int W>
__device__ __forceinline__ void sweep_histories(const SweepArgs& a, char* lds, int* hdr, int wave, int lane) {
    using TileT = tile::Tile<tile::bf16_t, D, kHistoryRows, true>;
    constexpr int TB = TileT::TB, NI = TileT::NI, PN = TileT::PN, BLK = kBlock * D * 2, PAD = D + 4;
    struct alignas(16) Fold { float acc[W][kHistoryRows][PAD]; float2 ml[W][kHistoryRows]; int next; };   // (two in turn: one barrier a history)
    static_assert(2 * sizeof(Fold) <= (size_t)W * kStages * 4 * BLK, "fits the tile stages");
    static_assert(sizeof(Fold) % 16 == 0 && PAD % 4 == 0, "rows of the second one are written 16 bytes at a time as well");
    Fold* folds = reinterpret_cast<Fold*>(lds);
    const int n = lane & 15, kg = lane >> 4, tid = wave * 64 + lane;
    const int units = a.B * a.Hkv;
    const int* order = reinterpret_cast<const int*>(a.ws + a.lay.members);
    int turn = 0;
    for (int unit = blockIdx.x; unit < units; turn ^= 1) {
        Fold& f = folds[turn];
        int claimed = 0;
        if (tid == 0) claimed = (int)gridDim.x + atomicAdd(&hdr[H_QUEUE], 1);
        const int i = min(max(__builtin_amdgcn_readfirstlane(order[unit / a.Hkv]), 0), a.B - 1), g = unit % a.Hkv;   // (in range whatever plan is reused)
        const int32_t* row = a.bt + (size_t)i * a.stride;
        auto ids_from = [&](int t0) {              // lane TB x + b: block b of the x-th tile of this wave from t0 on
            const int col = TB * (t0 + (lane / TB) * W) + lane % TB;
            return row[min(col, a.stride - 1)];
        };
        const int raw_len = a.seq_lens[i];
        int ids = ids_from(wave);
        TileT A, Bt;
        A.load_q(static_cast<const char*>(a.q) + ((size_t)i * a.Hq + g * a.G) * (D * 2), a.G, n, kg);
        const int L = __builtin_amdgcn_readfirstlane(min(max(raw_len, 0), a.stride * kBlock));
        const int nb = (L + kBlock - 1) / kBlock, ntiles = (nb + TB - 1) / TB;
        const int count = (ntiles - wave + W - 1) / W;   // of this wave (its tile k: wave + k W); <= 0: none
        f32x4 o[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m = kLowest, l = 0.f;
        const char* kb[TB];
        const char* vb[TB];
        int base = 0;                              // the tile that lane 0's id belongs to
        auto locate = [&](int k) {
            if (k - base == 64 / TB) {
                ids = ids_from(wave + k * W);
                asm volatile("" : "+v"(ids));      // waited for here, once in 64 blocks
                base = k;
            }
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const int blk = max(__builtin_amdgcn_readlane(ids, TB * (k - base) + (TB * (wave + k * W) + b < nb ? b : 0)), 0);
                const size_t off = ((size_t)blk * a.Hkv + g) * BLK;
                kb[b] = static_cast<const char*>(a.k_cache) + off;
                vb[b] = static_cast<const char*>(a.v_cache) + off;
            }
        };
        auto ask_k = [&](TileT& t) {
#pragma unroll
            for (int b = 0; b < TB; ++b) t.load_k(b, kb[b], n, kg);
        };
        auto ask_v = [&](TileT& t) {
#pragma unroll
            for (int b = 0; b < TB; ++b) t.load_v(b, vb[b], n, kg);
        };
        auto scores = [&](TileT& t, float (&p)[PN]) {
#pragma unroll
            for (int j = 0; j < TileT::KC; ++j) t.q[j] = A.q[j];
            t.scores(p);
        };
        auto step = [&](TileT& t, int k) {         // tile k, and tile k + 2 asked for
            float p[PN];
            scores(t, p);
            locate(k + 2);
            ask_k(t);
            tile::weigh<TileT, tile::bf16_t>(p, o, m, l, a.scale_log2);
            t.accumulate(p, o, n);
            ask_v(t);
            asm volatile("; tile asked for" ::: "memory");
        };
        auto last = [&](TileT& t, int k) {
            float p[PN];
            scores(t, p);
            const int rest = L - (wave + k * W) * (TB * kBlock);
            if (rest < TB * kBlock) t.mask(p, rest, n, kg);
            tile::weigh<TileT, tile::bf16_t>(p, o, m, l, a.scale_log2);
            t.accumulate(p, o, n);
        };
        if (count > 0) {
            locate(0);
            ask_k(A);
            ask_v(A);
            asm volatile("; first tile asked for" ::: "memory");
            if (count > 1) {
                locate(1);
                ask_k(Bt);
                ask_v(Bt);
                asm volatile("; second tile asked for" ::: "memory");
                int k = 0;
                for (; k + 3 < count; k += 2) {
                    step(A, k);
                    step(Bt, k + 1);
                }
                if (count - k == 3) {
                    step(A, k);
                    last(Bt, k + 1);
                    last(A, k + 2);
                } else {
                    last(A, k);
                    last(Bt, k + 1);
                }
            } else {
                last(A, 0);
            }
            if (__builtin_expect(__any(tile::any_nan(o)), 0)) tile::sweep_apart<TileT, D>(A, o, m, l, a, row, g, L, wave, 1, W, n, kg);
        }
        TileT::template to_lds<PAD>(f.acc[wave], o, a.G, n, kg);
        l = TileT::row_sum(l);
        if (TileT::one_of_row(n, kg)) f.ml[wave][TileT::head(n)] = make_float2(m, l);
        if (tid == 0) f.next = claimed;
        __syncthreads();
        unit = __builtin_amdgcn_readfirstlane(f.next);
        for (int y = tid; y < a.G * (D / 8); y += 64 * W) {
            const int h = y / (D / 8), c = y - h * (D / 8);
            float M, den, num[8];
            tile::fold_waves(f.acc, f.ml, h, c, M, den, num);
            const float inv = L == 0 ? 0.f : 1.f / den;   // an empty history gives a zero row, one of scores of -inf alone 0/0
            u32x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = bf16_rne(num[2 * e] * inv) | (bf16_rne(num[2 * e + 1] * inv) << 16);
            *reinterpret_cast<u32x4*>(static_cast<char*>(a.out) + ((size_t)i * a.Hq + g * a.G + h) * (D * 2) + 16 * c) = w;
        }
    }
}

template <int D>
__global__ __launch_bounds__(64 * waves_per_group<D>()) void sweep_mfma_kernel(SweepArgs a, int g_rcp, int xcd_aware) {
    constexpr int WPG = waves_per_group<D>();
    constexpr int STG = 4 * kBlock * D * 2;          // bytes of a tile stage: K b0 | K b1 | V b0 | V b1
    // Every wave sweeps a share of its own and owns a quarter of the workgroup's LDS; the waves of a
    // workgroup never wait for one another on this path.  (They sit in one workgroup so that the row
    // tiles of a shared run's piece, which read the same KV bytes, can share what is fetched.)
    __shared__ __attribute__((aligned(1024))) char s_stage_all[WPG * kStages * STG];
    __shared__ __attribute__((aligned(256))) int s_cols_all[WPG * 3 * 64];
    __shared__ __attribute__((aligned(256))) int s_desc_all[WPG * kDescWindow * 8];     // the next few item descriptors
    __shared__ __attribute__((aligned(1024))) char s_q_all[WPG * kBlock * (D < 128 ? 128 : D) * 2];   // query rows of the next item (at least 4 KB per wave: a team keeps its block ids there)
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    char* s_stage = s_stage_all + wv * (kStages * STG);
    int* s_cols = s_cols_all + wv * (3 * 64);
    int* s_desc = s_desc_all + wv * (kDescWindow * 8);
    char* s_q = s_q_all + wv * (kBlock * (D < 128 ? 128 : D) * 2);
    int* hdr = reinterpret_cast<int*>(a.ws);
    const Item* items = reinterpret_cast<const Item*>(a.ws + a.lay.items);
    // Which shares this wave sweeps: share, share + grid, ...  Workgroups are dealt
    // round-robin to the 8 XCDs (workgroup id mod 8), each with its own L2, while
    // consecutive shares of a shared run are its row tiles over the same KV bytes.
    // Put every 8 consecutive shares on one XCD so that those bytes are fetched into
    // one L2 once.  (Pure performance: any permutation is correct.)
    int group = blockIdx.x;
    if (xcd_aware) {
        const int x = blockIdx.x & 7, k = blockIdx.x >> 3;
        group = 2 * ((k >> 1) * 8 + x) + (k & 1);
    }
    int share = WPG * group + wv;
    // (arguments, then header and first items: each in one round trip to memory, not word by word - four in line before the first
    // descriptor can be asked for)
    const int* wave_first = reinterpret_cast<const int*>(a.ws + a.lay.wave_first);
    FEA_TOGETHER(share, a.lay.items, a.q, a.stride);
    int n_items = hdr[H_ITEMS], first_item = wave_first[share];
    const int variant = hdr[H_VARIANT], made = hdr[H_WAVES], histories = hdr[H_HISTORIES], first_end = wave_first[share + 1];
    asm("" : "+s"(n_items), "+s"(first_item) : "s"(variant), "s"(made), "s"(histories), "s"(first_end));
    const int n_shares = variant == kNoPlan ? 0 : made;   // (a reused plan that is none: nothing is swept, the merge reports it)
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)s_stage);
    const uint32_t cols_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)s_cols);
    const uint32_t desc_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)s_desc);
    const uint32_t q_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)s_q);

    Lanes L;
    L.n = lane & 15;
    L.kg = lane >> 4;
    {
        const int row = 4 * L.kg + (L.n >> 2), sub = (L.n & 3) >> 1;   // chunk 2 i + sub of the row holds the lane's dims of product i
        L.v_off = row * (D * 2) + ((sub ^ row) & (D == 64 ? 7 : 15)) * 16 + (L.n & 1) * 8;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (D == 128) {
            const int row = 4 * (i & 3) + L.kg;                    // token row of the block this lane fetches in load i
            L.dma_off[i] = L.kg * 256 + ((L.n ^ row) & 15) * 16;   // LDS chunk position n receives global chunk n ^ row
            L.k_off[i] = L.n * 256 + (((4 * (i & 3) + L.kg) ^ L.n) & 15) * 16;   // token row n, chunk 4 ks + kg
        } else if constexpr (D == 64) {
            // head_dim 64: 128-byte token rows of 8 chunks, eight rows per load; position p of row r holds chunk p ^ (r % 8)
            const int row = lane >> 3, pos = lane & 7;
            L.dma_off[i] = row * 128 + ((pos ^ row) & 7) * 16;     // (both loads)
            L.k_off[i] = L.n * 128 + (((4 * (i & 1) + L.kg) ^ L.n) & 7) * 16;   // token row n, chunk 4 ks + kg (k-steps 0 and 1)
        } else {
            // head_dim 256: 512-byte token rows of 32 chunks, two rows per load; each half of a row is swizzled like a
            // 256-byte row (position p of row r holds chunk (p & 16) | ((p ^ r) & 15)); dims 128 on sit 256 bytes on
            const int row = 2 * i + (lane >> 5), pos = lane & 31;
            L.dma_off[i] = (lane >> 5) * 512 + ((pos & 16) | ((pos ^ row) & 15)) * 16 + (i >> 2) * 4096;
            const int c = 4 * i + L.kg;                                          // chunk of k-step i
            L.k_off[i] = L.n * 512 + ((c & 16) | ((c ^ L.n) & 15)) * 16;
        }
    }

    // Item descriptors come through LDS too, kDescWindow at a time (one load of 4
    // bytes per lane); a descriptor is made wave-uniform (scalar registers) when it
    // is taken out of the window.
    auto fetch_desc = [&](int first, Stream& sm) {
        dma4(sgpr(items), (uint32_t)min(first * 8 + lane, n_items * 8 - 1) * 4u, desc_base);
        sm.seq += 1;
    };
    int team = 0, rank = 0;   // of the descriptor read last: team size (0: a wave on its own) and rank of a shared run's piece
    auto read_desc = [&](int k) {
        const int4* p = reinterpret_cast<const int4*>(s_desc + k * 8);
        const int4 w0 = p[0], w1 = p[1];
        auto u = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
        Piece x;
        const int gt = u(w0.y);
        team = (gt >> 16) & 15;
        rank = (gt >> 20) & 15;
        x.who = u(w0.x); x.g = gt & 0xFFFF; x.once = gt & kOnce; x.nrows = u(w0.z); x.mlist_off = u(w0.w);
        x.c0 = u(w1.x); x.c1 = u(w1.y); x.pbase = u(w1.z); x.tok_end = u(w1.w);
        return x;
    };

    const int n_waves = WPG * (int)gridDim.x;
    if constexpr (D != 256) {   // (two tiles of 256 dims would spill)
        if (__builtin_expect(histories != 0, 0)) {   // (placed behind the rest: the other way must not fetch its instructions)
            sweep_histories<D, WPG>(a, s_stage_all, hdr, wv, lane);
            return;
        }
    }
    for (int it_of_share = first_item, end_of_share = first_end; share < n_shares;) {
        int it = it_of_share;
        const int it_end = min(n_items, end_of_share);
        share += n_waves;
        if (share < n_shares) {
            it_of_share = __builtin_amdgcn_readfirstlane(wave_first[share]);
            end_of_share = __builtin_amdgcn_readfirstlane(wave_first[share + 1]);
        }
        if (it >= it_end) continue;
        wait_vmcnt<0>();   // nothing of an earlier share is still on its way into LDS
        wait_lgkmcnt0();
        Stream sm;
        sm.phase = 0;
        sm.iss = 0;
        sm.cb0 = 0; sm.cb1 = 1; sm.cbn = 2;
        sm.cols_ready = false;
        sm.q_ready = false;
        sm.seq = sm.done = 0;
        sm.tmark0 = sm.tmark1 = sm.cmark0 = sm.cmark1 = sm.cmark2 = sm.qmark = 0;
        int win_first = it;
        fetch_desc(win_first, sm);
        wait_all(sm);
        Piece item = read_desc(0);
        // A piece of a shared run as this wave's only work, its row tiles on the neighbouring waves of this
        // workgroup: the team sweeps it together if it qualifies (every member sees the same columns, so
        // they all decide alike).  Members without rows of their own only take part in that.
        if constexpr (D == 128) {   // (the team sequence is written for head_dim 128)
            if (a.fast_shared && team >= 2 && it + 1 == it_end && share >= n_shares &&
                ((item.c1 - item.c0) & 1) == 0 && item.c1 - item.c0 >= 8 && item.c1 - item.c0 <= kTeamCols &&
                item.tok_end == item.c1 * kBlock && (wv & (team - 1)) == rank) {
                wait_lgkmcnt0();
                const uint32_t ring = sgpr((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)s_stage_all) +
                                      (team == 2 ? (uint32_t)(wv >> 1) * (2u * kStages * kStageBytes) : 0u);
                sweep_team_core(a, item, team, rank, g_rcp, ring, q_base, lane);
                __builtin_amdgcn_endpgm();   // (not `return`: control must not rejoin the loop, or the loop's values live across the sequence)
            }
        }
        if (item.nrows == 0 && it + 1 == it_end) continue;   // a slot that only exists for a team (or a filler)
        // The first item's query rows ahead of its tiles, so that not everything asked for has to be there before the first product:
        // 48 requests of head_dim 256 on 3000 tokens 44.6 -> 44.0 us, 128 of head_dim 64 in 8 groups 47.5 -> 47.0.  Not at head_dim 128:
        // beside teams, which are on their way then, it took 1.01 to 1.02 of the time (64 on 4096 48.9 -> 49.8; without any, 0.99).
        if constexpr (D != 128)
            if (rows_in_line(item) && item.nrows > 0) {
                fetch_rows<D>(a, item, q_base, lane, sm);
                sm.q_ready = true;
            }
        for (;;) {
            const bool has_next = it + 1 < it_end;
            if (has_next && it + 1 - win_first == kDescWindow) {   // window used up: fetch the next one (drains the stream once)
                wait_lgkmcnt0();
                win_first = it + 1;
                fetch_desc(win_first, sm);
                wait_all(sm);
            }
            const Piece next = has_next ? read_desc(it + 1 - win_first) : item;
            if (item.nrows <= 16) sweep_item<1, D>(a, item, next, has_next, g_rcp, s_stage, s_cols, s_q, lds_base, cols_base, q_base, L, lane, sm);
            else if (D == 256 || item.nrows <= 32) sweep_item<2, D>(a, item, next, has_next, g_rcp, s_stage, s_cols, s_q, lds_base, cols_base, q_base, L, lane, sm);   // (head_dim 256: the planner makes no item of more than 32 rows)
            else sweep_item<(D == 256 ? 2 : 4), D>(a, item, next, has_next, g_rcp, s_stage, s_cols, s_q, lds_base, cols_base, q_base, L, lane, sm);
            if (!has_next) break;
            ++it;
            item = next;
        }
    }
}

void launch_sweep_mfma(const SweepArgs& a, int head_dim, int grid, const Launch& L) {
    const int g_rcp = (65536 + a.G - 1) / a.G;   // (row * g_rcp) >> 16 == row / G for the 64 rows of an item
    static const int by_xcd = [] { const char* v = std::getenv("FEA_XCD_AWARE"); return v && *v ? std::atoi(v) : 1; }();
    const int xcd_aware = by_xcd && (grid / (head_dim == 256 ? 2 : 4)) % 16 == 0;   // (of whole sets of two workgroups for each XCD)
    hipStream_t st = static_cast<hipStream_t>(L.stream);
    hipEvent_t e0 = static_cast<hipEvent_t>(L.ev_start), e1 = static_cast<hipEvent_t>(L.ev_stop);
    if (head_dim == 64) hipExtLaunchKernelGGL(sweep_mfma_kernel<64>, dim3(grid / 4), dim3(256), 0, st, e0, e1, 0, a, g_rcp, xcd_aware);
    else if (head_dim == 256) hipExtLaunchKernelGGL(sweep_mfma_kernel<256>, dim3(grid / 2), dim3(128), 0, st, e0, e1, 0, a, g_rcp, xcd_aware);
    else hipExtLaunchKernelGGL(sweep_mfma_kernel<128>, dim3(grid / 4), dim3(256), 0, st, e0, e1, 0, a, g_rcp, xcd_aware);
}

}  // namespace fea
