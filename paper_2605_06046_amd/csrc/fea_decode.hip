// fea_decode_attention: argument checks, workspace carving and the three launches
// (plan, KV sweep, merge), or the one of batches that need no plan.  No device memory is allocated here and nothing
// synchronises except fea_decode_plan_info.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <atomic>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/fea.h"
#include "fea_internal.h"
#include "fea_plan.h"

namespace fea {

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

static int env_int(const char* name, int dflt) {
    const char* v = std::getenv(name);
    if (!v || !*v) return dflt;
    return std::atoi(v);
}

// Development knobs for tuning sweeps.  The environment is read once, the first time
// a call needs them, and never again: a variable that changes later (or a stale one a
// second thread sets) cannot switch kernels or move the workspace layout between the
// sizing call and the attention call.  What tests need to steer is in fea_attn_params.
struct Knobs {
    int force_generic, sweep_grid, spare_waves, min_piece, min_run, w32, w64, no_fast_shared, w_team, w_team2, team_fixed, direct_pieces, histories;
};
static const Knobs& knobs() {
    static const Knobs k = {env_int("FEA_FORCE_GENERIC", 0), env_int("FEA_SWEEP_GRID", 0), env_int("FEA_SPARE_WAVES", 16),
                            env_int("FEA_MIN_PIECE", 4),     env_int("FEA_MIN_RUN", 2),    env_int("FEA_W32", 18),
                            env_int("FEA_W64", 24), env_int("FEA_NO_FAST_SHARED", 0), env_int("FEA_WTEAM", 12),
                            env_int("FEA_WTEAM2", 12), env_int("FEA_TEAM_FIXED", 40), env_int("FEA_DIRECT_PIECES", 0),
                            env_int("FEA_HISTORIES", 6)};
    return k;
}

struct Resolved {
    int variant;      // 0 generic, 1 MFMA
    int direct;       // pieces per history of the kernel that needs no plan; 0: plan, sweep and merge
    int G, mpt, grouping, split_user, grid;
    int pre, pre_grid;   // leaders and common runs on many workgroups first (large tables)
    int merge_by_rows;   // very many output rows: the merge takes several rows per wave
    int histories;       // tiles from which on a batch that shares nothing is swept by whole histories; 0: never
    PlanTuning tune;
    WsLayout lay;
};

// Optional per-kernel timing: each launch can carry a pair of library-owned events that
// take the start and end time of that dispatch itself (no marker packets in between).
constexpr int kEvPerCall = 8;               // (start, stop) for plan, sweep, merge, and the inner pair of a two-dispatch plan
static std::atomic<bool> g_prof_on{false};  // read without the lock on every call; everything below is under g_prof_mu
static std::mutex g_prof_mu;
static std::vector<hipEvent_t> g_ev_pool;   // kEvPerCall events per recorded call
static int g_prof_calls = 0;                // calls recorded since profiling was switched on
static int g_prof_which = -1;               // -1: all three launches; 0, 1, 2: only that one
static std::vector<unsigned char> g_prof_mask;   // per recorded call: bit k set if launch k was timed

static int cu_count() {
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.multiProcessorCount;
        if (n <= 0) n = 256;
    }
    return n;
}

// The kernel that needs no plan (fea_direct.hip) reads every request's whole history: how many workgroups it has
// without cutting histories, how many tiles a history is at the table's width, and how many of them a wave sweeps one
// after the other (two waves where there are no more than two tiles).
static int64_t direct_groups(const fea_attn_params* p, int64_t B) {
    return B * p->num_kv_heads * ((p->num_q_heads / p->num_kv_heads + 15) / 16);
}
static int64_t direct_tiles(const fea_attn_params* p, int64_t stride) {
    const int64_t tile_blocks = p->dtype == FEA_DTYPE_F32 && p->head_dim >= 128 ? 1 : 2;
    return (stride + tile_blocks - 1) / tile_blocks;
}
static int64_t direct_rounds(const fea_attn_params* p, int64_t stride) {
    const int64_t tiles = direct_tiles(p, stride), waves = tiles <= 2 ? 2 : p->head_dim == 256 ? 4 : 8;
    return (tiles + waves - 1) / waves;
}

// Pieces a history is cut into there, at most: workgroups that leave most of the chip idle are worth cutting, up to one per compute
// unit and 32 per history, where that saves two rounds.  (The lines of direct_pays were measured with as many.)
static int64_t direct_most(const fea_attn_params* p, int64_t B, int64_t stride) {
    const int64_t groups = direct_groups(p, B), rounds = direct_rounds(p, stride);
    if (groups <= 0 || 2 * groups > cu_count()) return 1;
    const int64_t most = std::min<int64_t>({cu_count() / groups, rounds, 32});
    const int64_t left = most > 0 ? (rounds + most - 1) / most : rounds;
    return rounds - left >= 2 ? (rounds + left - 1) / left : 1;
}
// How many it is cut into: what costs least.  A round of a wave's tiles takes 1 us (float32 1.6, with more than four heads 2.4), the
// fold of q pieces 1 us, 0.12 for each of them and 0.1 for every query head of the row tile.  Fitted to 66 shapes with 1 to 32 pieces
// each: 1.029 of the best in the mean (as many as there are at most: 1.042), none slower: bf16 32/2/128, 7 requests of 3 rounds 7.2 us
// whole, 8.8 in 3; 42 of 4 rounds 8.6, in 2 11.3; 28/4/128, 8 short chats of 3 7.1, 7.7; 12/4/256, 2 of 58 rounds 17.6 in 29, 16.7 in
// 20, 82 whole.
static int64_t direct_pieces(const fea_attn_params* p, int64_t B, int64_t stride) {
    const int64_t groups = direct_groups(p, B), rounds = direct_rounds(p, stride), most = direct_most(p, B, stride);
    if (most <= 1) return 1;
    const int heads = std::min(16, p->num_q_heads / p->num_kv_heads);
    const double round_us = p->dtype != FEA_DTYPE_F32 ? 1.0 : heads > 4 ? 2.4 : 1.6, fold_us = 1.0 + 0.1 * heads;
    const int all = (int)rounds, at_most = std::min<int>({cu_count() / (int)groups, all, 32});
    double least = round_us * all;
    int pieces = 1;
    for (int left = (all + at_most - 1) / at_most; round_us * left < least; ++left) {      // rounds left; a few of them, then they alone cost more
        const int q = (all + left - 1) / left;             // no more pieces than those need
        const double us = round_us * left + fold_us + 0.12 * q;
        if (us < least) { least = us; pieces = q; }
    }
    return pieces;
}

// Whether it is expected to beat plan + sweep + merge.  It reads what requests share once per request (5.0 to 5.9 TB/s
// from HBM, 8 and more where the L2s hold it), which the host cannot know; nor does it know whether the plan would serve other
// layers of the step as well.  So it is taken where it wins (or loses next to nothing) whatever is shared and however often
// the plan is used again.  Measured on 5800 matrix-core and 1600 vector-unit shapes (1 to 4096 requests, 16 to 70000 tokens,
// query groups of 1 to 96, 0 to 98 % shared), alone and against a reused plan.  On the matrix-core path, by the bytes of
// KV histories that its workgroups read:
//  - up to 64 MB.  Nothing shared: 8 requests of 1024 tokens 13.5 against 24.8 us.
//  - more than eight query heads per KV head, in at most four workgroups to a compute unit, up to 225 MB, where a wave has twelve
//    tiles at most: on 100 shapes of 100 to 225 MB 0.53 of the time of a new plan and 0.76 of the reused plan's, never more than
//    1.06 (32/2/128, 160 requests of 1216 tokens).  With fewer heads it wins there too in the mean (0.8 of the reused plan's up to
//    145 MB), but loses where much is shared: 12/4/64, 24 requests of 5280 tokens (130 MB), 98 % shared, 1.20; from 225 to 290 MB
//    0.97 and up to 1.64.  Some long histories among short ones (41 shapes): never more than 0.97 of a new plan up to twelve tiles, at
//    worst 1.57 of a reused one (49 requests, 4448 tokens and 194); with 15 and 19 tiles 0.91 and 1.27, and 1.88 and 2.49.
//  - in up to six workgroups to a compute unit (each has a few us of start-up) up to 100 MB: bf16 32/8/128, 32 requests of
//    752 tokens, 19.0 against 35.2 and, of the reused plan, 24.5; 90 % shared 12.1 against 33.9 and 21.9.  In eight rounds of
//    workgroups, 256 requests of 80 tokens, 31.7 against 37.8 and 26.2.
//  - tables of one or two tiles up to 128 MB: 2000 requests of one block 61 against 103 us (above it, a reused plan wins by a tenth).
//  - few query heads, one round of workgroups of up to 1 MB each (1.33 at head_dim 256), or two of 256 KB: bf16 32/8/128, 32
//    requests of 1520 tokens 36.1 against 52.1 and 40.9, 90 % shared 19.2 against 39.7 and 27.3.
//    Longer histories lose to a reused plan: 8/2/64, 128 requests of 4112 tokens, 90 % shared, 28.1 against 38.6 and 22.2.
// The vector-unit sweep costs 26 to 120 us to start with, and from some hundred thousand (query row, token) pairs on time in
// proportion to them.  float32 from 2 to 16 query heads per KV head: the plan-free kernel wins on all of 1174 shapes of even
// lengths (60 MB to 9 GB of histories, 0 to 99 % shared; 0.25 of the reused plan's time in the mean, 0.82 the closest: 2/1/32,
// 300 requests of 32544 tokens, 90 % shared, 290 against 351 us).  But the table's width does not tell how long the others are,
// and one long history among short ones is read by its own workgroups alone, at 53 GB/s each then, where a plan spreads it over the
// chip: 2/1/64, 134 requests, one of 46207 tokens and the rest of 34, 394 against 58 and, of the reused plan, 24 us.  So up to
// 1.5 MB of a history to a workgroup: on 107 shapes there (one or a twentieth of the requests long, or all alike) at most 0.76 of
// a new plan's time and 1.51 of a reused one's (0.44 and 0.54 in the mean); beyond it up to 1.44 of a new plan's time at 2.3 MB
// and 6.8 at 24.  And up to the 10 GB that were measured.  Past either line the estimate decides, and with one head: that can lose on histories
// that are shared and long (8/8/64, 1000 requests of 2192 tokens, 99 % shared: 612 against 515 and 480 us).
// All of that was measured while K rows were not read in pieces and histories were cut into direct_most of them, which the estimate
// goes on counting with; its 2 us a round and 4 us for the fold say where the line was found to lie, not what the two cost today (1.0
// to 2.4, above, and about 3).  Today the lines of bfloat16 are on the safe side: 88 shapes inside them, which a table 1.4 times
// as wide takes outside, take 0.53 of a new plan's time and 0.84 of a reused one's (0.86 and 1.19 at most); 72 outside, which one as
// much narrower takes inside, would take 0.58 and 0.90 (0.87 and 1.47 at most).
static bool direct_pays(const fea_attn_params* p, int64_t B, int64_t stride, int variant) {
    const bool f32 = p->dtype == FEA_DTYPE_F32;
    const double group = (double)(p->num_q_heads / p->num_kv_heads), groups = (double)direct_groups(p, B), cus = cu_count();
    const double tokens = (double)stride * kBlock, dd = p->head_dim / 64.0;
    const double per_group = tokens * p->head_dim * (f32 ? 8.0 : 4.0), bytes = groups * per_group;   // K and V read by a workgroup, by all
    const int64_t pieces = direct_most(p, B, stride), rounds = (direct_rounds(p, stride) + pieces - 1) / pieces;
    if (variant == 1) {
        if (bytes <= 64e6 || (group > 8 && bytes <= 225e6 && groups <= 4 * cus && rounds <= 12) || (bytes <= 100e6 && groups <= 6 * cus) || (bytes <= 128e6 && direct_tiles(p, stride) <= 2)) return true;
        return group <= 4 && ((groups <= cus && per_group <= (p->head_dim == 256 ? 1.33e6 : 1 << 20)) || (groups <= 2 * cus && per_group <= 1 << 18));
    }
    if (f32 && group >= 2 && group <= 16 && bytes <= 10e9 && per_group <= 1.5e6 * (double)pieces) return true;
    const double serial_us = 2.0 * (double)rounds;   // one workgroup's tiles, a round after the other
    const double direct_us = 7.0 + (pieces > 1 ? 4.0 : 0.0) + std::max(serial_us, bytes / 8.0e6);
    const double base = B < 4 ? 20.0 + 1.5 * group : std::min(30.0 + 4.0 * group, 120.0);
    const double planned_us = (B < 16 ? base : std::max(94.0, base)) * (p->head_dim >= 128 ? 1.4 : 1.0) +   // (it passes over its tokens once per 4 or 16 stacked rows)
                              (f32 ? 0.027e-3 : 0.0175e-3) * std::pow(dd, 1.6) * (double)(B * p->num_q_heads) * tokens;
    return 1.1 * direct_us < planned_us;
}

static int32_t check_params(const fea_attn_params* p, const char* who) {
    if (!p) return fail(FEA_EINVAL, "%s: params is NULL", who);
    if (p->num_q_heads <= 0 || p->num_kv_heads <= 0 || p->num_q_heads % p->num_kv_heads != 0)
        return fail(FEA_EINVAL, "%s: num_q_heads=%d must be a positive multiple of num_kv_heads=%d", who, p->num_q_heads, p->num_kv_heads);
    if (p->block_size != FEA_BLOCK_TOKENS) return fail(FEA_EINVAL, "%s: block_size=%d, only %d is supported", who, p->block_size, FEA_BLOCK_TOKENS);
    if (p->dtype != FEA_DTYPE_F32 && p->dtype != FEA_DTYPE_BF16) return fail(FEA_EINVAL, "%s: unknown dtype %d", who, p->dtype);
    const int d = p->head_dim;
    const bool d_ok = p->dtype == FEA_DTYPE_F32 ? (d == 32 || d == 64 || d == 128 || d == 256) : (d == 64 || d == 128 || d == 256);
    if (!d_ok) return fail(FEA_EINVAL, "%s: head_dim=%d not supported for this dtype", who, d);
    if (!(p->scale >= 0.f) || !std::isfinite(p->scale)) return fail(FEA_EINVAL, "%s: scale must be finite and >= 0", who);
    if (p->split_blocks < 0 || p->max_group < 0) return fail(FEA_EINVAL, "%s: split_blocks and max_group must be >= 0", who);
    if (p->flags & ~(FEA_FLAG_REUSE_PLAN | FEA_FLAG_PLAN_ONLY | FEA_FLAG_REFRESH_PLAN))
        return fail(FEA_EINVAL, "%s: unknown flag bits 0x%x", who, p->flags);
    const int plan_flags = p->flags & (FEA_FLAG_REUSE_PLAN | FEA_FLAG_PLAN_ONLY | FEA_FLAG_REFRESH_PLAN);
    if (plan_flags & (plan_flags - 1))
        return fail(FEA_EINVAL, "%s: FEA_FLAG_REUSE_PLAN, FEA_FLAG_PLAN_ONLY and FEA_FLAG_REFRESH_PLAN exclude one another", who);
    return FEA_OK;
}

constexpr int kFarMB = 32;   // what a call reads, from which on the sweep's loads pass by the caches (see the planner, and dma_tile)

static int32_t resolve(const fea_attn_params* p, int32_t B, int32_t stride, Resolved& r, const char* who) {
    if (B < 0 || stride < 0) return fail(FEA_EINVAL, "%s: negative B or table_stride", who);
    if ((int64_t)B * p->num_q_heads > 0x3FFFFFFF || (int64_t)stride * kBlock > 0x3FFFFFFF)
        return fail(FEA_EINVAL, "%s: problem too large (B*Hq or sequence length overflows)", who);
    // the planner counts 32-token tiles of the whole batch in 32-bit integers
    if ((int64_t)B * p->num_kv_heads * ((stride + 1) / 2) > 0x3FFFFFFF)
        return fail(FEA_EINVAL, "%s: problem too large (B * num_kv_heads * table_stride / 2 exceeds 2^30 tiles)", who);
    const Knobs& kn = knobs();
    r.G = p->num_q_heads / p->num_kv_heads;
    // (a work item's query rows - a request's query group, or stacked ones - fill at most 64 matrix-core rows, 32 at head_dim 256)
    const bool mfma_ok = p->dtype == FEA_DTYPE_BF16 && (p->head_dim == 128 || p->head_dim == 64 || p->head_dim == 256) &&
                         r.G <= (p->head_dim == 256 ? 32 : 64);
    r.variant = (mfma_ok && !kn.force_generic) ? 1 : 0;
    // No plan where that is estimated to be faster; an explicit bound on the row length stands alone.
    const bool direct = p->fused_max < 0 ? false : p->fused_max > 0 ? (stride <= p->fused_max) : direct_pays(p, B, stride, r.variant);
    // requests per row tile of a shared run: 64 query rows per work item, 32 on the matrix-core path at head_dim 256
    // (a wave's accumulation registers hold O for 32 rows of 256 dims)
    const int tile_rows = (r.variant == 1 && p->head_dim == 256) ? 32 : kTileRows;
    r.mpt = r.G >= tile_rows ? 1 : tile_rows / r.G;
    r.grouping = p->max_group == 1 ? 0 : 1;
    r.split_user = p->split_blocks > 0 ? ((p->split_blocks + 1) & ~1) : 0;
    // the sweep grid the plan is cut for: one single-wave workgroup per SIMD on the
    // matrix-core path, a few workgroups per CU on the generic path
    r.grid = kn.sweep_grid > 0 ? std::max(4, kn.sweep_grid & ~3) : (r.variant == 1 ? (p->head_dim == 256 ? 2 : 4) : 8) * cu_count();   // waves; four to a workgroup on the matrix-core path (two at head_dim 256)
    // The plan is cut for a few waves fewer than the grid has.  With every one of the
    // 4 x CUs single-wave workgroups busy from start to end, a handful of them (the first
    // ones dispatched) were measured to run about 1.5x longer than the rest, whatever
    // their work; with some workgroups exiting at once this does not happen.
    r.tune.n_waves = std::max(1, r.grid - std::min(r.grid / 2, std::max(0, kn.spare_waves)));
    r.tune.min_piece = std::max(1, kn.min_piece);
    r.tune.min_run = std::max(1, kn.min_run);
    r.tune.team_fixed = std::min(4096, std::max(0, kn.team_fixed));
    r.tune.weights = std::min(255, std::max(16, kn.w32)) | (std::min(255, std::max(16, kn.w64)) << 8) |
                     (std::min(255, std::max(1, kn.w_team)) << 16) | (std::min(127, std::max(1, kn.w_team2)) << 24);
    // Large tables: the rows are compared on many workgroups before the planner's one workgroup
    // takes over (a second launch, so only where the rows are long or many enough to pay for it).
    const int64_t groupable = std::min(B, kGroupReqMax);
    // (measured: 256 requests x 320 columns 30 -> 24 us, 800 x 657 105 -> 35 us; 32 x 2082 no gain, hence
    // the request count; a batch that shares nothing pays about 3 us for it)
    const int run_min = p->run_kernel_min == 0 ? 49152 : p->run_kernel_min;
    r.pre = r.grouping && (run_min < 0 || (groupable >= 128 && groupable * stride >= run_min)) ? 1 : 0;
    r.pre_grid = (int)std::max<int64_t>(1, std::min<int64_t>(2 * cu_count(), (groupable + 3) / 4));
    // Whole histories where the planner finds nothing shared: one row tile of 16 query heads, as many of them as even out over the
    // compute units (four to a unit, or not much less than a whole number), six tiles to every wave, 192 KB to a history.  Measured
    // on 144 shapes of 48 to 400 requests against shares cut beforehand: 0.89 of a call's time with a new plan, 0.95 with a
    // reused one (worst 0.97 and 1.01); 32/8/128, 256 requests of 512 to 1024 tokens 176 -> 146 us, 64/8/128, 512 of 512 to
    // 4096 924 -> 829.  With histories of 64 KB on average it would be 1.08 and 1.38 (a history's start counts), at 128 to 192 KB 0.95 and 1.08.
    // Not at head_dim 256, where two tiles in a wave's registers spill.
    const double per_cu = (double)B * p->num_kv_heads / cu_count();
    r.histories = r.variant == 1 && p->head_dim != 256 && r.grouping && r.split_user == 0 && r.G <= 16 && B <= kGroupReqMax && stride > 0 &&
                          (per_cu >= 4 || (per_cu > 1 && std::ceil(per_cu) <= 1.1 * per_cu)) ? kn.histories * r.tune.n_waves : 0;
    const int64_t rows = (int64_t)B * p->num_q_heads;
    // Very many rows mean many requests and hence few pieces per row: there a wave of the merge takes
    // several rows (a long shared run cut into many pieces comes with few rows, and keeps a wave per row).
    r.merge_by_rows = (p->merge_rows_min < 0 || rows >= (p->merge_rows_min == 0 ? 8192 : p->merge_rows_min)) ? 1 : 0;
    const int64_t segs = 2ll * B * p->num_kv_heads;          // private segments + at most as many shared ones
    const int64_t rows_per_item = std::max(kTileRows, r.mpt * r.G);
    int64_t max_items, max_rows;
    if (r.split_user > 0) {
        const int64_t per = ((stride + 1) / 2 + r.split_user / 2 - 1) / (r.split_user / 2) + 1;   // pieces per segment
        max_items = segs * per + 64;
        max_rows = 2 * rows * per + 64;
    } else {
        max_items = segs + 5ll * r.grid + 2ll * B + 64;      // pieces of shared runs (with team slots) + cuts of the private stream
        max_rows = 2 * rows + (int64_t)r.grid * (rows_per_item + 2 * r.G) + 64;
    }
    if (max_items > 0x3FFFFFFF || max_rows > 0x3FFFFFFF) return fail(FEA_EINVAL, "%s: split_blocks too small for this problem size", who);
    WsLayout& l = r.lay;
    size_t off = up256(H_WORDS * sizeof(int32_t));
    l.req = off;      off += up256((size_t)B * sizeof(ReqDesc));
    l.grp = off;      off += up256((size_t)B * sizeof(GroupDesc));
    l.members = off;  off += up256((size_t)B * sizeof(int32_t));       // member lists of the groups
    l.segs = off;     off += up256((size_t)segs * sizeof(SegDesc));
    l.wave_first = off; off += up256((size_t)(max_items + 2) * sizeof(int32_t));
    l.items = off;    off += up256((size_t)max_items * sizeof(Item));
    l.ml = off;       off += up256((size_t)max_rows * 2 * sizeof(float));
    l.acc = off;      off += up256((size_t)max_rows * p->head_dim * sizeof(float));
    l.pre = off;      off += up256((size_t)kGroupReqMax * (sizeof(uint64_t) + sizeof(int32_t)));
    l.total = off;
    l.max_items = (int32_t)max_items;
    l.max_rows = (int32_t)max_rows;
    // (the pieces of a history are counted in the workspace's section `pre`, up to 128 of them)
    int64_t pieces = kn.direct_pieces > 0 ? kn.direct_pieces : direct_pieces(p, B, stride);
    pieces = direct_groups(p, B) > kGroupReqMax ? 1 : std::min<int64_t>({pieces, 128, max_rows / std::max<int64_t>(1, rows)});
    r.direct = direct ? (int)std::max<int64_t>(1, pieces) : 0;
    return FEA_OK;
}

}  // namespace fea

using namespace fea;

extern "C" {

int32_t fea_decode_workspace_bytes(const fea_attn_params* p, int32_t B, int32_t table_stride, size_t* out_bytes) {
    if (!out_bytes) return fail(FEA_EINVAL, "fea_decode_workspace_bytes: out_bytes is NULL");
    return decode_workspace_bytes(p, B, table_stride, out_bytes, "fea_decode_workspace_bytes");
}

}  // extern "C"

namespace fea {

int32_t decode_workspace_bytes(const fea_attn_params* p, int32_t B, int32_t table_stride, size_t* out_bytes, const char* who) {
    int32_t rc = check_params(p, who);
    if (rc != FEA_OK) return rc;
    Resolved r;
    rc = resolve(p, B, table_stride, r, who);
    if (rc != FEA_OK) return rc;
    *out_bytes = r.lay.total;
    return FEA_OK;
}

int32_t decode_impl(const fea_attn_params* p, const void* q, const void* k_cache, const void* v_cache,
                    const int32_t* block_tables, int32_t table_stride, const int32_t* seq_lens, int32_t B,
                    void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    int32_t rc = check_params(p, "fea_decode_attention");
    if (rc != FEA_OK) return rc;
    Resolved r;
    rc = resolve(p, B, table_stride, r, "fea_decode_attention");
    if (rc != FEA_OK) return rc;
    if (B == 0) return FEA_OK;
    const bool plan_only = (p->flags & FEA_FLAG_PLAN_ONLY) != 0;
    if (!block_tables || !seq_lens || !workspace || (!plan_only && (!q || !k_cache || !v_cache || !out)))
        return fail(FEA_EINVAL, "fea_decode_attention: NULL device pointer");
    if (((uintptr_t)workspace & 255) != 0) return fail(FEA_EINVAL, "fea_decode_attention: workspace must be 256-byte aligned");
    if (((uintptr_t)q & 15) || ((uintptr_t)k_cache & 15) || ((uintptr_t)v_cache & 15) || ((uintptr_t)out & 15))
        return fail(FEA_EINVAL, "fea_decode_attention: q, caches and out must be 16-byte aligned");
    if (workspace_bytes < r.lay.total)
        return fail(FEA_ERANGE, "fea_decode_attention: workspace has %zu bytes, %zu needed", workspace_bytes, r.lay.total);

    const float scale = p->scale > 0.f ? p->scale : 1.0f / std::sqrt((float)p->head_dim);
    Launch where[3] = {{hip_stream, nullptr, nullptr}, {hip_stream, nullptr, nullptr}, {hip_stream, nullptr, nullptr}};
    std::unique_lock<std::mutex> prof_lock(g_prof_mu, std::defer_lock);
    if (g_prof_on.load(std::memory_order_relaxed)) prof_lock.lock();   // (calls of several threads take their slots one after the other)
    if (prof_lock.owns_lock() && g_prof_on.load() && !g_ev_pool.empty()) {
        const size_t slot = (size_t)(g_prof_calls % (int)(g_ev_pool.size() / kEvPerCall));
        hipEvent_t* ev = &g_ev_pool[kEvPerCall * slot];
        unsigned char mask = 0;
        for (int k = 0; k < 3; ++k) {
            if (g_prof_which >= 0 && g_prof_which != k) continue;
            if (k == 0 && ((p->flags & FEA_FLAG_REUSE_PLAN) || (r.direct && !plan_only))) continue;
            if (k > 0 && plan_only) continue;
            if (k == 2 && r.direct) continue;
            where[k].ev_start = ev[2 * k];
            where[k].ev_stop = ev[2 * k + 1];
            if (k == 0) { where[0].ev_mid[0] = ev[6]; where[0].ev_mid[1] = ev[7]; }
            mask |= (unsigned char)(1u << k);
        }
        g_prof_mask[slot] = mask;
        ++g_prof_calls;
    }
    if (prof_lock.owns_lock()) prof_lock.unlock();
    if (!(p->flags & FEA_FLAG_REUSE_PLAN) && (plan_only || !r.direct)) {   // a new plan, or the one in the workspace stretched to the lengths of now
        PlanArgs pa;
        std::memset(&pa, 0, sizeof pa);
        pa.bt = block_tables;
        pa.seq_lens = seq_lens;
        pa.ws = static_cast<char*>(workspace);
        pa.lay = r.lay;
        pa.tune = r.tune;
        pa.stride = table_stride;
        pa.B = B;
        pa.Hq = p->num_q_heads;
        pa.Hkv = p->num_kv_heads;
        pa.G = r.G;
        pa.mpt = r.mpt;
        pa.grouping = r.grouping;
        pa.split_user = r.split_user;
        pa.variant = r.variant;
        pa.teams = (r.variant == 1 && p->head_dim == 128 && !knobs().no_fast_shared) ? 1 : 0;
        pa.pre = r.pre;
        pa.pre_grid = r.pre_grid;
        pa.histories = r.histories;
        // (A plan alone has no caches to read.  At head_dim 256 the sweep waits less for memory: 48 requests on one prefix of 3000 43.9 ->
        // 45.2 us with it, five other shapes 0.98 to 1.03 of the time.)
        if (r.variant == 1 && p->head_dim != 256 && !plan_only) set_read_ahead(pa, k_cache, v_cache, p->head_dim, cu_count());
        pa.histories_each = 1536 / p->head_dim;
        pa.far_tiles = (kFarMB * 1000000 + 128 * p->head_dim - 1) / (128 * p->head_dim);   // (a tile: two blocks of K and of V)
        if (p->flags & FEA_FLAG_REFRESH_PLAN) launch_refresh(pa, where[0]);
        else launch_plan(pa, where[0]);
    }
    if (plan_only) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(FEA_EHIP, "fea_decode_attention: launch failed: %s", hipGetErrorString(e));
        return FEA_OK;
    }
    SweepArgs sa;
    std::memset(&sa, 0, sizeof sa);
    sa.q = q;
    sa.k_cache = k_cache;
    sa.v_cache = v_cache;
    sa.bt = block_tables;
    sa.seq_lens = seq_lens;
    sa.out = out;
    sa.ws = static_cast<char*>(workspace);
    sa.lay = r.lay;
    sa.scale_log2 = scale * 1.4426950408889634f;
    sa.stride = table_stride;
    sa.B = B;
    sa.Hq = p->num_q_heads;
    sa.Hkv = p->num_kv_heads;
    sa.G = r.G;
    sa.mpt = r.mpt;
    sa.fast_shared = (p->head_dim == 128 && (int64_t)B * p->num_q_heads < (1 << 23) && !knobs().no_fast_shared) ? 1 : 0;
    if (r.direct) {
        launch_decode_direct(sa, p->dtype, p->head_dim, r.direct, where[1]);
    } else {
        if (r.variant == 1) launch_sweep_mfma(sa, p->head_dim, r.grid, where[1]);
        else launch_sweep_generic(sa, p->dtype, p->head_dim, r.grid, where[1]);
        launch_merge(sa, p->dtype, p->head_dim, r.merge_by_rows != 0, where[2]);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FEA_EHIP, "fea_decode_attention: launch failed: %s", hipGetErrorString(e));
    return FEA_OK;
}

}  // namespace fea

extern "C" {

int32_t fea_decode_attention(const fea_attn_params* p, const void* q, const void* k_cache, const void* v_cache,
                             const int32_t* block_tables, int32_t table_stride, const int32_t* seq_lens, int32_t B,
                             void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return decode_impl(p, q, k_cache, v_cache, block_tables, table_stride, seq_lens, B, out, workspace, workspace_bytes,
                       hip_stream);
}

// A tool that intercepts the launches (rocprofv3 loads its library through this variable)
// times every dispatch itself; the library's own per-dispatch events are not attached then.
static bool profiler_attached() {
    const char* v = std::getenv("ROCP_TOOL_LIBRARIES");
    return v && *v;
}

int32_t fea_profile_enable(int32_t max_calls, int32_t which) {
    if (max_calls < 0 || max_calls > 65536) return fail(FEA_EINVAL, "fea_profile_enable: max_calls=%d out of range", max_calls);
    if (which < -1 || which > 2) return fail(FEA_EINVAL, "fea_profile_enable: which=%d, expected -1, 0, 1 or 2", which);
    if (max_calls > 0 && profiler_attached())
        return fail(FEA_EINVAL, "fea_profile_enable: a profiling tool is attached to this process (ROCP_TOOL_LIBRARIES); "
                                "it times the dispatches itself, the library's events stay off");
    return guarded("fea_profile_enable", [&]() -> int32_t {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    g_prof_which = which;
    while ((int)g_ev_pool.size() < kEvPerCall * max_calls) {
        hipEvent_t ev;
        const hipError_t e = hipEventCreate(&ev);
        if (e != hipSuccess) return fail(FEA_EHIP, "fea_profile_enable: %s", hipGetErrorString(e));
        g_ev_pool.push_back(ev);
    }
    g_prof_mask.assign(g_ev_pool.size() / kEvPerCall, 0);
    g_prof_on = max_calls > 0;
    g_prof_calls = 0;
    return FEA_OK;
    });
}

int32_t fea_profile_read(int32_t call, float* ms) {
    if (!ms) return fail(FEA_EINVAL, "fea_profile_read: ms is NULL");
    std::lock_guard<std::mutex> lock(g_prof_mu);
    const int slots = (int)(g_ev_pool.size() / kEvPerCall);
    if (call < 0 || call >= g_prof_calls || g_prof_calls - call > slots)
        return fail(FEA_EINVAL, "fea_profile_read: call %d was not recorded (or its events were reused)", call);
    const size_t slot = (size_t)(call % slots);
    hipEvent_t* ev = &g_ev_pool[kEvPerCall * slot];
    hipError_t e = hipSuccess;
    for (int k = 0; k < 3; ++k) {
        ms[k] = 0.f;
        if (!(g_prof_mask[slot] & (1u << k)) || e != hipSuccess) continue;
        e = hipEventSynchronize(ev[2 * k + 1]);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms[k], ev[2 * k], ev[2 * k + 1]);
    }
    if (e != hipSuccess) return fail(FEA_EHIP, "fea_profile_read: %s", hipGetErrorString(e));
    return FEA_OK;
}

int32_t fea_decode_plan_info(const void* workspace, void* hip_stream, int32_t* info) {
    if (!workspace || !info) return fail(FEA_EINVAL, "fea_decode_plan_info: NULL pointer");
    int32_t hdr[H_WORDS];
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipMemcpyAsync(hdr, workspace, sizeof hdr, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(FEA_EHIP, "fea_decode_plan_info: %s", hipGetErrorString(e));
    info[0] = hdr[H_ITEMS];
    info[1] = hdr[H_GROUPS];
    info[2] = hdr[H_GROUPED];
    info[3] = hdr[H_SPLIT];
    info[4] = hdr[H_ROWS];
    info[5] = hdr[H_SHARED_BLOCKS];
    info[6] = hdr[H_VARIANT] == kHistories ? 1 : hdr[H_VARIANT];
    info[7] = hdr[H_OVERFLOW];
    info[8] = hdr[H_WAVES];
    return FEA_OK;
}

}  // extern "C"
