// Host side of the C ABI: argument validation, launch plans, workspace carving.  No device work
// is done here other than enqueuing kernels on the caller's stream; nothing synchronises.
#include "ygg_internal.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>

namespace ygg {
namespace {

// Launch-plan override for tuning runs (ygg_debug_set_attention_plan): waves << 24 | rblocks << 16 | kshares << 8 in the
// upper word, the forced split count in the lower; 0 = no override.
std::atomic<uint64_t> g_plan_override{0};

// One-time set-up per device: every kernel variant that needs more dynamic shared memory than the default gets its limit
// raised, so that no later call (possibly under stream capture) has to.
constexpr int kMaxDevices = 64;
std::atomic<bool> g_device_ready[kMaxDevices];
std::mutex g_init_mutex;

// Library-owned workspace of ygg_equal_growth_expand_static, for callers that cannot provide one.  Every device
// holds its own copy at its own address (looked up once per device, below); host code only ever uses that
// address.  Nothing in it has to start at zero: every call writes what it reads.
constexpr size_t kStaticScratchBytes = YGG_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
unsigned char* g_scratch_ptr[kMaxDevices];

// What a segment of a balanced batch costs beside its key tiles (Q, masks, an empty pipeline, the partial rows), in tiles.
// us per call, 0 / 3 / 6 / 8 tiles: 16 sequences of 512 to 8192 tokens with 392 rows on 8 kv heads 165 / 157 / 152 / 149, 8 of 256 to
// 8192 with 516 rows 115 / 111 / 110 / 112, 4 of 1024 to 16384 with 196 rows 59 / 57 / 54 / 53, 40 of 100 to 3000 with 392 rows 169 /
// 165 / 159 / 156, 9 of 1 to 4000 with 164 rows 42 / 33 / 29 / 29; six equal ones of 1024 with 516 rows 41 / 39 / 40 / 41.
constexpr int32_t kSegmentLead = 6;

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

bool common_shape_ok(const ygg_shape& s) {
    if (s.batch < 1 || s.batch > 65535) return false;
    if (s.n_q_heads < 1 || s.n_kv_heads < 1 || s.n_q_heads % s.n_kv_heads != 0) return false;
    if (s.depth < 0 || s.width < 1 || s.n_nodes < 1) return false;
    if (s.max_seq_len < 0 || s.kv_capacity < (int64_t)s.max_seq_len + s.depth + 1) return false;
    return true;
}

int32_t check_shape(const ygg_shape* s, bool need_kv, bool need_vocab) {
    if (!s) return YGG_ERR_NULL;
    if (!common_shape_ok(*s)) return YGG_ERR_SHAPE;
    if (s->n_nodes > kMaxNodes || s->width > kMaxWidth) return YGG_ERR_UNSUPPORTED;
    if (need_kv) {
        if (s->kv_dtype != YGG_F32 && s->kv_dtype != YGG_BF16 && s->kv_dtype != YGG_FP8_E4M3) return YGG_ERR_UNSUPPORTED;
        if (s->head_dim != 64 && s->head_dim != 128) return YGG_ERR_UNSUPPORTED;
        if (s->kv_dtype == YGG_FP8_E4M3 && s->head_dim != 128) return YGG_ERR_UNSUPPORTED;
        // the matrix-core kernel takes row maxima before scaling, which needs a positive finite scale
        if (!(s->softmax_scale > 0.f) || !std::isfinite(s->softmax_scale)) return YGG_ERR_SHAPE;
    }
    if (need_vocab && s->vocab < 1) return YGG_ERR_SHAPE;
    return YGG_OK;
}

int32_t check_workspace(const void* ws, size_t have, size_t need) {
    if (need == 0) return YGG_OK;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || have < need) return YGG_ERR_WORKSPACE;
    return YGG_OK;
}

}  // namespace

// K/V streams -- (sequence, kv head, split) or (kv head, run) -- whose workgroups all run at once: the kernel keeps a stream's row
// tiles on one XCD, which has 32 compute units, and deals the streams out over eight.  Counting all 256 compute units instead let
// 12 heads with three row tiles have seven splits: 84 streams, eleven on some XCDs, 33 workgroups and so a second round.  us per
// call by that count -> by this one: 129 rows x 4096 tokens on 12 kv heads 27.0 -> 19.4, 257 rows x 16384 on 12 82.5 -> 52.9,
// 776 rows x 8192 on 4 42.0 -> 28.1.  (Beyond 32 row tiles one round does not hold a stream; what fills the chip is left.)
static int64_t streams_at_once(int64_t row_tiles) { return row_tiles <= 32 ? 8 * (32 / row_tiles) : 256 / row_tiles; }

// Splits of every sequence's key tiles for a workgroup shape: fill the 256 CUs once -- the tile buffers leave room for one
// workgroup per CU, and a second round of workgroups pays the start-up latency again while more splits add partial-result
// traffic -- with about three key tiles per split at least (17 tiles of 49 rows on 32 kv heads: 5 / 6 / 8 splits measured
// 16.4 / 15.7 / 16.4 us per layer).
static int64_t equal_splits(const ygg_shape& s, int row_tiles, int64_t tiles) {
    int64_t ns = streams_at_once(row_tiles) / ((int64_t)s.batch * s.n_kv_heads);
    if (ns > (tiles + 2) / 3) ns = (tiles + 2) / 3;
    return ns < 1 ? 1 : ns;   // (plan_attention keeps to 64, which the merge takes)
}
// At least this many key tiles to a workgroup of the longest sequence: a batch is cut into equal runs instead (plan_attention).
static constexpr int64_t kTilesForRuns = 8;
// At least this many tiles of one sequence to a workgroup: opposite phases (plan_attention).
static constexpr int64_t kTilesForPhases128 = 10, kTilesForPhases64 = 24;
static constexpr int64_t kTilesForPhasesInRuns128 = 20, kTilesForPhasesInRuns64 = 64;

// The padded rows decide where a workgroup streams many key tiles.  Where its share of them is short, a workgroup of fewer rows
// is the better one: it starts sooner (fewer rows of Q, fewer wavefronts to meet) and its tiles take less time, so with the
// compute units filled either way the call is done sooner although each K/V byte is fetched for fewer rows.  The estimate is a
// start and a time per tile of 64 keys for each shape, in us, fitted per head_dim on calls of 129 to 516 rows, plus the merge.  On 252
// calls per head_dim (65 to 1284 rows on 4, 8, 12, 32 and 40 kv heads over 256 to 16384 tokens) its mean error is 7 % (head_dim 64:
// 11 %); the plan's shape is 1.4 % (1.7 %) slower than the best of the five on average and at most 32 % (36 %), that of fewest padded
// rows 8.9 % (8.8 %) and 43 % (54 %).  (Fitted and counted with the kernels before the last split's share and opposite phases in
// short streams, which made the first two shapes up to 10 % faster.)  The shape of fewest padded rows stays unless another promises 4 %
// less.  Measured then, us per call with the shape of fewest padded rows -> with this rule's, 8 kv heads: 196 rows x 633 tokens 17.4 -> 12.7 (tiles of 256 rows -> 64), x 4096 20.4 -> 16.6, 176 x 2078 17.8 -> 14.7 (192 -> 64), 516 x 1024
// 17.8 -> 16.7 (192 -> 64), 392 x 4096 21.7 -> 20.9 (256 -> 128); 32 kv heads: 321 rows x 4096 48.1 -> 43.2 (128 -> 192).  At
// 16384 tokens tiles of 256 lead again (392 rows: 39.0, of 128 44.3).
static void short_run_shape(const ygg_shape& s, int R, int64_t tiles, AttnPlan& p) {
    struct Kind { int32_t waves, kshares; float start, tile; };
    static constexpr Kind kinds128[] = {{8, 1, 14.0f, 1.30f}, {6, 1, 11.5f, 1.41f}, {4, 1, 10.6f, 1.15f}, {8, 2, 11.9f, 0.87f}, {4, 2, 10.5f, 0.69f}};
    static constexpr Kind kinds64[] = {{8, 1, 13.0f, 0.95f}, {6, 1, 11.3f, 1.00f}, {4, 1, 10.6f, 0.85f}, {8, 2, 11.0f, 0.66f}, {4, 2, 9.7f, 0.50f}};
    const Kind(&kinds)[5] = s.head_dim == 128 ? kinds128 : kinds64;
    constexpr float kNo = 1e30f;
    auto estimate = [&](const Kind& k) {
        const int rows = k.waves / k.kshares * 32, row_tiles = (R + rows - 1) / rows;
        if ((int64_t)s.batch * s.n_kv_heads > streams_at_once(row_tiles)) return kNo;   // more than one round of workgroups: not fitted
        int64_t ns = equal_splits(s, row_tiles, tiles);
        if (s.batch >= 2 && tiles / ns >= kTilesForRuns) return kNo;   // a batch in equal runs
        if (s.batch >= 2 && p.kshares == 1 && k.kshares > 1) return kNo;   // stays a plan that runs can serve (pairs cannot), whatever the length bound
        if (ns > 64) ns = 64;
        const float merge = ns > 1 ? 4e-7f * (float)ns * (float)s.batch * (float)s.n_kv_heads * (float)R * (float)s.head_dim : 0.f;
        return k.start + k.tile * (float)((tiles + ns - 1) / ns) + merge;
    };
    const Kind* best = nullptr;
    float least = 0.f;
    for (const Kind& k : kinds)
        if (k.waves == p.waves && k.kshares == p.kshares) least = 0.96f * estimate(k);
    if (least > 0.9f * kNo) return;
    for (const Kind& k : kinds)
        if (estimate(k) < least) { best = &k; least = estimate(k); }
    if (best) { p.waves = best->waves; p.kshares = best->kshares; }
}

// matrix-core kernels: fp16 partial outputs with one fp32 scale per row; vector kernel: fp32 partial outputs
static size_t part_o_bytes(const ygg_shape& s, bool half, int64_t nsplit) {
    return align256((size_t)nsplit * (size_t)s.batch * (size_t)s.n_nodes * (size_t)s.n_q_heads * (size_t)s.head_dim * (half ? 2 : 4));
}
static size_t part_rec_bytes(const ygg_shape& s, int64_t nsplit) {
    return align256((size_t)nsplit * (size_t)s.batch * (size_t)s.n_nodes * (size_t)s.n_q_heads * sizeof(float3));
}

AttnPlan plan_attention(const ygg_shape& s) {
    AttnPlan p{};
    const int64_t rows = (int64_t)s.batch * s.n_nodes * s.n_q_heads;
    const int64_t T = (int64_t)s.max_seq_len + s.n_nodes;
    const int64_t tiles = (T + kKeyTile - 1) / kKeyTile;
    int64_t ns;
    const bool kv8 = s.kv_dtype == YGG_FP8_E4M3;  // K/V as 8-bit codes, Q and O bf16 (head_dim 128 only)
    p.use_mfma = (s.kv_dtype == YGG_BF16 && (s.head_dim == 128 || s.head_dim == 64)) || (kv8 && s.head_dim == 128);
    if (p.use_mfma) {
        // query rows that share one K/V stream, and the workgroup shape that wastes the fewest of them
        const int R = s.n_nodes * (s.n_q_heads / s.n_kv_heads);
        p.rblocks = 1;
        p.kshares = 1;
        // Workgroup shapes, by rows per workgroup: 256 (8 wavefronts), 192 (6), 128 (8 wavefronts in
        // pairs that split every key tile), 64 and 32 (4 and 2 wavefronts in pairs).  More rows per
        // workgroup amortise the K/V tile traffic and the per-tile barrier over more matrix work, so
        // a smaller shape is taken only when it saves a good share of padded rows.
        auto padded = [R](int rw) { return (R + rw - 1) / rw * rw; };
        if (R <= 32) { p.waves = 2; p.kshares = 2; }
        else if (R <= 64) { p.waves = 4; p.kshares = 2; }
        else if (kv8) { p.waves = 4; }  // 8-bit K/V: at most four computing wavefronts, the loaders take the other slots
        else if (R <= 128) { p.waves = 8; p.kshares = 2; }
        else {
            p.waves = 8;
            int best = padded(256);
            if (padded(128) * 100 <= best * 85) { best = padded(128); p.kshares = 2; }
            // 192 rows: two of the four SIMDs carry one wavefront only, so against 256-row workgroups it has to save a
            // fifth of the rows (1284 rows x 32768 keys with 1344 instead of 1536 padded rows: 210 vs 202 us); against the
            // paired 128-row shape, which meets a barrier every 16 matrix instructions, a tenth is enough (516 rows x 4096
            // keys with 576 instead of 640 padded rows and 10 instead of 6 key splits: 27.5 vs 28.1 us per call)
            if (padded(192) * 100 <= best * (p.kshares == 2 ? 92 : 80)) { p.waves = 6; p.kshares = 1; }
        }
        if (!kv8 && R > 64) short_run_shape(s, R, tiles, p);
        int64_t ns_forced = 0;
        if (const uint64_t ov = g_plan_override.load(std::memory_order_relaxed)) {
            const int w = (int)(ov >> 56), r = (int)(ov >> 48) & 0xff, k = (int)(ov >> 40) & 0xff;
            const bool known = r == 1 && (kv8 ? (w == 4 && (k == 1 || k == 2)) || (w == 2 && k == 2)
                                              : k == 2 ? (w == 2 || w == 4 || w == 8) : (k == 1 && (w == 4 || w == 6 || w == 8)));
            if (known) { p.waves = w; p.rblocks = r; p.kshares = k; }
            ns_forced = (int64_t)(ov & 0xffffffffu);
        }
        // the widest trees (more than 900 nodes, one query head per kv head) leave no room for their masks beside 256 rows
        const int G = s.n_q_heads / s.n_kv_heads;
        while (p.kshares == 1 && p.waves > 4 && attn_mfma_smem(p.waves, 1, s.head_dim, G, s.n_nodes) > kAttnMfmaMaxSmem) p.waves -= 2;
        const int rw = p.waves / p.kshares * p.rblocks * 32;
        p.row_tiles = (R + rw - 1) / rw;
        ns = equal_splits(s, p.row_tiles, tiles);
        if (ns_forced) ns = ns_forced < tiles ? ns_forced : tiles;
        // Batches: sequence lengths live on the device and may be ragged, so instead of giving every sequence the same
        // number of splits the key tiles of all sequences are laid end to end and cut into equal runs, one per workgroup
        // of a (kv head, row tile): 256 workgroups in all, each with the same number of tiles whatever the lengths.  A
        // workgroup whose run spans two sequences starts its pipeline twice, about as long as three tiles take; where the
        // longest sequence leaves a workgroup fewer than eight tiles anyway, that costs more than the raggedness (3
        // sequences of up to 1531 tokens, 8 kv heads x 36 nodes: 21 us per call in runs, 16 in splits).
        const int64_t streams = (int64_t)s.n_kv_heads * p.row_tiles;
        const int64_t per_wg = ns > 0 ? tiles / ns : tiles;
        if (p.kshares == 1 && s.batch >= 2 && s.batch <= 256 && streams <= 128 && !ns_forced && per_wg >= kTilesForRuns) {
            int64_t slots = streams_at_once(p.row_tiles) / s.n_kv_heads;
            const int64_t most = (int64_t)s.batch * tiles;   // never more runs than tiles
            if (slots > most) slots = most;
            if (slots > 64) slots = 64;                      // the merge takes at most 64 splits per row
            if (slots >= 2) p.slots = (int32_t)slots;
        }
        // Opposite phases of the two wavefronts of a SIMD pay where a workgroup streams many tiles of one sequence: the first tile and
        // the last four go through a body with conditions, and a tile takes four barriers instead of one.  One sequence on 8 kv heads,
        // us per call without -> with them, by tiles to a workgroup, both with shares after tree_cost: 256 rows, head_dim 128, 7 tiles
        // (516 rows x 4096 tokens) 23.5 -> 23.2, 9 (1284 x 2600) 29.7 -> 30.1, 11 33.4 -> 32.3, 13 38.8 -> 36.9 and (516 x 8192) 34.8 ->
        // 32.8; head_dim 64, 13 tiles 27.4 -> 26.9, 16 (392 rows) 26.9 -> 27.4, 26 40.7 -> 39.4, 52 68.5 -> 65.9; 192 rows, head_dim 128, 4
        // tiles (516 x 2000) 19.2 -> 20.0, 7 23.1 -> 23.0, 9 (161 x 4096 on 32 kv heads) 29.9 -> 30.0, 11 (129 x 4096 on 40) 31.7 -> 29.9, 13
        // 33.0 -> 31.3.  Runs start a pipeline for every sequence they touch, their shares are not shorter for the tree's keys, and the
        // lengths may lie far below the bound that the tiles are counted from, so their line lies higher.  us per call without -> with
        // them, by tiles of the bound to a run: head_dim 128, 12 (24 sequences of 63 tokens, 208 rows on 40 kv heads) 93.5 -> 98.8, (23 of
        // 84, 776 rows on 8) 53.8 -> 56.6, 14 (7 of 203 to 407, 788 rows on 8) 35.7 -> 37.8, 10 (2 of 3000, 1284 rows on 8) 54.8 -> 55.4, 15
        // (3 of 5000, 392 rows on 8) 42.0 -> 40.6; head_dim 64, 27 (4 of 6000, 388 rows on 8) 39.8 -> 41.2, 33 (of 8192) 47.3 -> 48.2, 39 (2
        // of 6000, 1284 rows) 58.7 -> 61.4, 36 (8 of 2048, 804 rows) 51.1 -> 52.8.
        const int64_t segment = p.slots > 0 ? std::min(s.batch * tiles / p.slots, tiles) : tiles / std::clamp(ns, (int64_t)1, (int64_t)64);
        const int64_t phases_from = p.slots > 0 ? (s.head_dim == 128 ? kTilesForPhasesInRuns128 : kTilesForPhasesInRuns64)
                                                : (s.head_dim == 128 ? kTilesForPhases128 : kTilesForPhases64);
        p.phases = p.kshares == 1 && segment >= phases_from &&
                   (p.waves == 8 || (p.waves == 6 && s.head_dim == 128 && p.slots == 0));
        // What the tree's keys and their masks cost the workgroup of a sequence's last split beside their tiles, in tiles: the masks'
        // chain, and per tile of tree keys the masking, which with opposite phases lengthens both wavefronts' phases.  Such a workgroup
        // with an equal share ended 5.9 us after the others (1284 rows x 2048 tokens), 7.5 at 8192.  us per call with equal shares ->
        // these: 1284 rows x 4096 tokens on 8 kv heads 42.1 -> 36.5, x 8192 59.8 -> 55.0, x 32768 178 -> 174, 516 rows x 4096 in
        // tiles of 256 26.0 -> 24.2, 392 x 16384 41.1 -> 40.6; without opposite phases 1284 x 2048 27.6 -> 27.1.  8-bit K/V: 1284 x 4096
        // 49.6 -> 48.3, 516 x 4096 23.7 either way; where the shares stay the same the arithmetic for them shows, 140 rows x 522 on 4
        // 10.85 -> 10.95.
        const int32_t tree_tiles = (s.n_nodes + kKeyTile - 1) / kKeyTile;
        p.tree_cost = p.phases ? 1 + 6 * tree_tiles / 5 : 1 + tree_tiles / 4;
    } else {
        // vector path: one wavefront per (row, split); aim for ~4096 wavefronts
        ns = (4096 + rows - 1) / rows;
        if (ns > tiles) ns = tiles;
    }
    if (ns < 1) ns = 1;
    if (ns > 64) ns = 64;
    if (!p.use_mfma) {
        // vector kernel: equal chunks rounded up to whole key tiles; drop the splits that rounding leaves empty
        // (the matrix-core kernel deals whole tiles out evenly instead, and no split of at most `tiles` is empty)
        const int64_t chunk = ((T + ns - 1) / ns + kKeyTile - 1) / kKeyTile * kKeyTile;
        ns = (T + chunk - 1) / chunk;
    }
    p.nsplit = p.slots > 0 ? p.slots : (int32_t)ns;   // balanced batches: a sequence may span every run
    p.part_o_bytes = part_o_bytes(s, p.use_mfma, p.nsplit);
    p.part_rec_bytes = part_rec_bytes(s, p.nsplit);
    p.seq_splits_bytes = p.slots > 0 ? align256((size_t)s.batch * sizeof(int32_t)) : 0;
    return p;
}

// Workspace for this shape and every smaller max_seq_len.  More keys mean no fewer splits or runs for one workgroup shape, but
// short_run_shape changes the shape with the length, and a shorter call may take one that allows more splits: the bound is the
// workgroup shape with the most.
static size_t attention_scratch_bytes(const ygg_shape& s) {
    const AttnPlan p = plan_attention(s);
    const int R = s.n_nodes * (s.n_q_heads / s.n_kv_heads);
    int64_t most = p.nsplit;
    if (p.use_mfma && s.kv_dtype != YGG_FP8_E4M3 && R > 64) {
        const int64_t tiles = ((int64_t)s.max_seq_len + s.n_nodes + kKeyTile - 1) / kKeyTile;
        for (int rows : {256, 192, 128, 64}) most = std::max(most, std::min(equal_splits(s, (R + rows - 1) / rows, tiles), (int64_t)64));
    }
    return part_o_bytes(s, p.use_mfma, most) + part_rec_bytes(s, most) + p.seq_splits_bytes;
}

// Raises the shared-memory limits of the current device's kernels once; later calls cost one atomic load.
int32_t ensure_device_ready() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return YGG_ERR_LAUNCH;
    if (g_device_ready[dev].load(std::memory_order_acquire)) return YGG_OK;
    std::lock_guard<std::mutex> lock(g_init_mutex);
    if (g_device_ready[dev].load(std::memory_order_relaxed)) return YGG_OK;
    if (raise_limits_attn_mfma() != hipSuccess || raise_limits_expand() != hipSuccess) return YGG_ERR_LAUNCH;
    void* sp = nullptr;
    if (hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) != hipSuccess || !sp) return YGG_ERR_LAUNCH;
    g_scratch_ptr[dev] = static_cast<unsigned char*>(sp);
    g_device_ready[dev].store(true, std::memory_order_release);
    return YGG_OK;
}

}  // namespace ygg

using namespace ygg;

extern "C" {

int32_t ygg_init(void) { return ensure_device_ready(); }

int32_t ygg_debug_set_attention_plan(int32_t waves, int32_t rblocks, int32_t nsplit, int32_t kshares) {
    if (waves < 0 || waves > 255 || rblocks < 0 || rblocks > 255 || kshares < 0 || kshares > 255 || nsplit < 0) return YGG_ERR_SHAPE;
    g_plan_override.store(((uint64_t)waves << 56) | ((uint64_t)rblocks << 48) | ((uint64_t)kshares << 40) | (uint32_t)nsplit,
                          std::memory_order_relaxed);
    return YGG_OK;
}

int32_t ygg_debug_attention_plan(const ygg_shape* s, int32_t* plan) {
    if (int32_t rc = check_shape(s, true, false)) return rc;
    if (!plan) return YGG_ERR_NULL;
    const AttnPlan p = plan_attention(*s);
    plan[0] = p.use_mfma; plan[1] = p.waves; plan[2] = p.kshares; plan[3] = p.row_tiles; plan[4] = p.nsplit;
    return YGG_OK;
}

int32_t ygg_debug_attention_launch(const ygg_shape* s, int32_t* launch) {
    if (int32_t rc = check_shape(s, true, false)) return rc;
    if (!launch) return YGG_ERR_NULL;
    const AttnPlan p = plan_attention(*s);
    launch[0] = p.phases; launch[1] = p.tree_cost;
    launch[2] = p.use_mfma ? (int32_t)attn_mfma_smem(p.waves, p.kshares, s->head_dim, s->n_q_heads / s->n_kv_heads, s->n_nodes) : 0;
    return YGG_OK;
}

const char* ygg_status_string(int32_t status) {
    switch (status) {
        case YGG_OK: return "ok";
        case YGG_ERR_NULL: return "null pointer";
        case YGG_ERR_SHAPE: return "inconsistent shape";
        case YGG_ERR_UNSUPPORTED: return "unsupported dtype, head_dim or size";
        case YGG_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case YGG_ERR_LAUNCH: return "kernel launch failed";
        default: return "unknown status";
    }
}

size_t ygg_workspace_bytes(const ygg_shape* s, int32_t op, int32_t n_layers) {
    (void)n_layers;
    if (!s) return 0;
    switch (op) {
        case YGG_OP_ATTENTION: {
            if (check_shape(s, true, false) != YGG_OK) return 0;
            return attention_scratch_bytes(*s);
        }
        case YGG_OP_EXPAND:
        case YGG_OP_ATTACH: {
            if (check_shape(s, false, true) != YGG_OK) return 0;
            return expand_scratch_bytes(*s);
        }
        case YGG_OP_ACCEPT: {
            if (check_shape(s, false, true) != YGG_OK) return 0;
            return accept_scratch_bytes(*s);
        }
        default: return 0;
    }
}

static int32_t tree_attention_impl(const ygg_shape* s, const void* q, const void* k_cache, const void* v_cache,
                                   const int32_t* seq_lens, const void* k_tree, const void* v_tree,
                                   const float* k_scale, const float* v_scale,
                                   const int32_t* parent_idx, void* out, float* lse, void* workspace,
                                   size_t workspace_bytes, void* hip_stream, bool main_only = false) {
    if (!q || !k_tree || !v_tree || !seq_lens || !parent_idx || !out) return YGG_ERR_NULL;
    if (s->max_seq_len > 0 && (!k_cache || !v_cache)) return YGG_ERR_NULL;
    // the kernels index query rows with 31 bits and address one sequence's K/V slab with 32-bit byte offsets
    const int64_t elem = s->kv_dtype == YGG_F32 ? 4 : s->kv_dtype == YGG_BF16 ? 2 : 1;
    if ((int64_t)s->batch * s->n_nodes * s->n_q_heads > 0x7fffffffLL) return YGG_ERR_UNSUPPORTED;
    if (s->kv_capacity * s->n_kv_heads * s->head_dim * elem > 0xffffffffLL) return YGG_ERR_UNSUPPORTED;
    const AttnPlan p = plan_attention(*s);
    if (int32_t rc = check_workspace(workspace, workspace_bytes, p.part_o_bytes + p.part_rec_bytes + p.seq_splits_bytes)) return rc;
    if (int32_t rc = ensure_device_ready()) return rc;

    AttnArgs a{};
    a.q = q; a.k_cache = k_cache; a.v_cache = v_cache; a.k_tree = k_tree; a.v_tree = v_tree;
    a.seq_lens = seq_lens; a.parent_idx = parent_idx; a.k_scale = k_scale; a.v_scale = v_scale;
    a.part_o = workspace;
    a.part_rec = reinterpret_cast<float3*>(static_cast<char*>(workspace) + p.part_o_bytes);
    a.seq_splits = p.slots > 0 ? reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + p.part_o_bytes + p.part_rec_bytes) : nullptr;
    a.out = out; a.lse = lse;
    a.B = s->batch; a.N = s->n_nodes; a.Hq = s->n_q_heads; a.Hkv = s->n_kv_heads;
    a.G = s->n_q_heads / s->n_kv_heads; a.Dh = s->head_dim;
    a.nsplit = p.nsplit; a.max_seq_len = s->max_seq_len; a.cap = s->kv_capacity; a.scale = s->softmax_scale;
    a.slots = p.slots;
    a.lead = kSegmentLead;
    a.tree_cost = p.tree_cost;
    a.seq_runs = p.slots > 0 && p.slots % s->batch == 0 ? p.slots / s->batch : 0;
    a.S = p.slots > 0 ? a.Hkv * p.slots : a.B * a.Hkv * p.nsplit;
    a.rows_total = a.B * a.N * a.Hq;
    a.mul_nsplit = 0xffffffffu / (uint32_t)a.nsplit;
    a.mul_last = a.nsplit > 1 ? 0xffffffffu / (uint32_t)(a.nsplit - 1) : 0;   // the last split apart
    a.mul_hkv = 0xffffffffu / (uint32_t)a.Hkv;
    a.mul_g = 0xffffffffu / (uint32_t)a.G;
    a.row_tiles = p.row_tiles > 0 ? p.row_tiles : 1;
    a.mul_rt = 0xffffffffu / (uint32_t)a.row_tiles;

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int out_dtype = s->kv_dtype == YGG_F32 ? YGG_F32 : YGG_BF16;  // element type of Q and O
    hipError_t e = p.use_mfma ? launch_attn_mfma(a, p, st) : launch_attn_vector(a, p, s->kv_dtype, st);
    if (e != hipSuccess) return YGG_ERR_LAUNCH;
    if (main_only) return YGG_OK;
    if (p.use_mfma && p.nsplit == 1) return YGG_OK;  // the kernel wrote the final rows itself
    e = launch_attn_combine(a, p, out_dtype, st);
    return e == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

int32_t ygg_tree_attention(const ygg_shape* s, const void* q, const void* k_cache, const void* v_cache,
                           const int32_t* seq_lens, const void* k_tree, const void* v_tree,
                           const int32_t* parent_idx, void* out, float* lse, void* workspace,
                           size_t workspace_bytes, void* hip_stream) {
    if (int32_t rc = check_shape(s, true, false)) return rc;
    if (s->kv_dtype == YGG_FP8_E4M3) return YGG_ERR_UNSUPPORTED;  // codes need their scales: ygg_tree_attention_fp8kv
    return tree_attention_impl(s, q, k_cache, v_cache, seq_lens, k_tree, v_tree, nullptr, nullptr, parent_idx, out, lse,
                               workspace, workspace_bytes, hip_stream);
}

int32_t ygg_debug_tree_attention_main(const ygg_shape* s, const void* q, const void* k_cache, const void* v_cache,
                                      const int32_t* seq_lens, const void* k_tree, const void* v_tree,
                                      const int32_t* parent_idx, void* out, float* lse, void* workspace,
                                      size_t workspace_bytes, void* hip_stream) {
    if (int32_t rc = check_shape(s, true, false)) return rc;
    if (s->kv_dtype == YGG_FP8_E4M3) return YGG_ERR_UNSUPPORTED;
    return tree_attention_impl(s, q, k_cache, v_cache, seq_lens, k_tree, v_tree, nullptr, nullptr, parent_idx, out, lse,
                               workspace, workspace_bytes, hip_stream, /*main_only=*/true);
}

int32_t ygg_tree_attention_fp8kv(const ygg_shape* s, const void* q, const void* k_cache, const void* v_cache,
                                 const int32_t* seq_lens, const void* k_tree, const void* v_tree,
                                 const float* k_scale, const float* v_scale, const int32_t* parent_idx, void* out,
                                 float* lse, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (int32_t rc = check_shape(s, true, false)) return rc;
    if (s->kv_dtype != YGG_FP8_E4M3) return YGG_ERR_UNSUPPORTED;
    if (!k_scale || !v_scale) return YGG_ERR_NULL;
    return tree_attention_impl(s, q, k_cache, v_cache, seq_lens, k_tree, v_tree, k_scale, v_scale, parent_idx, out, lse,
                               workspace, workspace_bytes, hip_stream);
}

int32_t ygg_equal_growth_expand(const ygg_shape* s, int32_t d, const float* draft_logits, int32_t* parent_idx,
                                int32_t* token_ids, float* cum_logprob, void* workspace, size_t workspace_bytes,
                                void* hip_stream) {
    if (int32_t rc = check_shape(s, false, true)) return rc;
    if (!draft_logits || !parent_idx || !token_ids || !cum_logprob) return YGG_ERR_NULL;
    if (s->depth < 1 || d < 1 || d > s->depth) return YGG_ERR_SHAPE;
    if ((int64_t)s->n_nodes != 1 + (int64_t)s->depth * s->width) return YGG_ERR_SHAPE;
    const ExpandPlan p = plan_expand(*s, d);
    if ((int64_t)p.F * s->vocab < s->width) return YGG_ERR_SHAPE;
    const int64_t pages = ((int64_t)s->vocab + 4095) / 4096;
    if ((int64_t)p.F * pages > 4096) return YGG_ERR_UNSUPPORTED;  // 16 M logits per sequence and step
    if ((int64_t)p.F * s->vocab >= 0x7fffffffLL) return YGG_ERR_UNSUPPORTED;  // flat candidate index is 32 bits
    if ((int64_t)s->batch * p.F > 0x7fffffffLL) return YGG_ERR_UNSUPPORTED;
    if (int32_t rc = check_workspace(workspace, workspace_bytes, p.cand_bytes + p.stat_bytes)) return rc;
    if (int32_t rc = ensure_device_ready()) return rc;

    ExpandArgs a{};
    a.logits = draft_logits; a.parent_idx = parent_idx; a.token_ids = token_ids; a.cum_logprob = cum_logprob;
    a.cands = workspace;
    a.stats = static_cast<char*>(workspace) + p.cand_bytes;
    a.B = s->batch; a.D = s->depth; a.W = s->width; a.V = s->vocab; a.N = s->n_nodes; a.d = d;
    a.F = p.F; a.chunk = p.chunk; a.nchunk = p.nchunk;
    return launch_expand(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

int32_t ygg_equal_growth_expand_static(const ygg_shape* s, int32_t d, const float* draft_logits, int32_t* parent_idx,
                                       int32_t* token_ids, float* cum_logprob, void* hip_stream) {
    const size_t need = ygg_workspace_bytes(s, YGG_OP_EXPAND, 0);
    if (need > kStaticScratchBytes) return YGG_ERR_WORKSPACE;   // shape too large for the built-in scratch (0: invalid shape, reported below)
    if (int32_t rc = ensure_device_ready()) return rc;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices || !g_scratch_ptr[dev]) return YGG_ERR_LAUNCH;
    return ygg_equal_growth_expand(s, d, draft_logits, parent_idx, token_ids, cum_logprob, g_scratch_ptr[dev],
                                   kStaticScratchBytes, hip_stream);
}

size_t ygg_attach_pool_bytes(const ygg_shape* s) {
    if (!s || check_shape(s, false, true) != YGG_OK || s->depth < 1) return 0;
    return attach_pool_bytes(*s);
}

int32_t ygg_equal_growth_attach(const ygg_shape* s, int32_t t, const float* draft_logits, int32_t* parent_idx,
                                int32_t* token_ids, float* cum_logprob, void* pool, size_t pool_bytes,
                                void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (int32_t rc = check_shape(s, false, true)) return rc;
    if (!draft_logits || !parent_idx || !token_ids || !cum_logprob || !pool) return YGG_ERR_NULL;
    if (s->depth < 1 || t < 1 || t > s->depth) return YGG_ERR_SHAPE;
    if ((int64_t)s->n_nodes != 1 + (int64_t)s->depth * s->width) return YGG_ERR_SHAPE;
    if (s->vocab < s->width) return YGG_ERR_SHAPE;  // every row must be able to offer W tokens
    const ExpandPlan p = plan_expand(*s, t);
    if (((int64_t)s->vocab + 4095) / 4096 * s->width > 4096) return YGG_ERR_UNSUPPORTED;   // 16 M logits per sequence and step
    if ((int64_t)s->n_nodes * s->vocab > 0xffffffffLL) return YGG_ERR_UNSUPPORTED;  // node*V + token is 32 bits
    if ((int64_t)s->batch * p.F > 0x7fffffffLL) return YGG_ERR_UNSUPPORTED;
    // pool + offers are sorted in one workgroup's LDS: at most 4096 entries
    if ((int64_t)p.F * s->width + (int64_t)s->width * (s->depth - t + 1) > 4096) return YGG_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(pool) & 15u) != 0 || pool_bytes < attach_pool_bytes(*s)) return YGG_ERR_WORKSPACE;
    if (int32_t rc = check_workspace(workspace, workspace_bytes, p.cand_bytes + p.stat_bytes)) return rc;
    if (int32_t rc = ensure_device_ready()) return rc;

    ExpandArgs a{};
    a.logits = draft_logits; a.parent_idx = parent_idx; a.token_ids = token_ids; a.cum_logprob = cum_logprob;
    a.cands = workspace;
    a.stats = static_cast<char*>(workspace) + p.cand_bytes;
    a.pool = pool; a.pool_cap = (int32_t)attach_pool_capacity(*s);
    a.B = s->batch; a.D = s->depth; a.W = s->width; a.V = s->vocab; a.N = s->n_nodes; a.d = t;
    a.F = p.F; a.chunk = p.chunk; a.nchunk = p.nchunk;
    return launch_attach(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

int32_t ygg_prune_for_verification(const ygg_shape* s, int32_t w_verify, const int32_t* parent_idx,
                                   const int32_t* token_ids, const float* cum_logprob, const float* t_verifier,
                                   float t_draft, int32_t* kept_nodes, int32_t* new_parent, int32_t* new_token,
                                   float* expected_len, int32_t* best_width, void* hip_stream) {
    if (int32_t rc = check_shape(s, false, false)) return rc;
    if (!parent_idx || !token_ids || !cum_logprob || !kept_nodes || !new_parent || !new_token) return YGG_ERR_NULL;
    if (best_width && !t_verifier) return YGG_ERR_NULL;
    if (w_verify < 1 || w_verify > s->n_nodes) return YGG_ERR_SHAPE;
    if (!(t_draft >= 0.f)) return YGG_ERR_SHAPE;
    PruneArgs a{};
    a.parent_idx = parent_idx; a.token_ids = token_ids; a.cum_logprob = cum_logprob; a.t_verifier = t_verifier;
    a.kept_nodes = kept_nodes; a.new_parent = new_parent; a.new_token = new_token;
    a.expected_len = expected_len; a.best_width = best_width; a.t_draft = t_draft;
    a.B = s->batch; a.N = s->n_nodes; a.w = w_verify;
    return launch_prune(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

int32_t ygg_debug_validate(const ygg_shape* s, const int32_t* parent_idx, const int32_t* seq_lens,
                           const int32_t* token_ids, const float* logits, int32_t logit_rows, int32_t* flags,
                           void* hip_stream) {
    if (int32_t rc = check_shape(s, false, token_ids != nullptr || logits != nullptr)) return rc;
    if (!flags) return YGG_ERR_NULL;
    if (logits && logit_rows < 1) return YGG_ERR_SHAPE;
    if (s->batch > 65535) return YGG_ERR_UNSUPPORTED;
    ValidateArgs a{};
    a.parent_idx = parent_idx; a.seq_lens = seq_lens; a.token_ids = token_ids; a.logits = logits; a.flags = flags;
    a.B = s->batch; a.N = s->n_nodes; a.D = s->depth; a.V = s->vocab; a.max_seq_len = s->max_seq_len;
    a.logit_rows = logit_rows;
    return launch_validate(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

int32_t ygg_accept_and_compact(const ygg_shape* s, int32_t n_layers, const float* target_logits,
                               const int32_t* target_tokens, const int32_t* parent_idx, const int32_t* token_ids,
                               const void* k_tree, const void* v_tree, void* k_cache, void* v_cache,
                               int32_t* seq_lens, int32_t* accept_len, int32_t* accept_path, int32_t* bonus_token,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (int32_t rc = check_shape(s, n_layers > 0, target_logits != nullptr)) return rc;
    if (n_layers < 0 || n_layers > 65535) return YGG_ERR_SHAPE;
    if ((target_logits == nullptr) == (target_tokens == nullptr)) return YGG_ERR_NULL;
    if (!parent_idx || !token_ids || !seq_lens || !accept_len || !accept_path || !bonus_token) return YGG_ERR_NULL;
    if (n_layers > 0 && (!k_tree || !v_tree || !k_cache || !v_cache)) return YGG_ERR_NULL;
    const AcceptPlan p = plan_accept(*s);
    if ((int64_t)s->batch * s->n_nodes > 0x7fffffffLL || p.nchunk > 65535) return YGG_ERR_UNSUPPORTED;
    if (int32_t rc = check_workspace(workspace, workspace_bytes, p.part_bytes + p.oldlen_bytes)) return rc;

    AcceptArgs a{};
    a.target_logits = target_logits; a.target_tokens = target_tokens;
    a.parent_idx = parent_idx; a.token_ids = token_ids;
    a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_cache; a.v_cache = v_cache;
    a.seq_lens = seq_lens; a.accept_len = accept_len; a.accept_path = accept_path; a.bonus_token = bonus_token;
    a.part = workspace;
    a.old_len = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + p.part_bytes);
    a.B = s->batch; a.N = s->n_nodes; a.D = s->depth; a.V = s->vocab; a.Hkv = s->n_kv_heads; a.Dh = s->head_dim;
    a.n_layers = n_layers; a.chunk = p.chunk; a.nchunk = p.nchunk; a.max_seq_len = s->max_seq_len;
    a.elem_bytes = s->kv_dtype == YGG_F32 ? 4 : s->kv_dtype == YGG_BF16 ? 2 : 1; a.cap = s->kv_capacity;
    return launch_accept(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? YGG_OK : YGG_ERR_LAUNCH;
}

}  // extern "C"
