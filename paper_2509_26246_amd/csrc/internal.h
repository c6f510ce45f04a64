// Private declarations shared by the host builder, the table handle and the kernel launchers.
#pragma once
#include <cstdint>
#include <vector>

#include "../../include/slimattn.h"

namespace slimattn {

// Tile sizes for which work-lists are derived: query tiles of 64 (fp32 kernels) and 128 rows (bf16 forward,
// dQ), key tiles of 64 (fp32) and 256 rows (bf16 dK/dV).
constexpr int kNumTileSizes = 3;
constexpr int kTileSizes[kNumTileSizes] = {64, 128, 256};
inline bool is_query_tile(int rows) { return rows == 64 || rows == 128; }
inline bool is_key_tile(int rows) { return rows == 64 || rows == 256; }
inline int tile_index(int rows) {
  for (int i = 0; i < kNumTileSizes; ++i) if (kTileSizes[i] == rows) return i;
  return -1;
}

// A query tile: rows [q_row0, q_row0 + q_rows) of one sample whose first token is kv_start.
// Row i sees keys kv_start .. i.  The tile therefore needs keys [kv_start, q_row0 + q_rows).
struct QItem { int32_t q_row0, q_rows, kv_start, pad; };

// Groups of a list of 128-row query tiles, in list order: n[i] items for which one block of the one-head kernels takes 1 << share[i] query
// heads, as far as the size of the head group allows (four with groups of 4, 8, ..., two with other even ones).  The last tile of a sample
// leaves waves without rows where it has at most 64 (32); a block costs nearly the same, so there it takes a second head (three more)
// against the same keys.  16K tokens, 32/8 heads of 128, forward / dQ, us: samples of 64 rows 99 / 183 -> 72 / 125, 160 rows 109 / 203 ->
// 87 / 134, 272 rows 123 / 200 -> 103 / 161.  (The blocks that are saved must not be launched: as blocks that end at once the 64-row samples
// took 125 / 203.)  Only for lists without a tile of more than kSharedKeys keys: groups are heavy-first in themselves only, tails first, and
// with long samples beside them that order costs more than the few tails save (forward of a 32K pack of 18 samples by units: 1120 -> 1128 us).
// Launches that share no heads walk the list heavy-first (in groups, 32K tokens of short samples, forward: 40/40 heads of 128 457 -> 472 us,
// 32/32 353 -> 361).
constexpr int kSharedKeys = 1024;
struct QGroups {
  int n[3], share[3];
  int total() const { return n[0] + n[1] + n[2]; }
  static QGroups plain(int n_items) { return QGroups{{n_items, 0, 0}, {0, 0, 0}}; }
};
// The query tiles of a launch: heavy-first and, where tails may share blocks, the same tiles in groups (otherwise groups.total() is 0).
struct QList {
  const QItem* items;
  int n;
  const QItem* grouped;
  QGroups groups;
};
inline int query_share(const QItem& it) {
  return it.q_rows > 64 ? 0 : it.q_rows > 32 ? 1 : 2;
}

// A run of query rows [q_lo, q_hi) of one sample that belong to the launch scope.
struct Seg { int32_t q_lo, q_hi; };

// A key tile: rows [kv_row0, kv_row0 + kv_rows) of one sample, and the scope's query runs of that
// sample that end after kv_row0 (segs[seg_begin .. seg_end), ascending).  slot < 0: the item covers
// every such run and its block owns the tile's dK/dV.  slot >= 0: the item is one part of a heavy
// tile whose query rows were divided among several blocks; it covers only its own runs and stores
// its sums as fp32 partial tile number `slot`, which a reduction launch adds up in slot order.
// load_until, final_from: where the rows' sums come from and go to (below).  number: the item's place when every item of
// the list stores a partial tile (launches divided by query heads): a tile's items have consecutive numbers, in slot order.
struct KvItem { int32_t kv_row0, kv_rows, seg_begin, seg_end, slot, load_until, final_from, number; };

// A key row collects from every unit of the backward list that has query rows of the sample at or after it
// (a slice's dK/dV are complete only when all later slices have run: the paper's inter-slice dependency of
// the backward pass).  Units run in list order, and a unit reaches the rows before the end of its last query
// row in the sample.  So for the rows of a unit's key tile: rows below `load_until` (the furthest reach of an
// earlier unit) continue a partial sum that unit left in the fp32 accumulators, the others start from zero
// (nothing has to be cleared beforehand); rows from `final_from` on (the furthest reach of a later unit) get no
// further contribution and are written as dK/dV in the output type, the others go to the accumulators.  A
// row's gradient is thus released by its last contributor, not at the end of the list.  Whole-list scope:
// load_until = 0, final_from = 0.

// A divided key tile: partial tiles first_slot .. first_slot + n_parts - 1 are its parts.
struct KvReduce { int32_t kv_row0, kv_rows, first_slot, n_parts, load_until, final_from, pad0, pad1; };

// Divided lists exist for the 256-row key tile (the bf16 dK/dV kernels) and seven classes
// of KV-head count (a half, 1, 2, 4, 8, 16, >= 32): a launch has items x KV heads blocks, so the fewer KV heads, the
// fewer blocks share the work and the more a single long sample's first tiles dominate the makespan.
constexpr int kNumSplitTiles = 1;                               // key-tile sizes for which divided lists are built
constexpr int kSplitTileRows[kNumSplitTiles] = {256};           // the bf16 dK/dV kernels' item
// Slots the per-slot share of the work is taken over: 3/4 of the one-wave kernel's 256 resident blocks (measured: a
// part costs a V tile, K fragments and an fp32 partial tile to set up, and dividing more finely lost 1-4 %).
constexpr int kSplitBlockSlots[kNumSplitTiles] = {192};
inline int split_tile_index(int rows) { return rows == 256 ? 0 : -1; }
constexpr int kNumSplitClasses = 7;
// (The share of a class is taken over its lower end; with 8 as the last one a launch on 32 KV heads was divided four times too
// finely: 10567-token pack, 32/32 heads, dK/dV 499 + reduction 79 us against 458.)
inline int split_class(int n_kv_heads) {
  int c = 1;
  while (c + 1 < kNumSplitClasses && (1 << c) <= n_kv_heads) ++c;
  return c;
}
// The class of a launch (dkdv_launch below).  At head dim 64 six half items share a compute unit, and few KV heads leave little beside the divided tiles to even the
// parts out: 1 to 3 of them take the class below (one 32K sample of 8/1 heads 2329 -> 2153 us, a 32K pack of long ones 489 -> 466), unless
// its partial tiles alone would lift the workspace above the built-in scratch array's size.  (From 4 on no gain: 32K pack of 32/8 heads 2783 -> 2818.)

// Blocks of a dK/dV launch that share one item by query heads: a launch of few items (one small unit, a small pack, few KV
// heads) leaves most compute units idle while each of its blocks walks the item's rows once per head of the group.  Every
// block then stores a partial tile and all tiles go through the reduction, so the walk that is saved has to be worth
// that: a step takes about 1.35 us, the reduction launch and the partial tiles about 15 (876-row pack, 8 heads on one KV
// head: 5 blocks of up to 128 steps, 177 us; 40 blocks of up to 16, 40 us and 6 for the reduction).
// max_blocks: one per compute unit, or fewer where their partial tiles would lift a workspace that fits the built-in scratch array above
// its size (slimattn_bwd_static then still takes the pack, and computes the same).
constexpr int kHeadPartBlocks = 256;
inline int head_parts(int n_items, int n_kv_heads, int group, int longest_rows, int64_t max_blocks) {
  const int64_t blocks = (int64_t)n_items * n_kv_heads;
  const int parts = blocks > 0 ? (int)(max_blocks / blocks < group ? max_blocks / blocks : group) : 1;
  const int64_t steps = (int64_t)longest_rows * group / 32;
  return parts > 1 && steps - steps / parts >= 20 ? parts : 1;
}

// Whether a dK/dV launch at head dim 128 takes the kernel with 128 keys and two blocks per compute unit (dkdv_pair_bf16.hip): what an item costs
// beside its steps is then hidden by the other block, and steps before a wave's keys are skipped; a step of the one-wave kernel
// (dkdv_wide_bf16.hip) is cheaper.  What decides is therefore the steps an item has on average (its last part's where blocks share it).  Where
// the lines lie is measured, 16K to 32K tokens in samples of one length, one-wave kernel / this one, us:
//   one query head per KV head: 36 steps 883 / 829 (32 KV heads), 60 steps alike (18 launches, this one 0.99 of the other on average, 0.90 to 1.05), 68 steps 483
//   / 494, 229 / 242 (8);
//   two: 56 steps 857 / 815 (16), 72 and 80 steps alike, 88 steps 283 / 302 (4), 1202 / 1196, 112 steps 333 / 354, 1440 / 1469;
//   three and more: 84 steps 793 / 776 (10 KV heads of 3), 112 steps 829 / 768 (8 of 4), 247 / 256 (2 of 4), 120 steps 572 / 517 (5 of 6), 144 steps
//   984 / 997 (8 of 4).
// With one or two heads the lines are for launches of more than 256 items and KV heads.  Below that the one-wave kernel leaves compute units without a block, and
// the halves pay at any of these lengths: two heads, 112 steps, 2 samples on 4 KV heads 148 / 128, 4 on one 108 / 84.
inline bool short_walks(int64_t walk_rows, int n_items, int n_kv_heads, int group, int head_parts) {
  const bool fills = (int64_t)n_items * n_kv_heads * head_parts > 256;
  const int64_t most = group > 2 ? 112 : group == 2 ? (fills ? 80 : 112) : fills ? 64 : 68;
  return walk_rows * group <= most * 32 * n_items * head_parts;
}

// Blocks that share an item: `heads` by the query heads of the group, each of them `rows` by the steps of its walk (kernel of
// dkdv_pair_bf16.hip only).  What is left of the longest walk of a launch of few blocks then runs on compute units that are otherwise idle, a
// step in about 1.2 us; a further part costs its share of the item's first loads, 256 KB of partial tile to write and read (kRowPartTiles
// bounds them), and the reduction launch where there was none.  dK/dV and reduction, us: 876 rows of 8/1 heads of 128, 16 steps in 40 blocks 34.5,
// 8 in 80 29.0, 5 in 120 29; 1428 rows of 3/1 heads 29.1 -> 26.8; 900 rows of 16/4 heads, 64 blocks 35.1, 128 30.5.
constexpr int kRowPartTiles = 128;
struct DkdvParts {
  int heads, rows;
  bool pair;                                                    // the kernel of dkdv_pair_bf16.hip
  int total() const { return heads * rows; }
};
inline DkdvParts dkdv_parts(int n_items, int n_kv_heads, int group, int64_t walk_rows, int longest_rows, int head_dim, int64_t max_blocks) {
  DkdvParts p{head_parts(n_items, n_kv_heads, group, longest_rows, max_blocks), 1, false};
  p.pair = head_dim == 64 || short_walks(walk_rows, n_items, n_kv_heads, group, p.heads);
  const int64_t blocks = (int64_t)n_items * n_kv_heads * p.heads, tiles = max_blocks < kRowPartTiles ? max_blocks : kRowPartTiles;
  if (p.pair && blocks > 0 && blocks <= tiles / 2) {
    const int64_t steps = (int64_t)longest_rows * group / p.heads / 32;
    const int64_t rows = tiles / blocks < steps / 4 ? tiles / blocks : steps / 4;
    if (rows > 1 && steps - steps / rows >= (p.heads > 1 ? 6 : 12)) p.rows = (int)rows;
  }
  return p;
}

struct Range { int32_t begin, end; };

// A launch scope is either one unit or the whole list ("fused").  Its items are stored heavy-first.
struct ScopeLists {
  std::vector<int32_t> q_off[kNumTileSizes];    // per-unit offsets into q_items (size n_units + 1)
  std::vector<QItem> q_items[kNumTileSizes];    // unit-major, each unit heavy-first
  std::vector<int32_t> grouped_off;             // the 128-row tiles of units with tails that share blocks, once more in groups
  std::vector<QItem> grouped_items;
  std::vector<QGroups> q_groups;                // per unit
  std::vector<int32_t> kv_off[kNumTileSizes];
  std::vector<KvItem> kv_items[kNumTileSizes];
  std::vector<Seg> segs;                        // all units' runs (and the parts' cut runs), referenced by the items
  // key tiles with heavy tiles divided, per tile size; per KV-head class and unit a range of them (a class in which no tile of
  // the unit is divided shares the range of the class below if that one has none either)
  std::vector<Range> split_rng[kNumSplitTiles][kNumSplitClasses];
  std::vector<KvItem> split_items[kNumSplitTiles];
  std::vector<int32_t> reduce_off[kNumSplitTiles][kNumSplitClasses];
  std::vector<KvReduce> reduce_items[kNumSplitTiles][kNumSplitClasses];
  int32_t max_slots[kNumSplitTiles][kNumSplitClasses] = {};   // most partial tiles any one scope needs
  // the same lists when every item stores a partial tile (head_parts below): one reduction per tile, and per unit the rows
  // of the longest item's walk
  std::vector<Range> tile_rng[kNumSplitTiles][kNumSplitClasses];
  std::vector<KvReduce> tile_items[kNumSplitTiles];
  std::vector<int32_t> longest[kNumSplitTiles][kNumSplitClasses];
  std::vector<int64_t> walk_rows[kNumSplitTiles];             // per unit: rows of all the tiles' walks
};

struct DeviceLists {                            // device mirrors (pointers into one allocation)
  const QItem* q_items[kNumTileSizes];
  const QItem* grouped_items;
  const KvItem* kv_items[kNumTileSizes];
  const Seg* segs;
  const KvItem* split_items[kNumSplitTiles];
  const KvReduce* reduce_items[kNumSplitTiles][kNumSplitClasses];
  const KvReduce* tile_items[kNumSplitTiles];
};

}  // namespace slimattn

struct slimattn_tables {
  int32_t n_samples = 0, n_slices = 0, n_units[2] = {0, 0};
  int64_t total_tokens = 0;
  int32_t max_sample_len = 0;
  int32_t mean_keys = 0;          // keys a row sees, on average over the pack's rows
  std::vector<int32_t> cu;
  std::vector<slimattn_slice> slices;
  std::vector<int32_t> unit_ptr[2], unit_slices[2];      // [0] forward list, [1] backward list
  slimattn::ScopeLists per_unit[2];                       // one scope per unit of each list
  slimattn::ScopeLists fused;                             // one scope: every slice (same for both passes)
  slimattn::DeviceLists d_per_unit[2], d_fused;
  const int32_t* d_cu = nullptr;
  const slimattn_slice* d_slices = nullptr;
  void* d_blob = nullptr;
  void* h_staging = nullptr;      // pinned copy of the tables for an upload queued on a stream (kept until destroy)
  int device = -1;
};

namespace slimattn {

// A launch may have at most 2^32 - 1 threads in a dimension, and the kernels' lists one item per sample: packs of very many short
// samples are launched in runs of the list.  f(first, count) launches a run and returns a hipError_t.
constexpr int64_t kMaxBlocks = int64_t(1) << 22;
template <class F>
int in_runs(int n_items, int64_t blocks_per_item, F&& f) {
  const int run = (int)(kMaxBlocks / blocks_per_item > 0 ? kMaxBlocks / blocks_per_item : 1);
  int e = 0;
  for (int a = 0; a < n_items && e == 0; a += run) e = f(a, n_items - a < run ? n_items - a : run);
  return e;
}

struct LaunchCtx {
  const slimattn_params* p;
  void* stream;           // hipStream_t
  int64_t T;
  int mean_keys;          // keys a row of the pack sees on average
};

// ---- forward launches whose keys are divided among blocks ------------------------------------------------------------
// A few query tiles against a long prefix (prefill by slices) are a launch of few blocks with a long serial walk: 1024 rows of
// 8 heads after 31K keys are 32 blocks of 500 key tiles for 256 compute units.  The launch then has `parts` blocks per
// (item, heads), each walking a run of the item's key tiles and moving its reference by itself (all start at the row's score against
// the sample's first key), and stores unnormalised O, reference and row sum in fp32; a second kernel adds the parts up in order.
// Row sums and O are sums over fewer terms than before.
//
// The forward has no workspace argument and allocates nothing, so the partial results live in one of kSplitRegions arrays
// (34 MB each) built into the library, one set per device.
// A region belongs to a launch from its claim kernel to its last finishing block, both on the caller's stream: the claim is an
// atomic compare-and-swap of a region's owner from 0 to the launch's ticket (a process-wide counter), decided on the
// device each time the launch runs, so calls on any streams and threads and replays of captured graphs never share a region.
// A launch that finds all of them taken, by launches that run at the same time, is not divided among blocks: its parts are
// walked one after another by the finishing kernel's blocks and added up in the same order by the same operations, so that
// o and lse have the same bits either way.  No launch waits for another.  (Executable graphs made from one capture carry
// one ticket; they also write the same o and lse, and may not run at the same time.)
constexpr int kSplitRegions = 2;
constexpr int kSplitUnits = 512;                                // (item, part, head) results of 128 rows per region: 256 compute
                                                                // units x 2 heads per block, or 2 blocks per unit x 1 head
constexpr int kSplitMinRows = 48 * 64;                          // shortest prefix that is divided
template <int D> constexpr int kSplitUnitFloats = 128 * D + 256;   // O^T, then per wave 32 references and 32 row sums
constexpr size_t kSplitRegionFloats = (size_t)kSplitUnits * kSplitUnitFloats<128>;
struct SplitState {
  unsigned long long owner[kSplitRegions];
  unsigned done[kSplitRegions];   // finishing blocks that are through
  unsigned long long launches[2]; // launches so far: added up from a region, walked part by part (slimattn_fwd_divided_counts)
};
struct FwdSplit {
  float* data;                    // the device's regions
  SplitState* state;
  unsigned long long ticket;
  int parts;                      // blocks per (item, heads): 1 = not divided
  int target;                     // key tiles per part (at least; shorter items take fewer parts)
};

// Fills in `sp` for a launch of n_items query tiles and claims a region on the stream; parts = 1 where division does not pay.
int split_begin(const LaunchCtx&, int n_items, int divide_rows, FwdSplit* sp);
// For a launch that fails behind split_begin: gives back, on the stream, what its claim may have taken.
void split_abandon(const LaunchCtx&, const FwdSplit& sp);
// Looks up the current device's regions (at table creation, so that launches find them ready, also under stream capture); hipError_t.
int prepare_split_regions();

// Kernel launchers (defined in the .hip files).  Each returns a hipError_t as int.
int launch_fwd_f32(const LaunchCtx&, const float* q, const float* k, const float* v, float* o, float* lse,
                   const QItem* items, int n_items);
// also writes delta = rowsum(dO * O) of the rows of the listed query tiles, which the dK/dV launch reads
int launch_bwd_dq_f32(const LaunchCtx&, const float* q, const float* k, const float* v, const float* o, const float* dO,
                      const float* lse, float* delta, float* dQ, const QItem* items, int n_items);
// longest: rows of the longest walk of a whole-list launch, whose accumulators may be used to divide the walks; 0 otherwise
int launch_bwd_dkdv_f32(const LaunchCtx&, const float* q, const float* k, const float* v, const float* dO, const float* lse,
                        const float* delta, float* acc_dk, float* acc_dv, float* dK, float* dV, const KvItem* items,
                        int n_items, const Seg* segs, int longest);

// divide_rows: keys the longest item sees, if the keys of the items may be divided among blocks (below); 0: one block walks them
int launch_fwd_bf16(const LaunchCtx&, const void* q, const void* k, const void* v, void* o, float* lse, const QList& list, int divide_rows);
// even group sizes at head dim 128: one wave per SIMD, two heads per wave (fwd_wide_bf16.hip)
int launch_fwd_wide_bf16(const LaunchCtx&, const void* q, const void* k, const void* v, void* o, float* lse,
                         const QItem* items, int n_items, const FwdSplit& sp);
// Row statistics of the bf16 backward (-lse*log2e and -delta = -dO.O per row and head, as bf16 triples):
// either the dQ kernel computes and stores them for the rows it owns (own_stats != 0; `o`, `lse` read), or
// the prepass below has stored them for the rows of the same query tiles and the dQ kernel reads them
// (own_stats == 0).  Either way only rows of the launch scope are read.
int launch_bwd_stat_bf16(const LaunchCtx&, const void* o, const void* dO, const float* lse, void* stat3, const QItem* items,
                         int n_items);
int launch_bwd_dq_bf16(const LaunchCtx&, const void* q, const void* k, const void* v, const void* dO, const void* o,
                       const float* lse, void* stat3, int own_stats, void* dQ, const QList& list);
// head_dim 128, long walks: one wave per SIMD, 256 key rows per block (dkdv_wide_bf16.hip)
int launch_bwd_dkdv_wide_bf16(const LaunchCtx&, const void* q, const void* k, const void* v, const void* dO, const void* stat3,
                            float* acc_dk, float* acc_dv, void* dK, void* dV, const KvItem* items, int n_items, const Seg* segs,
                            float* parts, int head_parts);
// head_dim 64, and 128 with short walks: two or three blocks of 128 key rows per compute unit (dkdv_pair_bf16.hip); same arguments
int launch_bwd_dkdv_pair_bf16(const LaunchCtx&, const void* q, const void* k, const void* v, const void* dO, const void* stat3,
                              float* acc_dk, float* acc_dv, void* dK, void* dV, const KvItem* items, int n_items, const Seg* segs,
                              float* parts, const DkdvParts& by);
// adds up the partial tiles (tile_rows rows each) of divided key tiles, in slot order, into dK/dV or the
// fp32 accumulators; per_slot: partial tiles per slot (the blocks that share an item by query heads)
int launch_bwd_reduce_bf16(const LaunchCtx&, const float* parts, float* acc_dk, float* acc_dv, void* dK, void* dV,
                           const KvReduce* items, int n_items, int tile_rows, int per_slot);

// How the bf16 dK/dV launch of a scope runs, unit u of t->per_unit[1] or t->fused (u = 0): the division class of its items and the blocks that
// share one.  The launch, the workspace's size and slimattn_bwd_dkdv_plan all go by it.
struct DkdvLaunch { int cls; DkdvParts by; };
DkdvLaunch dkdv_launch(const slimattn_tables* t, const ScopeLists& scope, int u, int32_t hq, int32_t hkv, int32_t d);

// Looks up the built-in scratch array of slimattn_bwd_static on the current device (so that the first such call
// finds it ready); returns a SLIMATTN_* code.
int prepare_static_scratch();

// Tile sizes each kernel family uses (must be one of kTileSizes).
int fwd_q_tile(int dtype, int head_dim);
int dq_q_tile(int dtype, int head_dim);
int dkdv_kv_tile(int dtype, int head_dim);
}  // namespace slimattn
