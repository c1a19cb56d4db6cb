// Host-side planning for the paged attention kernels: validation of host metadata and the split-KV /
// shared-prefix work lists the kernels consume.  Pure C++ (no HIP), so it builds and tests on a CPU.
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/kvpattn.h"

namespace kvp {

constexpr int kPage = 16;
constexpr int kMaxColsPerWave = 16;   // query columns one wave's MFMA tile holds (members x heads)
constexpr int kMaxColsPerGroup = 64;  // query columns one shared-prefix workgroup holds (4 waves)
constexpr int kMinSegmentPages = 8;   // smallest page count of a decode wave segment
// A wave chunk's start (its item, query fragments and first page ids are dependent reads) in pages of
// streaming: bf16 pages, and FP8 pages (half the bytes, so a start is worth more of them).
constexpr int kChunkStartPages = 3;
constexpr int kChunkStartPagesFp8 = 5;
constexpr int kGroupChunkPages = 16;  // pages per workgroup of the LDS-staged shared-prefix kernel
// Decode waves per call: one round of the waves resident at once on 256 CUs (4 SIMDs x 2 waves each).
// Sweeps of 1024-16384 put the optimum here on the target workloads.
constexpr int kDecodeWaves = 2048;

// One unit of decode work: one KV head of it is processed by one wave (private, <= 16 query columns)
// or one 4-wave workgroup (shared prefix, <= 64 query columns).  Mirrors kvp_plan_decode's 8 ints.
struct DecodeItem {
  int32_t kind;      // 0 = private range of one sequence, 1 = shared prefix of a group (or subgroup)
  int32_t row;       // block-table row the pages are read from
  int32_t page_lo;   // first logical page
  int32_t page_hi;   // one past the last logical page
  int32_t tok_end;   // tokens [0, tok_end) of the row are valid
  int32_t mem_off;   // first entry in the member list (sequence ids owning the query columns)
  int32_t n_mem;     // member count; query columns = n_mem * G
  int32_t slot;      // partial index within each member's list, -1 = write the final output directly
};
static_assert(sizeof(DecodeItem) == 32, "DecodeItem is uploaded as raw bytes");

// A wave-path chunk as the kernel reads it, over the bus from pinned host memory: what a wave needs before its first
// page in one record, so that a chunk of one member starts after one such read.  The segment's chunk range, the item
// and its member list were three dependent reads of 1.3 us each (and the partial index a fourth, at the chunk's
// end): one sequence of 131,007 tokens 58.1 -> 54.5 us, RLHF 178.0 -> 174.9 us, mixed 369.8 -> 363.6 us, RLVR 1392.8
// -> 1376.5 us.  The other members of a chunk stay in the call's member list: records that hold them all (160 bytes
// for 16) leave RLHF at 175.2 us and cost the host 3 us per 1000 short sequences.
struct DecodeRec {
  int32_t row, page_lo, page_hi, tok_end;  // as in DecodeItem
  uint32_t kind_mem;          // kind, n_mem - 1 and mem_off (0 for one member) in 1, 4 and 27 bits
  int32_t next;               // record of the segment's next chunk, -1 = none
  int32_t seq, part;          // the first member and the index of its partial, -1 = write the output
};
static_assert(sizeof(DecodeRec) == 32, "two 16-byte reads");

constexpr int64_t kMaxSharedMembers = int64_t(1) << 27;  // offsets that kind_mem holds

struct DecodePlan {
  std::vector<DecodeItem> wave_items;   // chunks in segment order (private and <= 16-column prefix)
  std::vector<int32_t> seg_off;         // [segments + 1]: chunks of segment s are seg_off[s]..seg_off[s+1]
  std::vector<DecodeItem> group_items;  // prefix items with 16 < n_mem * G <= 64 (LDS-staged kernel)
  std::vector<int32_t> members;         // member lists referenced by items
  std::vector<int32_t> part_base;       // [B] first partial index of each sequence
  std::vector<int32_t> n_parts;         // [B] partial count of each sequence
  std::vector<int32_t> merge_seqs;      // sequences whose output the merge kernel writes (0 or >= 2 parts)
  int32_t total_parts = 0;
  int32_t pages_per_split = 0;          // pages per wave segment
  int32_t group_reserved_blocks = 0;    // block slots the wave budget leaves to the shared-prefix path
};

// Prefill: one workgroup per (session, kv head, 256-row query tile, key range).  The key range is
// a run of 64-key stages [st_lo, st_hi) (st_hi is clamped to the tile's own last stage); a tile whose
// history is split over several workgroups writes one partial softmax state per range, merged per query
// row by log-sum-exp afterwards.
struct PrefillItem {
  int32_t seq;       // session index (block-table row)
  int32_t kvh;       // KV head
  int32_t row0;      // first flattened query row (position * G + head-in-group) of the tile
  int32_t st_lo;     // first 64-key stage of the range (st_lo * 64 <= the session's cached length)
  int32_t st_hi;     // one past the last stage of the range
  int32_t slot;      // partial index of the range within each query row's list, -1 = write the output
};

// An item as the kernels read it: the planner's item with what they would otherwise look up.
struct PrefillWork {
  int32_t seq, kvh, row0, st_lo;  // as in PrefillItem
  int32_t nst;       // stages of the range (>= 1)
  int32_t slot;      // as in PrefillItem
  int32_t ctx;       // the session's cached length
  int32_t q0;        // row of its first chunk token in q / out
  int32_t nrows;     // its flattened query rows
  int32_t n_keys;    // keys that any row of the tile sees
  int32_t part0;     // split sessions: first partial (row r owns part0 + r * nsplit ..)
  int32_t nsplit;    // key ranges per query row of the session
};
static_assert(sizeof(PrefillWork) == 48, "PrefillWork is uploaded as raw bytes");

struct PrefillPlan {
  std::vector<PrefillItem> items;  // blockIdx order (XCD-aware, empty entries have seq = -1)
  int64_t real_items = 0;
  std::vector<int32_t> nsplit;     // [B] key ranges per query row of each session (1 = not split)
  std::vector<int32_t> part_base;  // [B] first partial of each session (its row r owns part_base + r * nsplit)
  std::vector<int32_t> merge_info; // per merged query row: {row in q / out, first partial, nsplit, 0}
  int32_t total_parts = 0;
};

struct Status {
  int code = KVP_OK;
  std::string msg;
  bool ok() const { return code == KVP_OK; }
};

Status validate_group_prefix(const int32_t* lens, int B, const kvp_group_prefix* gp);
// chunk_start_pages: the start cost a segment's budget charges per chunk (kChunkStartPages for bf16
// pools, kChunkStartPagesFp8 for FP8 pools).
Status plan_decode(const int32_t* seq_lens, int B, int maxp, const kvp_group_prefix* gp, int Hq, int Hkv,
                   DecodePlan* plan, int chunk_start_pages = kChunkStartPages,
                   int64_t max_shared_members = kMaxSharedMembers);
// The wave path's records, one per chunk: segment s's first chunk is record s, its further chunks follow all the
// first ones.
void write_decode_recs(const DecodePlan& plan, DecodeRec* recs);
Status plan_prefill(const int32_t* ctx_lens, const int32_t* cu_q, int B, int maxp, int Hq, int Hkv,
                    PrefillPlan* plan);
// A plan's items as the kernels read them (ctx_lens, cu_q and G = Hq / Hkv as given to plan_prefill).
std::vector<PrefillWork> prefill_work(const PrefillPlan& plan, const int32_t* ctx_lens, const int32_t* cu_q, int G);
// 64-key stages of a plan's items on average, rounded down.
int64_t prefill_mean_stages(const PrefillPlan& plan);
Status check_tables(const int32_t* bt, int maxp, const int32_t* lens, int B, int num_pages,
                    const kvp_group_prefix* gp);

constexpr int kPrefillWaves = 8;                    // waves per prefill workgroup, 32 query rows each
constexpr int kPrefillRows = 32 * kPrefillWaves;    // flattened query rows per prefill workgroup
// A call whose tiles (x their 64-key stages) would not give about this many equal workgroups splits
// tile histories into key ranges: the resident prefill workgroups of 256 CUs (8 waves per CU).
constexpr int kPrefillSplitTarget = 256 * 8 / kPrefillWaves;
// Items of at least this many stages on average go to the kernel for long key ranges (bf16 pages, d = 128).  Its
// start must be paid back by what it saves per stage, which is the less the fewer query rows read each page: with
// fewer than 8 query heads per KV head more of a stage is the page itself.  700 calls of 1-32 sessions, chunks of
// 4-2048 tokens, histories of 200-65536 and 1-16 KV heads, that kernel's time over the other's (median, most):
//   8 or 16 heads: 18-30 stages 1.09, 1.19; 30-52: 1.02, 1.11; 52-64: 0.99, 1.04; 64-100: 0.97, 1.02; 100+: 0.94, 0.98
//   1, 2 or 4:     18-30 stages 1.12, 1.41; 30-52: 1.05, 1.14; 52-96: 1.01, 1.12; 96-150: 0.97, 1.00; 150+: 0.95, 0.99
constexpr int kPrefillLongStages = 64, kPrefillLongStagesFewHeads = 96;
inline bool prefill_long(bool bf16, int D, int G, int64_t mean_stages) {
  return bf16 && D == 128 && mean_stages >= (G >= 8 ? kPrefillLongStages : kPrefillLongStagesFewHeads);
}
// In the other kernel, items of fewer stages than this on average get a workgroup per half tile (twice the
// staging, but two workgroups on a CU overlap their starts and outputs).  Whole tiles' time over half tiles',
// d = 128: 2 stages 1.12, 4.5: 1.04, 8 (36 items) 1.10, 8 (128 items) 1.00, 8.5: 0.99, FP8 pages 12.5: 0.99, 68: 0.94.
constexpr int kPrefillHalfTileStages = 9;
constexpr int kPrefillMinSplitStages = 8;  // smallest key range of a split (512 keys)

}  // namespace kvp
