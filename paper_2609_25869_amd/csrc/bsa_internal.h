// Internal declarations shared by the host runtime and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bsa {

constexpr int kHeadDim = 128;

// SplitMix64 finaliser (Steele, Lea and Flood, "Fast splittable pseudorandom
// number generators", OOPSLA 2014).
__device__ inline uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// One workgroup task (Section 4.3): a contiguous slice [tile_begin, tile_end)
// of the active KV tiles of physical query tile `pq` of head `bh`
// (= b * heads + h).  `split` is the slice's ordinal among the row's `nsplit`
// slices; nsplit > 1 means the row is reduced by Split-K.
struct Task {
  int32_t bh, pq, tile_begin, tile_end, split, nsplit, pad0, pad1;
};
static_assert(sizeof(Task) == 32, "Task is 32 bytes");

// Per-head facts for the mask kernels.
struct HeadDesc {
  int64_t mask_off;  // offset of the head's mask inside one batch
  int32_t nqb, nkb;  // logical block grid
  int32_t seg;       // geometry segment
  int32_t pad;
};

// Device-side statistics of one segment (integer atomics only).
struct SegStats {
  unsigned long long nnz, run_blocks, max_row_nnz, pad;
};

// A range of logical rows inside one (b, h), reduced by one workgroup.
struct RowChunk {
  int64_t begin, end;
  int32_t bh, seg;
};

struct MaskStateArgs {
  const uint8_t* mask;
  int64_t stride_b;
  const HeadDesc* heads;
  const int64_t* row_base;  // [B*H + 1], logical rows of (b, h) start here
  int32_t H, nbh;
  int64_t R;
  int32_t* counts;          // [R]   (count pass)
  int32_t* runs;            // [R]   (count pass) active blocks of the row in runs of length >= 2
  const RowChunk* chunks;   // [nchunks] (count pass) reduction ranges
  int32_t nchunks;
  int64_t* chunk_sum;       // [nchunks] (count pass) active blocks of each chunk
  const int64_t* row_ptr;   // [R+1] (fill pass)
  int32_t* col_idx;         // [nnz] (fill pass)
  uint64_t* row_hash;       // [R] (fill pass, may be null) see RowHash in plan_kernels.hip
  SegStats* seg_stats;      // [nseg]
  unsigned long long* bh_nnz;  // [B*H]
  int32_t wide;             // every mask row starts 4-byte aligned and nkb % 4 == 0
};

struct MapArgs {
  const uint8_t* mask;
  int64_t stride_b;
  const HeadDesc* heads;
  const int32_t* seg_heads;  // heads of the segment, ascending
  int32_t nsh, H;
  int32_t npq, npk;          // physical grid of one head
  int32_t nqb, nkb;          // logical grid of one head
  int32_t gq, gkv, rq, rkv;  // members per tile / tiles per block along Q and KV
  int64_t Rp;                // physical rows of the segment = B * nsh * npq
  int32_t* counts;           // count pass
  const int64_t* tile_ptr;   // fill pass
  int32_t* tile_kv;
  uint64_t* member;          // may be null (no membership metadata)
  // Compacted list of a tile list with gkv == 2 (null: none): one entry per
  // KV block of the row with an active member, bit a of its member word for
  // query block a.
  int32_t* counts2;          // count pass
  const int64_t* tile_ptr2;  // fill pass
  int32_t* tile_kv2;
  uint64_t* member2;         // may be null
  // Fill pass, plans without Split-K (null: none): the row's task, and the
  // hash of its list for the dispatch order.
  Task* tasks;
  uint64_t* row_hash;
  int32_t wide;              // mask rows 4-byte aligned and nkb % 4 == 0 (see MaskStateArgs)
};

struct TaskArgs {
  const int64_t* tile_ptr;   // physical (or, for Direct, logical) row offsets
  const int64_t* row_base;   // logical row base per (b, h); used when direct
  const int32_t* seg_heads;
  int32_t nsh, H, npq, split;
  int32_t direct;
  int32_t grain;             // list entries that stay together (2 for compacted lists, else 1)
  int64_t Rp;
  int32_t* counts;           // count pass (split > 1)
  const int64_t* task_ptr;   // fill pass (split > 1), null when split == 1
  Task* tasks;
};

// Dispatch order of a segment's tasks (task_order.hip): a permutation of the
// task indices, row order with every task moved up to the first task that
// has the same KV tile list (and member bits).  Work arrays are [ntasks].
struct OrderArgs {
  const Task* tasks;
  const int64_t* ntasks_dev;  // device task count (may be null)
  int64_t ntasks;             // exact count, or the bound when ntasks_dev is set
  const int32_t* tile_kv;
  const uint64_t* member;     // may be null
  uint64_t* table_key;        // [table_size] list hashes (0: free slot)
  int32_t* table_min;         // [table_size] lowest task index per hash
  int64_t table_size;         // a power of two >= 2 * ntasks
  int32_t* task_slot;         // table slot of each task
  int32_t* idx_in;
  uint32_t* rep;              // representative task of each task
  uint32_t* rep_sorted;
  int32_t* order;             // out; the first (device count) entries are the real tasks
  Task* tasks_out;            // out (may be null): tasks[order[i]] at i; only without a device count
  void* temp;
  size_t temp_bytes;
};

// The same order for plans without Split-K, whose tasks are the physical rows
// ((b, head) by (b, head), npq rows each), from the rows' list hashes.
struct RowOrderArgs {
  const uint64_t* row_hash;   // by segment row, or (direct) by logical row
  const int64_t* row_base;    // logical row base per (b, h); used when direct
  const int32_t* seg_heads;
  int32_t nsh, H, npq, direct;
  int32_t nbh;                // (b, head) pairs of the segment
  const Task* tasks;
  int32_t* order;             // out
  Task* tasks_out;            // out: tasks[order[i]] at i
};
constexpr int32_t kRowOrderMax = 2048;  // most rows per (b, head)

struct AttnArgs {
  const Task* tasks;
  int32_t ntasks;              // exact count, or an upper bound when ntasks_dev is set
  const int64_t* ntasks_dev;   // device count (may be null)
  const int32_t* order;        // dispatch order of the tasks (may be null: as built)
  const int32_t* kv_tile;
  const uint64_t* member;      // null: every tile is fully active
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* o;
  float* lse;                  // may be null
  float* ws;                   // Split-K partial states (may be null when no row splits)
  const int64_t* row_task;     // Split-K: first task of each physical row (may be null otherwise)
  int64_t nrows;               // physical rows
  int64_t qs0, qs1, qs2, ks0, ks1, ks2, vs0, vs1, vs2, os0, os1, os2;
  int32_t H, Nq, Nkv;
  int32_t bq_shift, bkv_shift;  // log2 of the logical block sizes
  int32_t gq, gkv;              // membership grid of a list entry
  int32_t unit;                 // 16: the list entries are 16-token columns (gkv = 1); else whole tiles
  float scale_log2;             // log2(e) / sqrt(d)
  int32_t slot_group, slot_run; // launch-slot to task map: XCDs per group (1, 2, 4 or 8) and run length
  int32_t balanced;             // nonzero: group g's share of the task list is [share_lo[g], share_lo[g + 1])
  int32_t share_lo[5];
  int64_t slot0;                // first launch slot of this launch
  int64_t launch_slots;         // slots per launch (0: all in one)
  int64_t nslots;               // launch slots (0: the task count rounded up to 8)
};

// Kernel launchers (defined in the .hip files).
hipError_t launch_mask_count(const MaskStateArgs& a, hipStream_t s);
hipError_t launch_mask_fill(const MaskStateArgs& a, hipStream_t s);
hipError_t launch_mask_scan(const MaskStateArgs& a, int64_t* row_ptr, int64_t* scan_tmp, int32_t nseg,
                            unsigned long long* stats_host, hipStream_t s);
hipError_t launch_row_order(const RowOrderArgs& a, hipStream_t s);
hipError_t launch_scan_i32(const int32_t* in, int64_t* out, int64_t n, int64_t* block_tmp, hipStream_t s);
int64_t scan_tmp_elems(int64_t n);
hipError_t launch_map_count(const MapArgs& a, hipStream_t s);
hipError_t launch_map_fill(const MapArgs& a, hipStream_t s);
hipError_t launch_task_count(const TaskArgs& a, hipStream_t s);
hipError_t launch_task_fill(const TaskArgs& a, hipStream_t s);
// Count, offsets and fill of at most kTasksOneBlock rows in one launch.
constexpr int64_t kTasksOneBlock = 1024;
hipError_t launch_tasks_one_block(const TaskArgs& a, int64_t* task_ptr, hipStream_t s);
hipError_t launch_attention(int tq, int tkv, int waves, int stages, const AttnArgs& a, hipStream_t s);
int64_t task_order_table_size(int64_t n);
hipError_t task_order_temp_bytes(int64_t n, size_t* bytes);
hipError_t launch_task_order(const OrderArgs& a, hipStream_t s);
hipError_t launch_splitk_merge(int tq, const AttnArgs& a, hipStream_t s);

// Top-k sparsifier (sparsify.hip) over heads [bh0, bh0 + nbh): block means
// (fp64, [nbh][nb][128]) of Q (index 0) and K (index 1), bf16 [B, N, H, 128]
// tensors; fp32 scores [nbh][nqb][nkb] with, per head, `nparts` partial
// maxima of the mean keys' 2-norms; the uint8 mask rows they select.
struct MeanArgs {
  const uint16_t* x[2];
  int64_t s0[2], s1[2], s2[2];
  int32_t n[2], blk[2], nb[2];
  int32_t H, bh0, nbh;
  double* out[2];
};
struct SelectArgs {
  float* scores;  // room for sparsify_score_rows(rows) rows; not kept
  const float* knorm;
  int32_t nparts;
  const double* pq;
  const double* pk;
  int64_t rows;  // nbh * nqb
  int32_t nqb, nkb, k, diagonal, nq, nkv, bq, bkv, bh0;
  uint8_t* mask;
};
int32_t sparsify_max_kv_blocks();
int64_t sparsify_score_rows(int64_t rows);  // score rows of whole selection workgroups
int32_t sparsify_norm_parts(int32_t nkb);  // room per head for the partial maxima
hipError_t launch_block_mean(const MeanArgs& a, hipStream_t s);
hipError_t launch_block_scores(const double* pq, const double* pk, int32_t nqb, int32_t nkb, int32_t nbh,
                               float* scores, float* knorm, int32_t* nparts, hipStream_t s);
hipError_t launch_topk_select(const SelectArgs& a, hipStream_t s);

}  // namespace bsa
