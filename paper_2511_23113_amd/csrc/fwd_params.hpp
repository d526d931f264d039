// Kernel argument block of the forward pass (device pointers and sizes only).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

constexpr int kTilesInPlace = 14;       // a wave merges a split row in place up to so many tiles, see launch_fwd
constexpr int kMaxTilesPerWave = 4;     // and has at most so many of every chunk (Cfg::TPW)

struct dbsp_fwd_params {
  const uint16_t* q;   // bf16 [B,H,nQ*BLK,D]
  const uint16_t* k;   // bf16 [B,H,nK*BLK,D]
  const uint16_t* v;   // bf16 [B,H,nK*BLK,D]
  uint16_t* o;         // bf16 [B,H,nQ*BLK,D]
  float* lse;          // f32  [B,H,nQ*BLK] or null
  const int32_t* kv_idx;
  const int32_t* empty_rows;
  const int32_t* part_ptr;    // [P + 1] where in sched the workgroups' lists begin
  const int32_t* sched;       // 8 x int32 per item: the partitions' lists, then the shared queue: head, row, first KV word, blocks, slot; of split rows also index of the row, its chunks, its first slot
  uint32_t* queue;            // [0] next queue position, [1 + t] times tail item t was taken
  float* part_o;       // f32 [B][n_slots][BLK][D], every chunk as its waves' lanes hold it
  float* part_lse;     // f32 [B][n_slots][BLK]
  uint32_t* split_cnt; // [B][n_split][waves of a workgroup] chunks of a split row that are done; zero between launches
  const int32_t* split_rows;  // 4 x int32 per split row: row, first slot, chunks, 0
  uint64_t* busy;      // [P]
  uint32_t* hw_id;     // [P]
  int32_t B, H, nQ, nK;     // nQ: rows per head of the plan (pair mode: pairs of query blocks); nK: KV blocks
  int32_t Nq, Nk;           // tokens per head
  int32_t n_slots, n_split, n_empty, n_tail;
  int32_t n_placed;         // items the partitions' lists hold (all of them but the shared queue's)
  int32_t max_chunks;       // the most chunks a split row has; 0: no split rows
  int32_t in_place_ok;      // split_cnt may be used, and there are no more items than partitions, all batch entries counted
  int32_t local;            // a slice's barrier may leave two slices' copies under way, see dbsp_launch_fwd: the plan's placement is the
                            // round-based one, or a greedy one that has more than an item for a workgroup or leaves an eighth of the chip idle
  int32_t merge_later;      // set by dbsp_launch_fwd: split rows are merged by a kernel of their own behind this one
  float scale;         // softmax scale
  float scale_log2;    // softmax scale * log2(e)
};

// Enqueues the persistent kernel, and behind it a merge kernel for split rows where that is faster: `grid`
// workgroups, enough to reach every partition that has items (all of them unless the plan has fewer items
// than partitions).
// pair: the plan's rows are pairs of 64-token query blocks and its units pairs of 64-token KV blocks (d = 128 only).
hipError_t dbsp_launch_fwd(const dbsp_fwd_params& p, int block, int d, bool pair, int grid, hipStream_t stream);
