// Internal helpers shared by the HIP sources of the library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// XCD segment [s0, s1) of a head: the entries x, x+1 of its segment table (clamped into [0, m] and
// made non-decreasing), or without a table n_xcd segments of equal row count, the first m mod n_xcd
// one row longer.
__host__ __device__ inline void xcd_segment(int x, int m, int n_xcd, const int32_t* seg, int* s0, int* s1) {
  if (seg) {
    const int a = min(max(seg[x], 0), m);
    *s0 = a;
    *s1 = min(max(seg[x + 1], a), m);
  } else {
    const int base = m / n_xcd, extra = m % n_xcd;
    *s0 = x * base + (x < extra ? x : extra);
    *s1 = *s0 + base + (x < extra ? 1 : 0);
  }
}

// Workgroups per compute unit of a wave (Sec. IV-D): part of the definition of the default permutation and of
// the tail order, so fixed per shape rather than following the kernel's occupancy as it changes.
__host__ __device__ constexpr int wave_wgs(int d, int block) { return block == 128 ? 2 : d == 128 ? 4 : 6; }

// Scheduler state of one attention call, in the caller's workspace: a task counter per queue (queue x holds segment x of
// every head, heads in order; see spread_counters) and, per queue, from 64, the prefix sums of its segment lengths
// over the heads.
__host__ __device__ inline size_t sched_ints(int64_t bh, int n_xcd) { return 64 + (size_t)n_xcd * (bh + 1); }

// The last tail_heads(bh, m) heads of every queue run in an order built at each call (the tail
// order table, n_xcd x tail_heads x m int32 after the prefix tables): at most kTailEntries entries
// and kTailMaxHeads heads per queue.
constexpr int kTailEntries = 16384;
constexpr int kTailMaxHeads = 256;
__host__ __device__ inline int tail_heads(int64_t bh, int m) {
  if (bh <= 0 || m <= 0) return 0;
  int64_t w = kTailEntries / m;
  if (w > kTailMaxHeads) w = kTailMaxHeads;
  return (int)(bh < w ? bh : w);
}
__host__ __device__ inline size_t tail_offset(int64_t bh, int n_xcd) { return (sched_ints(bh, n_xcd) + 63) / 64 * 64; }
// Head-interleaved queue order (the alternative to heads in order): after the tail table, 64 queue
// offsets, then one entry h * m + slot per task, each queue's tasks round-robin over the heads.
__host__ __device__ inline size_t ilv_offset(int64_t bh, int m, int n_xcd) {
  return (tail_offset(bh, n_xcd) + (size_t)n_xcd * tail_heads(bh, m) * (m > 0 ? m : 0) + 63) / 64 * 64;
}
__host__ __device__ inline size_t sched_state_ints(int64_t bh, int m, int n_xcd) {
  return ilv_offset(bh, m, n_xcd) + 64 + (size_t)(bh > 0 ? bh : 0) * (m > 0 ? m : 0);
}

// The task counters: spread evenly over kCounterInts int32 behind the state where the memory has room for them (it does
// in a workspace, which is sized for 64 queues, but for the smallest calls with many queues), else the first 64
// int32. Atomics on one line serialise across the device, and a launch takes thousands. Eight counters in 32
// bytes, 32 bytes apart and 512 bytes apart: 70 x 83 rows (d 128) 454, 383 and 366 us, 20 x 338 rows of 64-token
// blocks (d 128) 648, 556 and 515 us.
constexpr int kCounterInts = 1024;
inline void spread_counters(int32_t* sched, size_t have_ints, int64_t bh, int m, int n_xcd, int32_t** counters, int32_t* step) {
  const size_t end = (sched_state_ints(bh, m, n_xcd) + 63) / 64 * 64;
  const bool room = end + kCounterInts <= have_ints;
  *counters = room ? sched + end : sched;
  *step = room ? kCounterInts / n_xcd : 1;
}

// Split rows. A launch with few rows ends when its longest row does, so a row of more than L kept
// blocks is computed in chunks by several workgroups: each chunk leaves its unnormalised O, row
// maxima and row sums in a float32 tile, and the workgroup that finishes a row's last chunk merges the
// tiles in chunk order. L follows from the lists and the device alone (see split_plan), so a row is
// split the same way in every execution order. The tiles take at most kPartBytes; L grows until
// the chunks fit. Launches of more than kSplitMaxTokens / block rows never split: their rows are short
// next to the launch (a row there outlasts its share of the launch only below 0.5% density).
// Shortest L. At 8 a launch of 44 x 29 rows of 4.6 of 64 blocks on average takes 47 us instead of 38 and one of 8 x 120
// rows of 11 blocks 82 instead of 43 (the merge costs about as much as ten blocks); 2 x 64 rows take 29
// instead of 31.
constexpr int kSplitMinBlocks = 12;
constexpr size_t kPartBytes = (size_t)32 << 20;
constexpr int64_t kSplitMaxTokens = (int64_t)1 << 22;
__host__ __device__ inline size_t part_tile_floats(int block, int d) { return (size_t)block * (d + 2); }
__host__ __device__ inline int split_cap(int64_t bh, int m, int block, int d) {
  if (m <= kSplitMinBlocks || bh * m > kSplitMaxTokens / block) return 0;
  const int64_t cap = (int64_t)(kPartBytes / (part_tile_floats(block, d) * 4));
  const int64_t most = bh * m * ((m + kSplitMinBlocks - 1) / kSplitMinBlocks);
  return (int)(most < cap ? most : cap);
}
// Split state: [0] chunk tasks, [1] L; the counters of chunks taken, one per shard of them, spread as the queues' are;
// from kSplitHead the tasks {head, row, chunk | chunks << 16, the row's first tile}; then one arrival
// counter per tile (the row's first tile counts the row), 64 bytes apart.
constexpr int kSplitShards = 8;
constexpr int kSplitHead = 64 + kCounterInts;
__host__ __device__ inline int split_counter(int shard) { return 64 + shard * (kCounterInts / kSplitShards); }
__host__ __device__ inline size_t split_arrival(int cap, int tile) { return kSplitHead + 4 * (size_t)cap + 16 * (size_t)tile; }
__host__ __device__ inline size_t split_ints(int cap) { return (split_arrival(cap, cap) + 63) / 64 * 64; }

// Lane moves through DPP (a few cycles, where a lane shuffle is an LDS round trip): lanes that the
// control leaves without a source, or that the row mask excludes, take `old`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp32(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xf, false);
}
// Inclusive prefix sum over the lanes: shifts by 1, 2, 4 and 8 within each row of 16, then the
// broadcasts of lane 15 into rows 1 and 3 and of lane 31 into rows 2 and 3.
__device__ __forceinline__ int lane_prefix_sum(int x) {
  x += dpp32<0x111, 0xf>(0, x);  // row_shr:1
  x += dpp32<0x112, 0xf>(0, x);  // row_shr:2
  x += dpp32<0x114, 0xf>(0, x);  // row_shr:4
  x += dpp32<0x118, 0xf>(0, x);  // row_shr:8
  x += dpp32<0x142, 0xa>(0, x);  // row_bcast:15
  x += dpp32<0x143, 0xc>(0, x);  // row_bcast:31
  return x;
}

}  // namespace wa

// Launch helpers (implemented in the .hip sources, called by the ABI layer).
struct WaAttnLaunch {
  const void* q;
  const void* k;
  const void* v;     // null when the caller passes V already transposed (vt)
  void* vt;          // V transposed to [bh][head_dim][mb*block], zero-padded: the caller's, or the
                     // workspace copy that the launch writes from v
  int32_t* sched;    // workspace: sched_state_ints(bh, mb, n_xcd) int32 (prefix tables at 64, the tail order
                     // table at tail_offset(bh, n_xcd))
  int32_t* counters;      // queue x's task counter at counters[x * counter_step]
  int32_t counter_step;
  int32_t split_cap;      // 0: no row is split
  int32_t* split;    // workspace: split_ints(split_cap) int32, then the tiles
  float* part;       // workspace: split_cap tiles of part_tile_floats(block, head_dim)
  const int32_t* row_ptr;  // [bh][mb+1], row r's list at col_idx + head mb^2 + row_ptr[r]; null:
  const int32_t* row_cnt;  // [bh][mb], row r's list at col_idx + head mb^2 + r mb
  const int32_t* col_idx;
  const int32_t* perm;
  const int32_t* seg;  // [bh][n_xcd+1] XCD segment starts, nullable
  void* o;
  float* lse;
  int32_t bh;        // batch * heads
  int32_t seq_len;
  int32_t mb;        // blocks per sequence
  int32_t head_dim;
  int32_t block;
  int32_t n_xcd;
  int32_t head_order;  // 0 heads in order within each queue, 1 round-robin over the heads
  int32_t* status;     // device word, nullable: bit 0 an invalid perm entry, bit 1 an invalid KV index
  float scale;         // softmax scale
};

namespace wa {
// List entries [beg, end) of row r of head h, relative to the head's list area. ARGS: a pointer to a
// WaAttnLaunch in any address space.
template <typename ARGS>
__device__ __forceinline__ void row_range(ARGS a, int h, int r, int32_t* beg, int32_t* end) {
  if (a->row_ptr) {
    const int32_t* rp = a->row_ptr + (int64_t)h * (a->mb + 1) + r;
    *beg = rp[0];
    *end = rp[1];
  } else {
    *beg = r * a->mb;
    *end = *beg + a->row_cnt[(int64_t)h * a->mb + r];
  }
}
}  // namespace wa

hipError_t wa_launch_attention(const WaAttnLaunch& a, hipStream_t stream);
// Order tables, split plan, cleared status word and, with a.v, the transposed copy of V, in one launch.
// grid: workgroups of the tail-order rule; slots: workgroups of the attention kernel the chip holds.
hipError_t wa_launch_attn_prep(const WaAttnLaunch& a, int grid, int slots, hipStream_t stream);
// device addresses and sizes of the calling device's static scheduler scratch and split-row scratch
// (looked up on first use)
hipError_t wa_noalloc_scratch(int32_t** ptr, size_t* bytes, int32_t** split, size_t* split_bytes);
hipError_t wa_launch_transpose_v(const void* v, void* vt, int64_t bh, int seq_len, int mb, int head_dim, int block,
                                 hipStream_t stream);
size_t wa_vt_bytes(int64_t bh, int mb, int head_dim, int block);

// row_ptr and the packed lists of every head
hipError_t wa_launch_compact(const uint8_t* mask, int bh, int mb, int32_t* row_ptr, int32_t* col_idx,
                             hipStream_t stream);
hipError_t wa_launch_row_count(const uint8_t* mask, int64_t rows, int n, int32_t* counts, int64_t count_stride_rows,
                               int counts_offset, int mb, hipStream_t stream);
hipError_t wa_launch_head_scan(int32_t* row_ptr, int bh, int mb, hipStream_t stream);
// row_ptr: the lists packed per head; null: row r's list at col_idx + r n and its length in counts[r]
hipError_t wa_launch_row_write(const uint8_t* mask, int bh, int mb, int n, const int32_t* row_ptr, int32_t* counts,
                               int32_t* col_idx, hipStream_t stream);
