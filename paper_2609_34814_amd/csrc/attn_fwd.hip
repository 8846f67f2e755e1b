// Block-sparse attention forward for gfx950 (MI355X).
//
// One workgroup computes one query block (Sec. II-C: query blocks in the outer
// loop, the mask-selected KV blocks in the inner loop, the online-softmax state
// and partial O kept on chip). The workgroup has BLK/32 wavefronts; wavefront w
// owns query rows [32w, 32w+32) of the block. Two workgroups share a CU.
//
// Data movement. K_j (natural [token][d] layout) and V_j^T (from a transposed,
// zero-padded [d][N_pad] copy of V made once per call) are copied from global
// memory straight into LDS with global_load_lds_dwordx4 (no register staging;
// K rows past the end of the sequence are clamped to the last row and masked). Only explicit vmcnt waits order these copies against LDS
// reads, so the copy into one tile stays in flight while the other tile is read.
// The LDS tiles are XOR-swizzled at 16-byte granularity so that the MFMA operand
// reads are free of bank conflicts; the swizzle is applied by choosing each
// lane's global source chunk. The loads of K_{j+1} are issued as soon as every
// wavefront has finished reading K_j and overlap the softmax and P V of block j;
// the loads of V_{j+1} overlap the next Q K^T.
//
// Arithmetic (per wavefront, per KV block):
//   * S^T = K_j Q^T with v_mfma_f32_32x32x16_bf16: A = 32 key rows of K_j from
//     LDS, B = the wavefront's 32 query columns held in registers. MFMA row r of
//     a 32-key tile holds key 16(r/16) + pi(r mod 16), pi(4a+t) = {0,8,4,12}[a] + t,
//     so that in the output layout each lane holds, per 16 keys, 8 consecutive
//     keys of one query (lane mod 32): the softmax max and sum are lane-local plus
//     one exchange with lane^32, and
//   * P^T in bf16 is the B operand of O^T += V^T P^T directly from those
//     registers; the matching A operand is one 16-byte row chunk of V^T (8 keys
//     of one d), so every operand read is one ds_read_b128. (Reading V in its
//     natural layout with ds_read_b64_tr_b16 takes two LDS instructions per
//     operand instead of one and measured slower.)
//   * O^T rows use the same permutation, so each lane finally holds 8 consecutive
//     output columns and O is written with 16-byte stores at the block's original
//     rows (the inverse permutation is fused into the store).
// Keys past the end of the sequence (ragged last block) get score -inf.
//
// Scheduling. The kernel is persistent: one workgroup per resident slot of the
// chip. Queue x holds, head after head, the slots of XCD segment x; a workgroup
// takes the next slot of the queue of the XCD it runs on (hardware XCC id), so
// that the query blocks that run together on one XCD, and share its L2, are
// consecutive slots of one segment (Sec. IV-D), and when that queue is empty
// it takes slots from the other queues. Slot s of head bh computes original
// query block perm[bh][s] (identity when perm is null). Row lengths are
// heavy-tailed (a row can hold ten times the mean number of blocks), and a launch
// whose last task is a long row ends with every other workgroup idle; so the last
// heads of each queue run in an order built at each call: a row that could still
// be running once the rest of the queue is done starts first, longest first, and
// every other row keeps its place (tail_order). In a launch of few rows even that leaves the
// longest row running alone, so rows of more than L blocks are computed in chunks (split_plan).

#include "common.h"
#include "wavealign.h"

#include <algorithm>
#include <atomic>
#include <cfloat>
#include <cmath>
#include <type_traits>

namespace {

using wa::bf16x8;
using wa::f32x16;

typedef __attribute__((address_space(3))) void lds_void_t;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// Probabilities are taken against the first block's row maximum; a row in which one reaches this
// bound is recomputed against its exact maximum (fp32 and bf16 hold values up to it exactly scaled).
constexpr float kProbLimit = 4294967296.0f;  // 2^32

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding)
#define WA_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
// workgroup barrier after this wavefront's LDS reads have completed; the compiler may not move
// memory accesses across it
#define WA_BARRIER() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

// Scheduling fence: no instruction moves across it. Placed between the operand reads of k-step s+1
// and the MFMAs of k-step s, it keeps those reads in flight while the MFMAs run (left alone, the
// scheduler sinks every read to just before its MFMA, and each MFMA then waits out an LDS latency).
#define WA_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats -> two bf16 (round to nearest even; one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Row r (0..15) of an MFMA 16-row group -> tile row, so that the output layout
// gives each lane half 8 consecutive tile rows.
__device__ __forceinline__ int perm16(int r) { return ((r >> 2) & 1) * 8 + ((r >> 3) & 1) * 4 + (r & 3); }

// Tiles have rows of RB bytes (256 or 128) in 16-byte chunks. Physical chunk of (row, chunk): both tiles are read
// one row per lane (ds_read_b128), 16 rows per wavefront quarter.
template <int RB>
__device__ __forceinline__ int swz(int row, int chunk) {
  return RB == 256 ? (chunk ^ (row & 15)) : (chunk ^ ((row >> 1) & 7));
}

template <int D, int BLK>
struct Cfg {
  static constexpr int NW = BLK / 32;
  static constexpr int NT = NW * 64;
  static constexpr int RB = D * 2;        // K tile row bytes
  static constexpr int VRB = BLK * 2;     // V^T tile row bytes (one row per d)
  static constexpr int TBYTES = BLK * RB;  // K tile bytes = V^T tile bytes
  static constexpr int NK = TBYTES / (NT * 16);  // DMA instructions per thread and tile
  static constexpr int KT = BLK / 32;
  static constexpr int DT = D / 32;
  static constexpr int KS = D / 16;
};

// One 16-byte-per-lane copy from global memory (uniform base + per-lane byte offset) into LDS at the
// uniform address lds (lane i writes lds + 16 i). Written as inline assembly so that only the
// explicit vmcnt waits of the pipeline order it against LDS reads of the other tile; M0 (the LDS
// base of the copy) is restored afterwards.
__device__ __forceinline__ void dma16(const void* gbase, uint32_t voff, const unsigned char* lds) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "global_load_lds_dwordx4 %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(m0), "v"(voff), "s"(gbase)
      : "memory");
}

// A device-scope 16-byte store: it goes through to the level every XCD sees. The caller waits for its
// completion (vmcnt) before it publishes the data. The instruction after a store of more than 8 bytes
// must not write the registers of its data; the compiler does not look for that inside assembly.
__device__ __forceinline__ void store_through(float* p, float x, float y, float z, float w) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const f32x4 v = {x, y, z, w};
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// DMA geometry of a tile with rows of RB bytes copied by NW wavefronts: instruction i of wavefront w
// writes tile rows [(i*NW + w)*RPI, +RPI), lane l the chunk (l mod LPR) of row (l / LPR) among them.
// The global source of that slot is chunk swz(row, slot) of the row (each swizzle is an involution).
template <int RB, int NW>
struct Dma {
  static constexpr int RPI = 1024 / RB;   // rows per instruction
  static constexpr int LPR = RB / 16;     // lanes per row
  // the swizzle of a lane's slot is the same for every instruction when the row step is a multiple of
  // the swizzle's row period
  static constexpr bool kInvariant = (NW * RPI) % 16 == 0;
  __device__ static __forceinline__ int row(int i, int w, int lane) { return (i * NW + w) * RPI + lane / LPR; }
  // per-lane source bytes relative to tile row (i*NW)*RPI, for source rows `stride` bytes apart
  __device__ static __forceinline__ uint32_t lane_bytes(int i, int w, int lane, uint32_t stride = RB) {
    const int r0 = w * RPI + lane / LPR;
    const int rs = kInvariant ? r0 : row(i, w, lane);
    return (uint32_t)r0 * stride + (uint32_t)(swz<RB>(rs, lane % LPR) * 16);
  }
};

// DMA of rows [key0, key0 + BLK) of a K head (g: its first row) into a swizzled tile. In the
// ragged last block, rows past the end of the sequence are clamped to the last row (their scores
// are masked, so their probabilities are 0).
template <int D, int BLK>
__device__ __forceinline__ void issue_tile(unsigned char* tile, const unsigned char* g, int key0, int n, int w,
                                           int lane) {
  using C = Cfg<D, BLK>;
  using G = Dma<C::RB, C::NW>;
  if (key0 + BLK <= n) {
#pragma unroll
    for (int i = 0; i < C::NK; ++i)
      dma16(g + (int64_t)(key0 + i * C::NW * G::RPI) * C::RB, G::lane_bytes(i, w, lane),
            tile + (i * C::NW + w) * 1024);
  } else {
#pragma unroll
    for (int i = 0; i < C::NK; ++i) {
      const int r = G::row(i, w, lane);
      const uint32_t off = (uint32_t)min(key0 + r, n - 1) * (uint32_t)C::RB +
                           (uint32_t)(swz<C::RB>(r, lane % G::LPR) * 16);
      dma16(g, off, tile + (i * C::NW + w) * 1024);
    }
  }
}

// DMA of the V^T tile: rows d of the transposed copy (row stride row_bytes), keys [key0, key0 + BLK),
// into a tile with the K-tile swizzle (rows of VRB bytes, read one row chunk per lane).
template <int D, int BLK>
__device__ __forceinline__ void issue_vt(unsigned char* tile, const unsigned char* vtg, uint32_t row_bytes, int key0,
                                         int w, int lane) {
  using C = Cfg<D, BLK>;
  using G = Dma<C::VRB, C::NW>;
#pragma unroll
  for (int i = 0; i < C::NK; ++i)
    dma16(vtg + (int64_t)key0 * 2 + (int64_t)(i * C::NW * G::RPI) * row_bytes, G::lane_bytes(i, w, lane, row_bytes),
          tile + (i * C::NW + w) * 1024);
}

// The attention kernel reads its arguments where they are used, through the kernel-argument pointer
// made opaque at that point: hoisted out of the task loop they would hold some 40 scalar registers,
// which the compiler then spills into vector registers that the block loop needs.
typedef const __attribute__((address_space(4))) WaAttnLaunch* Args;
__device__ __forceinline__ Args kernel_args() {
  Args a = (Args)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// What a workgroup computes next: chunk `chunk` of the `chunks` chunks of a row's list (1: the whole
// row), list entries [beg, end) of a list that starts at entry `list`.
struct Task {
  int32_t bh, row, list, beg, end, chunks, chunk, tile;
};

// The first task of workgroup b is fixed: the chunks of the split rows go to workgroups 0, 1, ..., and the
// first entries of queue x to the workgroups after them with b mod n_xcd = x, in order. Only later
// tasks are taken with atomic counters: an atomic on one address costs about 0.1 us of device time,
// whoever issues it, so a launch whose 512 to 1,536 workgroups all began with one spent 50 us and more. The
// chunks past the first of each workgroup have a counter per shard (workgroups b mod kSplitShards), read
// before it is added to: with one counter for all, 8 x 120 rows of 11 blocks of 64 in 1,850 chunks (a shortest chunk of 8
// blocks, with which the lines were compared) took 182 us, with eight 82. At 12 those rows stay whole: 43 us.
__device__ __forceinline__ int first_wg(int x, int split, int n_xcd) {  // of queue x's first entry
  return split + (x + n_xcd - split % n_xcd) % n_xcd;
}

// Entry t of queue x as a task; false if it needs no work (an invalid perm entry, which is reported, or a
// row computed in chunks).
__device__ bool queue_task(Args a, int x, int t, int longest, Task* out) {
  const int32_t* px = a->sched + 64 + (int64_t)x * (a->bh + 1);
  const int th = wa::tail_heads(a->bh, a->mb);
  int bh, slot;
  if (a->head_order) {  // round-robin over the heads: the call's order table
    const int32_t* ilv = a->sched + wa::ilv_offset(a->bh, a->mb, a->n_xcd);
    const int ent = ilv[64 + ilv[x] + t];
    bh = ent / a->mb;
    slot = ent - bh * a->mb;
  } else {
    const int tb = px[a->bh - th];
    if (t >= tb) {  // the last heads: the call's tail order
      const int e = a->sched[wa::tail_offset(a->bh, a->n_xcd) + (int64_t)x * th * a->mb + (t - tb)];
      bh = a->bh - th + (e >> 16);
      slot = e & 0xFFFF;
    } else {
      // head h with px[h] <= t < px[h+1]: with segments of about equal length its share of the queue
      // tells, else a binary search
      bh = (int)((int64_t)t * a->bh / px[a->bh]);
      if (px[bh] > t || px[bh + 1] <= t) {
        int lo = 0, hi = a->bh - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (px[mid] <= t) lo = mid; else hi = mid - 1;
        }
        bh = lo;
      }
      int s0, s1;
      wa::xcd_segment(x, a->mb, a->n_xcd, a->seg ? a->seg + (int64_t)bh * (a->n_xcd + 1) : nullptr, &s0, &s1);
      slot = s0 + (t - px[bh]);
    }
  }
  const int row = a->perm ? a->perm[(int64_t)bh * a->mb + slot] : slot;
  if ((unsigned)row >= (unsigned)a->mb) {  // not a valid block index: nothing to compute, reported
    if (a->status) atomicOr(a->status, 1);
    return false;
  }
  int beg, end;
  wa::row_range(a, bh, row, &beg, &end);
  *out = {bh, row, beg, beg, end, 1, 0, 0};
  return end - beg <= longest;
}

__device__ void split_task(Args a, int k, Task* out) {
  const int4 e = ((const int4*)(a->split + wa::kSplitHead))[k];
  int beg, end;
  wa::row_range(a, e.x, e.y, &beg, &end);
  // the first n mod chunks chunks are one block longer (n times c does not fit 32 bits for the longest lists)
  const int n = end - beg, c = e.z & 0xFFFF, chunks = e.z >> 16, per = n / chunks, more = n - per * chunks;
  const int b = beg + c * per + min(c, more);
  *out = {e.x, e.y, beg, b, b + per + (c < more ? 1 : 0), chunks, c, e.w};
}

// Next task of this workgroup, run by one wavefront (t: its first lane's): the chunks of the split rows first
// (the longest work), then the queue of the workgroup's XCD, then the others. bh = -1 when nothing is left.
// Lane x reads queue x's counter; with eight reads one after another the calls of 4 x 254 and 78 x 29 rows (d 128)
// took 125 and 158 us, so 120 and 152.
__device__ void fetch_task(Args a, bool first, Task* t) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));  // opaque: nothing per lane is held across the block loop
  const int b = blockIdx.x, wgs = gridDim.x;
  const int split = a->split_cap > 0 ? a->split[0] : 0;
  const int longest = split > 0 ? a->split[1] : INT32_MAX;  // rows of more blocks are split
  const int32_t* pre = a->sched + 64;
  bool got = false;  // lane 0's
  if (first) {
    if (b < split) {
      if (lane == 0) split_task(a, b, t);
      return;
    }
    const int x = b % a->n_xcd, k = (b - first_wg(x, split, a->n_xcd)) / a->n_xcd;
    if (k < pre[(int64_t)x * (a->bh + 1) + a->bh]) {
      if (lane == 0) got = queue_task(a, x, k, longest, t);
      if (__ballot(got)) return;
    }
  }
  if (split > wgs) {
    const int shards = min(wa::kSplitShards, wgs), s = b % shards;
    const int count = (split - wgs - s + shards - 1) / shards;  // chunks wgs + s, wgs + s + shards, ...
    int32_t* cnt = a->split + wa::split_counter(s);
    if (lane == 0 && __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < count) {
      const int k = atomicAdd(cnt, 1);
      got = k < count;
      if (got) split_task(a, wgs + s + k * shards, t);
    }
    if (__ballot(got)) return;
  }
  const int home = (int)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 0xF) % a->n_xcd;
  int given = 0, total = 0;
  if (lane < a->n_xcd) {
    total = pre[(int64_t)lane * (a->bh + 1) + a->bh];
    const int w0 = first_wg(lane, split, a->n_xcd);
    given = w0 < wgs ? (wgs - w0 + a->n_xcd - 1) / a->n_xcd : 0;  // entries with a fixed workgroup
  }
  for (;;) {
    // queues with entries left; a counter only grows, so the loop ends when every queue is drained
    bool left = given < total;
    if (left) left = given + __hip_atomic_load(a->counters + lane * a->counter_step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < total;
    const uint64_t mask = __ballot(left);
    if (mask == 0) break;
    const uint64_t from_home = mask >> home << home;
    const int x = __ffsll((unsigned long long)(from_home ? from_home : mask)) - 1;
    const int x_given = __shfl(given, x), x_total = __shfl(total, x);
    if (lane == 0) {
      const int k = x_given + atomicAdd(a->counters + x * a->counter_step, 1);
      got = k < x_total && queue_task(a, x, k, longest, t);
    }
    if (__ballot(got)) return;
  }
  t->bh = -1;
}

// Wavefronts a SIMD: 256 registers a lane leave room for two; the smallest tiles fit in 168 (three).
template <int D, int BLK>
__global__ __launch_bounds__(BLK * 2, D == 64 && BLK == 64 ? 3 : 2) void attn_fwd_kernel(WaAttnLaunch) {
  using C = Cfg<D, BLK>;
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[C::TBYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds[C::TBYTES];
  __shared__ Task task;
  __shared__ int redo;  // the current row is recomputed against its exact maximum

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform within the wavefront
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  // byte offsets of this lane's K-operand chunk of k-step s in the K tile (key tile kt adds kt 32 RB)
  uint32_t kofs[C::KS];
  {
    const int kr = 16 * ((lane & 31) >> 4) + perm16(lane & 15);
#pragma unroll
    for (int s = 0; s < C::KS; ++s) kofs[s] = (uint32_t)(kr * C::RB + swz<C::RB>(kr, 2 * s + hf) * 16);
  }
  // the same for the V^T operand of k-step ks (16 keys; d tile dt adds dt 32 VRB)
  uint32_t vofs[2 * C::KT];
  {
    const int kr = 16 * ((lane & 31) >> 4) + perm16(lane & 15);
#pragma unroll
    for (int ks = 0; ks < 2 * C::KT; ++ks)
      vofs[ks] = (uint32_t)(kr * C::VRB + swz<C::VRB>(kr, 2 * ks + hf) * 16);
  }

  for (bool first = true;; first = false) {
    if (w == 0) {
      Task t;
      fetch_task(kernel_args(), first, &t);
      if (tid == 0) {
        task = t;
        redo = 0;
      }
    }
    __syncthreads();
    const int bh = __builtin_amdgcn_readfirstlane(task.bh);
    const int row = __builtin_amdgcn_readfirstlane(task.row);
    const int list = __builtin_amdgcn_readfirstlane(task.list);  // the row's first entry
    const int beg = __builtin_amdgcn_readfirstlane(task.beg);
    const int end = __builtin_amdgcn_readfirstlane(task.end);
    const int chunks = __builtin_amdgcn_readfirstlane(task.chunks);
    const int tile = __builtin_amdgcn_readfirstlane(task.tile);    // the row's first partial tile
    const int chunk = __builtin_amdgcn_readfirstlane(task.chunk);
    __syncthreads();  // every wavefront has read the task before it is overwritten
    if (bh < 0) break;

    const Args a = kernel_args();
    const int n = a->seq_len;
    const int mb = a->mb;
    const float c2 = a->scale * kLog2e;
    const uint16_t* qg = (const uint16_t*)a->q + (int64_t)bh * n * D;
    const unsigned char* kg = (const unsigned char*)a->k + (int64_t)bh * n * D * 2;
    const int64_t npad = (int64_t)mb * BLK;
    const unsigned char* vtg = (const unsigned char*)a->vt + (int64_t)bh * D * npad * 2;
    const uint32_t vt_row_bytes = (uint32_t)(npad * 2);

    // read-only for the whole kernel: the constant address space lets the list be read with scalar loads
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    const const_i32_ptr cols = (const_i32_ptr)(a->col_idx + (int64_t)bh * mb * mb);

    // Q columns of this wavefront: B operand of S^T = K Q^T
    const int qi = row * BLK + w * 32 + l32;
    bf16x8 qf[C::KS];
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      uint4 val = make_uint4(0, 0, 0, 0);
      if (qi < n) val = *(const uint4*)(qg + (int64_t)qi * D + 16 * s + 8 * hf);
      qf[s] = as_bf16x8(val);
    }

    f32x16 oacc[C::DT];
    int bad_kv = 0;           // the row's list held an index outside 0..mb-1 (uniform)
    float m_run = -INFINITY;  // reference maximum (log2 units), set by the row's first block
    float l_run = 0.f;
    int j_cur = 0;

    // S^T = K_j Q^T from the K tile in LDS. Consecutive MFMAs go to different accumulators (a chain on
    // one accumulator would wait for each result), and the operand reads of k-step s+1 are in flight
    // during the MFMAs of step s.
    auto scores = [&](f32x16 (&sacc)[C::KT]) {
#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[kt][v] = 0.f;
      uint4 a_cur[C::KT], a_nxt[C::KT];
#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt) a_cur[kt] = *(const uint4*)(k_lds + kofs[0] + kt * 32 * C::RB);
#pragma unroll
      for (int s = 0; s < C::KS; ++s) {
        if (s + 1 < C::KS) {
#pragma unroll
          for (int kt = 0; kt < C::KT; ++kt) a_nxt[kt] = *(const uint4*)(k_lds + kofs[s + 1] + kt * 32 * C::RB);
        }
        WA_SCHED_FENCE();
#pragma unroll
        for (int kt = 0; kt < C::KT; ++kt)
          sacc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a_cur[kt]), qf[s], sacc[kt], 0, 0, 0);
        WA_SCHED_FENCE();
#pragma unroll
        for (int kt = 0; kt < C::KT; ++kt) a_cur[kt] = a_nxt[kt];
      }
    };
    // keys past the end of the sequence (ragged last block) score -inf
    auto mask_tail = [&](f32x16 (&sacc)[C::KT], int nvalid, int lane_o) {
      const int hf_o = lane_o >> 5;  // from the opaque lane copy: no key table held across blocks
#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = kt * 32 + 16 * (v >> 3) + 8 * hf_o + (v & 7);
          if (key >= nvalid) sacc[kt][v] = -INFINITY;
        }
    };
    // row maximum of a score tile, in log2 units (shared by the two lanes of a query)
    auto tile_max = [&](const f32x16 (&sacc)[C::KT]) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[kt][v]);
      return fmaxf(mx, __shfl_xor(mx, 32)) * c2;
    };

    // One KV block: wait for its tiles, S^T = K_j Q^T, softmax numerators, O^T += V_j^T P^T, and keep
    // the copies of the next block in flight. MASKED handles the ragged last block; the lists are
    // ascending, so it can only be a row's last block. FIRST takes the block's row maximum as the
    // softmax reference of the row: every later probability is taken against it, so O and l are never
    // rescaled (a row whose probabilities outgrow the reference is recomputed, below).
    int e = beg;
    auto kv_block = [&](auto masked_tag, auto first_tag) {
      constexpr bool MASKED = decltype(masked_tag)::value;
      constexpr bool FIRST = decltype(first_tag)::value;
      // The per-lane copy offsets are recomputed in every block from an opaque copy of the lane index
      // (hoisted out of the loop they would hold registers that the operand reads need); the operand
      // read offsets, one per k-step, are computed once per kernel (kofs, vofs).
      int lane_o = lane;
      asm volatile("" : "+v"(lane_o));
      const bool has_next = e + 1 < end;
      int j_next = 0;
      if (has_next) {
        j_next = cols[e + 1];
        if ((unsigned)j_next >= (unsigned)mb) {  // invalid KV index: block 0 is read, reported
          j_next = 0;
          bad_kv = 1;
        }
      }

      // K_j resident (V_j may still be in flight)
      WA_WAIT_VM(C::NK);
      WA_BARRIER();
      f32x16 sacc[C::KT];
      scores(sacc);
      // every wavefront is done with K_j: start K_{j+1}
      WA_BARRIER();
      if (has_next) issue_tile<D, BLK>(k_lds, kg, j_next * BLK, n, w, lane_o);

      // ---- softmax numerators (log2 domain) ----
      if constexpr (MASKED) mask_tail(sacc, n - j_cur * BLK, lane_o);
      if constexpr (FIRST) m_run = tile_max(sacc);
      float lsum = 0.f;
      uint32_t pb[C::KT][8];
#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt][v], c2, -m_run));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt][v + 1], c2, -m_run));
          lsum += p0 + p1;
          pb[kt][v >> 1] = pack_bf16x2(p0, p1);
        }
      l_run += lsum;

      // V_j resident (K_{j+1} may still be in flight)
      if (has_next) {
        WA_WAIT_VM(C::NK);
      } else {
        WA_WAIT_VM(0);
      }
      WA_BARRIER();

      // ---- O^T += V_j^T P^T ----
      {
        // k-step ks = 2 kt + k2 (16 keys); operand reads of step ks+1 in flight during step ks
        uint4 a_cur[C::DT], a_nxt[C::DT];
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt) a_cur[dt] = *(const uint4*)(v_lds + vofs[0] + dt * 32 * C::VRB);
#pragma unroll
        for (int ks = 0; ks < 2 * C::KT; ++ks) {
          if (ks + 1 < 2 * C::KT) {
#pragma unroll
            for (int dt = 0; dt < C::DT; ++dt)
              a_nxt[dt] = *(const uint4*)(v_lds + vofs[ks + 1] + dt * 32 * C::VRB);
          }
          const uint32_t* p = &pb[ks >> 1][4 * (ks & 1)];
          const bf16x8 bv = as_bf16x8(make_uint4(p[0], p[1], p[2], p[3]));
#pragma unroll
          for (int dt = 0; dt < C::DT; ++dt)
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a_cur[dt]), bv, oacc[dt], 0, 0, 0);
#pragma unroll
          for (int dt = 0; dt < C::DT; ++dt) a_cur[dt] = a_nxt[dt];
        }
      }
      // every wavefront is done with V_j: start V_{j+1}
      WA_BARRIER();
      if (has_next) issue_vt<D, BLK>(v_lds, vtg, vt_row_bytes, j_next * BLK, w, lane_o);
      j_cur = j_next;
    };
    const bool ragged_last = end > beg && (n % BLK) != 0 && cols[end - 1] == mb - 1;
    const int e_plain = end - (ragged_last ? 1 : 0);

    // Pass 0 takes the maximum of the row's first block as the reference. If some probability reached
    // kProbLimit (a later score above the reference by log2(kProbLimit) or more, in log2 units), the
    // whole workgroup recomputes the row: the exact row maximum over all its blocks first, then
    // pass 1 against it (every probability <= 1). The decision is per workgroup, since its wavefronts
    // share the tile copies. A later chunk of a split row computes the scores of the row's first block
    // before pass 0 (pass -1), so its probabilities are, rounded to bf16, those of the unsplit row: against the
    // first block of its own, O differed from the unsplit row's in a third of its values (2e-3 in the 2-norm; now 3e-4 of them) and an
    // unnormalised chunk of small weight could overflow. A chunk that is recomputed takes the exact maximum of its own
    // blocks (with a later half of K 32 times larger, 4e-4 in the 2-norm).
    for (int pass = chunk > 0 ? -1 : 0;; ++pass) {
      int m0 = list, m1 = list + 1;  // blocks of the maximum that the next pass takes as its reference
      if (pass >= 0) {
        if (beg < end) {
          j_cur = cols[beg];
          if ((unsigned)j_cur >= (unsigned)mb) {
            j_cur = 0;
            bad_kv = 1;
          }
          issue_tile<D, BLK>(k_lds, kg, j_cur * BLK, n, w, lane);
          issue_vt<D, BLK>(v_lds, vtg, vt_row_bytes, j_cur * BLK, w, lane);
        }
        // the Q loads (issued first) are complete; the first tiles stay in flight
        WA_WAIT_VM(2 * C::NK);
#pragma unroll
        for (int t = 0; t < C::DT; ++t)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[t][v] = 0.f;
        l_run = 0.f;
        e = beg;
        if (e < e_plain) {
          if (pass == 0 && chunk == 0) {
            kv_block(std::false_type{}, std::true_type{});
          } else {
            kv_block(std::false_type{}, std::false_type{});
          }
          for (++e; e < e_plain; ++e) kv_block(std::false_type{}, std::false_type{});
          if (ragged_last) kv_block(std::true_type{}, std::false_type{});
        } else if (ragged_last) {
          if (pass == 0 && chunk == 0) {
            kv_block(std::true_type{}, std::true_type{});
          } else {
            kv_block(std::true_type{}, std::false_type{});
          }
        }
        if (pass > 0) break;
        if (__builtin_amdgcn_ballot_w64(!(l_run < kProbLimit)) && lane == 0) redo = 1;  // also inf / NaN
        __syncthreads();
        const int again = __builtin_amdgcn_readfirstlane(redo);
        __syncthreads();  // every wavefront has read the flag before the next row clears it
        if (!again) break;
        m0 = beg;
        m1 = end;
      }
      // exact maximum: K tiles one at a time, scores only
      float mx = -INFINITY;
      for (int e2 = m0; e2 < m1; ++e2) {
        int j = cols[e2];
        if ((unsigned)j >= (unsigned)mb) j = 0;
        issue_tile<D, BLK>(k_lds, kg, j * BLK, n, w, lane);
        WA_WAIT_VM(0);
        WA_BARRIER();
        f32x16 sacc[C::KT];
        scores(sacc);
        if (j * BLK + BLK > n) mask_tail(sacc, n - j * BLK, lane);
        mx = fmaxf(mx, tile_max(sacc));
        WA_BARRIER();  // every wavefront is done with the tile before the next copy
      }
      // A chunk may hold only scores of -inf where its row does not: against the lowest float its
      // probabilities are 0 (NaN scores stay NaN), and so is its weight next to any finite score.
      m_run = fmaxf(mx, chunks > 1 ? -FLT_MAX : -INFINITY);
    }

    // ---- epilogue: merge the chunks of a split row, normalise and store at the original rows ----
    const float ltot = l_run + __shfl_xor(l_run, 32);
    // the thread's offsets from an opaque copy of its index, so that none is held across the block loop
    int tid_o = threadIdx.x;
    asm volatile("" : "+v"(tid_o));
    const int hf_o = (tid_o >> 5) & 1;
    const int qloc = (tid_o >> 6) * 32 + (tid_o & 31);
    const int qi_o = row * BLK + qloc;
    if (chunks > 1) {
      const Args a = kernel_args();
      // Partial tile of this chunk: O in 16-byte pieces [register quad][thread], then the row maxima and
      // the row sums. Device-scope stores (they go through to the level every XCD sees), completed before
      // the arrival is counted; the last arrival acquires and merges every tile in chunk order.
      constexpr int NQ = C::DT * 4;
      const size_t tile_floats = wa::part_tile_floats(BLK, D);
      float* mine = a->part + (size_t)(tile + chunk) * tile_floats;
#pragma unroll
      for (int r = 0; r < NQ; ++r)
        store_through(mine + 4 * (r * C::NT + tid_o), oacc[r >> 2][4 * (r & 3)], oacc[r >> 2][4 * (r & 3) + 1],
                      oacc[r >> 2][4 * (r & 3) + 2], oacc[r >> 2][4 * (r & 3) + 3]);
      if (hf_o == 0) {
        __hip_atomic_store(mine + BLK * D + qloc, m_run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(mine + BLK * D + BLK + qloc, ltot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (bad_kv && tid_o == 0 && a->status) atomicOr(a->status, 2);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid_o == 0) redo = atomicAdd(a->split + wa::split_arrival(a->split_cap, tile), 1);
      __syncthreads();
      const int arrived = __builtin_amdgcn_readfirstlane(redo);
      __syncthreads();  // every wavefront has read the count before the next task clears it
      if (arrived != chunks - 1) continue;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const float* first = a->part + (size_t)tile * tile_floats;
      const int qrow = BLK * D + qloc;
      // Each step reads the pieces of MC chunks together (a serial walk over the chunks costs a memory
      // latency each); past the last chunk the last one again, with its bits cleared (its sums may be infinite, so
      // weight 0 is not enough; a select compiles to branches, 32.4 us instead of 31.1 for 2 x 64 rows of 64-token blocks).
      constexpr int MC = 4;
      auto at = [&](int c) { return first + (size_t)min(c, chunks - 1) * tile_floats; };
      float m = -INFINITY, l = 0.f;
      for (int c0 = 0; c0 < chunks; c0 += 2 * MC) {
        float u[2 * MC];
#pragma unroll
        for (int c = 0; c < 2 * MC; ++c) u[c] = at(c0 + c)[qrow];
#pragma unroll
        for (int c = 0; c < 2 * MC; ++c) m = fmaxf(m, u[c]);
      }
      float inv = 0.f;
      uint16_t* og = (uint16_t*)a->o + ((int64_t)bh * n + qi_o) * D + 8 * hf_o;
#pragma unroll 1
      for (int g = 0; g < 2 * C::DT; g += 2) {  // 2 x 8 consecutive columns of this lane
        float acc[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = 0.f;
        l = 0.f;
#pragma unroll 1
        for (int c0 = 0; c0 < chunks; c0 += MC) {
          float4 u[MC][4];
          float um[MC], ul[MC];
#pragma unroll
          for (int c = 0; c < MC; ++c) {
            const float* pt = at(c0 + c);
            um[c] = pt[qrow];
            ul[c] = pt[qrow + BLK];
#pragma unroll
            for (int j = 0; j < 4; ++j) u[c][j] = ((const float4*)pt)[(2 * g + j) * C::NT + tid_o];
          }
#pragma unroll
          for (int c = 0; c < MC; ++c) {
            uint32_t keep = c0 + c < chunks ? ~0u : 0u;
            asm volatile("" : "+v"(keep));
            auto in = [&](float x) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & keep); };
            const float wgt = in(__builtin_amdgcn_exp2f(um[c] - m));
            l += wgt * in(ul[c]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              acc[4 * j] += wgt * in(u[c][j].x);
              acc[4 * j + 1] += wgt * in(u[c][j].y);
              acc[4 * j + 2] += wgt * in(u[c][j].z);
              acc[4 * j + 3] += wgt * in(u[c][j].w);
            }
          }
        }
        inv = l > 0.f ? 1.f / l : NAN;  // a split row is not empty: its scores are -inf or NaN
        if (qi_o < n)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            *(uint4*)(og + 16 * (g + j)) =
                make_uint4(pack_bf16x2(acc[8 * j] * inv, acc[8 * j + 1] * inv),
                           pack_bf16x2(acc[8 * j + 2] * inv, acc[8 * j + 3] * inv),
                           pack_bf16x2(acc[8 * j + 4] * inv, acc[8 * j + 5] * inv),
                           pack_bf16x2(acc[8 * j + 6] * inv, acc[8 * j + 7] * inv));
      }
      if (a->lse && hf_o == 0 && qi_o < n) a->lse[(int64_t)bh * n + qi_o] = l > 0.f ? (m + __log2f(l)) * kLn2 : -INFINITY;
      continue;
    }
    const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
    const Args ae = kernel_args();
    if (qi_o < n) {
      uint16_t* og = (uint16_t*)ae->o + ((int64_t)bh * n + qi_o) * D;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          const int col = dt * 32 + 16 * h2 + 8 * hf_o;
          uint4 st;
          st.x = pack_bf16x2(oacc[dt][8 * h2 + 0] * inv, oacc[dt][8 * h2 + 1] * inv);
          st.y = pack_bf16x2(oacc[dt][8 * h2 + 2] * inv, oacc[dt][8 * h2 + 3] * inv);
          st.z = pack_bf16x2(oacc[dt][8 * h2 + 4] * inv, oacc[dt][8 * h2 + 5] * inv);
          st.w = pack_bf16x2(oacc[dt][8 * h2 + 6] * inv, oacc[dt][8 * h2 + 7] * inv);
          *(uint4*)(og + col) = st;
        }
      if (ae->lse && hf_o == 0)
        ae->lse[(int64_t)bh * n + qi_o] = ltot > 0.f ? (m_run + __log2f(ltot)) * kLn2 : -INFINITY;
    }
    if (bad_kv && tid_o == 0 && ae->status) atomicOr(ae->status, 2);
  }
}

int resident_cus() {
  static int cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] <= 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Workgroups of the attention kernel resident on one compute unit (looked up once per device).
template <int D, int BLK>
hipError_t occ_t(int* n) {
  static std::atomic<int> cached[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool keep = dev >= 0 && dev < 64;
  if (keep && (*n = cached[dev].load(std::memory_order_relaxed)) > 0) return hipSuccess;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(n, attn_fwd_kernel<D, BLK>, BLK * 2, 0);
  if (e == hipSuccess && keep) cached[dev].store(*n, std::memory_order_relaxed);
  return e;
}

template <int D, int BLK>
hipError_t launch_t(const WaAttnLaunch& a, hipStream_t stream) {
  const int64_t tasks = (int64_t)a.bh * a.mb;
  int occ = 0;
  hipError_t e = occ_t<D, BLK>(&occ);
  if (e != hipSuccess) return e;
  const int64_t slots = (int64_t)resident_cus() * std::max(occ, 1);
  // the tail order's rule counts the workgroups of a wave
  const int64_t grid = std::min<int64_t>(tasks, (int64_t)resident_cus() * wa::wave_wgs(D, BLK));
  if ((e = wa_launch_attn_prep(a, (int)grid, (int)slots, stream)) != hipSuccess || tasks <= 0) return e;
  // split rows give work to every resident workgroup, however few the rows
  hipLaunchKernelGGL((attn_fwd_kernel<D, BLK>), dim3((unsigned)(a.split_cap > 0 ? slots : std::min(tasks, slots))), dim3(BLK * 2), 0,
                     stream, a);
  return hipGetLastError();
}

}  // namespace

size_t wa_vt_bytes(int64_t bh, int mb, int head_dim, int block) {
  return (size_t)bh * head_dim * (size_t)mb * block * 2;
}

hipError_t wa_launch_attention(const WaAttnLaunch& a, hipStream_t stream) {
  if (a.head_dim == 128 && a.block == 128) return launch_t<128, 128>(a, stream);
  if (a.head_dim == 64 && a.block == 128) return launch_t<64, 128>(a, stream);
  if (a.head_dim == 128 && a.block == 64) return launch_t<128, 64>(a, stream);
  if (a.head_dim == 64 && a.block == 64) return launch_t<64, 64>(a, stream);
  return hipErrorInvalidValue;
}
