// What an attention call needs before its kernel: the order tables of the task queues, the split plan and,
// when V comes in its natural layout, the transposed copy.

#include "common.h"
#include "wavealign.h"

namespace {

// L of the split plan: this share of the kept blocks per resident workgroup. Without the split, a launch
// of few rows lasts as long as its longest row: 2 x 64 rows of 64-token blocks (d 64, 24% kept) took
// 61 us in this kernel, 8 x 61 ragged rows (d 128, 25%) 148 us; with it 20 and 86 us. A smaller share
// makes more chunks than the launch has workgroups, a larger one longer ends: at 3/4, 1, 5/4 and 3/2 calls
// of 20 x 317 rows of 64 blocks (21% kept) took 720, 648, 632 and 631 us, 12 x 512 rows (d 128) of 64-token
// blocks 836, 850, 845 and 881, 8 x 208 rows (d 64) 195, 187, 186 and 182 us.
constexpr int kSplitNum = 5, kSplitDen = 4;

// Whether splitting pays. Whole, the launch takes about 9/10 of its longest row; split, each workgroup's share of the
// kept blocks, on average half a chunk more at the end, and the chunks' cost: writing and merging partial tiles takes as long
// as 16 kept blocks a chunk (24 for the smallest tiles, whose blocks are the shortest next to the fixed part). So rows are
// split if
//   0.9 longest > kept / slots + L / 2 + m chunks / slots + k,   m = 16 or 24, k = 4 (block 64) or 0.
// Over 5,994 launches (14 to 400 blocks a head, 3% to 20 times as many rows as workgroups, equal and log-normal row
// lengths, the four kernels) splitting whenever a row exceeded L was more than 3% slower than not splitting in 11%, up to
// 2.8 times (equal rows, about half as many as workgroups: 768 rows of 24 of 64-token blocks, d 64, 77 us for 44); by
// this rule in 0.4%, at most 1.12 times, and the geometric mean gain over not splitting is 1.614 for 1.589.
struct SplitCost {
  int merge, fixed;
};
__device__ __forceinline__ SplitCost split_cost(int d, int block) {
  return {d == 64 && block == 64 ? 24 : 16, block == 64 ? 4 : 0};
}

// ---------------------------------------------------------------------------------------------
// Preparation: everything a call needs before the attention kernel, in one launch, so that the latency
// of the order tables (a few workgroups) hides behind the copy of V. Workgroups [0, n_xcd) build
// the prefix table and the order of one queue each, the next one the split plan (and clears the status
// word), the others transpose V.
constexpr int PT = 1024;
constexpr int PW = PT / 64;

// Inclusive prefix sum over the workgroup's threads, and the total. One barrier pair.
__device__ __forceinline__ int wg_scan(int v, int32_t* part, int* all) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = wa::lane_prefix_sum(v);
  if (lane == 63) part[w] = v;
  __syncthreads();
  const int mine = lane < PW ? part[lane] : 0;
  const int incl = wa::lane_prefix_sum(mine);
  const int before = w ? __builtin_amdgcn_readlane(incl, w - 1) : 0;
  *all = __builtin_amdgcn_readlane(incl, PW - 1);
  __syncthreads();  // the partials are read before the next scan writes them
  return v + before;
}

// Maximum of nonnegative values over the workgroup's threads. One barrier pair.
__device__ __forceinline__ int wg_max(int v, int32_t* part) {
  for (int o = 1; o < 64; o <<= 1) v = max(v, __shfl_xor(v, o));
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  v = 0;
  for (int w = 0; w < PW; ++w) v = max(v, part[w]);
  __syncthreads();
  return v;
}

// Late entries up to this many are placed by counting (four wavefronts: 1.3 us at 256, where the bitonic stages
// take 4), more by a bitonic sort.
constexpr int kRankLate = 256;

struct OrderLds {
  int32_t hstart[wa::kTailMaxHeads + 1];  // first entry of each head's segment
  int32_t hslot0[wa::kTailMaxHeads];      // its first slot
  int32_t part[PW];
  __attribute__((aligned(16))) uint32_t key[wa::kTailEntries];
};
struct TransposeLds {
  uint16_t t[PT / 256][64][64 + 8];
};
union PrepLds {
  OrderLds order;
  TransposeLds tr;
};

__device__ __forceinline__ void queue_segment(const WaAttnLaunch& a, int h, int x, int* s0, int* s1) {
  wa::xcd_segment(x, a.mb, a.n_xcd, a.seg ? a.seg + (int64_t)h * (a.n_xcd + 1) : nullptr, s0, s1);
}

// Counter and prefix table of queue x: the prefix sums of its segment lengths over the heads.
__device__ void queue_prefix(const WaAttnLaunch& a, OrderLds& L, int x) {
  const int t = threadIdx.x;
  int32_t* px = a.sched + 64 + (int64_t)x * (a.bh + 1);
  if (t == 0) {
    a.counters[x * a.counter_step] = 0;
    px[0] = 0;
  }
  int carry = 0;
  for (int h0 = 0; h0 < a.bh; h0 += PT) {
    int s0 = 0, s1 = 0, all;
    if (h0 + t < a.bh) queue_segment(a, h0 + t, x, &s0, &s1);
    const int incl = wg_scan(s1 - s0, L.part, &all);
    if (h0 + t < a.bh) px[h0 + t + 1] = carry + incl;
    carry += all;
  }
}

// Tail order of queue x: entries e = 0, 1, ... enumerate, in queue order,
// the slots of segment x of the last th heads. A row of n blocks that starts with fewer than
// 2 n (grid / n_xcd) blocks queued after it could outlast the rest of the queue; such rows go first,
// by descending n (ties in queue order), and the others follow in queue order. Each entry is
// (head offset << 16) | slot. The order is a permutation of the queue's slots, so every row still
// runs exactly once.
__device__ void tail_order(const WaAttnLaunch& a, OrderLds& L, int x, int grid) {
  constexpr int PER = wa::kTailEntries / PT;
  const int t = threadIdx.x;
  const int th = wa::tail_heads(a.bh, a.mb);
  const int hb = a.bh - th;
  int32_t* tail = a.sched + wa::tail_offset(a.bh, a.n_xcd) + (int64_t)x * th * a.mb;
  int total;
  {
    int s0 = 0, s1 = 0;
    if (t < th) queue_segment(a, hb + t, x, &s0, &s1);
    const int incl = wg_scan(s1 - s0, L.part, &total);
    if (t < th) {
      L.hslot0[t] = s0;
      L.hstart[t + 1] = incl;
    }
    if (t == 0) L.hstart[0] = 0;
  }
  __syncthreads();
  // head offset of entry e: the last k with hstart[k] <= e
  auto head_of = [&](int e) {
    int lo = 0, hi = th - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (L.hstart[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  // Block counts of this thread's consecutive entries, per a thread (independent loads first): entry
  // e0 + i in nb[i], its head offset in kh[i].
  const int per = (total + PT - 1) / PT;
  const int e0 = t * per;
  uint16_t nb[PER], kh[PER];
  int sum = 0;
  {
    int k = e0 < total ? head_of(e0) : 0;
#pragma unroll
    for (int i0 = 0; i0 < PER; i0 += 4) {  // four entries' loads in flight together
      int row[4];
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        const int e = e0 + i;
        row[i - i0] = -1;
        kh[i] = 0;
        nb[i] = 0;
        if (i < per && e < total) {
          while (e >= L.hstart[k + 1]) ++k;
          kh[i] = (uint16_t)k;
          const int slot = L.hslot0[k] + (e - L.hstart[k]);
          row[i - i0] = a.perm ? a.perm[(int64_t)(hb + k) * a.mb + slot] : slot;
        }
      }
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        if (i < per && (unsigned)row[i - i0] < (unsigned)a.mb) {
          int beg, end;
          wa::row_range(&a, hb + kh[i], row[i - i0], &beg, &end);
          nb[i] = (uint16_t)min(max(end - beg, 0), WA_MAX_BLOCKS);
        }
        sum += nb[i];
      }
    }
  }
  // blocks queued after each entry, then the late entries and their ranks (workgroup-wide scans)
  const int64_t wgs = max(grid / a.n_xcd, 1);
  int all = 0;
  const int incl = wg_scan(sum, L.part, &all);
  int64_t after = (int64_t)all - incl;  // blocks of the entries after this thread's
  uint32_t late_bits = 0;
  int nlate_mine = 0;
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    if (i < per && e0 + i < total && 2 * (int64_t)nb[i] * wgs > after) {
      late_bits |= 1u << i;
      ++nlate_mine;
    }
    after += nb[i];
  }
  int nlate = 0;
  const int late_incl = wg_scan(nlate_mine, L.part, &nlate);
  int late_before = late_incl - nlate_mine;
  int lg = 0;
  while ((1 << lg) < nlate) ++lg;
  const int P = 1 << lg;
  for (int i = nlate + t; i < max(P, (nlate + 3) & ~3); i += PT) L.key[i] = 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = e0 + i;
    if (i < per && e < total) {
      if (late_bits >> i & 1u) {
        L.key[late_before++] = ((uint32_t)(WA_MAX_BLOCKS - nb[i]) << 14) | (uint32_t)e;
      } else {
        tail[nlate + (e - late_before)] = ((int)kh[i] << 16) | (L.hslot0[kh[i]] + (e - L.hstart[kh[i]]));
      }
    }
  }
  // Late entries ascending by key = descending block count, ties in queue order.
  auto place = [&](int pos, uint32_t key) {
    const int e = (int)(key & 0x3FFFu);
    const int k = head_of(e);
    tail[pos] = (k << 16) | (L.hslot0[k] + (e - L.hstart[k]));
  };
  __syncthreads();
  if (nlate <= kRankLate) {
    // few: an entry's place is the number of smaller keys (padded to four a read with the largest key)
    if (t < nlate) {
      const uint32_t mine = L.key[t];
      int r = 0;
      for (int i = 0; i < nlate; i += 4) {
        const uint4 x = *(const uint4*)&L.key[i];
        r += (x.x < mine) + (x.y < mine) + (x.z < mine) + (x.w < mine);
      }
      place(r, mine);
    }
    return;
  }
  // Bitonic sort. A pair at a distance of at most 64 lies within the 128 entries of one wavefront's threads,
  // so those stages need no workgroup barrier (a wavefront's LDS operations complete in order).
  for (int kk = 1; kk <= lg; ++kk)
    for (int lj = kk - 1; lj >= 0; --lj) {
      const int j = 1 << lj;
      for (int q = t; q < P / 2; q += PT) {
        const int i = ((q >> lj) << (lj + 1)) | (q & (j - 1));
        const uint32_t u = L.key[i], v = L.key[i + j];
        if ((u > v) == (((i >> kk) & 1) == 0)) {
          L.key[i] = v;
          L.key[i + j] = u;
        }
      }
      // the next stage pairs across wavefronts, or this one did
      if (lj > 6 || (lj == 0 && kk > 6)) {
        __syncthreads();
      } else {
        asm volatile("" ::: "memory");
      }
    }
  __syncthreads();
  for (int i = t; i < nlate; i += PT) place(i, L.key[i]);
}

// Head-interleaved order of queue x: the queue's tasks round-robin over the
// heads, round r taking slot s0_h + r of every head h whose segment of the queue has more than r
// slots, heads ascending. Entry (h, r) therefore sits at C(r) + #{h' < h : L_h' > r}, with L_h the
// segment length and C(r) = sum_h min(L_h, r) the entries of the rounds before r. Entries are
// h * mb + slot; queue x's entries start at the total of queues 0..x-1 (ilv[x]).
__device__ void ilv_order(const WaAttnLaunch& a, OrderLds& L, int x) {
  constexpr int RPT = WA_MAX_BLOCKS / PT;  // rounds per thread: r = t + k PT < mb <= WA_MAX_BLOCKS
  const int t = threadIdx.x;
  int32_t* ilv = a.sched + wa::ilv_offset(a.bh, a.mb, a.n_xcd);
  int len = 0, off;
  for (int64_t p = t; p < (int64_t)a.bh * x; p += PT) {  // segment lengths of the queues before x
    int s0, s1;
    queue_segment(a, (int)(p / x), (int)(p % x), &s0, &s1);
    len += s1 - s0;
  }
  wg_scan(len, L.part, &off);
  if (t == 0) ilv[x] = off;
  int32_t* out = ilv + 64 + off;
  int c[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) c[k] = 0;
  for (int h = 0; h < a.bh; ++h) {
    int s0, s1;
    queue_segment(a, h, x, &s0, &s1);
#pragma unroll
    for (int k = 0; k < RPT; ++k) c[k] += min(s1 - s0, t + k * PT);
  }
  for (int h = 0; h < a.bh; ++h) {
    int s0, s1;
    queue_segment(a, h, x, &s0, &s1);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int r = t + k * PT;
      if (r < s1 - s0) out[c[k]++] = h * a.mb + s0 + r;
    }
  }
}

// Split plan (one workgroup): L from the kept blocks per resident workgroup, grown until the chunks of
// the rows above it fit the tiles; then one task per chunk, enumerated over the slots that a queue holds (a row
// that no slot names, or only a slot outside every segment of the caller's table, is not computed). Counted over the
// rows as well, so that L is the same for every order.
__device__ void split_plan(const WaAttnLaunch& a, OrderLds& S, int slots) {
  const int t = threadIdx.x;
  if (t == 0 && a.status) *a.status = 0;
  if (a.split_cap <= 0) return;
  const int rows = a.bh * a.mb;
  int kept = 0, all;
  if (a.row_ptr) {
    for (int h = t; h < a.bh; h += PT) kept += a.row_ptr[(int64_t)h * (a.mb + 1) + a.mb];
  } else {
    for (int i = t; i < rows; i += PT) kept += a.row_cnt[i];
  }
  wg_scan(kept, S.part, &all);
  int L = max(wa::kSplitMinBlocks, (int)(((int64_t)all * kSplitNum / kSplitDen + slots - 1) / slots));
  auto blocks = [&](int h, int r) {
    int beg, end;
    wa::row_range(&a, h, r, &beg, &end);
    return end - beg;
  };
  auto slot_blocks = [&](int i, int* h, int* r) {
    *h = i / a.mb;
    *r = i - *h * a.mb;
    if (a.perm) *r = a.perm[i];
    return (unsigned)*r < (unsigned)a.mb ? blocks(*h, *r) : 0;
  };
  auto queued = [&](int i, int h) {  // slot i - h mb lies in a segment
    if (!a.seg) return true;
    for (int x = 0; x < a.n_xcd; ++x) {
      int s0, s1;
      queue_segment(a, h, x, &s0, &s1);
      if (s0 <= i - h * a.mb && i - h * a.mb < s1) return true;
    }
    return false;
  };
  const SplitCost cost = split_cost(a.head_dim, a.block);
  auto pays = [&](int longest, int chunks) {
    return (int64_t)slots * (9ll * longest - 5ll * L - 10 * cost.fixed) > 10 * ((int64_t)all + (int64_t)cost.merge * chunks);
  };
  int mine = 0, total = 0;
  for (;;) {
    total = 0;
    if (L >= a.mb || (!a.row_ptr && !pays(a.mb, 0))) break;  // (a caller's lists may name blocks repeatedly)
    int by_row = 0, longest = 0, h, r;
    mine = 0;
    for (int i = t; i < rows; i += PT) {
      int n = slot_blocks(i, &h, &r);
      if (n > L && queued(i, h)) mine += (n + L - 1) / L;
      if (a.perm) {
        n = blocks(h, i - h * a.mb);
        if (n > L) by_row += (n + L - 1) / L;
      }
      longest = max(longest, n);
    }
    int row_total;
    wg_scan(by_row, S.part, &row_total);
    mine = wg_scan(mine, S.part, &total) - mine;  // chunks of the threads before this one
    const bool fits = max(total, row_total) <= a.split_cap;
    if (!pays(wg_max(longest, S.part), fits ? max(total, row_total) : 0)) {
      total = 0;
      break;
    }
    if (fits) break;
    L += (L + 1) / 2;
  }
  if (t < wa::kSplitShards) a.split[wa::split_counter(t)] = 0;
  if (t == 0) {
    a.split[0] = total;
    a.split[1] = L;
  }
  if (total == 0) return;
  int4* tasks = (int4*)(a.split + wa::kSplitHead);
  int at = mine, h, r;
  for (int i = t; i < rows; i += PT) {
    const int n = slot_blocks(i, &h, &r);
    if (n <= L || !queued(i, h)) continue;
    const int chunks = (n + L - 1) / L;
    a.split[wa::split_arrival(a.split_cap, at)] = 0;
    for (int c = 0; c < chunks; ++c) tasks[at + c] = make_int4(h, r, c | (chunks << 16), at);
    at += chunks;
  }
}

// V [bh][n][D] -> V^T [bh][D][npad], zero for keys >= n. One 64-key x 64-column tile per 256 threads,
// 16-byte loads and stores, transposed through LDS. tid: 0..255; every thread of the workgroup calls.
template <int D>
__device__ __forceinline__ void transpose_tile(const uint16_t* __restrict__ v, uint16_t* __restrict__ vt, int n,
                                               int64_t npad, int tiles_n, int64_t index, int64_t count,
                                               uint16_t (*t)[64 + 8], int tid) {
  const bool any = index < count;
  const int tile = (int)(index % tiles_n);
  const int dtile = (int)(index / tiles_n % (D / 64));
  const int64_t bh = index / ((int64_t)tiles_n * (D / 64));
  const int key0 = tile * 64, d0 = dtile * 64;
  const uint16_t* src = v + bh * n * D;
  uint16_t* dst = vt + bh * D * npad;
  // load: thread -> (key r, 8-column group c8), two passes of 32 keys
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = pass * 32 + tid / 8, c8 = tid % 8;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (any && key0 + r < n) val = *(const uint4*)(src + (int64_t)(key0 + r) * D + d0 + c8 * 8);
    const uint32_t wv[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) t[r][c8 * 8 + e] = (uint16_t)(wv[e >> 1] >> ((e & 1) * 16));
  }
  __syncthreads();
  if (!any) return;
  // store: thread -> (column d, 8-key group k8), two passes of 32 columns
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int d = pass * 32 + tid / 8, k8 = tid % 8;
    uint32_t wv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      wv[e] = (uint32_t)t[k8 * 8 + 2 * e][d] | ((uint32_t)t[k8 * 8 + 2 * e + 1][d] << 16);
    *(uint4*)(dst + (int64_t)(d0 + d) * npad + key0 + k8 * 8) = make_uint4(wv[0], wv[1], wv[2], wv[3]);
  }
}

template <int D>
__global__ __launch_bounds__(256) void transpose_v_kernel(const uint16_t* __restrict__ v, uint16_t* __restrict__ vt,
                                                         int n, int64_t npad, int tiles_n, int64_t count) {
  __shared__ uint16_t t[64][64 + 8];
  transpose_tile<D>(v, vt, n, npad, tiles_n, blockIdx.x, count, t, threadIdx.x);
}

template <int D>
__global__ __launch_bounds__(PT, 8) void prep_kernel(WaAttnLaunch a, int grid, int slots, int tiles_n, int64_t tiles) {
  __shared__ PrepLds lds;
  const int x = blockIdx.x;
  if (x < a.n_xcd) {
    queue_prefix(a, lds.order, x);
    if (a.head_order) {
      ilv_order(a, lds.order, x);
    } else {
      tail_order(a, lds.order, x, grid);
    }
  } else if (x == a.n_xcd) {
    split_plan(a, lds.order, slots);
  } else {
    const int64_t index = (int64_t)(x - a.n_xcd - 1) * (PT / 256) + threadIdx.x / 256;
    transpose_tile<D>((const uint16_t*)a.v, (uint16_t*)a.vt, a.seq_len, (int64_t)a.mb * a.block, tiles_n, index, tiles,
                      lds.tr.t[threadIdx.x / 256], threadIdx.x & 255);
  }
}

template <int D>
hipError_t launch_transpose(const void* v, void* vt, int64_t bh, int n, int mb, int blk, hipStream_t stream) {
  const int64_t npad = (int64_t)mb * blk;
  const int tiles_n = (int)((npad + 63) / 64);
  const int64_t tgrid = bh * (D / 64) * tiles_n;
  if (tgrid <= 0) return hipSuccess;
  hipLaunchKernelGGL((transpose_v_kernel<D>), dim3((unsigned)tgrid), dim3(256), 0, stream, (const uint16_t*)v,
                     (uint16_t*)vt, n, npad, tiles_n, tgrid);
  return hipGetLastError();
}

template <int D>
hipError_t launch_prep(const WaAttnLaunch& a, int grid, int slots, hipStream_t stream) {
  const int tiles_n = (int)(((int64_t)a.mb * a.block + 63) / 64);
  const int64_t tiles = a.v ? (int64_t)a.bh * (D / 64) * tiles_n : 0;
  const int64_t wgs = a.n_xcd + 1 + (tiles + PT / 256 - 1) / (PT / 256);
  hipLaunchKernelGGL((prep_kernel<D>), dim3((unsigned)wgs), dim3(PT), 0, stream, a, grid, slots, tiles_n, tiles);
  return hipGetLastError();
}

}  // namespace

hipError_t wa_launch_attn_prep(const WaAttnLaunch& a, int grid, int slots, hipStream_t stream) {
  if (a.head_dim == 128) return launch_prep<128>(a, grid, slots, stream);
  if (a.head_dim == 64) return launch_prep<64>(a, grid, slots, stream);
  return hipErrorInvalidValue;
}

hipError_t wa_launch_transpose_v(const void* v, void* vt, int64_t bh, int seq_len, int mb, int head_dim, int block,
                                 hipStream_t stream) {
  if (head_dim == 128) return launch_transpose<128>(v, vt, bh, seq_len, mb, block, stream);
  if (head_dim == 64) return launch_transpose<64>(v, vt, bh, seq_len, mb, block, stream);
  return hipErrorInvalidValue;
}
