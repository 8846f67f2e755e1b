// Mask scans for gfx950: row counts, per-row KV-index lists, and the bit-packed
// row and column masks that the permutation builder iterates over.
//
// The scans are bound by memory: a wavefront walks rows at a fixed stride and has the loads of its next
// row in flight while it works on the current one (one short-lived wavefront per row, each waiting out
// a memory latency, read 323 MB in 71 us; this form takes 61). Rows start at any byte, so a
// lane takes the aligned 16-byte chunks 64 t + lane of the row's span, one load each, and the bytes
// before and after the row are dropped from its bits; each load covers at least one byte of the row, so
// it never leaves the pages that hold the mask. Kept-column counts are popcounts; the lanes' exclusive
// prefix sum ranks their columns, so indices are written in ascending column order (the order in which
// the attention kernel visits KV blocks) and the result is independent of scheduling.

#include "common.h"
#include "perm_launch.h"
#include "wavealign.h"

#include <algorithm>

namespace {

constexpr int kWavesPerWG = 4;

constexpr int kScanWGs = 2048;  // workgroups of a scan, at most: eight wavefronts per SIMD

// Nonzero mask of 16 bytes (bit b = byte b): each byte's high bit is set if the byte is nonzero, and two
// byte dot products with the weights 1, 2, 4, ..., 128 gather them, 128 times too large.
__device__ __forceinline__ uint32_t nz16(const uint4& c) {
  auto high = [](uint32_t w) { return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u; };
  auto gather = [&](uint32_t w0, uint32_t w1) {
    return __builtin_amdgcn_udot4(high(w1), 0x80402010u, __builtin_amdgcn_udot4(high(w0), 0x08040201u, 0u, false), false);
  };
  const uint32_t lo = gather(c.x, c.y), hi = gather(c.z, c.w);
  return (lo >> 7) | (hi << 1);
}

// A mask row as aligned 16-byte chunks: chunk c holds columns [16 c - off, 16 c - off + 16).
struct RowSpan {
  const uint8_t* base;
  int off, chunks, n;
};
__device__ __forceinline__ RowSpan row_span(const uint8_t* mask, int64_t row, int n) {
  const uint8_t* p = mask + row * n;
  const int off = (int)((uintptr_t)p & 15);
  return {p - off, off, (off + n + 15) >> 4, n};
}
// Steps of 64 chunks that cover any row of n bytes.
constexpr int kMaxSteps = (WA_MAX_BLOCKS + 15 + 1023) / 1024;
template <int STEPS>
__device__ __forceinline__ void load_span(const RowSpan& r, int lane, uint4 (&c)[STEPS]) {
#pragma unroll
  for (int t = 0; t < STEPS; ++t) {
    const int k = 64 * t + lane;
    c[t] = k < r.chunks ? *(const uint4*)(r.base + 16 * (int64_t)k) : make_uint4(0u, 0u, 0u, 0u);
  }
}
// Kept bits of chunk k: bit b = column 16 k - off + b.
__device__ __forceinline__ uint32_t span_bits(const RowSpan& r, int k, const uint4& c) {
  uint32_t bits = nz16(c);
  if (k == 0) bits &= 0xFFFFu << r.off;
  const int end = r.off + r.n - 16 * k;  // bytes of the row from this chunk's start on
  if (end < 16) bits &= end > 0 ? (1u << end) - 1u : 0u;
  return bits & 0xFFFFu;
}

// Calls f(row, span, chunks) for the rows of this wavefront, the loads of the next row in flight. DOWN: from the last
// row to the first.
template <int STEPS, bool DOWN, typename F>
__device__ __forceinline__ void for_rows(const uint8_t* mask, int rows, int n, F&& f) {
  const int lane = threadIdx.x & 63;
  const int stride = (int)gridDim.x * kWavesPerWG;
  int row = (int)blockIdx.x * kWavesPerWG + (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= rows) return;
  auto at = [&](int i) { return DOWN ? rows - 1 - i : i; };
  RowSpan cur = row_span(mask, at(row), n);
  uint4 c[STEPS];
  load_span<STEPS>(cur, lane, c);
  for (;;) {
    const int next = row > INT32_MAX - stride ? INT32_MAX : row + stride;
    RowSpan nr = cur;
    uint4 nc[STEPS];
    if (next < rows) {
      nr = row_span(mask, at(next), n);
      load_span<STEPS>(nr, lane, nc);
    }
    f(at(row), cur, c);
    if (next >= rows) break;
    row = next;
    cur = nr;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) c[t] = nc[t];
  }
}

// counts[(row / mb) * stride + offset + row % mb] = n_row. From the last row to the first: the list writing that
// follows starts at the rows read last, which the memory-side cache still holds (323 MB of mask, counts and
// lists together: 150.7 us with both passes ascending, 144.1 so).
template <int STEPS>
__global__ __launch_bounds__(256) void row_count_kernel(const uint8_t* __restrict__ mask, int rows, int n,
                                                         int32_t* __restrict__ counts, int64_t stride, int offset,
                                                         int mb) {
  const int lane = threadIdx.x & 63;
  for_rows<STEPS, true>(mask, rows, n, [&](int row, const RowSpan& r, const uint4 (&c)[STEPS]) {
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) cnt += __popc(span_bits(r, 64 * t + lane, c[t]));
    cnt = wa::lane_prefix_sum(cnt);
    if (lane == 63) counts[(int64_t)(row / mb) * stride + offset + row % mb] = cnt;
  });
}

// In place: row_ptr[h][1..mb] holds counts on entry, the inclusive scan on exit (row_ptr[h][0] = 0). Bound by
// latency: one round of loads in flight together, scans within wavefronts, one barrier for the totals of
// the 16 wavefronts' pieces. Against a run of counts a thread and a scan of ten barrier pairs, the compaction of
// 40 heads of 591 blocks takes 15.8 us instead of 17.0, of 2841 blocks 141.9 instead of 143.9.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void head_scan_kernel(int32_t* __restrict__ row_ptr, int mb) {
  constexpr int PER = WA_MAX_BLOCKS / kScanThreads;  // pieces of 1024 counts
  static_assert(PER * (kScanThreads / 64) == 64, "one lane a partial");
  __shared__ int32_t part[64];
  int32_t* rp = row_ptr + (int64_t)blockIdx.x * (mb + 1);
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  int v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * kScanThreads + t;
    v[k] = i < mb ? rp[i + 1] : 0;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    v[k] = wa::lane_prefix_sum(v[k]);
    if (lane == 63) part[k * (kScanThreads / 64) + w] = v[k];
  }
  __syncthreads();
  const int mine = part[lane];
  const int before = wa::lane_prefix_sum(mine) - mine;  // of the piece that this lane's partial ends
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * kScanThreads + t;
    const int off = __builtin_amdgcn_readlane(before, k * (kScanThreads / 64) + w);
    if (i < mb) rp[i + 1] = off + v[k];
  }
  if (t == 0) rp[0] = 0;
}

// The rows' index lists. CSR: row i of head h at out[h mb n + row_ptr[h][i]]; otherwise (row_ptr null) at
// out[(h mb + i) n], with its length in counts[h mb + i]. The indices are gathered in LDS and written
// from there, 64 consecutive entries per store: a store per kept bit of each lane costs the
// address unit a pass over 64 scattered addresses (16 of them for a run of 16 blocks), which bound the
// list writing at 111 us for 16 M indices of 323 MB of mask against 77.
template <int STEPS>
__global__ __launch_bounds__(256) void row_write_kernel(const uint8_t* __restrict__ mask, int rows, int mb, int n,
                                                         const int32_t* __restrict__ row_ptr,
                                                         int32_t* __restrict__ counts, int32_t* __restrict__ col_idx) {
  __shared__ uint16_t stage[kWavesPerWG][STEPS * 1024];
  const int lane = threadIdx.x & 63;
  uint16_t* st = stage[threadIdx.x >> 6];
  for_rows<STEPS, false>(mask, rows, n, [&](int row, const RowSpan& r, const uint4 (&c)[STEPS]) {
    const int h = row / mb;
    int32_t* out = row_ptr ? col_idx + (int64_t)h * mb * n + row_ptr[(int64_t)h * (mb + 1) + (row - h * mb)]
                           : col_idx + (int64_t)row * n;
    int base = 0;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const int k = 64 * t + lane;
      uint32_t bits = span_bits(r, k, c[t]);
      const int cnt = __popc(bits);
      const int incl = wa::lane_prefix_sum(cnt);
      int pos = base + incl - cnt;
      const int col = 16 * k - r.off;
      while (bits) {
        st[pos++] = (uint16_t)(col + __ffs((int)bits) - 1);
        bits &= bits - 1u;
      }
      base += __builtin_amdgcn_readlane(incl, 63);
    }
    asm volatile("" ::: "memory");  // (a wavefront's LDS operations complete in order)
    for (int e = lane; e < base; e += 64) out[e] = st[e];
    asm volatile("" ::: "memory");
    if (!row_ptr && lane == 0) counts[row] = base;
  });
}

// Lists of short heads (at most kOneWgBlocks blocks) in one launch, one workgroup a head: the rows' bits into
// registers and their counts into LDS, the scan, then the lists. 2 x 64 blocks 13.1 -> 8.3 us, 12 x 128 12.8 ->
// 9.4 us against the three launches; at 256 blocks the 16 rows of a wavefront take longer than the launches
// (16.1 us against 12.5).
constexpr int kOneWgBlocks = 128;
constexpr int kOneWgWaves = 16;
__global__ __launch_bounds__(64 * kOneWgWaves) void compact_head_kernel(const uint8_t* __restrict__ mask, int mb,
                                                                        int32_t* __restrict__ row_ptr,
                                                                        int32_t* __restrict__ col_idx) {
  constexpr int PER = kOneWgBlocks / kOneWgWaves;  // rows a wavefront: wave, wave + 16, ...
  __shared__ int32_t scan[kOneWgBlocks];
  __shared__ int32_t part[kOneWgBlocks / 64];
  __shared__ uint16_t stage[kOneWgWaves][kOneWgBlocks];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t h = blockIdx.x;
  const uint8_t* base = mask + h * mb * mb;
  uint32_t bits[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int r = w + kOneWgWaves * k;
    bits[k] = 0u;
    if (r < mb) {
      const RowSpan s = row_span(base, r, mb);
      uint4 c[1];
      load_span<1>(s, lane, c);
      bits[k] = span_bits(s, lane, c[0]);
    }
  }
  int incl[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    incl[k] = wa::lane_prefix_sum(__popc(bits[k]));
    const int r = w + kOneWgWaves * k;
    if (lane == 63 && r < mb) scan[r] = incl[k];
  }
  __syncthreads();
  // inclusive scan of the counts, 64 rows a wavefront
  int v = 0;
  if (w < kOneWgBlocks / 64) {
    v = wa::lane_prefix_sum(tid < mb ? scan[tid] : 0);
    if (lane == 63) part[w] = v;
  }
  __syncthreads();
  if (w < kOneWgBlocks / 64) {
    for (int i = 0; i < w; ++i) v += part[i];
    if (tid < mb) {
      scan[tid] = v;
      row_ptr[h * (mb + 1) + tid + 1] = v;
    }
    if (tid == 0) row_ptr[h * (mb + 1)] = 0;
  }
  __syncthreads();
  uint16_t* st = stage[w];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int r = w + kOneWgWaves * k;
    if (r < mb) {
      const int start = r > 0 ? scan[r - 1] : 0, count = __builtin_amdgcn_readlane(incl[k], 63);
      const RowSpan s = row_span(base, r, mb);
      int pos = incl[k] - __popc(bits[k]);
      uint32_t b = bits[k];
      while (b) {
        st[pos++] = (uint16_t)(16 * lane - s.off + __ffs((int)b) - 1);
        b &= b - 1u;
      }
      asm volatile("" ::: "memory");  // (a wavefront's LDS operations complete in order)
      int32_t* out = col_idx + h * mb * mb + start;
      for (int e = lane; e < count; e += 64) out[e] = st[e];
      asm volatile("" ::: "memory");
    }
  }
}

// The bit-packed mask of the permutation builder: one workgroup packs 64 rows of a head into words in
// LDS and writes them in both layouts, in 512-byte runs:
//   rows     rowbits[(h nw + w) m + i], bit b = M[h][i][64 w + b]
//   columns  colbits[(h mw + v) n + j], bit r = M[h][64 v + r][j]
// with row_nnz[h m + i] = n_i, and per 64-row group v the adjacent-row overlap within it,
// adj[h mw + v] = {sum |M_i & M_i+1|, sum |M_i | M_i+1|} over its rows i and i + 1 (the pairs that straddle two
// groups are left to the statistics). Packing row by row wrote each word by itself (8 bytes of a line
// whose other rows other XCDs wrote) and re-read the words for the columns: 94 + 33 us for 323 MB of
// mask against 90.
constexpr int kPackWaves = 16;
template <int STEPS>
__global__ __launch_bounds__(64 * kPackWaves, 8) void pack_kernel(const uint8_t* __restrict__ mask, int m, int n,
                                                                  int nw, int mw, uint64_t* __restrict__ rowbits,
                                                                  uint64_t* __restrict__ colbits,
                                                                  int32_t* __restrict__ row_nnz,
                                                                  int2* __restrict__ adj) {
  constexpr int W = (16 * STEPS < WA_MAX_BLOCKS / 64 ? 16 * STEPS : WA_MAX_BLOCKS / 64) + 1;  // (+1: bank conflicts)
  __shared__ uint64_t words[64][W];
  __shared__ int2 part[kPackWaves];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t h = blockIdx.x / mw;
  const int v = (int)(blockIdx.x % mw);
  const int r0 = 64 * v, rows = min(64, m - r0);
  const uint8_t* base = mask + (h * m + r0) * n;
  RowSpan cur = {};
  uint4 c[STEPS];
  if (wv < rows) {
    cur = row_span(base, wv, n);
    load_span<STEPS>(cur, lane, c);
  }
  for (int r = wv; r < 64; r += kPackWaves) {
    RowSpan nr = cur;
    uint4 nc[STEPS];
    const int next = r + kPackWaves;
    if (next < rows) {
      nr = row_span(base, next, n);
      load_span<STEPS>(nr, lane, nc);
    }
    uint32_t b[STEPS + 1];
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      b[t] = r < rows ? span_bits(cur, 64 * t + lane, c[t]) : 0u;
      cnt += __popc(b[t]);
    }
    b[STEPS] = 0u;
    cnt = wa::lane_prefix_sum(cnt);
    if (lane == 63 && r < rows) row_nnz[h * m + r0 + r] = cnt;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      // columns [16 k, 16 k + 16) of chunk position k: the end of this chunk and the start of the next
      const uint32_t up = (uint32_t)wa::dpp32<0x130, 0xf>(0, (int)b[t]);  // wave_shl:1: lane + 1's bits
      const uint32_t nx = lane == 63 ? (uint32_t)__builtin_amdgcn_readlane((int)b[t + 1], 0) : up;
      const uint32_t x = ((b[t] | (nx << 16)) >> cur.off) & 0xFFFFu;
      // lanes 4k .. 4k+3 hold the 64 columns of word 16 t + k
      const uint32_t lo = x | ((uint32_t)wa::dpp32<0x101, 0xf>(0, (int)x) << 16);  // row_shl:1
      const uint32_t hi = (uint32_t)wa::dpp32<0x102, 0xf>(0, (int)lo);             // row_shl:2
      const int w = 16 * t + (lane >> 2);
      if ((lane & 3) == 0 && w < nw) words[r][w] = (uint64_t)lo | ((uint64_t)hi << 32);
    }
    cur = nr;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) c[t] = nc[t];
  }
  __syncthreads();
  int both = 0, any = 0;
  for (int w = wv; w < nw; w += kPackWaves) {
    uint64_t x = words[lane][w];  // row r0 + lane (zero past the head)
    if (lane < rows) rowbits[(h * nw + w) * m + r0 + lane] = x;
    const uint64_t y = (uint64_t)(uint32_t)wa::dpp32<0x130, 0xf>(0, (int)(uint32_t)x) |
                       ((uint64_t)(uint32_t)wa::dpp32<0x130, 0xf>(0, (int)(uint32_t)(x >> 32)) << 32);
    if (lane < 63 && lane + 1 < rows) {
      both += __popcll(x & y);
      any += __popcll(x | y);
    }
    // 64 x 64 bit transpose (lane = row -> lane = column) by the recursive block swap: at distance s,
    // a lane in the lower half of each 2s group trades its columns with bit s set for the partner's
    // columns with bit s clear
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
      const uint64_t lo = s == 32 ? 0x00000000FFFFFFFFull : s == 16 ? 0x0000FFFF0000FFFFull
                        : s == 8 ? 0x00FF00FF00FF00FFull : s == 4 ? 0x0F0F0F0F0F0F0F0Full
                        : s == 2 ? 0x3333333333333333ull : 0x5555555555555555ull;  // columns with bit s clear
      const uint32_t tlo = (uint32_t)__shfl_xor((int)(uint32_t)x, s);
      const uint32_t thi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), s);
      const uint64_t t = ((uint64_t)thi << 32) | tlo;
      x = (lane & s) ? ((x & ~lo) | ((t >> s) & lo)) : ((x & lo) | ((t & lo) << s));
    }
    const int j = 64 * w + lane;
    if (j < n) colbits[(h * mw + v) * n + j] = x;
  }
  both = wa::lane_prefix_sum(both);
  any = wa::lane_prefix_sum(any);
  if (lane == 63) part[wv] = make_int2(both, any);
  __syncthreads();
  if (threadIdx.x == 0) {
    int2 s = make_int2(0, 0);
    for (int k = 0; k < kPackWaves; ++k) {
      s.x += part[k].x;
      s.y += part[k].y;
    }
    adj[h * mw + v] = s;
  }
}

// Permutation check: one workgroup per head marks each entry in an LDS bitmap; an entry out of
// range or already marked, or a bitmap with fewer than m marks, makes the head bad. bad[0] counts
// bad heads (zeroed by the first workgroup's predecessor kernel); head_ok (nullable) gets 1 / 0.
__global__ __launch_bounds__(64) void zero_counter_kernel(int32_t* c) {
  if (threadIdx.x == 0) c[0] = 0;
}

__global__ __launch_bounds__(256) void check_perm_kernel(const int32_t* __restrict__ perm, int m,
                                                         int32_t* __restrict__ bad, int32_t* __restrict__ head_ok) {
  __shared__ uint32_t seen[WA_MAX_BLOCKS / 32];
  __shared__ int fault;
  const int64_t h = blockIdx.x;
  const int tid = threadIdx.x;
  for (int i = tid; i < (m + 31) / 32; i += 256) seen[i] = 0u;
  if (tid == 0) fault = 0;
  __syncthreads();
  const int32_t* p = perm + h * m;
  for (int s = tid; s < m; s += 256) {
    const int32_t r = p[s];
    if (r < 0 || r >= m) {
      fault = 1;
    } else {
      const uint32_t bit = 1u << (r & 31);
      if (atomicOr(&seen[r >> 5], bit) & bit) fault = 1;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (head_ok) head_ok[h] = fault ? 0 : 1;
    if (fault) atomicAdd(bad, 1);
  }
}

// Each workgroup records the XCD it runs on (hardware register XCC_ID, bits [3:0]).
__global__ void xcc_probe_kernel(int32_t* out, int n) {
  if (threadIdx.x == 0 && (int)blockIdx.x < n)
    out[blockIdx.x] = (int32_t)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 0xF);
}

}  // namespace

hipError_t wa_launch_check_perm(const int32_t* perm, int bh, int m, int32_t* bad, int32_t* head_ok,
                                hipStream_t stream) {
  hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(64), 0, stream, bad);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || bh <= 0) return e;
  hipLaunchKernelGGL(check_perm_kernel, dim3(bh), dim3(256), 0, stream, perm, m, bad, head_ok);
  return hipGetLastError();
}

hipError_t wa_launch_xcc_probe(int32_t* out, int n_wg, hipStream_t stream) {
  if (n_wg <= 0) return hipSuccess;
  hipLaunchKernelGGL(xcc_probe_kernel, dim3(n_wg), dim3(64), 0, stream, out, n_wg);
  return hipGetLastError();
}

// Instantiates a scan for the steps that a row of n bytes at any alignment takes.
#define WA_SCAN(kernel, rows, n, ...)                                                                            \
  do {                                                                                                           \
    const int64_t wgs_ = std::min<int64_t>(((rows) + kWavesPerWG - 1) / kWavesPerWG, kScanWGs);                  \
    const int steps_ = ((n) + 15 + 1023) / 1024;                                                                 \
    const dim3 g_((unsigned)wgs_), t_(64 * kWavesPerWG);                                                         \
    if (steps_ <= 1) hipLaunchKernelGGL((kernel<1>), g_, t_, 0, stream, __VA_ARGS__);                            \
    else if (steps_ <= 2) hipLaunchKernelGGL((kernel<2>), g_, t_, 0, stream, __VA_ARGS__);                       \
    else if (steps_ <= 3) hipLaunchKernelGGL((kernel<3>), g_, t_, 0, stream, __VA_ARGS__);                       \
    else hipLaunchKernelGGL((kernel<kMaxSteps>), g_, t_, 0, stream, __VA_ARGS__);                                \
  } while (0)

hipError_t wa_launch_row_count(const uint8_t* mask, int64_t rows, int n, int32_t* counts, int64_t count_stride_rows,
                               int counts_offset, int mb, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  WA_SCAN(row_count_kernel, rows, n, mask, (int)rows, n, counts, count_stride_rows, counts_offset, mb);
  return hipGetLastError();
}

hipError_t wa_launch_compact(const uint8_t* mask, int bh, int mb, int32_t* row_ptr, int32_t* col_idx,
                             hipStream_t stream) {
  if (bh <= 0) return hipSuccess;
  if (mb <= kOneWgBlocks) {
    hipLaunchKernelGGL(compact_head_kernel, dim3(bh), dim3(64 * kOneWgWaves), 0, stream, mask, mb, row_ptr, col_idx);
    return hipGetLastError();
  }
  hipError_t e = wa_launch_row_count(mask, (int64_t)bh * mb, mb, row_ptr, mb + 1, 1, mb, stream);
  if (e == hipSuccess) e = wa_launch_head_scan(row_ptr, bh, mb, stream);
  if (e == hipSuccess) e = wa_launch_row_write(mask, bh, mb, mb, row_ptr, nullptr, col_idx, stream);
  return e;
}

hipError_t wa_launch_head_scan(int32_t* row_ptr, int bh, int mb, hipStream_t stream) {
  if (bh <= 0) return hipSuccess;
  hipLaunchKernelGGL(head_scan_kernel, dim3(bh), dim3(kScanThreads), 0, stream, row_ptr, mb);
  return hipGetLastError();
}

hipError_t wa_launch_row_write(const uint8_t* mask, int bh, int mb, int n, const int32_t* row_ptr, int32_t* counts,
                               int32_t* col_idx, hipStream_t stream) {
  const int64_t rows = (int64_t)bh * mb;
  if (rows <= 0) return hipSuccess;
  WA_SCAN(row_write_kernel, rows, n, mask, (int)rows, mb, n, row_ptr, counts, col_idx);
  return hipGetLastError();
}

hipError_t wa_launch_pack(const uint8_t* mask, int bh, int m, int n, uint64_t* rowbits, uint64_t* colbits,
                          int32_t* row_nnz, int2* adj, hipStream_t stream) {
  const int nw = (n + 63) / 64, mw = (m + 63) / 64;
  if (bh <= 0 || m <= 0 || n <= 0) return hipSuccess;
  const int steps = (n + 15 + 1023) / 1024;
  const dim3 g((unsigned)((int64_t)bh * mw)), t(64 * kPackWaves);
  auto* f = steps <= 1 ? pack_kernel<1> : steps <= 2 ? pack_kernel<2> : steps <= 3 ? pack_kernel<3> : pack_kernel<kMaxSteps>;
  hipLaunchKernelGGL(f, g, t, 0, stream, mask, m, n, nw, mw, rowbits, colbits, row_nnz, adj);
  return hipGetLastError();
}
