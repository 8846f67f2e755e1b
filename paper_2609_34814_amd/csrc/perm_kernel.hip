// Cache-aware query-row permutation for gfx950.
//
// Phases (Sec. IV-C..IV-E, Alg. 1, Alg. 2):
//   0  mask statistics from the bit-packed rows and columns (n_i, c_j, nnz,
//      distinct columns, adjacent-row overlap, sum c_j^2);
//   1  skip cases 1-3 (fits in cache, too little work, already local);
//   2  matrix-free centred subspace iteration in exact fixed point: the centred
//      products are exact integer products of the packed mask with X (or Ys)
//      plus the rank-one centring corrections scaled by m (Alg. 1); the
//      2-column QR is a Cholesky-QR of the exactly summed Gram matrix (one IEEE
//      fp64 rounding per operation, no contraction); then Rayleigh-Ritz with
//      one Jacobi rotation and a canonical column sign;
//   3  skip case 4 (the rank-2 embedding keeps too little of ||M~||_F^2);
//   4  Stage 1: sort of the rows by polar angle (Eq. 4) in the order of an exact
//      integer comparator (half-plane class, then the sign of the cross product,
//      then the row index);
//   5  Stage 2: the order is cut into n_xcd contiguous segments of equal work
//      (w_i = n_i + 1, a prefix sum over the order decides each row's segment)
//      and each segment into buckets of W rows; one bitonic sort over
//      (bucket, -n_i, position) keys sorts every bucket by descending n_i,
//      stably. The segment table is an output: the attention kernel runs
//      segment x on XCD x.
// Two forms, both exact, so the same result bit for bit:
//   * heads of at most 1024 rows and columns: perm_mfma_kernel, one workgroup per head
//     and one launch for all heads; the centred products are int8 matrix-core products of the
//     mask bits with the base-256 digits of X and Ys (see the kernel);
//   * larger heads: per subspace step mfma_gather_kernel (QR and M^T X) and mfma_scatter_kernel (M Ys),
//     several workgroups per head, the first pair also phases 0-1; phases 3-5 in perm_finish_kernel (one
//     workgroup per head). Per-head state between the kernels lives in the workspace.
// Every sum is an exact integer, so neither the order of parallel reductions nor the slicing nor the
// form matters. Supports m, n <= 4096.

#pragma clang fp contract(off)

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "perm_launch.h"

namespace {

constexpr int MAXB = 4096;

constexpr int FLAG_FITS_CACHE = 1, FLAG_LITTLE_WORK = 2, FLAG_LOCAL = 4, FLAG_UNSTRUCTURED = 8, FLAG_DEGENERATE = 16,
              FLAG_IDENTITY = 64;
constexpr int SKIP_AUTO = 0, SKIP_ALWAYS = 2;

// A workgroup of NT threads on a head of at most CAP rows and columns, PER a thread.
template <int NT_, int CAP_>
struct Cfg {
  static constexpr int NT = NT_, CAP = CAP_, NW = NT / 64, PER = CAP / NT;
};

template <typename C>
struct Shared {
  int32_t cc[C::CAP];        // column counts; later the Stage-1 order
  int32_t xs[2 * C::CAP];    // X (2^30 fixed point), later U
  uint64_t key[2][C::CAP];   // sort scratch
  int64_t red[2][5][C::NW];  // wavefront partials of the reductions, two alternating slot sets
  int32_t seg[65];           // XCD segment starts of the current order
};

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ int bitlen_u64(uint64_t v) { return v ? 64 - __clzll((long long)v) : 0; }
__device__ __forceinline__ uint64_t uabs64(int64_t v) { return v < 0 ? (uint64_t)(-v) : (uint64_t)v; }

// Wavefront reductions with DPP lane moves (a few cycles each, where a lane shuffle goes through
// LDS): xor 1 and xor 2 within quads, then the half-row and row mirrors, then the row broadcasts of
// lane 15 and lane 31, which leave the total in lane 63; it is read back to every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROW_MASK, 0xf, false);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t lane63(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ int64_t wave_sum(int64_t v) {
  uint64_t u = (uint64_t)v;  // two's complement: the sum modulo 2^64 is the exact sum
  u += dpp64<0xB1, 0xf>(u);   // quad_perm [1,0,3,2]
  u += dpp64<0x4E, 0xf>(u);   // quad_perm [2,3,0,1]
  u += dpp64<0x141, 0xf>(u);  // row_half_mirror
  u += dpp64<0x140, 0xf>(u);  // row_mirror
  u += dpp64<0x142, 0xa>(u);  // row_bcast15 into rows 1 and 3
  u += dpp64<0x143, 0xc>(u);  // row_bcast31 into rows 2 and 3
  return (int64_t)lane63(u);
}
__device__ __forceinline__ uint32_t wave_max32(uint32_t v) {
  v = max(v, (uint32_t)wa::dpp32<0xB1, 0xf>(0, (int)v));
  v = max(v, (uint32_t)wa::dpp32<0x4E, 0xf>(0, (int)v));
  v = max(v, (uint32_t)wa::dpp32<0x141, 0xf>(0, (int)v));
  v = max(v, (uint32_t)wa::dpp32<0x140, 0xf>(0, (int)v));
  v = max(v, (uint32_t)wa::dpp32<0x142, 0xa>(0, (int)v));
  v = max(v, (uint32_t)wa::dpp32<0x143, 0xc>(0, (int)v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Scheduling fence between the phases of a kernel: no instruction moves across it. Left alone, the
// compiler interleaves the phases (the products, the reductions, the fp64 Cholesky factor) in a way that
// made the one-workgroup kernel three times slower than the same code with these fences.
#define WA_PHASE_FENCE() __builtin_amdgcn_sched_barrier(0)

// Reductions over the workgroup, returned to every thread: each wavefront reduces its lanes and parks
// its partial in LDS, and after the barrier the first lanes of every wavefront read the NW partials (one
// read each) and reduce them within their DPP row. Consecutive reductions alternate between the two slot
// sets (turn), so a wavefront that writes the partials of the next reduction never overwrites ones that
// another is still reading. One barrier, which also publishes every LDS write made before the call.
template <int NW, typename T, typename F>
__device__ __forceinline__ T lanes_reduce(T v, F&& dpp) {  // over NW = 4, 8 or 16 lanes; the result in lane 0
  static_assert(NW == 4 || NW == 8 || NW == 16, "the partials are reduced within one DPP row");
  v = dpp(v, std::integral_constant<int, 0xB1>{});             // quad_perm [1,0,3,2]
  v = dpp(v, std::integral_constant<int, 0x4E>{});             // quad_perm [2,3,0,1]
  if (NW > 4) v = dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  if (NW > 8) v = dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror
  return v;
}
template <typename C, int K>
__device__ __forceinline__ void wg_sum(int64_t (&red)[2][5][C::NW], int& turn, int64_t (&v)[K]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, buf = turn++ & 1;
  WA_PHASE_FENCE();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) red[buf][k][w] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t t = lanes_reduce<C::NW>((uint64_t)red[buf][k][lane < C::NW ? lane : 0], [](uint64_t x, auto ctrl) {
      return x + dpp64<decltype(ctrl)::value, 0xf>(x);
    });
    v[k] = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(t >> 32), 0) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)t, 0));
  }
  WA_PHASE_FENCE();
}
// Maximum of K uint32 values each.
template <typename C, int K>
__device__ __forceinline__ void wg_max(int64_t (&red)[2][5][C::NW], int& turn, uint32_t (&v)[K]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, buf = turn++ & 1;
  WA_PHASE_FENCE();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_max32(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) red[buf][k][w] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint32_t t = lanes_reduce<C::NW>((uint32_t)red[buf][k][lane < C::NW ? lane : 0], [](uint32_t x, auto ctrl) {
      return max(x, (uint32_t)wa::dpp32<decltype(ctrl)::value, 0xf>(0, (int)x));
    });
    v[k] = (uint32_t)__builtin_amdgcn_readlane((int)t, 0);
  }
  WA_PHASE_FENCE();
}
// Bit length of the largest of the values whose bitwise or is v.
template <typename C>
__device__ __forceinline__ int wg_bitlen(int64_t (&red)[2][5][C::NW], int& turn, uint64_t v) {
  uint32_t b[1] = {(uint32_t)bitlen_u64(v)};
  wg_max<C, 1>(red, turn, b);
  return (int)b[0];
}

struct Head {
  const uint64_t* rowbits;  // [nw][m] word-major: word w of row i at w * m + i
  const uint64_t* colbits;  // [mw][n] word-major: word v of column j at v * n + j
  const int32_t* row_nnz;   // [m]
  int m, n, nw, mw;
};

// Cholesky factor of the 2 x 2 Gram matrix g of a block Z (exact sums of its entries shifted to 24
// bits): r11, r12, r22, and whether the second column keeps a direction of its own (its residual u
// above G22 2^-30). One IEEE fp64 rounding per operation, no contraction.
struct Chol {
  double r11, r12, r22;
  bool rank2;
};
__device__ __forceinline__ Chol chol2(const int64_t (&g)[3]) {
  const double G11 = (double)g[0], G12 = (double)g[1], G22 = (double)g[2];
  Chol c;
  c.r11 = __builtin_sqrt(G11);
  c.r12 = G12 / c.r11;
  const double u = G22 - c.r12 * c.r12;
  c.rank2 = u > G22 * 0x1p-30;
  c.r22 = c.rank2 ? __builtin_sqrt(u) : 0.0;
  return c;
}

// Row (x0, x1) of the orthonormal factor X = Z R^-1 in 2^30 fixed point, from the row of Z shifted
// right by the Gram shift (z0s, z1s); the second entry is 0 when Z has rank one.
__device__ __forceinline__ void orth_row(const Chol& c, int64_t z0s, int64_t z1s, int32_t& x0, int32_t& x1) {
  const double q0 = (double)z0s / c.r11;
  x0 = (int32_t)__builtin_rint(q0 * 1073741824.0);
  if (c.rank2) {
    const double q1 = ((double)z1s - c.r12 * q0) / c.r22;
    x1 = (int32_t)__builtin_rint(q1 * 1073741824.0);
  } else {
    x1 = 0;
  }
}

// Threads that share one row in a rank sort: the largest power of two up to 16 with threads * rows <= nt.
// They are consecutive lanes of one wavefront.
__device__ __forceinline__ int lanes_per_line(int lines, int nt) {
  int t = 1;
  while (t < 16 && 2 * t * lines <= nt) t *= 2;
  return t;
}

// Sum over groups of t consecutive lanes (t a power of two up to 64); every lane of a group receives its
// group's sum.
__device__ __forceinline__ int group_sum(int v, int t) {
  for (int o = 1; o < t; o <<= 1) v += __shfl_xor(v, o);
  return v;
}

// Heads of at most this many rows are ordered by rank sorts (no barriers; m^2 / NT compares a thread),
// larger ones by bitonic sorts.
constexpr int kRankSortMax = 128;

__device__ __forceinline__ Head head_of(const WaPermLaunch& a, int h) {
  Head H;
  H.m = a.m;
  H.n = a.n;
  H.nw = (a.n + 63) / 64;
  H.mw = (a.m + 63) / 64;
  H.rowbits = a.rowbits + (int64_t)h * a.m * H.nw;
  H.colbits = a.colbits + (int64_t)h * a.n * H.mw;
  H.row_nnz = a.row_nnz + (int64_t)h * a.m;
  return H;
}

__device__ __forceinline__ int angle_class(int64_t x, int64_t y) {
  if (y < 0) return 0;
  if (y == 0) return x >= 0 ? 1 : 3;
  return 2;
}

// true if row a precedes row b in ascending polar angle (ties: smaller index); xs: (x, y) of each row
__device__ __forceinline__ bool angle_less(const int32_t* xs, int a, int b) {
  const int64_t xa = xs[2 * a], ya = xs[2 * a + 1];
  const int64_t xb = xs[2 * b], yb = xs[2 * b + 1];
  const int ca = angle_class(xa, ya), cb = angle_class(xb, yb);
  if (ca != cb) return ca < cb;
  if (ca == 0 || ca == 2) {
    const int64_t cross = xa * yb - ya * xb;
    if (cross != 0) return cross > 0;
  }
  return a < b;
}

// Sort key of a row: angle class, 50 bits of a monotone function of the angle within the class, and the
// row. In the half-planes that function is +-x / (|x| + |y|), one correctly rounded fp64 division, so a row
// of smaller angle never has the larger value; rows whose upper 52 bits agree are then put in the exact
// order. A key compare costs a fraction of the exact one (two 64-bit cross products).
__device__ __forceinline__ uint64_t angle_key(int32_t x, int32_t y, int row) {
  const int c = angle_class(x, y);
  uint64_t u = 0;
  if (c == 0 || c == 2) {
    const double den = (double)((int64_t)(x < 0 ? -(int64_t)x : x) + (int64_t)(y < 0 ? -(int64_t)y : y));
    const double q = (c == 0 ? (double)x : -(double)x) / den;
    const uint64_t b = (uint64_t)__double_as_longlong(q + 0.0);  // (-0 and 0 are one value)
    u = (b >> 63) ? ~b : b | 0x8000000000000000ull;
  }
  return ((uint64_t)c << 62) | (u >> 14 << 12) | (uint64_t)row;
}

// Work-balanced XCD segments of the order held in sh.cc[0..m): position p belongs to segment
// min(n_xcd - 1, n_xcd * W_p / W_m) with W_p the sum of (n_i + 1) over the first p positions.
// Fills sh.seg[0..n_xcd] (and seg_out, if given). Uses sh.xs as scratch.
template <typename C>
__device__ void compute_segments(Shared<C>& sh, const int32_t* row_nnz, int m, int n_xcd, int32_t* seg_out) {
  constexpr int NT = C::NT, NWAVE = C::NW;
  int32_t* part = reinterpret_cast<int32_t*>(sh.key[0]);
  const int tid = threadIdx.x;
  const int per = (m + NT - 1) / NT;
  const int lo = min(tid * per, m), hi = min(lo + per, m);
  int32_t local = 0;
  for (int p = lo; p < hi; ++p) local += row_nnz[sh.cc[p]] + 1;
  // prefix sums of the thread totals: within the wavefront by lane shifts, then over the wavefront totals
  const int lane = tid & 63, w = tid >> 6;
  const int32_t incl = wa::lane_prefix_sum(local);
  if (lane == 63) part[w] = incl;
  __syncthreads();
  int32_t before = 0, sum = 0;
  for (int i = 0; i < NWAVE; ++i) {
    const int32_t t = part[i];
    before += i < w ? t : 0;
    sum += t;
  }
  const int64_t total = sum;
  int32_t run = before + incl - local;   // W_lo
  int32_t* segof = sh.xs;
  for (int p = lo; p < hi; ++p) {
    const int64_t x = ((int64_t)n_xcd * run) / total;
    segof[p] = (int32_t)(x < n_xcd - 1 ? x : n_xcd - 1);
    run += row_nnz[sh.cc[p]] + 1;
  }
  __syncthreads();
  for (int p = tid; p < m; p += NT) {
    const int prev = p > 0 ? segof[p - 1] : -1;
    for (int x = prev + 1; x <= segof[p]; ++x) sh.seg[x] = p;
  }
  if (tid == 0)
    for (int x = segof[m - 1] + 1; x <= n_xcd; ++x) sh.seg[x] = m;
  __syncthreads();
  if (seg_out)
    for (int x = tid; x <= n_xcd; x += NT) seg_out[x] = sh.seg[x];
}

// Writes the identity order for head h (and its segments and flags).
template <typename C>
__device__ void write_identity(const WaPermLaunch& a, Shared<C>& sh, int h, int flags, bool zero_embedding) {
  constexpr int NT = C::NT;
  const int tid = threadIdx.x, m = a.m;
  int32_t* perm = a.perm + (int64_t)h * m;
  for (int i = tid; i < m; i += NT) {
    perm[i] = i;
    sh.cc[i] = i;
    if (a.stage1) a.stage1[(int64_t)h * m + i] = i;
    if (zero_embedding && a.embedding) {
      a.embedding[((int64_t)h * m + i) * 2] = 0;
      a.embedding[((int64_t)h * m + i) * 2 + 1] = 0;
    }
  }
  __syncthreads();
  compute_segments(sh, a.row_nnz + (int64_t)h * m, m, a.n_xcd,
                   a.seg_start ? a.seg_start + (int64_t)h * (a.n_xcd + 1) : nullptr);
  if (a.flags && tid == 0) a.flags[h] = (uint8_t)(flags | FLAG_IDENTITY);
}

// What the set-up of a head leaves for the subspace iteration (uniform over the workgroup).
struct HeadInit {
  int status;  // 0: iterate; 1: done (a skipped head with its identity order written)
  int flags;   // skip-rule flags of cases 1-3
  int64_t nnz, sum_c2;
  int64_t adj_and, adj_or;  // adjacent-row overlap of the natural order
};
constexpr int HEAD_ITERATE = 0, HEAD_DONE = 1;

// Skip-rule flags of cases 1-3.
__device__ int tier1_flags(const WaPermLaunch& a, int64_t nnz, int64_t distinct, int64_t adj_and, int64_t adj_or) {
  int f = 0;
  const double kvb = (double)(2 * a.block * a.head_dim * 2);
  if ((double)distinct * kvb <= a.prof.cache_bytes) f |= FLAG_FITS_CACHE;
  const double saving = (double)nnz * a.prof.gain_ns_per_block;
  // the cost curve of the form that builds this head: one workgroup for small heads, else sliced
  const bool fused = (double)a.m <= a.prof.fused_max_blocks;
  const double c0 = fused ? a.prof.ovh_fused_ns_fixed : a.prof.ovh_ns_fixed;
  const double c1 = fused ? a.prof.ovh_fused_ns_per_row : a.prof.ovh_ns_per_row;
  const double c2 = fused ? a.prof.ovh_fused_ns_per_nnz : a.prof.ovh_ns_per_nnz;
  const double cost = c0 + c1 * (double)a.m + c2 * (double)nnz;
  if (saving < cost) f |= FLAG_LITTLE_WORK;
  if (adj_or > 0 && (double)adj_and / (double)adj_or >= a.prof.j_max) f |= FLAG_LOCAL;
  return f;
}

// Entry (z0, z1) of the seeded start block.
__device__ __forceinline__ void start_row(const WaPermLaunch& a, int h, int i, int64_t& z0, int64_t& z1) {
  const uint64_t base = a.seed + 2ull * ((uint64_t)h * (uint64_t)a.m + (uint64_t)i);
  z0 = (int64_t)(splitmix64(base) >> 40) - (1ll << 23);
  z1 = (int64_t)(splitmix64(base + 1ull) >> 40) - (1ll << 23);
}

// Adds the overlap of the row pairs that straddle two 64-row groups, words [first, ...) by `step`.
__device__ __forceinline__ void straddling_overlap(const Head& H, int first, int step, int64_t& both, int64_t& any) {
  for (int e = first; e < (H.mw - 1) * H.nw; e += step) {
    const int g = e / H.nw, w = e - g * H.nw;
    const uint64_t* p = H.rowbits + (int64_t)w * H.m + 64 * g + 63;
    const uint64_t x = p[0], y = p[1];
    both += __popcll(x & y);
    any += __popcll(x | y);
  }
}

// Set-up of a head of the one-workgroup form (one row and column a thread): statistics, skip cases 1-3, and
// the seeded start block. cc: the thread's column count; z: its row of the start block.
template <typename C>
__device__ HeadInit init_head(const WaPermLaunch& a, Shared<C>& sh, int& turn, int h, int32_t& cc, int64_t (&z)[2]) {
  const int tid = threadIdx.x;
  const int m = a.m, n = a.n;
  const Head H = head_of(a, h);
  constexpr int WB = 8;  // words loaded together, so that their latencies overlap
  int64_t st[5] = {0, 0, 0, 0, 0};  // nnz, distinct, sum c^2, adjacent-row overlap
  int c = 0;
  if (tid < n)
    for (int v0 = 0; v0 < H.mw; v0 += WB) {
      uint64_t wd[WB];
#pragma unroll
      for (int u = 0; u < WB; ++u) wd[u] = v0 + u < H.mw ? H.colbits[(int64_t)(v0 + u) * n + tid] : 0ull;
#pragma unroll
      for (int u = 0; u < WB; ++u) c += __popcll(wd[u]);
    }
  cc = c;
  st[0] = c;
  st[1] = c > 0;
  st[2] = (int64_t)c * c;
  if (tid < H.mw) {
    const int2 g = a.adj[(int64_t)h * H.mw + tid];
    st[3] = g.x;
    st[4] = g.y;
  }
  straddling_overlap(H, tid, C::NT, st[3], st[4]);
  wg_sum<C, 5>(sh.red, turn, st);
  const int flags = tier1_flags(a, st[0], st[1], st[3], st[4]);
  if (a.skip_mode == SKIP_ALWAYS || (a.skip_mode == SKIP_AUTO && flags != 0)) {
    write_identity(a, sh, h, flags, true);
    return {HEAD_DONE, flags, st[0], st[2], st[3], st[4]};
  }
  z[0] = z[1] = 0;
  if (tid < m) start_row(a, h, tid, z[0], z[1]);
  return {HEAD_ITERATE, flags, st[0], st[2], st[3], st[4]};
}

// Lane l ^ S's value.
template <int S>
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v) {
  if constexpr (S == 1) return (uint32_t)wa::dpp32<0xB1, 0xf>(0, (int)v);
  if constexpr (S == 2) return (uint32_t)wa::dpp32<0x4E, 0xf>(0, (int)v);
  if constexpr (S == 4)  // half-row mirror (l ^ 7), then quad mirror (l ^ 3)
    return (uint32_t)wa::dpp32<0x1B, 0xf>(0, wa::dpp32<0x141, 0xf>(0, (int)v));
  if constexpr (S == 8) return (uint32_t)wa::dpp32<0x128, 0xf>(0, (int)v);  // row_ror:8
  if constexpr (S == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);
  if constexpr (S == 32) return (uint32_t)__shfl_xor((int)v, 32);
}
template <int S>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v) {
  return ((uint64_t)lane_xor32<S>((uint32_t)(v >> 32)) << 32) | lane_xor32<S>((uint32_t)v);
}

// Bitonic sort, ascending, of NT R keys held R a thread: key 64 (R wave + r) + lane in v[r]. Partners
// at a distance of up to 32 are reached by lane moves, up to 32 R within the thread, and only the others
// (10 of the 78 stages at 4,096 keys) through LDS, with one barrier each (buf: two buffers of NT R keys in turn).
// With every stage through LDS and a barrier after each, and the exact comparator in the first sort, the
// finishing phase of 2,841-block heads took 149 us; it takes 57.
template <typename C, int R>
__device__ __forceinline__ void sort_keys(uint64_t (&v)[R], uint64_t (*buf)[C::CAP]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int LG = __builtin_ctz(C::NT * R);
  int turn = 0;
  auto up = [&](int r, int k) { return ((64 * (R * w + r) + lane) >> k & 1) == 0; };
  // keeps the smaller (or larger) of own and partner's key
  auto keep = [&](uint64_t own, uint64_t other, bool smaller) { return (other < own) == smaller ? other : own; };
  auto lanes = [&](int k, auto dist) {
    constexpr int S = decltype(dist)::value;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = keep(v[r], lane_xor<S>(v[r]), ((lane & S) == 0) == up(r, k));
  };
#pragma unroll 1
  for (int k = 1; k <= LG; ++k) {
#pragma unroll 1
    for (int lj = k - 1; lj >= 6; --lj) {
      const int d = 1 << (lj - 6);  // distance in 64-key runs
      if (d >= R) {                 // another wavefront's
        uint64_t* b = buf[turn++ & 1];
#pragma unroll
        for (int r = 0; r < R; ++r) b[64 * (R * w + r) + lane] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int run = R * w + r;
          v[r] = keep(v[r], b[64 * (run ^ d) + lane], ((run & d) == 0) == up(r, k));
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
          for (int dd = 1; dd < R; dd *= 2)
            if (dd == d && (r & dd) == 0) {
              const uint64_t x = v[r], y = v[r | dd];
              const bool swap = (y < x) == up(r, k);
              v[r] = swap ? y : x;
              v[r | dd] = swap ? x : y;
            }
        }
      }
    }
    if (k > 5) lanes(k, std::integral_constant<int, 32>{});
    if (k > 4) lanes(k, std::integral_constant<int, 16>{});
    if (k > 3) lanes(k, std::integral_constant<int, 8>{});
    if (k > 2) lanes(k, std::integral_constant<int, 4>{});
    if (k > 1) lanes(k, std::integral_constant<int, 2>{});
    lanes(k, std::integral_constant<int, 1>{});
  }
}

// Rayleigh-Ritz on the last product Z (rows tid + k NT, zr) of X (in sh.xs), canonical sign, skip case 4,
// Stage 1 and Stage 2, then case 3 against the built order. bly: the bit length of the max |Ym| of that
// product's first half (it fixes sy); adj_and / adj_or: the natural order's adjacent-row overlap.
template <typename C>
__device__ void finish_head(const WaPermLaunch& a, Shared<C>& sh, int& turn, int h, bool degen, int64_t nnz,
                            int64_t sum_c2, int flags, int bly, const int64_t (&zr)[C::PER][2], int64_t adj_and,
                            int64_t adj_or) {
  constexpr int NT = C::NT, PER = C::PER;
  const int tid = threadIdx.x;
  const int m = a.m;
  const Head H = head_of(a, h);
  int32_t* perm = a.perm + (int64_t)h * m;
  int32_t* seg_out = a.seg_start ? a.seg_start + (int64_t)h * (a.n_xcd + 1) : nullptr;
  int64_t trace = 0;
  int scale_exp = 0;
  if (!degen) {
    const int sy = bly > 30 ? bly - 30 : 0;
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (tid + k * NT < m) any |= uabs64(zr[k][0]) | uabs64(zr[k][1]);
    const int bl = wg_bitlen<C>(sh.red, turn, any);  // its barrier also publishes sh.xs
    const int s_r = bl > 24 ? bl - 24 : 0;
    int64_t b[4] = {0, 0, 0, 0};
    int32_t x[PER][2];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + k * NT;
      x[k][0] = i < m ? sh.xs[2 * i] : 0;
      x[k][1] = i < m ? sh.xs[2 * i + 1] : 0;
      if (i < m) {
        const int64_t x0 = x[k][0] >> 6, x1 = x[k][1] >> 6;
        const int64_t z0 = zr[k][0] >> s_r, z1 = zr[k][1] >> s_r;
        b[0] += x0 * z0;
        b[1] += x0 * z1;
        b[2] += x1 * z0;
        b[3] += x1 * z1;
      }
    }
    wg_sum<C, 4>(sh.red, turn, b);
    trace = b[0] + b[3];
    scale_exp = sy + s_r + 6 - 60;
    const double A = (double)b[0], D = (double)b[3], B = (double)((b[1] + b[2]) >> 1);
    double t = 0.0, cs = 1.0, sn = 0.0;
    if (B != 0.0) {
      const double tau = (D - A) / (2.0 * B);
      const double sgn = tau >= 0.0 ? 1.0 : -1.0;
      t = sgn / (__builtin_fabs(tau) + __builtin_sqrt(1.0 + tau * tau));
      cs = 1.0 / __builtin_sqrt(1.0 + t * t);
      sn = t * cs;
    }
    const double lam0 = A - t * B, lam1 = D + t * B;
    const bool swp = lam1 > lam0;
    uint32_t mag[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const double x0 = (double)x[k][0], x1 = (double)x[k][1];
      const int32_t u0 = (int32_t)__builtin_rint(cs * x0 - sn * x1);
      const int32_t u1 = (int32_t)__builtin_rint(sn * x0 + cs * x1);
      x[k][0] = swp ? u1 : u0;
      x[k][1] = swp ? u0 : u1;
#pragma unroll
      for (int c = 0; c < 2; ++c) mag[c] = max(mag[c], (uint32_t)uabs64(x[k][c]));  // (0 past the head)
    }
    // canonical sign: the entry of largest magnitude (smallest row on ties) is positive
    const uint32_t own[2] = {mag[0], mag[1]};
    wg_max<C, 2>(sh.red, turn, mag);
    uint32_t first[2] = {0, 0};  // largest of 2 (~row) + (entry < 0) over the rows of that magnitude
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (own[c] == mag[c])
#pragma unroll
        for (int k = PER - 1; k >= 0; --k) {
          const int i = tid + k * NT;
          if (i < m && (uint32_t)uabs64(x[k][c]) == mag[c])
            first[c] = max(first[c], ((uint32_t)(0x7FFFFFFF - i) << 1) | (x[k][c] < 0 ? 1u : 0u));
        }
    wg_max<C, 2>(sh.red, turn, first);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + k * NT;
      if (i < m) {
        sh.xs[2 * i] = first[0] & 1u ? -x[k][0] : x[k][0];
        sh.xs[2 * i + 1] = first[1] & 1u ? -x[k][1] : x[k][1];
      }
    }
  }

  // ---- phase 3: skip case 4 ----
  if (degen) {
    flags |= FLAG_DEGENERATE;
  } else {
    const double den = (double)m * (double)((int64_t)m * nnz - sum_c2);
    const double eta = den <= 0.0 ? 0.0 : __builtin_ldexp((double)trace, scale_exp) / den;
    if (eta < a.prof.eta_min) flags |= FLAG_UNSTRUCTURED;
  }
  __syncthreads();
  if (a.embedding)
    for (int i = tid; i < m; i += NT) {
      a.embedding[((int64_t)h * m + i) * 2] = degen ? 0 : sh.xs[2 * i];
      a.embedding[((int64_t)h * m + i) * 2 + 1] = degen ? 0 : sh.xs[2 * i + 1];
    }
  if (a.skip_mode == SKIP_AUTO && (flags & FLAG_UNSTRUCTURED)) {
    __syncthreads();  // every thread has written its embedding rows (read from sh.xs)
    write_identity(a, sh, h, flags, false);
    return;
  }

  // ---- phase 4: Stage 1, exact polar-angle order ----
  const bool rank = m <= kRankSortMax;
  const int per_row = lanes_per_line(m, NT);  // of the rank sorts
  const int line = tid / per_row, sub = tid % per_row;
  // sorts the keys key(0), ..., key(m - 1) of distinct value and calls out(position, key)
  auto sort_all = [&](auto&& key, auto&& out) {
    auto run = [&](auto regs) {
      constexpr int R = decltype(regs)::value;
      uint64_t v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = 64 * (R * (tid >> 6) + r) + (tid & 63);
        v[r] = e < m ? key(e) : ~0ull;  // (orders last; no key has all bits set)
      }
      sort_keys<C, R>(v, sh.key);
      __syncthreads();  // every key and buffer is read before out writes
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = 64 * (R * (tid >> 6) + r) + (tid & 63);
        if (e < m) out(e, v[r]);
      }
    };
    if constexpr (PER == 4) {
      if (m <= 2 * NT) {
        run(std::integral_constant<int, 2>{});
        return;
      }
    }
    run(std::integral_constant<int, PER>{});
  };
  if (degen) {
    for (int i = tid; i < m; i += NT) sh.cc[i] = i;
  } else if (rank) {
    // rank sort: a row's position is the number of rows that precede it (a total order)
    int r = 0;
    if (line < m)
      for (int j = sub; j < m; j += per_row) r += angle_less(sh.xs, j, line) ? 1 : 0;
    r = group_sum(r, per_row);
    if (line < m && sub == 0) sh.cc[r] = line;
  } else {
    uint64_t* keys = sh.key[0];
    sort_all([&](int i) { return angle_key(sh.xs[2 * i], sh.xs[2 * i + 1], i); },
             [&](int e, uint64_t x) { keys[e] = x; });
    // Runs of keys that agree above the row are in row order; odd-even passes put them in the exact order (rows
    // of one angle stay as they are, so this is one pass over the neighbours unless 50 bits were too few).
    for (;;) {
      uint32_t moved[1] = {0};
      for (int odd = 0; odd < 2; ++odd) {
        __syncthreads();
        for (int e = 2 * tid + odd; e + 1 < m; e += 2 * NT) {
          const uint64_t x = keys[e], y = keys[e + 1];
          if ((x ^ y) >> 12 == 0 && angle_less(sh.xs, (int)(y & 0xFFF), (int)(x & 0xFFF))) {
            keys[e] = y;
            keys[e + 1] = x;
            moved[0] = 1;
          }
        }
      }
      wg_max<C, 1>(sh.red, turn, moved);
      if (!moved[0]) break;
    }
    for (int i = tid; i < m; i += NT) sh.cc[i] = (int32_t)(keys[i] & 0xFFF);
  }
  __syncthreads();
  if (a.stage1)
    for (int i = tid; i < m; i += NT) a.stage1[(int64_t)h * m + i] = sh.cc[i];

  // ---- phase 5: work-balanced segments, wave buckets, Stage 2 ----
  compute_segments(sh, H.row_nnz, m, a.n_xcd, seg_out);
  const int32_t* segof = sh.xs;  // segment of each position, left by compute_segments
  auto bucket_key = [&](int p) {
    const int x = segof[p];
    const int off = p - sh.seg[x];
    const uint64_t bucket = ((uint64_t)x << 12) | (uint64_t)(off / a.wave);
    const uint64_t nz = (uint64_t)H.row_nnz[sh.cc[p]];
    return (bucket << 32) | ((0xFFFFull - nz) << 16) | (uint64_t)p;
  };
  int32_t* fin = sh.xs + C::CAP;  // the built order (beside the segment map, in the half X leaves free)
  if (rank) {
    uint64_t* keys = sh.key[0];
    __syncthreads();  // the scan partials in the key buffer are read
    for (int p = tid; p < m; p += NT) keys[p] = bucket_key(p);
    __syncthreads();
    int r = 0;
    if (line < m) {
      const uint64_t kp = keys[line];
      for (int q = sub; q < m; q += per_row) r += keys[q] < kp ? 1 : 0;
    }
    r = group_sum(r, per_row);
    if (line < m && sub == 0) fin[r] = sh.cc[line];
  } else {
    sort_all(bucket_key, [&](int e, uint64_t x) { fin[e] = sh.cc[(int)(x & 0xFFFFull)]; });
  }
  __syncthreads();
  for (int s = tid; s < m; s += NT) perm[s] = fin[s];

  // ---- case 3 against the built order: it must raise the adjacent-row overlap ----
  if (a.skip_mode == SKIP_AUTO) {
    int64_t ov[2] = {0, 0};
    for (int t = tid; t < (m - 1) * H.nw; t += NT) {
      const int w = t / (m - 1), s = t % (m - 1);
      const uint64_t x = H.rowbits[(int64_t)w * m + fin[s]], y = H.rowbits[(int64_t)w * m + fin[s + 1]];
      ov[0] += __popcll(x & y);
      ov[1] += __popcll(x | y);
    }
    wg_sum<C, 2>(sh.red, turn, ov);
    if (ov[0] * adj_or <= adj_and * ov[1]) {  // J(built order) <= J(natural order), exactly
      __syncthreads();
      write_identity(a, sh, h, flags | FLAG_LOCAL, false);
      return;
    }
  }
  if (a.flags && tid == 0) a.flags[h] = (uint8_t)flags;
}

using FinishCfg = Cfg<1024, MAXB>;  // the finishing kernel of the larger heads
__global__ __launch_bounds__(FinishCfg::NT) void perm_finish_kernel(WaPermLaunch a) {
  using C = FinishCfg;
  __shared__ Shared<C> sh;
  const int h = blockIdx.x;
  const PermState* S = a.state + h;
  if (S->done) {
    write_identity(a, sh, h, S->flags, true);
    return;
  }
  const bool degen = S->degen != 0;
  int64_t zr[C::PER][2] = {};
  if (!degen) {
    const int2* xg = reinterpret_cast<const int2*>(a.xg) + (int64_t)h * a.m;
#pragma unroll
    for (int k = 0; k < C::PER; ++k) {
      const int i = (int)threadIdx.x + k * C::NT;
      if (i < a.m) {
        const int2 x = xg[i];
        sh.xs[2 * i] = x.x;
        sh.xs[2 * i + 1] = x.y;
        zr[k][0] = a.z[((int64_t)h * a.m + i) * 2];
        zr[k][1] = a.z[((int64_t)h * a.m + i) * 2 + 1];
      }
    }
  }
  int turn = 0;
  finish_head(a, sh, turn, h, degen, S->nnz, S->sum_c2, S->flags, S->bly, zr, S->adj_and, S->adj_or);
}

// ---------------------------------------------------------------------------------------------
// The centred products on the matrix cores.
//
// An integer v with |v| <= 2^31 - 2^25 is the sum of its four balanced base-256 digits,
// v = sum_b d_b 256^b with d_b in [-128, 127] (d_0 is the low byte read as a signed byte, then
// v <- (v - d_0) / 256, exactly, and so on; the last digit stays in range because the lower ones add
// at most 128 (1 + 256 + 65536) < 2^23 to it). X (2^30 per unit, a column of an orthonormal block) and
// Ys (30 significant bits) stay within 2^30 + 1. So M^T X = sum_b 256^b (M^T D_b), where D_b holds digit
// b of every entry of X: each term is a product of a 0/1 matrix and an int8 matrix, whose int32
// sums are exact (at most 4096 * 128 in magnitude), and the terms are combined exactly in int64.
// One v_mfma_i32_16x16x64_i8 takes 64 rows of 16 columns of M: A = the eight digit rows (two
// columns of X, four digits each; rows 8-15 repeat them), B = the 16 columns' bits. Lane l = 16 q + r
// loads the whole 64-bit word 4 g + q of line 16 t + r (one 8-byte load a lane for four MFMAs) and MFMA j
// takes 16 of its bits, so the contraction index of MFMA j, lane group q, slot 4 d + i is
// row 64 (4 g + q) + 32 (j / 2) + 4 (j mod 2) + d + 8 i: bits d, d + 8, d + 16, d + 24 of a half word are one
// shift and one mask, four bytes of 0 or 1. The digits are stored in that order (digit_column), so that
// A is a 16-byte LDS read. Lane l receives digit rows 4 q .. +3 of line r, so lanes 0-15 hold the line's
// product with the first column of X and lanes 16-31 with the second. M Ys reads the row words the same
// way. Every sum is exact, so the result is the same integers whatever the tiling.
constexpr int kMfmaMax = 1024;  // rows and columns of the heads built in one workgroup: one row or column a thread
typedef int v4i __attribute__((ext_vector_type(4)));

// A digit row holds digit b of column k of X for every row, at row 4 k + b; rows are 16 bytes longer than
// their entries, so that the eight rows one A read takes lie in distinct banks.
__host__ __device__ constexpr int digit_stride(int entries) { return entries + 16; }
// Digits of v: byte b is the balanced digit b.
__device__ __forceinline__ uint32_t digits4(int32_t v) { return ((uint32_t)v + 0x80808080u) ^ 0x80808080u; }

// Four bytes (0 or 1): bits `first`, + 8, + 16, + 24 of half, each 4-dword operand of MFMA j from one half word.
__device__ __forceinline__ v4i mask_bytes(uint64_t word, int j) {
  const uint32_t half = j < 2 ? (uint32_t)word : (uint32_t)(word >> 32);
  v4i r;
#pragma unroll
  for (int d = 0; d < 4; ++d) r[d] = (int)((half >> (4 * (j & 1) + d)) & 0x01010101u);
  return r;
}
__device__ __forceinline__ v4i digit_operand(const int8_t* dg, int stride, int g, int j) {
  const int lane = threadIdx.x & 63;
  return *(const v4i*)(dg + (lane & 7) * stride + 64 * (4 * g + (lane >> 4)) + 16 * j);
}
__device__ __forceinline__ int64_t combine_digits(const v4i& acc) {
  return (int64_t)acc[0] + 256ll * acc[1] + 65536ll * acc[2] + 16777216ll * acc[3];
}

// ---------------------------------------------------------------------------------------------
// Heads of at most kMfmaMax blocks: the whole permutation in one workgroup of NT threads, one row and column
// a thread (NT = 256, 512 or 1024). A wavefront takes up to four 16-line tiles of both products and holds their
// mask words in registers through every step, so a step touches no memory outside the compute unit; what
// bounds it is the chain of its five barriers, reductions and the fp64 factor, which every wavefront
// computes: with 16 wavefronts on a head of 256 blocks each reduction took 2,000 cycles or more, since
// the four of one SIMD issue the same instructions in turn (105 us a call of 12 heads against 52).
template <typename C>
struct MfmaLds {
  __attribute__((aligned(16))) int8_t xd[8 * digit_stride(C::CAP)];  // digit rows of X
  __attribute__((aligned(16))) int8_t yd[8 * digit_stride(C::CAP)];  // digit rows of Ys
  int64_t v[2 * C::CAP];  // Ym of the first product, then Z of the second: [line][column of X]
};

// Digits of the thread's entry (row or column tid) of one column of X or Ys into digit rows row0 .. row0 + 3:
// the four lanes whose entries are 8 apart share a dword in each digit row, so they transpose their 4 x 4
// bytes among themselves (two exchanges) and each writes one digit row's dword. Every thread takes part.
template <int STRIDE>
__device__ __forceinline__ void put_digits(int8_t* dg, int row0, int32_t v) {
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t o = digits4(v);
  uint32_t p = lane_xor32<8>(o);
  o = __builtin_amdgcn_perm(p, o, lane & 8 ? 0x03070105u : 0x06020400u);
  p = lane_xor32<16>(o);
  o = __builtin_amdgcn_perm(p, o, lane & 16 ? 0x03020706u : 0x05040100u);
  const int digit = (lane >> 3) & 3;
  *(uint32_t*)(dg + (row0 + digit) * STRIDE + 32 * (tid >> 5) + 4 * (lane & 7)) = o;
}

// T: tiles a wavefront takes at most.
template <typename C, int T>
struct WaveWords {
  static constexpr int G = C::CAP / 256;  // groups of four words a line
  uint64_t w[G][T];  // [word group g][tile k]: word 4 g + q of line 16 (wave + NW k) + r
  __device__ __forceinline__ void load(const uint64_t* bits, int lines, int words) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int k = 0; k < T; ++k) {
      // a line past the head reads the head's last line: its products are never used
      const int line = min(16 * (wv + C::NW * k) + r, lines - 1);
#pragma unroll
      for (int g = 0; g < G; ++g) w[g][k] = 4 * g + q < words ? bits[(int64_t)(4 * g + q) * lines + line] : 0ull;
    }
  }
  // f(line, column, value) in lanes 0-31 for every line of the wavefront's tiles (line may lie past `lines`)
  template <typename F>
  __device__ __forceinline__ void product(const int8_t* dg, int lines, int words, F&& f) const {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WA_PHASE_FENCE();
    if (16 * wv < lines) {
      v4i acc[T];
#pragma unroll
      for (int k = 0; k < T; ++k) acc[k] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (4 * g < words) {
          uint64_t x[T];
#pragma unroll
          for (int k = 0; k < T; ++k) {
            x[k] = w[g][k];
            // opaque here, so that the words' bytes are not expanded once outside the step loop and held
            asm volatile("" : "+v"(x[k]));
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const v4i av = digit_operand(dg, digit_stride(C::CAP), g, j);
#pragma unroll
            for (int k = 0; k < T; ++k)
              acc[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, mask_bytes(x[k], j), acc[k], 0, 0, 0);
          }
        }
      if (lane < 32)
#pragma unroll
        for (int k = 0; k < T; ++k) f(16 * (wv + C::NW * k) + (lane & 15), lane >> 4, combine_digits(acc[k]));
    }
    WA_PHASE_FENCE();
  }
};

template <int NT, int T>
__global__ __launch_bounds__(NT) void perm_mfma_kernel(WaPermLaunch a) {
  using C = Cfg<NT, NT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  Shared<C>& sh = *reinterpret_cast<Shared<C>*>(smem_raw);
  MfmaLds<C>& L = *reinterpret_cast<MfmaLds<C>*>(smem_raw + ((sizeof(Shared<C>) + 15) & ~(size_t)15));
  const int h = blockIdx.x;
  int turn = 0;  // reductions so far (selects the slot set)
  int32_t cc;    // column count of column tid
  int64_t z[2];  // the thread's row of Z
  const HeadInit hi = init_head(a, sh, turn, h, cc, z);
  if (hi.status == HEAD_DONE) return;
  const int tid = threadIdx.x;  // row tid (QR) and column tid (Ys) of the head
  const int m = a.m, n = a.n;
  const int64_t mm = m;
  const Head H = head_of(a, h);
  WaveWords<C, T> cols, rows;
  cols.load(H.colbits, n, H.mw);
  rows.load(H.rowbits, m, H.nw);
  sh.cc[tid] = cc;
  bool degen = false;
  int bly = 0;
  uint64_t anyz = uabs64(z[0]) | uabs64(z[1]);
  for (int it = 0;; ++it) {
    // ---- Cholesky-QR: X = Z R^-1 (Z: the seeded block at first) ----
    const int blz = wg_bitlen<C>(sh.red, turn, anyz);  // its barrier also publishes Z
    if (it > 0) {
      z[0] = tid < m ? L.v[2 * tid] : 0;
      z[1] = tid < m ? L.v[2 * tid + 1] : 0;
      if (it == a.iters + 1) break;  // the last product: Rayleigh-Ritz in the finishing phases
    }
    const int s = blz > 24 ? blz - 24 : 0;
    const int64_t z0s = z[0] >> s, z1s = z[1] >> s;
    int64_t g[3] = {z0s * z0s, z0s * z1s, z1s * z1s};
    wg_sum<C, 3>(sh.red, turn, g);
    if (g[0] == 0) {  // uniform: every thread holds the same sums
      degen = true;
      break;
    }
    const Chol c = chol2(g);
    int32_t x0 = 0, x1 = 0;
    if (tid < m) {
      orth_row(c, z0s, z1s, x0, x1);
      sh.xs[2 * tid] = x0;
      sh.xs[2 * tid + 1] = x1;
    }
    put_digits<digit_stride(C::CAP)>(L.xd, 0, x0);
    put_digits<digit_stride(C::CAP)>(L.xd, 4, x1);
    int64_t sx[2] = {x0, x1};            // 1^T X
    wg_sum<C, 2>(sh.red, turn, sx);  // its barrier also publishes X, its digits and the column counts
    // ---- Ym = m M^T X - c (1^T X), and the bit length of max |Ym| ----
    uint64_t any = 0;
    cols.product(L.xd, n, H.mw, [&](int j, int k, int64_t ya) {
      if (j < n) {
        const int64_t y = mm * ya - (int64_t)sh.cc[j] * (k == 0 ? sx[0] : sx[1]);
        L.v[2 * j + k] = y;
        any |= uabs64(y);
      }
    });
    bly = wg_bitlen<C>(sh.red, turn, any);  // its barrier also publishes Ym
    const int sy = bly > 30 ? bly - 30 : 0;
    // ---- Ys = Ym >> sy as digit rows, and c^T Ys ----
    const int32_t v0 = tid < n ? (int32_t)(L.v[2 * tid] >> sy) : 0, v1 = tid < n ? (int32_t)(L.v[2 * tid + 1] >> sy) : 0;
    put_digits<digit_stride(C::CAP)>(L.yd, 0, v0);
    put_digits<digit_stride(C::CAP)>(L.yd, 4, v1);
    int64_t py[2] = {(int64_t)cc * v0, (int64_t)cc * v1};
    wg_sum<C, 2>(sh.red, turn, py);  // its barrier also publishes the Ys digits (Ym is read)
    // ---- Z = m M Ys - 1 (c^T Ys) ----
    anyz = 0;
    rows.product(L.yd, m, H.nw, [&](int i, int k, int64_t za) {
      if (i < m) {
        const int64_t zi = mm * za - (k == 0 ? py[0] : py[1]);
        L.v[2 * i + k] = zi;
        anyz |= uabs64(zi);
      }
    });
  }
  const int64_t zr[1][2] = {{z[0], z[1]}};
  finish_head(a, sh, turn, h, degen, hi.nnz, hi.sum_c2, hi.flags, bly, zr, hi.adj_and, hi.adj_or);
}

// ---------------------------------------------------------------------------------------------
// Larger heads: many workgroups a head and two launches a subspace step, X -> Z = m * M~ Ys with
// Ys = (m * M~^T X) >> sy. A workgroup takes a slice of one head's 16-line tiles; the slices are chosen so
// that the heads fill the chip once.
//   gather:   the Cholesky-QR of Z (of the seeded block at first), the next X; its digit rows and 1^T X;
//             then Ym[j] = m * (M^T X)[j] - c_j * 1^T X for the columns of the slice;
//   scatter:  max |Ym|, the digit rows of Ys = Ym >> sy and c^T Ys; then Z[i] = m * (M Ys)[i] - c^T Ys for
//             the rows of the slice.
// Every workgroup of a head does the head's QR (or its Ys) itself, from exact sums, so the slicing does not
// change any result and no launch of its own is needed for it; each line is written by one lane. A step is
// bound by its two launches (about 4 us each), the latency of each workgroup's start (Z or Ym of the head,
// two reductions: about 7 us) and the read of the mask words, 41 MB a product at 40 x 2,841 blocks, from the
// last-level cache (6 us): 19.7 + 16.7 us a step at that size, against 28 + 28 + 7 with a third launch for
// the QR, workgroups of 128 lines that each built the digits byte by byte, and 2-byte mask loads.
using SliceCfg = Cfg<1024, MAXB>;
constexpr int PER = SliceCfg::PER, NWAVE = SliceCfg::NW;
struct SliceLds {
  __attribute__((aligned(16))) int8_t dg[8 * digit_stride(MAXB)];
  int64_t red[2][5][NWAVE];
};

// The thread's entries are 32 (tid / 8) + tid mod 8 + 8 k, k = 0..3: the four that share a dword of a digit
// row (dword tid), so it transposes their 4 x 4 digits alone.
__device__ __forceinline__ int slice_entry(int k) { return 32 * ((int)threadIdx.x >> 3) + ((int)threadIdx.x & 7) + 8 * k; }
__device__ __forceinline__ void put_digits4(int8_t* dg, int row0, const int32_t (&v)[PER]) {
  const uint32_t w0 = digits4(v[0]), w1 = digits4(v[1]), w2 = digits4(v[2]), w3 = digits4(v[3]);
  const uint32_t t0 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), t1 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
  const uint32_t u0 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), u1 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
  uint32_t* d = (uint32_t*)(dg + row0 * digit_stride(MAXB)) + threadIdx.x;
  constexpr int S = digit_stride(MAXB) / 4;
  d[0] = __builtin_amdgcn_perm(u0, t0, 0x05040100u);
  d[S] = __builtin_amdgcn_perm(u0, t0, 0x07060302u);
  d[2 * S] = __builtin_amdgcn_perm(u1, t1, 0x05040100u);
  d[3 * S] = __builtin_amdgcn_perm(u1, t1, 0x07060302u);
}
static_assert(PER == 4, "a thread's entries fill one dword of every digit row");

// f(line, column, value, kept), in lanes 0-31, for the lines of tiles [t0, t1) (line may lie past `lines`). A
// wavefront takes two tiles at a time, which share each digit operand, and loads the words of the next 16
// while it multiplies. (Loading them before the QR or the Ys instead delays the loads of Z or Ym that
// those wait for, and measured 1-2 us slower a launch.) kept: with COUNT, the line's kept blocks.
template <bool COUNT, typename F>
__device__ __forceinline__ void slice_product(const int8_t* dg, const uint64_t* bits, int lines, int words, int t0,
                                              int t1, F&& f) {
  constexpr int T = 2, CH = 4;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int chunks = (words + 4 * CH - 1) / (4 * CH);
  for (int tile = t0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); tile < t1; tile += T * NWAVE) {
    uint32_t off[T];  // of word q of the lane's lines (a head's words take at most 2 MB)
#pragma unroll
    for (int k = 0; k < T; ++k) off[k] = (uint32_t)(q * lines + min(16 * (tile + NWAVE * k) + r, lines - 1));
    auto load = [&](int c, uint64_t (&w)[CH][T]) {
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int g = CH * c + u;
        const uint64_t* row = bits + (int64_t)4 * g * lines;  // uniform
#pragma unroll
        for (int k = 0; k < T; ++k) w[u][k] = q < words - 4 * g ? row[off[k]] : 0ull;
      }
    };
    v4i acc[T];
    int kept[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
      acc[k] = v4i{0, 0, 0, 0};
      kept[k] = 0;
    }
    uint64_t cur[CH][T], nxt[CH][T];
    load(0, cur);
    for (int c = 0; c < chunks; ++c) {
      if (c + 1 < chunks) load(c + 1, nxt);
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (4 * (CH * c + u) < words) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const v4i av = digit_operand(dg, digit_stride(MAXB), CH * c + u, j);
#pragma unroll
            for (int k = 0; k < T; ++k)
              acc[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, mask_bytes(cur[u][k], j), acc[k], 0, 0, 0);
          }
          if (COUNT)
#pragma unroll
            for (int k = 0; k < T; ++k) kept[k] += __popcll(cur[u][k]);
        }
#pragma unroll
      for (int u = 0; u < CH; ++u)
#pragma unroll
        for (int k = 0; k < T; ++k) cur[u][k] = nxt[u][k];
    }
    if (COUNT)
#pragma unroll
      for (int k = 0; k < T; ++k) {  // the four lanes of a line hold a quarter of its words each
        kept[k] += (int)lane_xor32<16>((uint32_t)kept[k]);
        kept[k] += (int)lane_xor32<32>((uint32_t)kept[k]);
      }
    if (lane < 32)
#pragma unroll
      for (int k = 0; k < T; ++k)
        if (tile + NWAVE * k < t1) f(16 * (tile + NWAVE * k) + r, q, combine_digits(acc[k]), kept[k]);
  }
}

// Statistics of columns [kStatCols c, + kStatCols) of a head, and a share of its straddling row pairs.
__global__ __launch_bounds__(kStatCols) void perm_stats_kernel(WaPermLaunch a, int runs) {
  __shared__ int64_t red[kStatCols / 64][5];
  const int h = blockIdx.x / runs, c = blockIdx.x % runs;
  const int tid = threadIdx.x, lane = tid & 63;
  const Head H = head_of(a, h);
  const int j = kStatCols * c + tid;
  int64_t v[5] = {0, 0, 0, 0, 0};
  if (j < a.n) {
    constexpr int WB = 16;  // words loaded together, so that their latencies overlap
    int cnt = 0;
    for (int v0 = 0; v0 < H.mw; v0 += WB) {
      uint64_t wd[WB];
#pragma unroll
      for (int u = 0; u < WB; ++u) wd[u] = v0 + u < H.mw ? H.colbits[(int64_t)(v0 + u) * a.n + j] : 0ull;
#pragma unroll
      for (int u = 0; u < WB; ++u) cnt += __popcll(wd[u]);
    }
    a.cc[(int64_t)h * a.n + j] = cnt;
    if (a.col_cnt) a.col_cnt[(int64_t)h * a.n + j] = cnt;
    v[0] = cnt;
    v[1] = cnt > 0;
    v[2] = (int64_t)cnt * cnt;
  }
  straddling_overlap(H, kStatCols * c + tid, kStatCols * runs, v[3], v[4]);
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    v[k] = wave_sum(v[k]);
    if (lane == 0) red[tid >> 6][k] = v[k];
  }
  __syncthreads();
  if (tid < 5) {
    int64_t s = 0;
    for (int w = 0; w < kStatCols / 64; ++w) s += red[w][tid];
    (&a.stats[(int64_t)h * runs + c].nnz)[tid] = s;
  }
}

// A head's statistics: the sums of its runs' and of its row groups' overlaps. Every lane of the wavefront.
__device__ PermStats head_stats(const WaPermLaunch& a, int h, int runs) {
  const int lane = threadIdx.x & 63, mw = (a.m + 63) / 64;
  static_assert(MAXB / kStatCols <= 64 && MAXB / 64 <= 64, "one lane a run and a row group");
  PermStats s = {};
  if (lane < runs) s = a.stats[(int64_t)h * runs + lane];
  if (lane < mw) {
    const int2 g = a.adj[(int64_t)h * mw + lane];
    s.adj_and += g.x;
    s.adj_or += g.y;
  }
  s.nnz = wave_sum(s.nnz);
  s.distinct = wave_sum(s.distinct);
  s.sum_c2 = wave_sum(s.sum_c2);
  s.adj_and = wave_sum(s.adj_and);
  s.adj_or = wave_sum(s.adj_or);
  return s;
}

__global__ __launch_bounds__(64) void perm_head_stats_kernel(WaPermLaunch a, int runs) {
  const PermStats s = head_stats(a, blockIdx.x, runs);
  const int64_t v[6] = {s.nnz, s.distinct, s.adj_and, s.adj_or, s.sum_c2, 0};
  if (threadIdx.x == 0)
    for (int k = 0; k < 6; ++k) a.head_stats[(int64_t)blockIdx.x * 6 + k] = v[k];
}

// FIRST: the seeded block instead of Z, and the head's statistics on the way (the column counts are popcounts of
// the words that the product reads), which the first scatter decides on.
template <bool FIRST>
__global__ __launch_bounds__(SliceCfg::NT) void mfma_gather_kernel(WaPermLaunch a, int last) {
  __shared__ SliceLds L;
  const int h = blockIdx.x / a.slices, g = blockIdx.x % a.slices;
  const int tid = threadIdx.x;
  const int m = a.m, n = a.n;
  PermState* S = a.state + h;
  if (!FIRST && !S->active) return;
  const Head H = head_of(a, h);
  const int tiles = (n + 15) / 16, per = (tiles + a.slices - 1) / a.slices;
  const int t0 = g * per, t1 = min(g * per + per, tiles);
  int64_t zr[PER][2];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = slice_entry(k);
    zr[k][0] = zr[k][1] = 0;
    if (i < m) {
      if (FIRST) {
        start_row(a, h, i, zr[k][0], zr[k][1]);
      } else {
        const int64_t* z = a.z + ((int64_t)h * m + i) * 2;
        zr[k][0] = z[0];
        zr[k][1] = z[1];
      }
    }
  }
  // ---- Cholesky-QR: X = Z R^-1 ----
  uint64_t any = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) any |= uabs64(zr[k][0]) | uabs64(zr[k][1]);
  int turn = 0;
  const int bl = wg_bitlen<SliceCfg>(L.red, turn, any);
  const int s = bl > 24 ? bl - 24 : 0;
  int64_t gr[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t z0 = zr[k][0] >> s, z1 = zr[k][1] >> s;
    gr[0] += z0 * z0;
    gr[1] += z0 * z1;
    gr[2] += z1 * z1;
  }
  wg_sum<SliceCfg, 3>(L.red, turn, gr);
  const bool degen = gr[0] == 0;  // the same for every workgroup of the head
  if (g == 0 && tid == 0 && (FIRST || degen)) {
    S->active = degen ? 0 : 1;
    S->degen = degen ? 1 : 0;
  }
  if (!FIRST && degen) return;
  int32_t x0[PER], x1[PER];
  int64_t sx[2] = {0, 0};
#pragma unroll
  for (int k = 0; k < PER; ++k) x0[k] = x1[k] = 0;
  if (!degen) {
    const Chol c = chol2(gr);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      WA_PHASE_FENCE();  // (one row's divisions at a time: interleaved, their temporaries spill)
      if (slice_entry(k) < m) orth_row(c, zr[k][0] >> s, zr[k][1] >> s, x0[k], x1[k]);
      sx[0] += x0[k];
      sx[1] += x1[k];
    }
  }
  put_digits4(L.dg, 0, x0);
  put_digits4(L.dg, 4, x1);
  if (last && g == 0) {  // the finishing kernel reads the X of the last product
    int2* xg = reinterpret_cast<int2*>(a.xg) + (int64_t)h * m;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (slice_entry(k) < m) xg[slice_entry(k)] = make_int2(x0[k], x1[k]);
  }
  wg_sum<SliceCfg, 2>(L.red, turn, sx);  // its barrier also publishes the digits
  // ---- Ym of the slice ----
  int32_t* cc = a.cc + (int64_t)h * n;
  int64_t* ym = a.ym + (int64_t)h * n * 2;
  int64_t st[5] = {0, 0, 0, 0, 0};
  slice_product<FIRST>(L.dg, H.colbits, n, H.mw, t0, t1, [&](int j, int k, int64_t ya, int kept) {
    if (j >= n) return;
    const int c = FIRST ? kept : cc[j];
    ym[2 * j + k] = (int64_t)m * ya - (int64_t)c * (k == 0 ? sx[0] : sx[1]);
    if (FIRST && k == 0) {
      cc[j] = c;
      st[0] += c;
      st[1] += c > 0;
      st[2] += (int64_t)c * c;
    }
  });
  if (FIRST) {
    straddling_overlap(H, SliceCfg::NT * g + tid, SliceCfg::NT * a.slices, st[3], st[4]);
    wg_sum<SliceCfg, 5>(L.red, turn, st);
    if (tid == 0) a.stats[(int64_t)h * a.slices + g] = {st[0], st[1], st[2], st[3], st[4], 0};
  }
}

template <bool FIRST>
__global__ __launch_bounds__(SliceCfg::NT) void mfma_scatter_kernel(WaPermLaunch a) {
  __shared__ SliceLds L;
  const int h = blockIdx.x / a.slices, g = blockIdx.x % a.slices;
  PermState* S = a.state + h;
  if (FIRST) {
    const PermStats st = head_stats(a, h, a.slices);
    const int flags = tier1_flags(a, st.nnz, st.distinct, st.adj_and, st.adj_or);
    const bool done = a.skip_mode == SKIP_AUTO && flags != 0;
    if (g == 0 && threadIdx.x == 0) {
      S->done = done ? 1 : 0;
      S->flags = flags;
      S->nnz = st.nnz;
      S->sum_c2 = st.sum_c2;
      S->adj_and = st.adj_and;
      S->adj_or = st.adj_or;
      if (done) S->active = 0;
    }
    if (done) return;
  }
  if (!S->active) return;
  const int m = a.m, n = a.n;
  const Head H = head_of(a, h);
  const int tiles = (m + 15) / 16, per = (tiles + a.slices - 1) / a.slices;
  const int t0 = g * per, t1 = min(g * per + per, tiles);
  const int32_t* cc = a.cc + (int64_t)h * n;
  const int64_t* ym = a.ym + (int64_t)h * n * 2;
  int64_t y[PER][2];
  int32_t c[PER];
  uint64_t any = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int j = slice_entry(k);
    y[k][0] = j < n ? ym[2 * j] : 0;
    y[k][1] = j < n ? ym[2 * j + 1] : 0;
    c[k] = j < n ? cc[j] : 0;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) any |= uabs64(y[k][0]) | uabs64(y[k][1]);
  int turn = 0;
  const int bl = wg_bitlen<SliceCfg>(L.red, turn, any);
  if (g == 0 && threadIdx.x == 0) S->bly = bl;
  const int sy = bl > 30 ? bl - 30 : 0;
  int32_t y0[PER], y1[PER];
  int64_t py[2] = {0, 0};  // c^T Ys
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    y0[k] = (int32_t)(y[k][0] >> sy);
    y1[k] = (int32_t)(y[k][1] >> sy);
    py[0] += (int64_t)c[k] * y0[k];
    py[1] += (int64_t)c[k] * y1[k];
  }
  put_digits4(L.dg, 0, y0);
  put_digits4(L.dg, 4, y1);
  wg_sum<SliceCfg, 2>(L.red, turn, py);  // its barrier also publishes the digits
  int64_t* z = a.z + (int64_t)h * m * 2;
  slice_product<false>(L.dg, H.rowbits, m, H.nw, t0, t1, [&](int i, int k, int64_t za, int) {
    if (i < m) z[2 * i + k] = (int64_t)m * za - (k == 0 ? py[0] : py[1]);
  });
}

// The state of every head when no head is reordered (skip mode "always").
__global__ __launch_bounds__(64) void perm_skip_state_kernel(WaPermLaunch a, int runs) {
  const int h = blockIdx.x;
  const PermStats st = head_stats(a, h, runs);
  if (threadIdx.x == 0) {
    a.state[h].active = 0;
    a.state[h].done = 1;
    a.state[h].flags = tier1_flags(a, st.nnz, st.distinct, st.adj_and, st.adj_or);
  }
}

// Arithmetic self-check: the fp64 operations the permutation relies on, evaluated on the GPU.
__global__ void fp64_probe_kernel(const double* a, const double* b, const int64_t* c, double* out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = a[i], y = b[i];
  out[6 * i + 0] = __builtin_sqrt(__builtin_fabs(x));
  out[6 * i + 1] = x / y;
  out[6 * i + 2] = (double)c[i];
  out[6 * i + 3] = __builtin_rint(x * 1073741824.0);
  out[6 * i + 4] = x * y - y * 3.0;
  out[6 * i + 5] = __builtin_ldexp(x, (int)(c[i] & 31) - 16);
}

}  // namespace

template <int NT, int T>
static hipError_t launch_fused(const WaPermLaunch& a, hipStream_t stream) {
  using C = Cfg<NT, NT>;
  constexpr size_t smem = ((sizeof(Shared<C>) + 15) & ~(size_t)15) + sizeof(MfmaLds<C>);
  static_assert(smem <= 160 * 1024, "the one-workgroup form fits one workgroup's LDS");
  const hipError_t e =
      hipFuncSetAttribute((const void*)perm_mfma_kernel<NT, T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((perm_mfma_kernel<NT, T>), dim3(a.bh), dim3(NT), smem, stream, a);
  return hipGetLastError();
}

// Launch sequence on one stream: heads of at most kMfmaMax rows and columns by the one-workgroup kernel;
// larger ones by iters + 1 x (gather, scatter) and the finishing kernel. The statistics-only form and skip
// mode "always" run the statistics kernel instead of the products.
hipError_t wa_launch_perm(const WaPermLaunch& launch, hipStream_t stream) {
  WaPermLaunch a = launch;
  if (a.bh <= 0) return hipSuccess;
  if (a.m > MAXB || a.n > MAXB) return hipErrorInvalidValue;
  const int lines = a.m > a.n ? a.m : a.n;
  if (!a.stats_only && lines <= kMfmaMax) {
    // (512 threads for heads of 256 blocks: 61 us a call of 12 heads against 52)
    if (lines <= 64) return launch_fused<256, 1>(a, stream);
    if (lines <= 128) return launch_fused<256, 2>(a, stream);
    if (lines <= 256) return launch_fused<256, 4>(a, stream);
    if (lines <= 512) return launch_fused<512, 4>(a, stream);
    return launch_fused<1024, 4>(a, stream);
  }
  hipError_t e;
  if (a.stats_only || a.skip_mode == SKIP_ALWAYS) {
    const int runs = wa_perm_stat_runs(a.n);
    hipLaunchKernelGGL(perm_stats_kernel, dim3((unsigned)((int64_t)a.bh * runs)), dim3(kStatCols), 0, stream, a, runs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.stats_only) {
      hipLaunchKernelGGL(perm_head_stats_kernel, dim3(a.bh), dim3(64), 0, stream, a, runs);
      return hipGetLastError();
    }
    hipLaunchKernelGGL(perm_skip_state_kernel, dim3(a.bh), dim3(64), 0, stream, a, runs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else {
    // at most one workgroup a compute unit, at least one tile a wavefront (so at most one slice a statistics run). From
    // more than half as many heads as compute units on that is one slice: 130 heads of 1,100 blocks take 408 us a
    // call, 128 heads 334 (683 and 680 with a workgroup per 128 lines)
    const int most = ((lines + 15) / 16 + NWAVE - 1) / NWAVE;
    a.slices = std::max(1, std::min(most, a.cus / a.bh));
    const dim3 grid((unsigned)((int64_t)a.bh * a.slices)), block(SliceCfg::NT);
    for (int it = 0; it <= a.iters; ++it) {
      const int last = it == a.iters;
      if (it == 0) {
        hipLaunchKernelGGL(mfma_gather_kernel<true>, grid, block, 0, stream, a, last);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(mfma_scatter_kernel<true>, grid, block, 0, stream, a);
      } else {
        hipLaunchKernelGGL(mfma_gather_kernel<false>, grid, block, 0, stream, a, last);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(mfma_scatter_kernel<false>, grid, block, 0, stream, a);
      }
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  hipLaunchKernelGGL(perm_finish_kernel, dim3(a.bh), dim3(FinishCfg::NT), 0, stream, a);
  return hipGetLastError();
}

hipError_t wa_launch_fp64_probe(const double* a, const double* b, const int64_t* c, double* out, int n,
                                hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fp64_probe_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, a, b, c, out, n);
  return hipGetLastError();
}
