// Internal launch interface of the permutation kernels (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wavealign.h"

// Per-head state carried between the permutation kernels (workspace, 64 bytes a head).
struct PermState {
  int32_t bly;      // bit length of max |Ym| of the last centred product
  int32_t pad0;
  int32_t active;   // the subspace iteration still runs for this head
  int32_t degen;    // a QR found no direction
  int32_t done;     // a skipped head: the identity order
  int32_t flags;    // skip-rule flags of cases 1-3
  int64_t nnz, sum_c2;
  int64_t adj_and, adj_or;  // adjacent-row overlap of the natural order: sum |M_i & M_i+1|, sum |M_i | M_i+1|
  int64_t pad[1];
};
static_assert(sizeof(PermState) == 64, "PermState is 64 bytes");

// Statistics of one run of kStatCols columns of a head (workspace): the head's are their sums.
struct PermStats {
  int64_t nnz, distinct, sum_c2;
  int64_t adj_and, adj_or;  // of a share of the row pairs that straddle two 64-row groups
  int64_t pad;
};
constexpr int kStatCols = 256;
inline int wa_perm_stat_runs(int n) { return (n + kStatCols - 1) / kStatCols; }

struct WaPermLaunch {
  const uint64_t* rowbits;  // [bh][ceil(n/64)][m] word-major
  const uint64_t* colbits;  // [bh][ceil(m/64)][n] word-major
  const int32_t* row_nnz;   // [bh][m]
  int32_t* cc;              // workspace [bh][n]: column counts
  int32_t* col_cnt;         // [bh][n], nullable (a copy of the column counts for the caller)
  int32_t* xg;              // workspace [bh][m][2]: X of the subspace iteration (2^30 fixed point)
  int64_t* ym;              // workspace [bh][n][2]: m * M~^T X
  int64_t* z;               // workspace [bh][m][2]: m * M~ Ys
  PermState* state;         // workspace [bh]
  const int2* adj;          // workspace [bh][ceil(m/64)]: adjacent-row overlap within each 64-row group
  PermStats* stats;         // workspace [bh][wa_perm_stat_runs(n)]
  int64_t* head_stats;      // [bh][6], nullable
  int32_t* perm;            // [bh][m]
  uint8_t* flags;           // [bh], nullable
  int32_t* embedding;       // [bh][m][2], nullable
  int32_t* stage1;          // [bh][m], nullable
  int32_t* seg_start;       // [bh][n_xcd+1], nullable
  int32_t bh, m, n;
  int32_t cus;     // compute units of the device
  int32_t slices;  // workgroups per head of the centred-product kernels (set by wa_launch_perm)
  int32_t wave, n_xcd, iters, skip_mode, stats_only;
  int32_t block, head_dim;
  uint64_t seed;
  wa_skip_profile prof;
};

hipError_t wa_launch_perm(const WaPermLaunch& a, hipStream_t stream);
hipError_t wa_launch_fp64_probe(const double* a, const double* b, const int64_t* c, double* out, int n,
                                hipStream_t stream);
hipError_t wa_launch_pack(const uint8_t* mask, int bh, int m, int n, uint64_t* rowbits, uint64_t* colbits,
                          int32_t* row_nnz, int2* adj, hipStream_t stream);
hipError_t wa_launch_xcc_probe(int32_t* out, int n_wg, hipStream_t stream);
hipError_t wa_launch_check_perm(const int32_t* perm, int bh, int m, int32_t* bad, int32_t* head_ok,
                                hipStream_t stream);
