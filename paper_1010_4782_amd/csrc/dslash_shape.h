// What the Dslash kernels (dslash_kernel.h) and their host side (dslash.hip) share.
#pragma once

#include "launch.h"

namespace stag {

// Margin of the LDS window of a staged workgroup, in sites on each side.
__host__ __device__ constexpr int window_margin(int xh) { return 3 * xh; }

// The XCD-block tile order cuts z into kZBlocks x chunks blocks (xcd_block_tile).
constexpr int kZBlocks = 8;
__host__ __device__ inline bool xcd_order_ok(int ny, int nz, int xh, int wg, int nzb) {
  return nzb > 0 && nz % nzb == 0 && (ny * xh) % wg == 0;
}

// Positions per time slice (of S sites) and XCD in the XCD sweep (xcd_sweep_tile).
__host__ __device__ inline int sweep_tiles(int S, int wg) { return ceil_div((S + 7) / 8, wg); }

// Kernel arguments of a Dslash launch.  A call outside the solvers (one problem, at most kInlineRhs right-hand
// sides) carries its problem and masses here, with no table in device memory to fill first: inl = 1.
struct DslashArgs {
  Batch B;
  int inl;
  int pad;
  ProbDev one;
  double mass4[kInlineRhs];  // 4 m^2 per right-hand side
};

// One instantiation per storage precision and long-link storage (C12: two rows), each in its own source
// (dslash_f64.hip, dslash_f64_c12.hip, ...).  nt: non-temporal link loads.
template <int P, bool C12>
hipError_t dslash_pc(const DslashArgs& A, int nblk, int epi, int out_par, int in_id, int out_id, int x_id, int b_id,
                     int gate, const DslashShape& sh, bool nt, size_t lds_bytes, hipStream_t st);

}  // namespace stag
