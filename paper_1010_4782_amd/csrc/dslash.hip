// Host side of the even-odd Dslash (dslash_kernel.h): block map, valid launch shapes and dispatch.  The kernels
// are instantiated in dslash_f64.hip, dslash_f64_c12.hip and their FP32 and FP16 counterparts.
#include <algorithm>

#include "dslash_shape.h"

namespace stag {

Batch make_batch(const BatchHost& bh, int wg, int r) {
  Batch B{};
  B.probs = bh.d_probs;
  B.scal = bh.d_scal;
  B.partial = bh.d_partial;
  B.pstride = bh.pstride;
  B.nprob = (int)bh.probs.size();
  B.block_start[0] = 0;
  for (int p = 0; p < B.nprob; ++p) {
    B.tiles[p] = ceil_div(bh.probs[p].half, wg);
    B.groups[p] = ceil_div(bh.probs[p].nrhs, r);
    B.block_start[p + 1] = B.block_start[p] + B.tiles[p] * B.groups[p];
  }
  return B;
}

// The LDS window holds wg + 6 Xh sites (of the widest lattice of the batch) per RHS of a lane.
size_t dslash_lds_bytes(const BatchHost& bh, int prec, const DslashShape& sh) {
  if (!sh.lds) return 0;
  int xh = 0;
  for (const auto& p : bh.probs) xh = std::max(xh, p.xh);
  return (size_t)sh.r * (sh.wg + 2 * window_margin(xh)) * spinor_bytes(prec);
}

bool dslash_shape_valid(const BatchHost& bh, int prec, const DslashShape& sh) {
  if (sh.order == 2) return prec == P16 && sh.wg == 64 && sh.lds == 0 && dslash_t_ok(bh, sh.r, sh.chunks);
  if (sh.wg != 64 && sh.wg != 128 && sh.wg != 256) return false;
  if (sh.r != 1 && sh.r != 2 && sh.r != 4 && sh.r != 8) return false;
  if (sh.order != 0 && sh.order != 1) return false;
  if (sh.order == 0 && sh.chunks != 1) return false;
  if (sh.order)
    for (const auto& p : bh.probs)
      if (!xcd_order_ok(p.ny, p.nz, p.xh, sh.wg, kZBlocks * sh.chunks)) return false;
  return dslash_lds_bytes(bh, prec, sh) <= kMaxDslashLds;
}

hipError_t launch_dslash(const BatchHost& bh, int prec, int epi, int out_par, int in_id, int out_id, int x_id,
                         int b_id, int gate, const DslashShape& sh, hipStream_t st) {
  if (!dslash_shape_valid(bh, prec, sh)) return hipErrorInvalidValue;
  if (sh.order == 2 && bh.inl) return hipErrorInvalidValue;  // the time-streaming kernel reads the device table
  if (sh.order == 2) return launch_dslash_t(bh, epi, out_par, in_id, out_id, x_id, gate, sh.r, sh.chunks, st);
  DslashArgs A{};
  A.B = make_batch(bh, sh.wg, sh.r);
  const bool sweep = sh.order == 0 && sh.sweep;
  if (sweep)  // positions per XCD
    for (int p = 0; p < A.B.nprob; ++p)
      A.B.block_start[p + 1] = A.B.block_start[p] + sweep_tiles(bh.probs[p].half / bh.probs[p].lt, sh.wg) * bh.probs[p].lt * A.B.groups[p];
  const int nblk = (sweep ? 8 : 1) * A.B.block_start[A.B.nprob];
  if (nblk == 0) return hipSuccess;
  if (bh.inl) {
    A.inl = 1;
    A.one = *bh.inl;
    if (bh.inl_mass)
      for (int r = 0; r < bh.inl->nrhs; ++r) A.mass4[r] = 4.0 * bh.inl_mass[r] * bh.inl_mass[r];
  }
  // Where right-hand sides are spread over several groups of workgroups, the groups of a tile run next to each
  // other on one XCD and read the same links: with ordinary loads all but the first find them in L2.
  long alone = 0, shared = 0;
  for (int p = 0; p < A.B.nprob; ++p) (A.B.groups[p] > 1 ? shared : alone) += bh.probs[p].half;
  const bool nt = alone >= shared, c12 = bh.long12;
  const size_t lds = dslash_lds_bytes(bh, prec, sh);
#define STAG_DSLASH(P, C) dslash_pc<P, C>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh, nt, lds, st)
  switch (prec) {
    case P64: return c12 ? STAG_DSLASH(P64, true) : STAG_DSLASH(P64, false);
    case P32: return c12 ? STAG_DSLASH(P32, true) : STAG_DSLASH(P32, false);
    case P16: return c12 ? STAG_DSLASH(P16, true) : STAG_DSLASH(P16, false);
    default: return hipErrorInvalidValue;
  }
#undef STAG_DSLASH
}

}  // namespace stag
