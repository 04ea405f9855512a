// Even-odd staggered Dslash for gfx950 (Eq. (5) with folded phases plus the
// three-hop Naik term), one output site per lane and R right-hand sides per
// lane so that every link load serves R colour vectors.
//
//   out_p(n) = sum_{k<16} L_k(n) in_{1-p}(n + delta_k),  delta_k in {+-mu, +-3mu}
//
// L_k are the packed, phase-, sign- and c_N-folded matrices (pack.hip).  The
// link stream is the compulsory traffic (16 x 144 B per site in FP64), read
// with non-temporal loads where one workgroup serves all right-hand sides of
// its sites and with ordinary ones where several read the same links;
// neighbour colour vectors come through L1/L2, which the XCD-aware block order
// keeps local.  With 8 right-hand sides the
// loads of a site's 16 neighbours x R vectors keep the CU's vector-memory
// address and data units nearly always busy, mostly waiting on lines from
// beyond L2: the loads each CU keeps in flight, more than HBM, set the pace.  The output (and the epilogue's
// one read of x or b per site) also goes non-temporal, so that it does not take
// L2 lines from the neighbours: 9% off the FP16 launch inside the CG solve.
#pragma once

#include <cstddef>

#include "device.h"
#include "dslash_shape.h"

namespace stag {

// Issue the loads of link k of this lane's site and of the R colour vectors it multiplies (only for the
// active RHS; `on` is uniform over the workgroup).
template <int P, bool C12, int R, bool NT>
__device__ __forceinline__ void dslash_issue_r(int k, const Site& s, const Geo& g, const char* lbase, long blk,
                                               int lane, const char* in, long rstride_in, const bool on[R],
                                               RawLink<P>& l, RawSpinor<P> v[R]) {
  const int mu = k >> 2, j = k & 3;
  const int nb = neighbour(s, g, mu, j < 2 ? g.h1[mu] : g.h3[mu], (j & 1) == 0);
  const char* slot = lbase + link_slot_offset(P, C12, blk, k);
  if (C12 && j >= 2)
    raw_link_load<P, 2, NT>(slot, lane, l);
  else
    raw_link_load<P, 3, NT>(slot, lane, l);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (on[r]) raw_spinor_load<P>(in + r * rstride_in, nb, v[r]);
}

// The i-th matrix an output site accumulates: f16_link_order for FP16, index order otherwise.
template <int P> __device__ __forceinline__ constexpr int link_at(int i) { return P == P16 ? f16_link_order(i) : i; }

// FP16: acc += (link scale x vector scale) (L v) for one colour vector v of a link L in dot2 form.
template <bool C12>
__device__ __forceinline__ void apply_link_h(const LinkH& L, bool long_link, const RawSpinor<P16>& v, float lsc,
                                             Cx<float> acc[3]) {
  const float s = lsc * __uint_as_float(v.w.w);
  if (C12 && long_link)
    matvec_h_acc<2>(L, v.w.x, v.w.y, v.w.z, s, acc);
  else
    matvec_h_acc<3>(L, v.w.x, v.w.y, v.w.z, s, acc);
}
template <bool C12>
__device__ __forceinline__ void prepare_link_h(const RawLink<P16>& lr, bool long_link, float lsc, float row3,
                                               LinkH& L) {
  if (C12 && long_link)
    link_h_prepare<2>(lr, row3 * lsc, L);
  else
    link_h_prepare<3>(lr, 0.f, L);
}

// Prefetch distance (links) of the single right-hand-side kernel, per storage precision, from a
// sweep of 0-16 on the 28^3x96 lattice: the compiler's own schedule keeps 2-4 loads in flight,
// and these distances are 6% (f16), 8% (f32) and 9% (f64) faster.
template <int P> constexpr int dslash_pf() { return P == P16 ? 12 : (P == P32 ? 8 : 6); }
// With several RHS per lane the link loads are pipelined too, over fewer links, since each stage holds
// R colour vectors in flight.
template <int P, int R> constexpr int dslash_pf_r() {
  if (R == 1) return dslash_pf<P>();
  if (P == P16) return R == 2 ? 8 : (R == 4 ? 4 : 2);
  // FP32 and FP64, measured at 48^3x144 x 8 RHS: 4 and 2 links ahead at R = 4 and 8 (FP64: 7.1 and
  // 5.6 ms per launch against 8.1 and 6.4 ms at 2 and 1; FP32: 3.40 and 2.81 ms against 3.46 and 2.91 ms).
  // Every FP64 kernel here holds one wave per SIMD (268 to 419 registers)
  return R == 2 ? 4 : (R == 4 ? 4 : 2);
}

// LDS staging (LDS = true): before the link loop a workgroup copies into LDS the colour vectors of
// the window [c0 - 3 Xh, c0 + wg + 3 Xh) of its first site c0 (for each of its RHS); the x and y
// neighbours of its sites that fall in the window (all but the y neighbours that wrap around the
// lattice) are then read from LDS instead of through L1/L2.  Same arithmetic, same result.
extern __shared__ __align__(16) char dslash_window[];

// Tile order 1 (XCD blocks): the z extent is cut into nzb = 8 c blocks (c = the shape's chunks), c per
// XCD, and the workgroups of an XCD (a contiguous range of positions, xcd_remap) sweep t through one
// block, then the next: the colour vectors of the t +-1, +-3 neighbours of a block's slices are then
// still in that XCD's L2 when they are read again, which the lattice order (t slowest) loses once a slice
// of all RHS outgrows L2.  Thinner blocks keep more of the t window in L2 but read more z neighbours
// (3 planes on each side) from outside the block; the autotuner picks c.  Tiles stay contiguous site
// ranges (a whole number of them per z plane), so every tile is computed exactly as in the lattice
// order; the shape is valid only where that holds (xcd_order_ok).
__device__ __forceinline__ int xcd_block_tile(int pos, const Geo& g, int wg, int nzb) {
  const int tpz = g.L[1] * g.Xh / wg;  // tiles per z plane
  const int zbs = g.L[2] / nzb;
  const int j = pos % tpz;
  int rest = pos / tpz;
  const int zi = rest % zbs;
  rest /= zbs;
  const int t = rest % g.L[3];
  const int zb = rest / g.L[3];
  return (t * g.L[2] + zb * zbs + zi) * tpz + j;
}

// Store the wave's output vectors (rounded in place to the stored value), non-temporal.  FP32 and FP64 vectors
// take three pieces per lane, 24 or 48 bytes apart: a full wave's go through LDS (STAGED) so that each store
// covers whole cache lines.  Written piecewise, the FP64 output of the 8-RHS FP16 operator at 48^3x144 cost 680 us
// for 3 GB instead of 350.
template <int P, bool STAGED>
__device__ __forceinline__ void store_out(char* out, int cb, bool live, int half, Cx<typename RealOf<P>::T> v[3]) {
  if constexpr (P == P16 || !STAGED) {
    if (live) store_spinor<P, true, true>(out, cb, v);
  } else {
    __shared__ __align__(16) d2v stage[kMaxWG / kWave][3 * kWave];
    d2v* w = stage[threadIdx.x / kWave];
    const int wl = threadIdx.x % kWave;
    if (cb - wl + kWave > half) {  // uniform per wave: the ragged last one
      if (live) store_spinor<P, true>(out, cb, v);
      return;
    }
    constexpr int kWords = kWave * spinor_bytes(P) / 16;  // 16-byte words of a wave
    if constexpr (P == P64) {
#pragma unroll
      for (int c = 0; c < 3; ++c) w[3 * wl + c] = d2v{v[c].re, v[c].im};
    } else {
      f2v* f = reinterpret_cast<f2v*>(w);
#pragma unroll
      for (int c = 0; c < 3; ++c) f[3 * wl + c] = f2v{v[c].re, v[c].im};
    }
    __builtin_amdgcn_wave_barrier();
    gptr_w<d2v> o = as_global_w<d2v>(out + (long)(cb - wl) * spinor_bytes(P));
#pragma unroll
    for (int i = 0; i < kWords; i += kWave)
      if (i + wl < kWords) __builtin_nontemporal_store(w[i + wl], o + i + wl);
    __builtin_amdgcn_wave_barrier();
  }
}

// XCD sweep (nzb < 0): XCD x (workgroups go round-robin over the XCDs) takes the tiles that start in the
// positions [x S / 8, (x + 1) S / 8) of every time slice of S sites and walks t through them, for any extents;
// per slice and XCD sweep_tiles(S, wg) positions, of which the last may hold no tile (-1).
__device__ __forceinline__ int xcd_sweep_tile(int pos, const Geo& g, int wg) {
  const int S = g.stride[3], x = blockIdx.x & 7, m = sweep_tiles(S, wg);
  const int t = pos / m, j = pos - t * m;
  const int a = t * S + (int)((long)x * S >> 3), b = t * S + (int)((long)(x + 1) * S >> 3);
  const int tile = (a + wg - 1) / wg + j;
  return tile * (long)wg < b ? tile : -1;
}

// The problem a launch carries in its arguments, read where they lie (constant memory, like the table that
// B.probs points to): copying the struct into registers cost the 8-RHS kernel its third wave per SIMD.
// DslashArgs is the kernel's first argument.
template <typename T> using cptr = const __attribute__((address_space(4))) T*;
__device__ __forceinline__ cptr<ProbDev> kernarg_problem() {
  return (cptr<ProbDev>)((cptr<char>)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(DslashArgs, one));
}
__device__ __forceinline__ Geo load_geo(cptr<ProbDev> pd) {  // field by field: no copy leaves that address space
  Geo g;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    g.L[i] = pd->g.L[i];
    g.stride[i] = pd->g.stride[i];
    g.h1[i] = pd->g.h1[i];
    g.h3[i] = pd->g.h3[i];
  }
  g.antiper = pd->g.antiper;
  g.long12 = pd->g.long12;
  g.cn_inv = pd->g.cn_inv;
  g.Xh = pd->g.Xh;
  g.half = pd->g.half;
  g.t0 = pd->g.t0;
  g.lt_glob = pd->g.lt_glob;
  g.h3g = pd->g.h3g;
  g.t_open = pd->g.t_open;
  g.in_half = pd->g.in_half;
  return g;
}

template <int P, int R, int EPI, bool C12, int PF, bool LDS, bool NT>
__global__ __launch_bounds__(kMaxWG) void k_dslash(DslashArgs A, int out_par, int in_id, int out_id, int x_id,
                                                   int b_id, int gate, int nzb) {
  static_assert(!(LDS && PF > 0), "the staged path uses the plain link loop");
  using T = typename RealOf<P>::T;
  __shared__ double lds[R * 4];
  const Batch& B = A.B;
  // Asked for one by one where a branch first needs them, the launch's parameters are a chain of round trips to
  // memory in front of every wave (28^3x96 x 2, FP16: a launch that finds every right-hand side stopped takes 6.9
  // us).  FP32 and FP16 with one or two per lane ask for them at once: an FP16 iteration of 8^4 takes 32 us instead
  // of 37, of 16^3x32 x 4 77 instead of 83, of 28^3x96 303 instead of 308.  Longer lanes and FP64 are better off
  // with the chain on large lattices (FP16, three lattices at 4 per lane: 290 us a launch and 294; FP64, 28^3x96 x 2
  // with 18-real links: 1155 us an iteration and 1190).
  constexpr bool kAtOnce = P != P64 && R <= 2;
  int nblk = 0, wg0 = 0, inl0 = 0, nprob = 0, groups0 = 0;
  if constexpr (kAtOnce) {
    nblk = gridDim.x;
    wg0 = blockDim.x;
    inl0 = A.inl;
    nprob = B.nprob;
    groups0 = B.groups[0];
    asm volatile("" : "+s"(nblk), "+s"(wg0), "+s"(nzb), "+s"(inl0), "+s"(nprob), "+s"(groups0));
  }
  auto wg = [&] { return kAtOnce ? (unsigned)wg0 : blockDim.x; };
  const bool sweep = nzb < 0;
  const int bid = sweep ? (int)(blockIdx.x >> 3) : xcd_remap(blockIdx.x, kAtOnce ? nblk : (int)gridDim.x);
  const bool inl = (kAtOnce ? inl0 : A.inl) != 0;
  const bool first = kAtOnce && nprob == 1;
  const int p = inl || first ? 0 : find_problem(B, bid);
  const cptr<ProbDev> pd = inl ? kernarg_problem() : (cptr<ProbDev>)(B.probs + p);
  const Geo g = load_geo(pd);
  auto vec = [&](int id) { return reinterpret_cast<char*>(pd->vec[id]); };
  const int local = first ? bid : bid - B.block_start[p];
  const int groups = first ? groups0 : B.groups[p];
  const int pos = local / groups;
  const int r0 = (local - pos * groups) * R;
  int nrhs = pd->nrhs, slot0 = pd->slot0;
  if constexpr (kAtOnce) asm volatile("" : "+s"(nrhs), "+s"(slot0));
  const int tile = sweep ? xcd_sweep_tile(pos, g, wg()) : (nzb ? xcd_block_tile(pos, g, wg(), nzb) : pos);
  if (tile < 0) return;  // uniform: an unused position of the sweep

  bool on[R];
  bool any = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    on[r] = (r0 + r < nrhs) && slot_on(B.scal, slot0 + r0 + r, gate);
    any |= on[r];
  }
  if (!any) return;  // uniform over the workgroup

  const int cb_raw = tile * wg() + threadIdx.x;
  const bool live = cb_raw < g.half;
  const int cb = live ? cb_raw : g.half - 1;  // dead lanes read a valid site and store nothing
  const Site s = site_of(cb, out_par, g);
  const long gcb = cb + (long)g.t0 * g.stride[3];  // the site's index in the whole lattice: packed links
  const long blk = gcb >> 6;
  const int lane = (int)(gcb & 63);

  const long rstride = (long)g.half * spinor_bytes(P);
  const long rstride_in = (long)g.in_half * spinor_bytes(P);
  const char* in = vec(in_id) + (long)r0 * rstride_in;
  const char* lbase = reinterpret_cast<const char*>(pd->links[P][out_par]);
  const T cn_inv = (T)g.cn_inv;
  // FP16: the matrices stay in code units; each link's scale multiplies the colour vector instead
  float sc_fat = 1.f, sc_long = 1.f;
  if (P == P16) {
    gptr<float> ls = as_global<float>(pd->lscale[out_par]) + blk * 2 * kWave + lane;
    sc_fat = ls[0];
    sc_long = ls[kWave];
  }

  Cx<T> acc[R][3];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[r][c] = Cx<T>{T(0), T(0)};

  // LDS window: sites [w0, w0 + wn) of every active RHS, 8-byte units, loaded by the whole workgroup
  const int w0 = tile * (int)wg() - window_margin(g.Xh);
  const int wn = (int)wg() + 2 * window_margin(g.Xh);
  constexpr int SB = spinor_bytes(P);
  if constexpr (LDS) {
    const int units = wn * SB / 8;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!on[r]) continue;  // uniform over the workgroup
      // window sites outside [0, in_half) are never read back: every neighbour index is in range
      const char* src = in + r * rstride_in;
      char* dst = dslash_window + r * wn * SB;
      for (int u = threadIdx.x; u < units; u += wg()) {
        const int site = w0 + (u * 8) / SB;
        if (site >= 0 && site < g.in_half)
          *reinterpret_cast<u2v*>(dst + u * 8) = *as_global<u2v>(src + (long)w0 * SB + (long)u * 8);
      }
    }
    __syncthreads();
  }

  // The FP16 launches take the 16 matrices in f16_link_order and multiply binary16 codes with dot2
  // (apply_link_h); FP32 and FP64 take them in index order with decoded matrices.  Either way every
  // launch shape of a precision does the same arithmetic in the same order.
  if constexpr (PF > 0) {
    // Software pipeline over the 16 links: the loads of link i + PF are issued while link i is
    // multiplied.  An empty volatile asm that takes the accumulators closes each stage: the
    // products of link i must be done before it and the loads issued after it cannot move above
    // it, so the compiler can neither hoist all loads to the top nor sink them to their uses.
    RawLink<P> lb[PF];
    RawSpinor<P> vb[PF][R];
#pragma unroll
    for (int i = 0; i < PF; ++i)
      dslash_issue_r<P, C12, R, NT>(link_at<P>(i), s, g, lbase, blk, lane, in, rstride_in, on, lb[i], vb[i]);
#pragma unroll
    for (int i = 0; i < kLinks; ++i) {
      const int k = link_at<P>(i);
      const int mu = k >> 2, j = k & 3;
      const float lsc = j < 2 ? sc_fat : sc_long;
      if constexpr (P == P16) {
        LinkH L;
        prepare_link_h<C12>(lb[i % PF], j >= 2, lsc, (float)long_sign(s, g, mu, j == 2) * cn_inv, L);
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (on[r]) apply_link_h<C12>(L, j >= 2, vb[i % PF][r], lsc, acc[r]);
      } else {
        Cx<T> u[9];
        if (C12 && j >= 2) {
          raw_link_decode<P, 2>(lb[i % PF], 1.f, u);
          rebuild_row3(u, (T)long_sign(s, g, mu, j == 2) * cn_inv);
        } else {
          raw_link_decode<P, 3>(lb[i % PF], 1.f, u);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (!on[r]) continue;
          Cx<T> v[3];
          raw_spinor_decode<P>(vb[i % PF][r], 1.f, v);
          matvec_acc(u, v, acc[r]);
        }
      }
      if (i + PF < kLinks)
        dslash_issue_r<P, C12, R, NT>(link_at<P>(i + PF), s, g, lbase, blk, lane, in, rstride_in, on, lb[i % PF],
                                  vb[i % PF]);
#pragma unroll
      for (int r = 0; r < R; ++r)
        asm volatile("" : "+v"(acc[r][0].re), "+v"(acc[r][0].im), "+v"(acc[r][1].re), "+v"(acc[r][1].im),
                     "+v"(acc[r][2].re), "+v"(acc[r][2].im));
    }
  } else {
#pragma unroll
    for (int i = 0; i < kLinks; ++i) {
      const int k = link_at<P>(i);
      const int mu = k >> 2, j = k & 3;
      const int hop = j < 2 ? g.h1[mu] : g.h3[mu];
      const int nb = neighbour(s, g, mu, hop, (j & 1) == 0);
      const float lsc = j < 2 ? sc_fat : sc_long;
      const bool from_lds = LDS && mu < 2 && (unsigned)(nb - w0) < (unsigned)wn;
      const char* slot = lbase + link_slot_offset(P, C12, blk, k);
      RawLink<P> lr;
      if (C12 && j >= 2)
        raw_link_load<P, 2, NT>(slot, lane, lr);
      else
        raw_link_load<P, 3, NT>(slot, lane, lr);
      RawSpinor<P> vr[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!on[r]) continue;
        if (from_lds)
          raw_spinor_lds<P>(dslash_window + r * wn * SB, nb - w0, vr[r]);
        else
          raw_spinor_load<P>(in + r * rstride_in, nb, vr[r]);
      }
      if constexpr (P == P16) {
        LinkH L;
        prepare_link_h<C12>(lr, j >= 2, lsc, (float)long_sign(s, g, mu, j == 2) * cn_inv, L);
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (on[r]) apply_link_h<C12>(L, j >= 2, vr[r], lsc, acc[r]);
      } else {
        Cx<T> u[9];
        if (C12 && j >= 2) {
          raw_link_decode<P, 2>(lr, 1.f, u);
          rebuild_row3(u, (T)long_sign(s, g, mu, j == 2) * cn_inv);
        } else {
          raw_link_decode<P, 3>(lr, 1.f, u);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (!on[r]) continue;
          Cx<T> v[3];
          raw_spinor_decode<P>(vr[r], 1.f, v);
          matvec_acc(u, v, acc[r]);
        }
      }
    }
  }

  if constexpr (EPI == EPI_WIDE) {
    // the stored (rounded) value, widened to FP64
    char* out = vec(out_id) + (long)r0 * g.half * spinor_bytes(P64);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!on[r]) continue;  // uniform
      if constexpr (P == P16) (void)round_spinor_f16<true>(acc[r]);
      Cx<double> w[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) w[c] = Cx<double>{(double)acc[r][c].re, (double)acc[r][c].im};
      store_out<P64, !LDS>(out + (long)r * g.half * spinor_bytes(P64), cb_raw, live, g.half, w);
    }
    return;
  }
  if constexpr (EPI == EPI_NORM) {
    // |out|^2 of the site instead of the colour vector: one FP64 number per right-hand side
    char* out = vec(out_id) + (long)r0 * g.half * 8;
    if (live)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (on[r]) {
          double n2 = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) n2 += (double)acc[r][c].re * (double)acc[r][c].re + (double)acc[r][c].im * (double)acc[r][c].im;
          __builtin_nontemporal_store(n2, as_global_w<double>(out + (long)r * g.half * 8) + cb);
        }
    return;
  }

  // One right-hand side in FP64 with 18-real three-hop links stores piecewise: 22x28x26x50 162 us against 168
  // staged (28^3x96 425 and 433).  With 12-real links (137 us staged, 142 piecewise) and in FP32 (101 and 103)
  // staging is faster there too.
  constexpr bool kStaged = !LDS && !(P == P64 && R == 1 && !C12);
  // With 12-real links the launch that ends a CG iteration's operator stores piecewise too from 2^19 sites on
  // (an iteration of 28^3x96 826 us against 835, 26^3x60 416 and 421; below, 24^3x48 270 and 268).
  constexpr int kPiecewiseFrom = 1 << 19;
  constexpr bool kEither = kStaged && P == P64 && R == 1 && (EPI == EPI_XPAY_DOT || EPI == EPI_RESID);
  const bool piecewise = kEither && g.half >= kPiecewiseFrom;  // uniform
  char* out = vec(out_id) + (long)r0 * rstride;
  if (EPI == EPI_PLAIN) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (on[r]) store_out<P, kStaged>(out + r * rstride, cb_raw, live, g.half, acc[r]);
    return;
  }

  const char* xb = vec(x_id) + (long)r0 * rstride;
  double part[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    part[r] = 0.0;
    if (!on[r]) continue;
    const T a = (T)(inl ? A.mass4[r0 + r] : B.scal[slot0 + r0 + r].mass4);
    Cx<T> xv[3], o[3];
    load_spinor<P, true>(xb + r * rstride, cb, xv);
    if (EPI == EPI_RESID) {
      Cx<T> bv[3];
      load_spinor<P, true>(vec(b_id) + (long)(r0 + r) * rstride, cb, bv);
#pragma unroll
      for (int c = 0; c < 3; ++c)
        o[c] = Cx<T>{bv[c].re - a * xv[c].re + acc[r][c].re, bv[c].im - a * xv[c].im + acc[r][c].im};
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) o[c] = Cx<T>{a * xv[c].re - acc[r][c].re, a * xv[c].im - acc[r][c].im};
    }
    if (piecewise)
      store_out<P, false>(out + r * rstride, cb_raw, live, g.half, o);
    else
      store_out<P, kStaged>(out + r * rstride, cb_raw, live, g.half, o);
    if (live) {
      if (EPI == EPI_XPAY_DOT) {
#pragma unroll
        for (int c = 0; c < 3; ++c) part[r] += (double)xv[c].re * (double)o[c].re + (double)xv[c].im * (double)o[c].im;
      } else if (EPI == EPI_RESID) {
#pragma unroll
        for (int c = 0; c < 3; ++c) part[r] += (double)o[c].re * (double)o[c].re + (double)o[c].im * (double)o[c].im;
      }
    }
  }
  if (EPI == EPI_XPAY) return;
  block_sum<R>(part, lds);
  if (threadIdx.x == 0) {
    const int kind = EPI == EPI_XPAY_DOT ? 0 : 1;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (on[r]) B.partial[((long)(slot0 + r0 + r) * kPartialSlots + kind) * B.pstride + tile] = part[r];
  }
}

template <int P, int R, bool C12, bool LDS, bool NT>
hipError_t dslash_r(const DslashArgs& A, int nblk, int epi, int out_par, int in_id, int out_id, int x_id, int b_id,
                    int gate, int wg, int nzb, size_t lds_bytes, hipStream_t st) {
  constexpr int PF = !LDS ? dslash_pf_r<P, R>() : 0;
#define STAG_DSLASH(E)                                                                                              \
  k_dslash<P, R, E, C12, PF, LDS, NT><<<nblk, wg, lds_bytes, st>>>(A, out_par, in_id, out_id, x_id, b_id, gate, nzb); \
  return hipGetLastError()
  if (epi == EPI_PLAIN) { STAG_DSLASH(EPI_PLAIN); }
  if (epi == EPI_XPAY_DOT) { STAG_DSLASH(EPI_XPAY_DOT); }
  if constexpr (P == P64) {
    if (epi == EPI_RESID) { STAG_DSLASH(EPI_RESID); }
    if (epi == EPI_XPAY) { STAG_DSLASH(EPI_XPAY); }
    if (epi == EPI_NORM) { STAG_DSLASH(EPI_NORM); }
  } else {
    if (epi == EPI_WIDE) { STAG_DSLASH(EPI_WIDE); }
  }
#undef STAG_DSLASH
  return hipErrorInvalidValue;
}

template <int P, bool C12, bool LDS, bool NT>
hipError_t dslash_p(const DslashArgs& A, int nblk, int epi, int out_par, int in_id, int out_id, int x_id, int b_id,
                    int gate, const DslashShape& sh, size_t lds_bytes, hipStream_t st) {
  // z blocks of the XCD order, 0: lattice order, -1: XCD sweep
  const int nzb = sh.order == 1 ? kZBlocks * sh.chunks : (sh.sweep ? -1 : 0);
  switch (sh.r) {
    case 1: return dslash_r<P, 1, C12, LDS, NT>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh.wg, nzb, lds_bytes, st);
    case 2: return dslash_r<P, 2, C12, LDS, NT>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh.wg, nzb, lds_bytes, st);
    case 4: return dslash_r<P, 4, C12, LDS, NT>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh.wg, nzb, lds_bytes, st);
    case 8: return dslash_r<P, 8, C12, LDS, NT>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh.wg, nzb, lds_bytes, st);
    default: return hipErrorInvalidValue;
  }
}

// The LDS-staged shapes keep non-temporal link loads.
template <int P, bool C12>
hipError_t dslash_pc(const DslashArgs& A, int nblk, int epi, int out_par, int in_id, int out_id, int x_id, int b_id,
                     int gate, const DslashShape& sh, bool nt, size_t lds_bytes, hipStream_t st) {
#define STAG_DSLASH(L, N) dslash_p<P, C12, L, N>(A, nblk, epi, out_par, in_id, out_id, x_id, b_id, gate, sh, lds_bytes, st)
  return sh.lds ? STAG_DSLASH(true, true) : (nt ? STAG_DSLASH(false, true) : STAG_DSLASH(false, false));
#undef STAG_DSLASH
}

}  // namespace stag
