// CG iterations with the scalar steps inside the vector kernels.
//
// On a small lattice an iteration of the general path (Dslash, Dslash + <d, Ad>, finalize, r update,
// finalize, x and d update) is six launches of 3.3-6 us that each wait on a chain of memory round trips; the
// two finalize launches, one workgroup each, take 5.7 us of it apiece.  With at most kFusedTiles partial sums
// per right-hand side, every workgroup that needs alpha or beta adds the partials itself, in k_finalize's
// order, and one of them writes the slot's scalars:
//   k_resid  alpha from the <d, Ad> partials; r -= alpha Ad; |r|^2 partials
//   k_xd     beta from the |r|^2 partials and the stopping test; x += alpha d; d = r + beta d
// Every sum and product is taken in the order and precision of the general kernels: the same bits.  An FP64
// iteration at 8^4 takes 25 us instead of 37, an FP16 one at 16^3x32 44 instead of 54.  Forming
// r + beta d inside the first operator launch too (three launches) was slower from 12^4 on: 33.8 us against
// 29.4, the reads of two vectors at 16 neighbours cost more than a launch.
//
// The scalars are double-buffered: k_xd reads one bank and its writer fills the other, so no workgroup can see
// another's update of what it is still reading.  k_resid writes alpha, <d, Ad> and a state that only ever
// leaves 0 or 1 for 2, none of which its other workgroups act on differently: a state of 1 or 2 stops them
// either way, and a breakdown is in the sum they all form.
#include "device.h"
#include "launch.h"
#include "wide_grid.h"

namespace stag {

namespace {

// The sum of src[0..n), n <= kFusedTiles, as k_finalize forms it: 1024 lanes with one partial each, a butterfly
// per wave of 64, the waves in order.  Valid in every thread; blockDim.x is a multiple of 64.
__device__ __forceinline__ double sum_partials(const double* src, int n, double* lds /* >= 16 */) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, nw = blockDim.x / kWave;
  const int nv = ceil_div(n, kWave);
  for (int w = wave; w < nv; w += nw) {
    double v[1] = {w * kWave + lane < n ? src[w * kWave + lane] : 0.0};
    wave_sum<1>(v);
    if (lane == 0) lds[w] = v[0];
  }
  __syncthreads();
  double s = lds[0];
  for (int w = 1; w < nv; ++w) s += lds[w];
  return s;
}

struct Slot {
  const ProbDev* pd;
  int tile, r, slot;
};
__device__ __forceinline__ Slot slot_of_block(const Batch& B, int bid) {
  Slot m;
  const int p = find_problem(B, bid);
  m.pd = B.probs + p;
  const int local = bid - B.block_start[p], groups = B.groups[p];
  m.tile = local / groups;
  m.r = local - m.tile * groups;
  m.slot = m.pd->slot0 + m.r;
  return m;
}
__device__ __forceinline__ const double* partials(const Batch& B, int slot, int kind) {
  return B.partial + ((long)slot * kPartialSlots + kind) * B.pstride;
}

// Beta and the stopping test of a slot (k_finalize's FIN_BETA); r2() gives |r|^2.  Returns the state after it
// (2 if the slot was not running) and beta; the workgroup of tile 0 writes the slot's scalars to the other bank.
template <typename Sum>
__device__ __forceinline__ int beta_step(const Batch& B, const Slot& m, Scal* next, double* hist, int hist_stride,
                                         Sum&& r2, double& beta) {
  const Scal& pre = B.scal[m.slot];
  const int st = pre.state;
  const double delta0 = pre.delta, thr0 = pre.thr, rel0 = pre.rel_thr;
  const int iter0 = pre.iter, max0 = pre.max_iter;
  double sum = 0.0;
  int now = st, flags = pre.flags;
  beta = 0.0;
  if (st == 0) {  // uniform
    sum = r2();
    if (!isfinite(sum)) {
      now = 2;
      flags |= kFlagNaN;
    } else {
      beta = sum / delta0;
      if (sum <= thr0) now = 1;
      if (sum <= rel0) {
        now = 1;
        flags |= kFlagRelDue;
      }
      if (iter0 + 1 >= max0) {
        now = 1;
        flags |= kFlagMaxIter;
      }
    }
  }
  if (m.tile == 0 && threadIdx.x == 0) {
    // the whole slot, as bytes (a copy through another type need not be ordered with the members' stores), then
    // the members that changed
    __builtin_memcpy(next + m.slot, &pre, sizeof(Scal));
    if (st == 0) {
      Scal& sc = next[m.slot];
      sc.state = now;
      sc.flags = flags;
      if (now != 2) {
        sc.delta_old = delta0;
        sc.delta = sum;
        sc.beta = beta;
        sc.iter = iter0 + 1;
        if (hist && iter0 < pre.hist_len) hist[((long)m.slot * hist_stride + iter0) * 2 + 1] = beta;
      }
    }
  }
  return st == 0 ? now : 2;
}

// alpha (or, for a slot the stopping test ended, state 1 -> 2), r -= alpha Ad, partial |r|^2.  dot_wg: sites
// per <d, Ad> partial.
template <int P>
__global__ __launch_bounds__(kMaxWG) void k_resid(Batch B, int r_id, int dot_wg, double* hist, int hist_stride) {
  using T = typename RealOf<P>::T;
  constexpr bool kNT = P != P64;  // as in k_update_r
  __shared__ double lds[kFusedTiles / kWave];
  const Slot m = slot_of_block(B, blockIdx.x);
  Scal& sc = B.scal[m.slot];
  const int st = sc.state;
  const double delta = sc.delta;
  const bool writer = m.tile == 0 && threadIdx.x == 0;
  if (st != 0) {  // uniform
    if (st == 1 && writer) sc.state = 2;
    return;
  }
  const int half = m.pd->g.half;
  const long off = (long)m.r * half * spinor_bytes(P);
  const int cb_raw = m.tile * kMaxWG + threadIdx.x;
  const bool live = cb_raw < half;
  char* rp = reinterpret_cast<char*>(m.pd->vec[r_id]) + off;
  Cx<T> r[3], ad[3];
  if (live) {
    load_spinor<P, kNT>(rp, cb_raw, r);
    load_spinor<P, kNT>(reinterpret_cast<const char*>(m.pd->vec[V_AD]) + off, cb_raw, ad);
  }
  const double dAd = sum_partials(partials(B, m.slot, 0), ceil_div(half, dot_wg), lds);
  const bool ok = dAd > 0.0 && isfinite(dAd);
  const double alpha = delta / dAd;
  if (writer) {
    sc.dAd = dAd;
    if (ok) {
      sc.alpha = alpha;
      if (hist && sc.iter < sc.hist_len) hist[((long)m.slot * hist_stride + sc.iter) * 2] = alpha;
    } else {
      sc.flags |= kFlagNaN;
      sc.state = 2;
    }
  }
  if (!ok) return;  // uniform
  const T al = (T)alpha;
  double s[1] = {0.0};
  if (live) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c].re = fma(-al, ad[c].re, r[c].re);
      r[c].im = fma(-al, ad[c].im, r[c].im);
    }
    store_spinor<P, kNT>(rp, cb_raw, r);
#pragma unroll
    for (int c = 0; c < 3; ++c) s[0] += (double)r[c].re * r[c].re + (double)r[c].im * r[c].im;
  }
  __syncthreads();  // lds is read above
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) B.partial[((long)m.slot * kPartialSlots + 1) * B.pstride + m.tile] = s[0];
}

// beta and the stopping test, x += alpha d, d = r + beta d.
template <int P, int PX>
__global__ __launch_bounds__(kMaxWG) void k_xd(Batch B, Scal* next, int x_id, int r_id, double* hist,
                                               int hist_stride) {
  using T = typename RealOf<P>::T;
  using TX = typename RealOf<PX>::T;
  constexpr bool kNT = P != P64;  // as in k_update_xd
  __shared__ double lds[kFusedTiles / kWave];
  const Slot m = slot_of_block(B, blockIdx.x);
  const int half = m.pd->g.half;
  const int cb = m.tile * kMaxWG + threadIdx.x;
  const TX alpha = (TX)B.scal[m.slot].alpha;
  double b64;
  const int now = beta_step(
      B, m, next, hist, hist_stride,
      [&] { return sum_partials(partials(B, m.slot, 1), ceil_div(half, kMaxWG), lds); }, b64);
  if (now > 1 || cb >= half) return;
  const T beta = (T)b64;
  char* dp = reinterpret_cast<char*>(m.pd->vec[V_D]) + (long)m.r * half * spinor_bytes(P);
  char* xp = reinterpret_cast<char*>(m.pd->vec[x_id]) + (long)m.r * half * spinor_bytes(PX);
  Cx<T> d[3], r[3];
  Cx<TX> x[3];
  load_spinor<P, kNT>(dp, cb, d);
  load_spinor<P, kNT>(reinterpret_cast<const char*>(m.pd->vec[r_id]) + (long)m.r * half * spinor_bytes(P), cb, r);
  load_spinor<PX, kNT>(xp, cb, x);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    x[c].re = fma(alpha, (TX)d[c].re, x[c].re);
    x[c].im = fma(alpha, (TX)d[c].im, x[c].im);
    d[c].re = fma(beta, d[c].re, r[c].re);
    d[c].im = fma(beta, d[c].im, r[c].im);
  }
  store_spinor<PX, kNT>(xp, cb, x);
  store_spinor<P, kNT>(dp, cb, d);
}

// ---- larger problems ----------------------------------------------------------------------------------
// With more partials the same two kernels run as one 1024-lane workgroup per CU at most: each adds all partials
// of its slot, lane t the partials t, t + 1024, ... as k_finalize does, then walks its share of the slot's
// vectors.  Such a launch reads the partials once per workgroup (24^3x48: 41 KB, 10 MB in all, from L2) while its
// first sites are on their way, where the general path waits for a one-workgroup launch (6.4 us) twice an
// iteration.  An iteration takes, general -> wide: 24^3x48 FP16 111 -> 103 us, FP64 270 -> 262; 20^3x40 x 4
// FP16 122 -> 114; 32^3x64 FP32 451 -> 443; 28^3x96 FP16 270 -> 266.  With 512 workgroups the sums cost more than
// the second workgroup per CU gives: 3.5% on 24^3x48 in FP16, 2.5% on 28^3x96.
constexpr int kWideUnroll = 24;   // partials a lane has in flight

__device__ __forceinline__ double wide_sum(const double* src, int n, double* lds /* >= 16 */) {
  double s[1] = {0.0};
  for (int base = 0; base < n; base += kWideUnroll * kWideWG) {
    double v[kWideUnroll];
#pragma unroll
    for (int j = 0; j < kWideUnroll; ++j) {
      const int i = base + j * kWideWG + threadIdx.x;
      v[j] = i < n ? src[i] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kWideUnroll; ++j) s[0] += v[j];
  }
  wave_sum<1>(s);
  if (threadIdx.x % kWave == 0) lds[threadIdx.x / kWave] = s[0];
  __syncthreads();
  double t = lds[0];
  for (int w = 1; w < kWideWG / kWave; ++w) t += lds[w];
  return t;
}

// Workgroup of a wide launch: B.groups[p] workgroups per slot of problem p; `tile` is this one's number.
__device__ __forceinline__ Slot wide_slot(const Batch& B) {
  Slot m;
  const int p = find_problem(B, blockIdx.x);
  m.pd = B.probs + p;
  const int local = blockIdx.x - B.block_start[p], groups = B.groups[p];
  m.r = local / groups;
  m.tile = local - m.r * groups;
  m.slot = m.pd->slot0 + m.r;
  return m;
}

template <int P>
__global__ __launch_bounds__(kWideWG) void k_resid_wide(Batch B, int r_id, int dot_wg, double* hist,
                                                        int hist_stride) {
  using T = typename RealOf<P>::T;
  constexpr bool kNT = P != P64;  // as in k_update_r
  __shared__ double lds[kWideWG / kWave], tiles[2][kWideWG / kWave];
  const Slot m = wide_slot(B);
  const int p = find_problem(B, blockIdx.x), groups = B.groups[p];
  Scal& sc = B.scal[m.slot];
  const int st = sc.state;
  const double delta = sc.delta;
  const bool writer = m.tile == 0 && threadIdx.x == 0;
  if (st != 0) {  // uniform
    if (st == 1 && writer) sc.state = 2;
    return;
  }
  const int half = m.pd->g.half, ntiles = ceil_div(half, kMaxWG);
  const long off = (long)m.r * half * spinor_bytes(P);
  char* rp = reinterpret_cast<char*>(m.pd->vec[r_id]) + off;
  const char* ap = reinterpret_cast<const char*>(m.pd->vec[V_AD]) + off;
  // a tile's vectors are read while the tile before it (or the sum) is worked on
  const int step = groups * kWideWG;
  Cx<T> r[3], ad[3], r2[3], ad2[3];
  int cb = m.tile * kWideWG + threadIdx.x;
  if (cb < half) {
    load_spinor<P, kNT>(rp, cb, r);
    load_spinor<P, kNT>(ap, cb, ad);
  }
  const double dAd = wide_sum(partials(B, m.slot, 0), ceil_div(half, dot_wg), lds);
  const bool ok = dAd > 0.0 && isfinite(dAd);
  const double alpha = delta / dAd;
  if (writer) {
    sc.dAd = dAd;
    if (ok) {
      sc.alpha = alpha;
      if (hist && sc.iter < sc.hist_len) hist[((long)m.slot * hist_stride + sc.iter) * 2] = alpha;
    } else {
      sc.flags |= kFlagNaN;
      sc.state = 2;
    }
  }
  if (!ok) return;  // uniform
  const T al = (T)alpha;
  double* part = B.partial + ((long)m.slot * kPartialSlots + 1) * B.pstride;
  int buf = 0;
  for (int t4 = m.tile * (kWideWG / kMaxWG); t4 < ntiles; t4 += groups * (kWideWG / kMaxWG), buf ^= 1, cb += step) {
    double s[1] = {0.0};
    if (cb + step < half) {
      load_spinor<P, kNT>(rp, cb + step, r2);
      load_spinor<P, kNT>(ap, cb + step, ad2);
    }
    if (cb < half) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        r[c].re = fma(-al, ad[c].re, r[c].re);
        r[c].im = fma(-al, ad[c].im, r[c].im);
      }
      store_spinor<P, kNT>(rp, cb, r);
#pragma unroll
      for (int c = 0; c < 3; ++c) s[0] += (double)r[c].re * r[c].re + (double)r[c].im * r[c].im;
    }
    // one partial per 256 sites: four waves, in order
    wave_sum<1>(s);
    if (threadIdx.x % kWave == 0) tiles[buf][threadIdx.x / kWave] = s[0];
    __syncthreads();
    if (threadIdx.x < kWideWG / kMaxWG && t4 + (int)threadIdx.x < ntiles) {
      const double* w = &tiles[buf][threadIdx.x * (kMaxWG / kWave)];
      double v = w[0];
#pragma unroll
      for (int k = 1; k < kMaxWG / kWave; ++k) v += w[k];
      part[t4 + threadIdx.x] = v;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[c] = r2[c];
      ad[c] = ad2[c];
    }
  }
}

template <int P, int PX>
__global__ __launch_bounds__(kWideWG) void k_xd_wide(Batch B, Scal* next, int x_id, int r_id, double* hist,
                                                     int hist_stride) {
  using T = typename RealOf<P>::T;
  using TX = typename RealOf<PX>::T;
  constexpr bool kNT = P != P64;  // as in k_update_xd
  __shared__ double lds[kWideWG / kWave];
  const Slot m = wide_slot(B);
  const int p = find_problem(B, blockIdx.x), groups = B.groups[p];
  const int half = m.pd->g.half;
  const TX alpha = (TX)B.scal[m.slot].alpha;
  char* dp = reinterpret_cast<char*>(m.pd->vec[V_D]) + (long)m.r * half * spinor_bytes(P);
  char* xp = reinterpret_cast<char*>(m.pd->vec[x_id]) + (long)m.r * half * spinor_bytes(PX);
  const char* rp = reinterpret_cast<const char*>(m.pd->vec[r_id]) + (long)m.r * half * spinor_bytes(P);
  const int step = groups * kWideWG;
  Cx<T> d[3], r[3], d2[3], r2[3];
  Cx<TX> x[3], x2[3];
  int cb = m.tile * kWideWG + threadIdx.x;
  if (cb < half) {
    load_spinor<P, kNT>(dp, cb, d);
    load_spinor<P, kNT>(rp, cb, r);
    load_spinor<PX, kNT>(xp, cb, x);
  }
  double b64;
  const int now = beta_step(
      B, m, next, hist, hist_stride,
      [&] { return wide_sum(partials(B, m.slot, 1), ceil_div(half, kMaxWG), lds); }, b64);
  if (now > 1) return;  // uniform
  const T beta = (T)b64;
  for (; cb < half; cb += step) {
    if (cb + step < half) {
      load_spinor<P, kNT>(dp, cb + step, d2);
      load_spinor<P, kNT>(rp, cb + step, r2);
      load_spinor<PX, kNT>(xp, cb + step, x2);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c].re = fma(alpha, (TX)d[c].re, x[c].re);
      x[c].im = fma(alpha, (TX)d[c].im, x[c].im);
      d[c].re = fma(beta, d[c].re, r[c].re);
      d[c].im = fma(beta, d[c].im, r[c].im);
    }
    store_spinor<PX, kNT>(xp, cb, x);
    store_spinor<P, kNT>(dp, cb, d);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      d[c] = d2[c];
      r[c] = r2[c];
      x[c] = x2[c];
    }
  }
}

int blocks_of(const Batch& B) { return B.block_start[B.nprob]; }

Batch wide_batch(const BatchHost& bh) {
  Batch B = make_batch(bh, kWideWG, 1);
  int slots[kMaxProb];
  for (int p = 0; p < B.nprob; ++p) slots[p] = bh.probs[p].nrhs;
  const int per = wide_tiles(B.tiles, slots, B.nprob);
  for (int p = 0; p < B.nprob; ++p) {
    B.groups[p] = per ? ceil_div(B.tiles[p], per) : 0;  // none fit: refused below
    B.block_start[p + 1] = B.block_start[p] + B.groups[p] * slots[p];
  }
  return B;
}

}  // namespace

hipError_t launch_fused_resid(const BatchHost& bh, bool wide, int prec, int dot_wg, double* hist, int hist_stride,
                              hipStream_t st) {
  const Batch B = wide ? wide_batch(bh) : make_batch(bh, kMaxWG, 1);
  const int nb = blocks_of(B);
  if (nb == 0) return bh.nslots ? hipErrorInvalidValue : hipSuccess;
  const int r_id = prec == P64 ? V_R : V_RL;
#define STAG_RESID(P)                                                                                  \
  if (wide)                                                                                            \
    k_resid_wide<P><<<nb, kWideWG, 0, st>>>(B, r_id, dot_wg, hist, hist_stride);                       \
  else                                                                                                 \
    k_resid<P><<<nb, kMaxWG, 0, st>>>(B, r_id, dot_wg, hist, hist_stride);                             \
  return hipGetLastError()
  switch (prec) {
    case P64: STAG_RESID(P64);
    case P32: STAG_RESID(P32);
    case P16: STAG_RESID(P16);
    default: return hipErrorInvalidValue;
  }
#undef STAG_RESID
}

hipError_t launch_fused_xd(const BatchHost& bh, bool wide, Scal* next, int prec, int x_id, double* hist,
                           int hist_stride, hipStream_t st) {
  const Batch B = wide ? wide_batch(bh) : make_batch(bh, kMaxWG, 1);
  const int nb = blocks_of(B);
  if (nb == 0) return bh.nslots ? hipErrorInvalidValue : hipSuccess;
  const int r_id = prec == P64 ? V_R : V_RL;
#define STAG_XD(P, PX)                                                                                 \
  if (wide)                                                                                            \
    k_xd_wide<P, PX><<<nb, kWideWG, 0, st>>>(B, next, x_id, r_id, hist, hist_stride);                  \
  else                                                                                                 \
    k_xd<P, PX><<<nb, kMaxWG, 0, st>>>(B, next, x_id, r_id, hist, hist_stride);                        \
  return hipGetLastError()
  switch (prec) {
    case P64: STAG_XD(P64, P64);
    case P32: STAG_XD(P32, P32);
    case P16: STAG_XD(P16, P32);
    default: return hipErrorInvalidValue;
  }
#undef STAG_XD
}

}  // namespace stag
