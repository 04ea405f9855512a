// Link fattening in FP64: the one-hop (fat) links of the asqtad action and the three-hop (long)
// products, from a thin gauge field in the user layout [4][Lt][Lz][Ly][Lx][3][3] complex128.
//
// The improved staggered operator of the paper (Sec. 1 and Sec. 2, the MILC setting) takes smeared
// one-hop links and three-hop Naik links as input.  The smearing recipe is the published asqtad one
// (Orginos, Toussaint and Sugar 1999; Lepage 1999): for direction mu,
//   V_mu = c1 U_mu + c3 (3-link staples) + c5 (5-link staples) + c7 (7-link staples) + cL (Lepage paths)
// with c1 = 5/8, c3 = 1/16, c5 = 1/64, c7 = 1/384, cL = -1/16, each path of l links scaled by u0^(1-l),
// and W_mu(n) = U_mu(n) U_mu(n+mu) U_mu(n+2mu).
//
// The staples are built in stages, as products of whole fields, instead of walking 85 paths per site:
// a "wrap" of a field F (a path from n to n+mu) in a transverse direction nu and sign s is
//   s = +1:  U_nu(n) F(n+nu) U_nu(n+mu)^dag,        s = -1:  U_nu(n-nu)^dag F(n-nu) U_nu(n-nu+mu),
// the path that steps s nu, follows F, and steps back.  A wrap is linear in F, so everything whose
// outermost step is nu is summed before that step is taken.  With {nu, rho, si} the three transverse
// directions and both_nu = wrap_nu^+ + wrap_nu^-:
//   stage 1   X_nu = both_nu(U_mu)                                             (the 3-link staples)
//   stage 2   G_nu = c3 U_mu + c5 (X_rho + X_si) + c7 (both_rho(X_si) + both_si(X_rho))
//   stage 3   V_mu = c1 U_mu + sum_nu [ wrap_nu^+(G_nu + cL wrap_nu^+(U_mu)) + wrap_nu^-(G_nu + cL wrap_nu^-(U_mu)) ]
// (the Lepage paths take the same sign twice; their inner wrap is recomputed in stage 3, two products,
// rather than stored and read back, 288 B).  24 + 6 wraps per mu and site, in three launches.
//
// What bounds it: traffic beyond L2.  A field is 144 B per site (95 MB at 24^3x48) and the sites in flight on one
// XCD touch more of a stage's fields than its 4 MB L2 holds, so what matters is how few sites are in flight while
// enough bytes are.  Each kernel therefore runs as one wave per SIMD with 512 registers, and reads the matrices of
// its next product while it multiplies the current one: 27 to 36 KiB in flight per wave.  Against
// two to three waves per SIMD that each read, wait and multiply, the three stages fetch 0.61, 1.45 and 1.47 GB
// instead of 1.25, 1.97 and 2.04 at 24^3x48, and take 0.18, 0.26 and 0.25 ms instead of 0.22, 0.32 and 0.30
// (compulsory: 0.38, 0.67 and 0.67 GB read).  Three waves per CU instead of four are no faster, two are slower.
// One lane per site; the fields it works on are planar ([9][V] double2, one plane per matrix element), so that a
// wave's load of one element of 64 neighbour matrices is 1 KiB contiguous.  In the user layout the same load
// touches 64 cache lines for a sixth of their bytes.  What is written is not read again by the same launch: it
// goes past L2 (2% of the whole).  Workgroups are single waves: nothing is shared between waves, the last round of
// a launch drains a wave at a time, and a 16^3x32 field still fills the chip (0.59 ms against 0.71).
// The sum of each nu starts from zero and the larger term c1 U comes last: against extended precision the one-hop
// links of an 8^4 field are off by 0.9e-16 (relative, root mean square), 1.2e-16 as one running sum and 1.6e-16
// when every wrap was rounded to memory.
// Both link fields of a 24^3x48 field take 2.9 ms; 110 launches over matrices in the user layout, one wrap each,
// took 16.6 ms.
#include <hip/hip_runtime.h>

#include "device.h"
#include "fatten.h"

namespace stag {

namespace {

struct M3 {
  double2 e[9];  // row-major, (re, im)
};

// s += a b, s += a conj(b), s += conj(a) b
__device__ __forceinline__ void fma_nn(double2& s, double2 a, double2 b) {
  s.x = fma(a.x, b.x, s.x);
  s.x = fma(-a.y, b.y, s.x);
  s.y = fma(a.x, b.y, s.y);
  s.y = fma(a.y, b.x, s.y);
}
__device__ __forceinline__ void fma_nc(double2& s, double2 a, double2 b) { fma_nn(s, a, double2{b.x, -b.y}); }
__device__ __forceinline__ void fma_cn(double2& s, double2 a, double2 b) { fma_nn(s, double2{a.x, -a.y}, b); }

struct FGeo {
  int L[4];
  int stride[4];  // lex distance of one step: 1, Lx, Lx Ly, Lx Ly Lz
  int vol;        // at most 2^28: a planar element's byte offset fits 32 bits
};

// lex distance from n to n + d e_dir (periodic, |d| <= 2 <= L); c = coordinates of n
__device__ __forceinline__ int hop(const int c[4], const FGeo& g, int dir, int d) {
  int v = c[dir] + d;
  v = v >= g.L[dir] ? v - g.L[dir] : (v < 0 ? v + g.L[dir] : v);
  return (v - c[dir]) * g.stride[dir];
}

__device__ __forceinline__ void coords(int lex, const FGeo& g, int c[4]) {
  c[0] = lex % g.L[0];
  int r = lex / g.L[0];
  c[1] = r % g.L[1];
  r /= g.L[1];
  c[2] = r % g.L[2];
  c[3] = r / g.L[2];
}

__device__ __forceinline__ void st_past_l2(double2* p, double2 v) {
  __builtin_nontemporal_store(d2v{v.x, v.y}, reinterpret_cast<d2v*>(p));
}

// Element e of the matrix at `site` of a planar field.  The plane's base is uniform over the wave and the
// lane's offset 32 bits wide, so the loads take a scalar base.
__device__ __forceinline__ double2 ld_e(const double2* f, const FGeo& g, int e, int site) {
  const char* plane = reinterpret_cast<const char*>(f) + (long)e * g.vol * 16;
  return *reinterpret_cast<const double2*>(plane + (unsigned)site * 16u);
}
__device__ __forceinline__ void st_e(double2* f, const FGeo& g, int e, int site, double2 v) {
  char* plane = reinterpret_cast<char*>(f) + (long)e * g.vol * 16;
  st_past_l2(reinterpret_cast<double2*>(plane + (unsigned)site * 16u), v);
}
__device__ __forceinline__ M3 ld(const double2* f, const FGeo& g, int site) {
  M3 m;
#pragma unroll
  for (int i = 0; i < 9; ++i) m.e[i] = ld_e(f, g, i, site);
  return m;
}
__device__ __forceinline__ M3 zero() {
  M3 m;
#pragma unroll
  for (int i = 0; i < 9; ++i) m.e[i] = double2{0.0, 0.0};
  return m;
}

// acc += A F B^dag (PLUS) or A^dag F B, one row of the first product at a time
template <bool PLUS>
__device__ __forceinline__ void wrap_acc(M3& acc, const M3& a, const M3& f, const M3& b) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double2 t[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (PLUS)
          fma_nn(t[j], a.e[3 * i + k], f.e[3 * k + j]);
        else
          fma_cn(t[j], a.e[3 * k + i], f.e[3 * k + j]);
      }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (PLUS)
          fma_nc(acc.e[3 * i + j], t[k], b.e[3 * j + k]);
        else
          fma_nn(acc.e[3 * i + j], t[k], b.e[3 * k + j]);
      }
  }
}

// Closes a group of loads, or the product it feeds: loads stay on their side of it.  Left alone the compiler keeps
// two or three loads in flight and waits out a full memory latency for nearly every matrix row.
__device__ __forceinline__ void issue_all() { asm volatile("" ::: "memory"); }

// A B; an element is the sum of three complex products, each rounded by itself: against extended precision the
// long links are off by 0.95e-16 that way, 1.1e-16 as one chain of six fused products
__device__ __forceinline__ M3 mul(const M3& a, const M3& b) {
  M3 c = zero();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const double2 x = a.e[3 * i + k], y = b.e[3 * k + j];
        c.e[3 * i + j].x += x.x * y.x - x.y * y.y;
        c.e[3 * i + j].y += x.x * y.y + x.y * y.x;
      }
    __builtin_amdgcn_sched_barrier(0);  // row by row: interleaved, they cost k_long its third wave per SIMD
  }
  return c;
}

constexpr int kFatWG = 64;  // one wave
// LDS that holds a launch to one wave per SIMD (four of 160 KiB per CU) where the registers do not
constexpr int kOneWaveLds = 40000;

// The site of this lane in XCD-sweep order (xcd_sweep_site), or -1: workgroups go round-robin over the XCDs.
__device__ __forceinline__ int my_site(const FGeo& g) {
  return xcd_sweep_site(blockIdx.x & 7, (int)(blockIdx.x >> 3) * kFatWG + threadIdx.x, g.stride[3], g.L[3]);
}
inline int site_blocks(const FGeo& g) {
  return 8 * (int)((xcd_sweep_len(g.stride[3], g.L[3]) + kFatWG - 1) / kFatWG);
}

// The k-th transverse direction of mu, k = 0..2
__host__ __device__ constexpr int transverse(int mu, int k) { return k < mu ? k : k + 1; }

// The matrices of a wave between the user layout (9 double2 per site, contiguous) and one matrix per lane,
// through LDS, so that a load or store covers whole cache lines where the lanes' sites are neighbours.
// site < 0: nothing is stored.
__device__ __forceinline__ void store_user(double2* out, int site, int lane, const M3& m, double2* lds) {
#pragma unroll
  for (int e = 0; e < 9; ++e) lds[9 * lane + e] = m.e[e];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int u = i * 64 + lane, owner = u / 9;
    const int s = __shfl(site, owner, 64);
    if (s >= 0) st_past_l2(&out[9L * s + (u - 9 * owner)], lds[u]);
  }
  __builtin_amdgcn_wave_barrier();
}
// Every lane asks for a valid site.
__device__ __forceinline__ M3 load_user(const double2* f, int site, int lane, double2* lds) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int u = i * 64 + lane, owner = u / 9;
    const int s = __shfl(site, owner, 64);
    lds[u] = f[9L * s + (u - 9 * owner)];
  }
  __builtin_amdgcn_wave_barrier();
  M3 m;
#pragma unroll
  for (int e = 0; e < 9; ++e) m.e[e] = lds[9 * lane + e];
  __builtin_amdgcn_wave_barrier();
  return m;
}

// user layout -> planes, one direction per blockIdx.y
__global__ __launch_bounds__(kFatWG) void k_planes(const double2* __restrict__ U, double2* __restrict__ P, FGeo g) {
  __shared__ double2 lds[9 * kFatWG];
  const int raw = blockIdx.x * kFatWG + threadIdx.x;
  const long f = (long)blockIdx.y * 9 * g.vol;
  const M3 m = load_user(U + f, raw < g.vol ? raw : g.vol - 1, threadIdx.x, lds);
  if (raw >= g.vol) return;
#pragma unroll
  for (int e = 0; e < 9; ++e) st_e(P + f, g, e, raw, m.e[e]);
}

// Stage 1: X_nu = both_nu(U_mu), a group of three matrices per nu and sign
template <int MU>
__global__ __launch_bounds__(kFatWG, 1) void k_staple(const double2* __restrict__ U, double2* __restrict__ X, FGeo g) {
  const int n = my_site(g);
  if (n < 0) return;
  int c[4];
  coords(n, g, c);
  const long f9 = 9L * g.vol;
  const double2* Um = U + MU * f9;
  const int mu1 = hop(c, g, MU, 1);
  M3 m[2][3], acc;
  auto fetch = [&](int i, M3(&w)[3]) {
    const int nu = transverse(MU, i >> 1);
    const double2* Un = U + nu * f9;
    const int up = n + hop(c, g, nu, 1), dn = n + hop(c, g, nu, -1);
    const int at = (i & 1) == 0 ? n : dn;
    w[0] = ld(Un, g, at);
    w[1] = ld(Um, g, (i & 1) == 0 ? up : dn);
    w[2] = ld(Un, g, at + mu1);
    issue_all();
  };
  fetch(0, m[0]);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    if (i < 5) fetch(i + 1, m[(i + 1) & 1]);
    const M3(&w)[3] = m[i & 1];
    if ((i & 1) == 0) {
      acc = zero();
      wrap_acc<true>(acc, w[0], w[1], w[2]);
    } else {
      wrap_acc<false>(acc, w[0], w[1], w[2]);
#pragma unroll
      for (int e = 0; e < 9; ++e) st_e(X + (i >> 1) * f9, g, e, n, acc.e[e]);
    }
    issue_all();
  }
}

// Stage 2: G_nu = c3 U_mu + c5 (X_rho + X_si) + c7 (both_rho(X_si) + both_si(X_rho)), the three nu together:
// the four U_rho matrices of a wrap serve both X fields that rho wraps.  A group of four matrices per rho and
// sign, and a last one with the terms of the site itself.
template <int MU>
__global__ __launch_bounds__(kFatWG, 1) void k_inner(const double2* __restrict__ U, const double2* __restrict__ X,
                                                     double2* __restrict__ G, double c3, double c5, double c7, FGeo g) {
  const int n = my_site(g);
  if (n < 0) return;
  int c[4];
  coords(n, g, c);
  const long f9 = 9L * g.vol;
  const int mu1 = hop(c, g, MU, 1);
  M3 m[2][4], acc[3] = {zero(), zero(), zero()};
  auto fetch = [&](int i, M3(&w)[4]) {
    if (i == 6) {
      w[3] = ld(U + MU * f9, g, n);
      // unrolled late, by itself: with the pragma the allocator spills 16 registers (276 us instead of 254)
      for (int k = 0; k < 3; ++k) w[k] = ld(X + k * f9, g, n);
    } else {
      const int r = i >> 1, rho = transverse(MU, r), p = (r + 1) % 3, q = (r + 2) % 3;
      const double2* Ur = U + rho * f9;
      const int at = (i & 1) ? n + hop(c, g, rho, -1) : n, from = (i & 1) ? at : n + hop(c, g, rho, 1);
      w[0] = ld(Ur, g, at);
      w[1] = ld(Ur, g, at + mu1);
      w[2] = ld(X + p * f9, g, from);
      w[3] = ld(X + q * f9, g, from);
    }
    issue_all();
  };
  fetch(0, m[0]);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    fetch(i + 1, m[(i + 1) & 1]);
    const int r = i >> 1, p = (r + 1) % 3, q = (r + 2) % 3;
    const M3(&w)[4] = m[i & 1];
    if ((i & 1) == 0) {
      wrap_acc<true>(acc[q], w[0], w[2], w[1]);
      wrap_acc<true>(acc[p], w[0], w[3], w[1]);
    } else {
      wrap_acc<false>(acc[q], w[0], w[2], w[1]);
      wrap_acc<false>(acc[p], w[0], w[3], w[1]);
    }
    issue_all();
  }
  const M3(&w)[4] = m[0];
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    const double2 u = w[3].e[e];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double2 p = w[(k + 1) % 3].e[e], q = w[(k + 2) % 3].e[e], a = acc[k].e[e];
      st_e(G + k * f9, g, e, n, double2{c3 * u.x + c5 * (p.x + q.x) + c7 * a.x, c3 * u.y + c5 * (p.y + q.y) + c7 * a.y});
    }
  }
}

// Stage 3: V_mu in the user layout.  Two groups of three matrices per nu and sign: the inner wrap of U_mu at the
// site one step away, which reads one step further,
//   +: U_nu(n+nu) U_mu(n+2nu) U_nu(n+nu+mu)^dag,  -: U_nu(n-2nu)^dag U_mu(n-2nu) U_nu(n-2nu+mu),
// and the outer one; then U_mu of the site itself.
template <int MU>
__global__ __launch_bounds__(kFatWG, 1) void k_outer(const double2* __restrict__ U, const double2* __restrict__ G,
                                                     double2* __restrict__ V, double c1, double cl, FGeo g) {
  __shared__ double2 lds[9 * kFatWG];
  const int own = my_site(g);
  if (__ballot(own >= 0) == 0) return;  // the whole wave is past the lattice
  const int n = own >= 0 ? own : 0;
  int c[4];
  coords(n, g, c);
  const long f9 = 9L * g.vol;
  const double2* Um = U + MU * f9;
  const int mu1 = hop(c, g, MU, 1);
  M3 h, m[2][3], part, acc = zero();
  auto fetch = [&](int i, M3(&w)[3]) {
    if (i == 12) {
      w[0] = ld(Um, g, n);
      issue_all();
      return;
    }
    const int k = i >> 2, nu = transverse(MU, k);
    const bool plus = ((i >> 1) & 1) == 0, inner = (i & 1) == 0;
    const double2* Un = U + nu * f9;
    const int one = n + hop(c, g, nu, plus ? 1 : -1), two = n + hop(c, g, nu, plus ? 2 : -2);
    const int at = inner ? (plus ? one : two) : (plus ? n : one);
    w[0] = ld(Un, g, at);
    w[1] = inner ? ld(Um, g, two) : ld(G + k * f9, g, one);
    w[2] = ld(Un, g, at + mu1);
    issue_all();
  };
  fetch(0, m[0]);
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    fetch(i + 1, m[(i + 1) & 1]);
    const bool plus = ((i >> 1) & 1) == 0;
    const M3(&w)[3] = m[i & 1];
    if ((i & 1) == 0) {
      if ((i & 3) == 0) part = zero();
      h = zero();
      if (plus)
        wrap_acc<true>(h, w[0], w[1], w[2]);
      else
        wrap_acc<false>(h, w[0], w[1], w[2]);
    } else {
#pragma unroll
      for (int e = 0; e < 9; ++e) h.e[e] = double2{fma(cl, h.e[e].x, w[1].e[e].x), fma(cl, h.e[e].y, w[1].e[e].y)};
      if (plus)
        wrap_acc<true>(part, w[0], h, w[2]);
      else
        wrap_acc<false>(part, w[0], h, w[2]);
      if ((i & 3) == 3)
#pragma unroll
        for (int e = 0; e < 9; ++e) {
          acc.e[e].x += part.e[e].x;
          acc.e[e].y += part.e[e].y;
        }
    }
    issue_all();
  }
  // c1 U_mu, the largest term, last: the sum's roundings are then relative to the staples alone
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    const double2 u = m[0][0].e[e];
    acc.e[e] = double2{fma(c1, u.x, acc.e[e].x), fma(c1, u.y, acc.e[e].y)};
  }
  store_user(V, own, threadIdx.x, acc, lds);
}

// W_mu(n) = U_mu(n) U_mu(n + mu) U_mu(n + 2 mu), from and to the user layout, one mu per blockIdx.y
__global__ __launch_bounds__(kFatWG) void k_long(const double2* __restrict__ U, double2* __restrict__ W, FGeo g) {
  __shared__ double2 lds[9 * kFatWG];
  const int lane = threadIdx.x, own = my_site(g);
  if (__ballot(own >= 0) == 0) return;  // the whole wave is past the lattice
  const int n = own >= 0 ? own : 0, mu = blockIdx.y;
  int c[4];
  coords(n, g, c);
  int d1 = 0, d2 = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d)
    if (d == mu) {
      d1 = hop(c, g, d, 1);
      d2 = hop(c, g, d, 2);
    }
  const double2* Um = U + (long)mu * 9 * g.vol;
  const M3 a = load_user(Um, n, lane, lds);
  const M3 t = mul(a, load_user(Um, n + d1, lane, lds));
  const M3 w = mul(t, load_user(Um, n + d2, lane, lds));
  store_user(W + (long)mu * 9 * g.vol, own, lane, w, lds);
}

template <int MU>
void fat_direction(const double2* Up, double2* X, double2* G, double2* V, double u0, const FGeo& g, hipStream_t st) {
  const double u2 = 1.0 / (u0 * u0), u4 = u2 * u2, u6 = u4 * u2;
  const double c1 = 5.0 / 8.0, c3 = u2 / 16.0, c5 = u4 / 64.0, c7 = u6 / 384.0, cl = -u4 / 16.0;
  const dim3 nb(site_blocks(g)), wg(kFatWG);
  hipLaunchKernelGGL(k_staple<MU>, nb, wg, kOneWaveLds, st, Up, X, g);
  hipLaunchKernelGGL(k_inner<MU>, nb, wg, 0, st, Up, (const double2*)X, G, c3, c5, c7, g);
  hipLaunchKernelGGL(k_outer<MU>, nb, wg, 0, st, Up, (const double2*)G, V, c1, cl, g);
}

}  // namespace

size_t fatten_workspace_bytes(const int dims[4]) {
  const long vol = (long)dims[0] * dims[1] * dims[2] * dims[3];
  return (size_t)kFattenWsFields * vol * 9 * sizeof(double2);
}

hipError_t fatten_links(const int dims[4], const void* thin, double u0, void* fat, void* lng, void* ws,
                        hipStream_t st) {
  const long vol = (long)dims[0] * dims[1] * dims[2] * dims[3];
  if (vol > (1L << 28)) return hipErrorOutOfMemory;  // thin, fat and lng alone would take 464 GB
  FGeo g;
  for (int i = 0; i < 4; ++i) g.L[i] = dims[i];
  g.stride[0] = 1;
  for (int i = 1; i < 4; ++i) g.stride[i] = g.stride[i - 1] * dims[i - 1];
  g.vol = (int)vol;
  const long f9 = 9 * vol;
  const double2* U = static_cast<const double2*>(thin);
  double2* V = static_cast<double2*>(fat);
  // the planar copy of U lives in the long-link output until the last launch writes that
  double2* Up = static_cast<double2*>(lng);
  double2* X = static_cast<double2*>(ws);
  double2* G = X + 3 * f9;
  const dim3 nb4((g.vol + kFatWG - 1) / kFatWG, 4), wg(kFatWG);
  hipLaunchKernelGGL(k_planes, nb4, wg, 0, st, U, Up, g);
  fat_direction<0>(Up, X, G, V, u0, g, st);
  fat_direction<1>(Up, X, G, V + f9, u0, g, st);
  fat_direction<2>(Up, X, G, V + 2 * f9, u0, g, st);
  fat_direction<3>(Up, X, G, V + 3 * f9, u0, g, st);
  hipLaunchKernelGGL(k_long, dim3(site_blocks(g), 4), wg, 0, st, U, static_cast<double2*>(lng), g);
  return hipGetLastError();
}

}  // namespace stag
