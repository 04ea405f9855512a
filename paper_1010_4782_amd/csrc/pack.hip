// Link ingest and packing, and colour-vector precision conversions.
//
// Packing folds into each of the 16 matrices an output site uses (Sec. 2, Eq. (5):
// the staggered phases are absorbed into the stored links):
//   k = 4 mu + 0 : eta_mu(n) s(n,1) F_mu(n)                       (neighbour n + mu)
//   k = 4 mu + 1 : -eta_mu(n) s(n-mu,1) F_mu(n-mu)^dag            (neighbour n - mu)
//   k = 4 mu + 2 : c_N eta_mu(n) s(n,3) W_mu(n)                   (neighbour n + 3mu)
//   k = 4 mu + 3 : -c_N eta_mu(n) s(n-3mu,3) W_mu(n-3mu)^dag      (neighbour n - 3mu)
// with s(m,k) = (-1)^floor((m_t + k)/L_t) for the time direction when it is
// antiperiodic and 1 otherwise.  Back links are duplicated per output parity so
// the Dslash streams exactly 16 matrices per site, coalesced (Sec. 3.1).
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace stag {

Geo make_geo(const int dims[4]) {
  Geo g{};
  for (int i = 0; i < 4; ++i) {
    g.L[i] = dims[i];
    g.h1[i] = 1 % dims[i];
    g.h3[i] = 3 % dims[i];
  }
  g.Xh = dims[0] / 2;
  g.half = (int)((long)dims[0] * dims[1] * dims[2] * dims[3] / 2);
  g.stride[0] = 0;
  g.stride[1] = g.Xh;
  g.stride[2] = g.Xh * dims[1];
  g.stride[3] = g.Xh * dims[1] * dims[2];
  g.t0 = 0;
  g.lt_glob = dims[3];
  g.h3g = 3 % dims[3];
  g.t_open = 0;
  g.in_half = g.half;
  return g;
}

// binary16 code of v / s, the quotient in binary64 (the compiler contracts the two conversions into one
// rounding, to nearest even).
__device__ __forceinline__ _Float16 f16_code(double v, float s) {
  return s > 0.f ? (_Float16)(float)(v / (double)s) : (_Float16)0.f;
}

// The same code from y = RN(1 / s), s finite and positive, without a division and with the conversion
// instructions instead of the dozens of integer ones that a binary64 -> binary16 rounding expands to.
//  * q = RN(v y) is within two units of v / s in the last place, one step q + RN(v - q s) y brings it within
//    one, and the second then gives RN(v / s) itself (Markstein 1990: the remainder of a faithful quotient is
//    exact, and the corrected quotient correctly rounded when y is).
//  * q goes to binary32 rounded to odd (an inexact result takes the neighbour whose last bit is set), which
//    keeps enough of q for the rounding to binary16 to be the direct one (two more bits than the result
//    suffice, Boldo and Melquiond 2008).
__device__ __forceinline__ unsigned short f16_code_y(double v, double s, double y) {
  double q = v * y;
  q = fma(fma(-q, s, v), y, q);
  q = fma(fma(-q, s, v), y, q);
  const float f = (float)q;
  const double d = fabs((double)f), a = fabs(q);
  unsigned w = __float_as_uint(f);
  const unsigned moved = d < a ? w + 1u : (d > a ? w - 1u : w);
  w = (w & 1u) ? w : moved;
  return __builtin_bit_cast(unsigned short, (_Float16)__uint_as_float(w));
}

// Packs the links of one block of 64 output sites and both parities in every requested precision (FP64 always).
// A wave takes 32 sites of one parity with two lanes per site: lane half h loads, folds and stores the four
// matrices of directions 2h and 2h + 1 of a group (one-hop, then three-hop).  The four waves of a block read
// the same cache lines: the sites of the other parity lie in between.  A wave's 64 source matrices (144 B each,
// at sites that are neighbours but for lattice edges) are loaded as 9 x 1 KiB with consecutive lanes on
// consecutive 16-byte words, the next matrix already in flight, and handed to their lanes through LDS; one
// lane per matrix would touch 64 cache lines per load.
// The FP16 scales need all eight matrices of a group (largest |re|, |im| over the stored entries of an output
// site's one-hop and, separately, three-hop matrices, rounded to binary32), so with FP16 a lane's four stay in
// registers (144 of 256 VGPRs; 9 or 10 others of the kernel spill, 40 or 44 bytes per lane) instead of being read
// back from the FP64 blocks.
// Lanes past the lattice pack site 0 into the padding, which nothing reads.
// Bound by its traffic: 8.2 GB beyond L2 at 28^3x96 (FP64 + FP16, two-row long links: 5 GB of it the packed
// links) in 1.63 ms, 5 TB/s.  One pass per parity and precision, a lane per output site gathering 144-byte
// matrices and the FP16 pass reading the FP64 blocks back, took 3.02 ms.
template <bool W32, bool W16>
__global__ __launch_bounds__(4 * kWave, 2) void k_pack_links(const double2* fat, const double2* lng, double naik,
                                                             Geo g, PackOut out) {
  __shared__ d2v lds[4][9 * kWave];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int par = wave & 1, h = lane >> 5;
  const long blk = xcd_remap(blockIdx.x, gridDim.x);
  const int bl = 32 * (wave >> 1) + (lane & 31);  // this lane's site within the block
  const int cb_raw = (int)blk * kWave + bl;
  const Site s = site_of(cb_raw < g.half ? cb_raw : 0, par, g);
  const long vol9 = (long)g.half * 18;
  const long lex = (((long)s.t * g.L[2] + s.z) * g.L[1] + s.y) * g.L[0] + s.x;
  const bool c12 = g.long12 != 0;
  d2v* stage = lds[wave];
  // this lane's two directions, q = 0, 1: mu = 2 h + q
  int c[2], L[2], stride[2], eta[2];
  c[0] = h ? s.z : s.x;
  c[1] = h ? s.t : s.y;
  L[0] = h ? g.L[2] : g.L[0];
  L[1] = h ? g.L[3] : g.L[1];
  stride[0] = h ? g.L[0] * g.L[1] : 1;
  stride[1] = h ? g.L[0] * g.L[1] * g.L[2] : g.L[0];
  eta[0] = h ? (s.x + s.y) & 1 : 0;
  eta[1] = h ? (s.x + s.y + s.z) & 1 : s.x & 1;
  // which lane's matrix, and which of its words, this lane loads in step i
  int owner[9], word[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    owner[i] = (i * kWave + lane) / 9;
    word[i] = i * kWave + lane - 9 * owner[i];
  }
  // start coordinate of the lane's j-th matrix (direction q = j / 2, odd j backward: n - hop mu)
  auto start = [&](int j, int hop) {
    const int q = j >> 1;
    return (j & 1) ? ((c[q] - hop) % L[q] + L[q]) % L[q] : c[q];
  };
  auto load = [&](const double2* field, int j, int hop, d2v (&w)[9]) {
    const int q = j >> 1;
    const long at = (2 * h + q) * vol9 + 9 * (lex + (long)(start(j, hop) - c[q]) * stride[q]);
#pragma unroll
    for (int i = 0; i < 9; ++i) w[i] = as_global<d2v>(field)[__shfl(at, owner[i], kWave) + word[i]];
  };
  d2v next[9];
  load(fat, 0, 1, next);
  auto group = [&](auto which) {
    constexpr int grp = decltype(which)::value;  // 0: one-hop, 1: three-hop matrices
    constexpr int hop = grp ? 3 : 1;
    const bool two_rows = c12 && grp == 1, have = grp == 0 || lng != nullptr;
    d2v u[W16 ? 4 : 1][9];
    float scale = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      d2v(&v)[9] = u[W16 ? j : 0];
      const int k0 = 4 * (j >> 1) + (j & 1) + 2 * grp;  // matrix index of the lower half; the upper's is 8 more
      if (have) {  // uniform
#pragma unroll
        for (int i = 0; i < 9; ++i) stage[i * kWave + lane] = next[i];
        __builtin_amdgcn_wave_barrier();
        if (j < 3)
          load(grp ? lng : fat, j + 1, hop, next);
        else if (grp == 0 && lng)
          load(lng, 0, 3, next);
        // folded matrix: eta, boundary sign, c_N; the backward one daggered and negated
        double coef = eta[j >> 1] ? -1.0 : 1.0;
        if (grp == 1) coef *= naik;
        if (j & 1) coef = -coef;
        if ((j >> 1) == 1 && h && g.antiper && (((start(j, hop) + hop) / L[1]) & 1)) coef = -coef;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            // forward: U[a][b]; backward: (U^dag)[a][b] = conj(U[b][a])
            const d2v w = stage[9 * lane + ((j & 1) ? 3 * b + a : 3 * a + b)];
            v[3 * a + b] = d2v{coef * w.x, (j & 1) ? -coef * w.y : coef * w.y};
          }
        __builtin_amdgcn_wave_barrier();
      } else {
#pragma unroll
        for (int e = 0; e < 9; ++e) v[e] = d2v{0.0, 0.0};
      }
      gptr_w<d2v> o = as_global_w<d2v>(out.f64[par] + link_slot_offset(P64, c12, blk, k0 + 8 * h)) + bl;
#pragma unroll
      for (int e = 0; e < 9; ++e)
        if (!two_rows || e < 6) __builtin_nontemporal_store(v[e], o + e * kWave);
      if constexpr (W32) {
        char* base = out.f32[par] + link_slot_offset(P32, c12, blk, k0 + 8 * h);
        gptr_w<f4v> q = as_global_w<f4v>(base) + bl;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!two_rows || e < 3)
            __builtin_nontemporal_store(f4v{(float)v[2 * e].x, (float)v[2 * e].y, (float)v[2 * e + 1].x, (float)v[2 * e + 1].y},
                                        q + e * kWave);
        if (!two_rows)
          __builtin_nontemporal_store(f2v{(float)v[8].x, (float)v[8].y}, as_global_w<f2v>(base + 4 * kWave * 16) + bl);
      }
      if constexpr (W16) {
        double mx = 0.0;
#pragma unroll
        for (int e = 0; e < 9; ++e)
          if (!two_rows || e < 6) mx = fmax(mx, fmax(fabs(v[e].x), fabs(v[e].y)));
        scale = fmaxf(scale, (float)mx);
      }
    }
    if constexpr (W16) {
      scale = fmaxf(scale, __shfl_xor(scale, 32, kWave));
      if (h == 0)
        __builtin_nontemporal_store(scale, as_global_w<float>(out.scale[par]) + (blk * 2 + grp) * kWave + bl);
      const bool fast = scale > 0.f && scale < __builtin_inff();
      const double sd = (double)scale, y = 1.0 / sd;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned w[9];
        if (fast) {
#pragma unroll
          for (int e = 0; e < 9; ++e)
            w[e] = f16_code_y(u[j][e].x, sd, y) | (unsigned)f16_code_y(u[j][e].y, sd, y) << 16;
        } else {  // a zero group, or one past binary32's range
#pragma unroll 1
          for (int e = 0; e < 9; ++e) {
            h2v q;
            q.x = f16_code(u[j][0].x, scale);
            q.y = f16_code(u[j][0].y, scale);
            const d2v first = u[j][0];  // rotate: the registers are indexed statically
            const unsigned code = __builtin_bit_cast(unsigned, q);
#pragma unroll
            for (int i = 0; i < 8; ++i) u[j][i] = u[j][i + 1];
            u[j][8] = first;
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = w[i + 1];
            w[8] = code;
          }
        }
        char* base = out.f16[par] + link_slot_offset(P16, c12, blk, 4 * (j >> 1) + (j & 1) + 2 * grp + 8 * h);
        gptr_w<u4v> q = as_global_w<u4v>(base) + bl;
        __builtin_nontemporal_store(u4v{w[0], w[1], w[2], w[3]}, q);
        if (two_rows) {
          __builtin_nontemporal_store(u2v{w[4], w[5]}, as_global_w<u2v>(base + kWave * 16) + bl);
        } else {
          __builtin_nontemporal_store(u4v{w[4], w[5], w[6], w[7]}, q + kWave);
          __builtin_nontemporal_store(w[8], as_global_w<unsigned>(base + 2 * kWave * 16) + bl);
        }
      }
    }
  };
  group(std::integral_constant<int, 0>{});
  group(std::integral_constant<int, 1>{});
}

hipError_t launch_pack_links(const void* fat, const void* lng, double naik, const Geo& g, const PackOut& out,
                             hipStream_t st) {
  const int nblk = ceil_div(g.half, kWave);
  auto f = reinterpret_cast<const double2*>(fat);
  auto l = reinterpret_cast<const double2*>(lng);
  const bool w32 = out.f32[0] != nullptr, w16 = out.f16[0] != nullptr;
  if (w32 && w16)
    k_pack_links<true, true><<<nblk, 4 * kWave, 0, st>>>(f, l, naik, g, out);
  else if (w32)
    k_pack_links<true, false><<<nblk, 4 * kWave, 0, st>>>(f, l, naik, g, out);
  else if (w16)
    k_pack_links<false, true><<<nblk, 4 * kWave, 0, st>>>(f, l, naik, g, out);
  else
    k_pack_links<false, false><<<nblk, 4 * kWave, 0, st>>>(f, l, naik, g, out);
  return hipGetLastError();
}

// ---- colour-vector conversions ---------------------------------------------------
// complex128 -> storage format; f16 uses the per-site rule s = binary32(max |v|),
// code = binary16(binary32(v / s)).
template <int P>
__global__ __launch_bounds__(256) void k_from_f64(const double2* in, char* out, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2* v = in + 3 * i;
  double2 w[3] = {v[0], v[1], v[2]};
  if (P == P32) {
    float2* o = reinterpret_cast<float2*>(out) + 3 * i;
#pragma unroll
    for (int c = 0; c < 3; ++c) o[c] = make_float2((float)w[c].x, (float)w[c].y);
  } else if (P == P16) {
    double m = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) m = fmax(m, fmax(fabs(w[c].x), fabs(w[c].y)));
    const float s = (float)m;
    h2v h[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      h[c].x = f16_code(w[c].x, s);
      h[c].y = f16_code(w[c].y, s);
    }
    reinterpret_cast<uint4*>(out)[i] = make_uint4(__builtin_bit_cast(unsigned, h[0]), __builtin_bit_cast(unsigned, h[1]),
                                                  __builtin_bit_cast(unsigned, h[2]), __float_as_uint(s));
  } else {
    double2* o = reinterpret_cast<double2*>(out) + 3 * i;
#pragma unroll
    for (int c = 0; c < 3; ++c) o[c] = w[c];
  }
}

template <int P>
__global__ __launch_bounds__(256) void k_to_f64(const char* in, double2* out, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Cx<typename RealOf<P>::T> v[3];
  load_spinor<P>(in, i, v);
#pragma unroll
  for (int c = 0; c < 3; ++c) out[3 * i + c] = make_double2((double)v[c].re, (double)v[c].im);
}

hipError_t launch_convert_from_f64(int prec, const void* in, void* out, long nsites, hipStream_t st) {
  if (nsites == 0) return hipSuccess;
  const long nblk = (nsites + 255) / 256;
  auto i = reinterpret_cast<const double2*>(in);
  auto o = reinterpret_cast<char*>(out);
  switch (prec) {
    case P64: k_from_f64<P64><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    case P32: k_from_f64<P32><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    case P16: k_from_f64<P16><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_convert_to_f64(int prec, const void* in, void* out, long nsites, hipStream_t st) {
  if (nsites == 0) return hipSuccess;
  const long nblk = (nsites + 255) / 256;
  auto i = reinterpret_cast<const char*>(in);
  auto o = reinterpret_cast<double2*>(out);
  switch (prec) {
    case P64: k_to_f64<P64><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    case P32: k_to_f64<P32><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    case P16: k_to_f64<P16><<<nblk, 256, 0, st>>>(i, o, nsites); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace stag
