// Autotuner for the Dslash launch shape: workgroup size (sites per workgroup),
// right-hand sides per lane, LDS staging of the x/y neighbour window and the
// tile order (lattice order, or XCD blocks with their number of z blocks per XCD), and, for FP16
// batches of 8k right-hand sides, the time-streaming kernel with its number of time chunks; and the untuned
// default, whatever it is.  Candidates are timed with HIP events on the caller's stream on the real buffers of
// the call; winners are kept per key (lattice shapes, right-hand sides, storage precision) in memory and can be
// saved to / loaded from a small JSON file.
#include <algorithm>
#include <cstdio>
#include <fstream>
#include <map>
#include <mutex>
#include <sstream>

#include "runtime.h"

namespace stag {

namespace {

std::mutex g_mu;
std::map<std::string, DslashShape> g_table;   // tuned or pinned shapes

std::string key_of(const BatchHost& bh, const std::vector<const stag_lattice_s*>& lats, int prec) {
  std::ostringstream k;
  k << "p" << prec << (bh.long12 ? "c" : "");
  for (size_t i = 0; i < lats.size(); ++i) {
    const int* d = lats[i]->dims;
    k << ":" << d[0] << "x" << d[1] << "x" << d[2] << "x" << d[3] << "/" << bh.probs[i].nrhs;
  }
  return k.str();
}

int rhs_divisor(const BatchHost& bh) {
  int r = 8;
  for (const auto& p : bh.probs)
    while (r > 1 && p.nrhs % r) r >>= 1;
  return r;
}

// The most right-hand sides per lane that any problem of the batch can use: a lane with fewer left masks the rest.
int rhs_most(const BatchHost& bh) {
  int n = 1, r = 1;
  for (const auto& p : bh.probs) n = std::max(n, p.nrhs);
  while (r < 8 && r < n) r <<= 1;
  return r;
}

// The colour vectors of one time slice, all right-hand sides, of the largest lattice.
double slice_bytes(const BatchHost& bh, int prec) {
  double m = 0.0;
  for (const auto& p : bh.probs)
    if (p.lt > 0) m = std::max(m, (double)(p.half / p.lt) * p.nrhs * spinor_bytes(prec));
  return m;
}

// Whether FP16 below 2 MiB of colour vectors per time slice takes z blocks too, at r right-hand sides per lane.
bool f16_z_blocks(const BatchHost& bh, int r) {
  const bool power_of_two = (bh.max_half & (bh.max_half - 1)) == 0;
  return r <= 2 && bh.max_half >= 3 << 18 && !power_of_two;
}

// Without a tuned entry.  64-site workgroups (128 for FP16 at 8 RHS per lane); every choice gives the same bits.
//  * Right-hand sides per lane: up to 4; 8 for FP16 with 18-real three-hop links, and for FP32 and FP64 from 2^18
//    sites of one parity on, where each link is read once for all of them (28^3x96 x 8: FP64 803 us against 994 at
//    4, FP32 534 and 616; 24^3x48: 276 and 280, 178 and 187; at 16^3x32 4 is faster, 48 and 57).  Waves per SIMD do
//    not decide it: FP64 holds one at every count (268 to 419 registers), FP32 three at 2 per lane and two at 1, 4
//    and 8, FP16 two at 2 per lane and three at the others.  The FP16 kernel of 12-real links at 8 per lane keeps 120
//    bytes per lane in scratch memory, with 213 registers and none spilled.
//  * Fewer while that leaves less than two waves per SIMD (16^3x32 x 4, FP32: 25 us at 2 per lane, 28 at 4).  An FP64
//    launch holds one wave per SIMD, 1024 at once, and one that fits is not split over more (12^4 x 24: 28 us at 4
//    per lane, 972 waves, 42 at 1, four rounds of waves; 10x14x18x22 x 8: 22 us at 4, 36 at 1; the normal operator of
//    16^3x32 with 18-real links, x 2: 61 us at 2 per lane, 75 at 1, where a repeated one-parity operator, whose links
//    stay in the 256 MB cache, takes 30 and 28).
//  * Counts that are no multiple of 4 or 8 mask lanes of the last group instead of taking one or two per lane, where
//    that leaves at most two thirds of the groups: links are read, and x, y neighbours found in L1, once per
//    group.  28^3x96: 3 RHS FP64 739 -> 500 us, FP32 405 -> 313, FP16 247 -> 190; 5 RHS 982 -> 582, 609 -> 394,
//    378 -> 262; 7 RHS 1283 -> 728; 9 RHS 1582 -> 960.  8 per lane only if the last lane has 5 or more (9 RHS:
//    1072 us at 8 per lane, 960 at 4; 12: 1168 and 1105).  Enough waves must remain to hide the longer lane:
//    2048 in FP64 (16^3x32 x 5: 51 -> 43 us), 5120 in FP32 (20^3x40 x 3, 2500 waves: 57 us masked, 50 not), 7168
//    in FP16 (24^3x48 x 3, 5184 waves: 70 and 64), where 2 per lane gains nothing (64 -> 62..67).
//  * Tile order: on a small lattice the lattice order, whose t neighbours are in an XCD's 4 MiB L2 anyway
//    (16^3x32 x 8, FP64: 45 us, the z-block order 51).  From 2 MiB of colour vectors per time slice the orders
//    that sweep t through one XCD's share: z blocks where the lattice allows them (32^3x64 x 8: FP64 781 us
//    against 989, FP32 415 and 462), else the XCD sweep (28^3x96: FP64 x 12 RHS, 6.3 MB a slice, 1154 us against
//    1398; FP32 x 8, 2.1 MB, 591 and 626; at 2.0 MB, 24^3x48 FP32 x 12, 264 and 260).  FP32 and FP64 take z blocks
//    from 2^18 sites on (32^3x64 x 1: 349 us against 356 and 175 against 183).  FP16 takes
//    them with one or two per lane from 3 x 2^18 sites on: an iteration of CG, z blocks and lattice order, 48^3x144
//    x 1 1972 and 2049 us, 32^3x96 x 1 395 and 414, x 2 496 and 520, 32^3x48 x 2 267 and 283; below, 32^2x16x48
//    x 1 119 and 115.  Not where the sites are a power of two (32^3x64 x 1 341 and 337, x 2 356 and 342, where
//    32^3x72 has 303 and 323, 393 and 409), and not with four per lane (32^3x96 717 and 715).
DslashShape heuristic(const BatchHost& bh, int prec) {
  constexpr int kLargeHalf = 1 << 18;
  const bool r8_f16 = prec == P16 && !bh.long12, large = bh.max_half >= kLargeHalf;
  const bool sweep = slice_bytes(bh, prec) >= 2.0 * 1024 * 1024;
  DslashShape s;
  const int most = r8_f16 || (prec != P16 && large) ? 8 : 4;
  s.r = std::min(rhs_divisor(bh), most);
  auto waves = [&](int r) {
    long n = 0;
    for (const auto& p : bh.probs) n += (long)ceil_div(p.half, kWave) * ceil_div(p.nrhs, r);
    return n;
  };
  auto mostly_idle = [&](int r) {  // a last lane with half of its right-hand sides or more masked
    return std::any_of(bh.probs.begin(), bh.probs.end(), [&](const HostProb& p) { return (r - p.nrhs % r) % r >= r / 2; });
  };
  auto one_round = [&](int r) { return prec == P64 && waves(r) <= 1024; };
  while (s.r > 1 && waves(s.r) < 2048 && one_round(s.r) == one_round(s.r / 2)) s.r >>= 1;
  const long enough = prec == P64 ? 2048 : (prec == P32 ? 5120 : 7168);
  for (int r = std::min(rhs_most(bh), most); r > s.r && r >= (prec == P16 ? 4 : 2); r >>= 1)
    if (waves(r) >= enough && 3 * waves(r) <= 2 * waves(s.r) && !(r == 8 && mostly_idle(r))) {
      s.r = r;
      break;
    }
  s.wg = prec == P16 && s.r == 8 ? 128 : 64;
  s.order = sweep || (prec == P16 ? f16_z_blocks(bh, s.r) : large) ? 1 : 0;
  if (s.order && !dslash_shape_valid(bh, prec, s)) s.order = 0;
  if (!dslash_shape_valid(bh, prec, s)) s = DslashShape{64, 1, 0, 0};
  s.sweep = s.order == 0 && sweep;
  return s;
}

}  // namespace

std::string tune_key(const BatchHost& bh, const std::vector<const stag_lattice_s*>& lats, int prec) {
  return key_of(bh, lats, prec);
}

DslashShape lookup_shape(const BatchHost& bh, const std::string& key, int prec) {
  std::lock_guard<std::mutex> lk(g_mu);
  auto it = g_table.find(key);
  if (it != g_table.end()) {
    DslashShape s = it->second;
    s.r = std::min(s.r, rhs_most(bh));
    if (!dslash_shape_valid(bh, prec, s)) {  // a loaded entry that does not fit this batch
      s.lds = s.order = 0;
      s.chunks = 1;
    }
    return s;
  }
  return heuristic(bh, prec);
}

void pin_shape(const std::string& key, const DslashShape& s) {
  std::lock_guard<std::mutex> lk(g_mu);
  if (s.wg == 0)
    g_table.erase(key);
  else
    g_table[key] = s;
}

bool has_shape(const std::string& key) {
  std::lock_guard<std::mutex> lk(g_mu);
  return g_table.count(key) != 0;
}

// Time every candidate shape on the batch's Dslash (in_id -> out_id, output parity 1, plain epilogue).  The untuned
// default is always among them, so that a tuned shape is never the slower one: where it masks lanes or sweeps t per
// XCD it is timed besides the listed shapes and kept if it is the fastest; best_out and all hold shapes that
// stag_set_dslash_shape takes (28^3x96 FP64 x 12: default 1108 us, the fastest of those 1322).
hipError_t tune_batch(const BatchHost& bh, const std::string& key, int prec, hipStream_t st, DslashShape* best_out,
                      std::vector<std::pair<DslashShape, float>>* all, int in_id, int out_id) {
  const int rmax = rhs_divisor(bh);
  hipEvent_t e0, e1;
  hipError_t e = hipEventCreate(&e0);
  if (e != hipSuccess) return e;
  e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    (void)hipEventDestroy(e0);
    return e;
  }
  DslashShape best{};
  float best_us = 1e30f;
  const int reps = 5;
  std::vector<DslashShape> cands;
  for (int wg : {64, 128, 256})
    for (int r = 1; r <= rmax; r *= 2)
      for (int v = 0; v < 4; ++v) cands.push_back(DslashShape{wg, r, v & 1, v >> 1});
  // thinner XCD z blocks (2, 3, 4 or 6 per XCD) for the shapes without LDS staging
  for (int wg : {64, 128})
    for (int r = 1; r <= rmax; r *= 2)
      for (int c : {2, 3, 4, 6}) cands.push_back(DslashShape{wg, r, 0, 1, c});
  for (int r : {8, 4})
    for (int chunks : {1, 2, 4}) cands.push_back(DslashShape{64, r, 0, 2, chunks});
  const size_t settable = cands.size();
  const DslashShape untuned = heuristic(bh, prec);
  if (untuned.r > rmax || untuned.sweep) cands.push_back(untuned);
  DslashShape keep{};
  float keep_us = 1e30f;
  for (size_t i = 0; i < cands.size(); ++i) {
    const DslashShape& sh = cands[i];
    if (e != hipSuccess) break;
    if (!dslash_shape_valid(bh, prec, sh)) continue;
    for (int w = 0; w < 2 && e == hipSuccess; ++w)
      e = launch_dslash(bh, prec, EPI_PLAIN, 1, in_id, out_id, 0, 0, 3, sh, st);
    if (e == hipSuccess) e = hipEventRecord(e0, st);
    for (int k = 0; k < reps && e == hipSuccess; ++k)
      e = launch_dslash(bh, prec, EPI_PLAIN, 1, in_id, out_id, 0, 0, 3, sh, st);
    if (e == hipSuccess) e = hipEventRecord(e1, st);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess) break;
    const float us = 1e3f * ms / reps;
    if (us < keep_us) {
      keep_us = us;
      keep = sh;
    }
    if (i >= settable) continue;
    if (all) all->push_back({sh, us});
    if (us < best_us) {
      best_us = us;
      best = sh;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e == hipSuccess) {
    pin_shape(key, keep);
    if (best_out) *best_out = best;
  }
  return e;
}

bool save_table(const char* path) {
  std::lock_guard<std::mutex> lk(g_mu);
  std::ofstream f(path);
  if (!f) return false;
  f << "{\n";
  size_t i = 0;
  for (const auto& kv : g_table) {
    f << "  \"" << kv.first << "\": [" << kv.second.wg << ", " << kv.second.r << ", " << kv.second.lds << ", "
      << kv.second.order << ", " << kv.second.chunks << (kv.second.sweep ? ", 1]" : "]")
      << (++i < g_table.size() ? ",\n" : "\n");
  }
  f << "}\n";
  return (bool)f;
}

// Reads the format save_table writes: one "key": [wg, r, lds, order, chunks, sweep] entry per line (lds, order and
// sweep may be absent: 0; chunks: 1).
bool load_table(const char* path, int* n_loaded) {
  std::ifstream f(path);
  if (!f) return false;
  std::string line;
  int n = 0;
  std::map<std::string, DslashShape> tmp;
  while (std::getline(f, line)) {
    const size_t q0 = line.find('"');
    if (q0 == std::string::npos) continue;
    const size_t q1 = line.find('"', q0 + 1);
    const size_t b0 = line.find('[', q1);
    if (q1 == std::string::npos || b0 == std::string::npos) return false;
    int wg = 0, r = 0, lds = 0, order = 0, chunks = 1, sweep = 0;
    const int got =
        std::sscanf(line.c_str() + b0, "[%d , %d , %d , %d , %d , %d]", &wg, &r, &lds, &order, &chunks, &sweep);
    if (got < 2) return false;
    if ((wg != 64 && wg != 128 && wg != 256) || (r != 1 && r != 2 && r != 4 && r != 8) || (lds != 0 && lds != 1) ||
        (order < 0 || order > 2) || chunks < 1 || chunks > 64 || (sweep != 0 && sweep != 1) || (sweep && (lds || order)))
      return false;
    tmp[line.substr(q0 + 1, q1 - q0 - 1)] = DslashShape{wg, r, lds, order, chunks, sweep != 0};
    ++n;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  for (const auto& kv : tmp) g_table[kv.first] = kv.second;
  if (n_loaded) *n_loaded = n;
  return true;
}

}  // namespace stag
