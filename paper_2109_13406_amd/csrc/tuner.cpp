// tuner.cpp -- the tuning table of a handle (see tuner.hpp).
#include "tuner.hpp"

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "kernels.hpp"

namespace mpdd {

int shape_bucket(int64_t x) {
  int b = 0;
  while (b < 62 && ((int64_t)1 << b) < x) ++b;
  return b;
}

static int op_code(const char* s) {
  if (std::strcmp(s, "gemm") == 0) return 0;
  if (std::strcmp(s, "syrk") == 0) return 1;
  return -1;
}

bool TuneTable::load(const char* path) {
  FILE* f = std::fopen(path, "r");
  if (!f) return false;
  char line[512];
  bool ok = true;
  while (std::fgets(line, sizeof line, f)) {
    const char* p = std::strstr(line, "{\"op\"");
    if (!p) continue;
    char op[8] = {0}, tr[4] = {0};
    int mb, nb, kb, tile, splitk, nsl = 0;
    int got = std::sscanf(p,
                          "{\"op\": \"%7[a-z]\", \"trans\": \"%3[NT]\", \"mb\": %d, \"nb\": %d, "
                          "\"kb\": %d, \"tile\": %d, \"splitk\": %d, \"nslices\": %d",
                          op, tr, &mb, &nb, &kb, &tile, &splitk, &nsl);
    const int code = op_code(op);
    if (got < 7 || code < 0 || std::strlen(tr) != 2 || !tile_info(tile) || splitk < 1) {
      ok = false;
      break;
    }
    TuneEntry e;
    e.tile = tile;
    e.splitk = splitk;
    e.nslices = nsl;
    if (const char* st = std::strstr(p, "\"serve_tile\":")) {
      int t = -1;
      if (std::sscanf(st, "\"serve_tile\": %d", &t) != 1 || (t >= 0 && !tile_info(t))) {
        ok = false;
        break;
      }
      e.serve_tile = t;
    }
    map_[Key(code, tr[0] == 'T', tr[1] == 'T', mb, nb, kb)] = e;
  }
  std::fclose(f);
  return ok;
}

bool TuneTable::lookup(int op, bool ta, bool tb, int64_t m, int64_t n, int64_t k,
                       TuneEntry& out) const {
  auto it = map_.find(Key(op, ta, tb, shape_bucket(m), shape_bucket(n), shape_bucket(k)));
  if (it == map_.end()) return false;
  out = it->second;
  return true;
}

// The built-in choice.  Products whose 64 x 64 tiles (entry 4), split along k
// into ranges of >= 512, give 512 workgroups (1024 for a triangle) take those,
// with a k-split (default_split) that aims at 1024 workgroups (2048) and ranges
// of >= 256 (512).  The others go by the time that each of the square tiles
// (entries 2, 4 and 5) would take with each k-split S, in microseconds:
//   base + (k / S) max(alone, L shared) + (S > 1: reduce + partials / bandwidth)
// with L = ceil(tiles S / 256) workgroups per CU, `alone` the time per term of
// a workgroup that has its CU for itself (its serial chain) and `shared` that
// of one among several (FP64 issue and LDS reads: 1.4, 1.2 and 1.6 times the
// 10 issue slots per multiply-add).  Measured: entry 5 at 64^3 8.9 us, 256^3
// 16.9, 512^3 62; entry 2 at 64^3 13.5, 200^3 30.3, 512^3 split in 4 64; entry
// 4 at 64^3 34, 8192 x 64 x 2000 split in 4 368.  Against every (tile, split)
// pair the choice is within 10 % of the best; the rule before it (by the
// number of 64 x 64 tiles alone, k-ranges of 256 and more) lost up to 3.5x:
// 64 x 64 x 1000 69 -> 18 us, 300 x 60 x 1500 55 -> 28.
namespace {

struct TileTime {
  int tile, edge;
  double base, alone, shared;
};
constexpr TileTime kTileTimes[] = {{5, 16, 5.5, 0.043, 0.0283},
                                   {2, 32, 5.0, 0.125, 0.0955},
                                   {4, 64, 5.0, 0.45, 0.335}};
constexpr double kReduceUs = 6.0, kPartialBytesPerUs = 3.0e6;

double plan_time(const TileTime& t, int64_t m, int64_t n, int64_t k, bool tri, int s) {
  const int64_t tm = (m + t.edge - 1) / t.edge, tn = (n + t.edge - 1) / t.edge;
  const double tiles = tri ? 0.5 * (double)tm * (double)(tm + 1) : (double)tm * (double)tn;
  const double load = (double)(int64_t)((tiles * s + 255.0) / 256.0);
  double us = t.base + (double)((k + s - 1) / s) * std::max(t.alone, load * t.shared);
  if (s > 1) us += kReduceUs + 32.0 * s * (double)m * (double)n / kPartialBytesPerUs;
  return us;
}

}  // namespace

double estimated_us(int tile, int64_t m, int64_t n, int64_t k, bool tri, int splitk) {
  for (const TileTime& t : kTileTimes)
    if (t.tile == tile) return plan_time(t, m, n, k, tri, splitk);
  return 0.0;
}

int default_split(int64_t tiles, int64_t k, bool tri) {
  const int64_t target = tri ? 2048 : 1024, min_range = tri ? 512 : 256;
  int s = 1;
  while (s < 32 && tiles * s < target && k / (2 * s) >= min_range) s *= 2;
  return s;
}

TilePlan default_plan(int64_t m, int64_t n, int64_t k, bool tri, int max_split) {
  const int64_t tm = (m + 63) / 64, tn = (n + 63) / 64;
  const int64_t tiles = tri ? tm * (tm + 1) / 2 : tm * tn;
  if (tiles * std::min<int64_t>(32, std::max<int64_t>(1, k / 512)) >= (tri ? 1024 : 512)) {
    const int s = std::min(max_split, default_split(tiles, k, tri));
    return TilePlan{4, s, plan_time(kTileTimes[2], m, n, k, tri, s)};
  }
  return timed_plan(m, n, k, tri, max_split);
}

TilePlan timed_plan(int64_t m, int64_t n, int64_t k, bool tri, int max_split, int max_edge) {
  TilePlan best{2, 1, 0.0};
  for (const TileTime& t : kTileTimes)
    for (int s = 1; t.edge <= max_edge && s <= max_split && (s == 1 || k / s >= 32); s *= 2) {
      const double us = plan_time(t, m, n, k, tri, s);
      if (best.us == 0.0 || us < best.us) best = TilePlan{t.tile, s, us};
    }
  return best;
}

int64_t split_chunk(int64_t k, int bk, int& splits) {
  auto range = [&] { return ((k + splits - 1) / splits + bk - 1) / bk * bk; };
  const int64_t asked = range();
  while (splits > 1 && (int64_t)(splits - 1) * asked >= k) splits >>= 1;
  return splits > 1 ? range() : k;
}

int default_tile(int64_t m, int64_t n, int64_t k, bool tri) {
  return default_plan(m, n, k, tri, 1).tile;
}

}  // namespace mpdd
