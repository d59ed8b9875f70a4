// Choice of the bf16 LM head's kernel for a launch: positions per workgroup
// and how W is loaded.  Host code without HIP, so that the rules can be checked
// by themselves.
#pragma once

#include <stdint.h>

namespace fork {

// Positions per workgroup; narrow: gemm_narrow.hip's kernel, with nontemporal
// W loads and the two-slot W ring (two workgroups per CU) as given.
struct TileChoice {
  bool narrow;
  int positions;
  bool nontemporal, two_per_cu;
};

constexpr long long kCus = 256;

// Rows of W are whole 128-byte cache lines.  If not, a row's 128-byte slab of
// a stage ends inside a line whose rest the next stage needs.
inline bool whole_lines(const void* W, int d) {
  return d % 64 == 0 && (reinterpret_cast<uintptr_t>(W) & 127) == 0;
}

// Tiles of 256 positions left in a last round that takes at most a quarter of
// the CUs after a few whole rounds: such tiles run as four workgroups of 64
// positions each, at the end of the same launch, so that they start on the
// CUs that finish first (M = 903, d = 1544, V = 50257, 788 tiles: step 192 ->
// 180 us; in a launch of their own 190).  Kernels with this path run their
// 256-position tiles 4% slower than those without, so it pays for at most six
// rounds.  0 if there are none.
inline int tail_tiles(long long n) {
  const long long rem = n % kCus, full = n / kCus;
  return full >= 1 && full <= 6 && rem > 0 && rem <= kCus / 4 ? (int)rem : 0;
}

// A tile of 64, 128 or 256 positions takes 1 : 1.45 : 2.1 (measured over d =
// 256 .. 4096, V = 2000 .. 32000, one round of tiles: 9.4 / 12.2 / 16.2 us,
// 14.3 / 19.9 / 27.5 us, 36.5 / 53 / 73 us; with every CU busy 39 / 58 / 94
// us), and the 256 CUs take one tile each per round, so the cost of a launch is
// the rounds times the tile's.  Rows that are not whole cache lines, and long
// rows, make the smaller tiles, which load more per flop, dearer once more than
// one round runs (d = 3504, M = 1294, V = 23341: 392 / 257 / 228 us; d = 3584, M =
// 142, V = 85185 202 / 172 / 159, M = 266, V = 48270 160 / 134 / 133).  Over 5663
// random sizes (d = 64 .. 4096, M to 3000, V to 130000) the choice is 0.6% slower
// than the best tile for each, and nowhere more than 4% slower than 256 positions.  Examples (us, 64 / 128
// / 256 positions): V = 8000, d = 1024: M = 512 16 / 22 / 28, M = 1024 28 / 23 /
// 29; V = 32000, d = 1024: M = 128 20 / 24 / 25, M = 256 30 / 27 / 30, M = 1024
// 98 / 79 / 63.
inline TileChoice choose_tile(int M, int d, int nvt, bool lines, long long w_bytes) {
  auto tiles = [&](int p) { return ((long long)M + p - 1) / p; };
  auto cost = [&](int p, int per_round) {
    const long long n = nvt * tiles(p);
    const bool dear = p < 256 && n > kCus && (!lines || d >= 2560);
    return (n + kCus - 1) / kCus * per_round * (dear ? 12 : 10);
  };
  const long long c64 = cost(64, 100), c128 = cost(128, 145);
  const long long c256 = cost(256, 210) - (tail_tiles(nvt * tiles(256)) ? 1050 : 0);
  const int best = c256 < c64 && c256 < c128 ? 256 : c128 < c64 ? 128 : 64;
  // One position tile reads W once: past the 256 MB last-level cache it is
  // loaded nontemporally (M = 64, d = 4096, one W for every step: 130 MB 37 us
  // cached and 51 nontemporal, 262 MB 52 and 60, 412 MB 80 and 73).  With 256
  // positions the same holds for the narrow kernel's four-column variant
  // (M = 256, V = 126464: 239 against 223 us; 412 MB 92 against 94 us).  Not
  // where rows are not whole lines: a line loaded past the caches is fetched
  // again for its rest (V = 126464, cached / nontemporal, us: d = 4088, M = 64
  // 220 / 271, M = 128 238 / 291, M = 256 281 / 317; d = 2056, M = 64 112 / 146).
  const bool nt = lines && tiles(best) == 1 && w_bytes > (320LL << 20);
  if (best == 256 && !(nt && w_bytes > (512LL << 20))) return {false, 256, false, false};
  // Two workgroups per CU fetch twice the lines at a time: with long rows that
  // are not whole lines the rest of a line is gone when its stage comes (V =
  // 126464, M = 64, three slots / two, us: d = 4088 220 / 236, 3504 178 / 195).
  const bool two = best == 64 && nvt * tiles(64) > kCus && (lines || d <= 1024);
  return {true, best, nt, two};
}

}  // namespace fork
