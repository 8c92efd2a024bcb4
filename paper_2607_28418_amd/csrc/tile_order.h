// Which tile, chunk or place each workgroup of the large kernels takes: index
// arithmetic only, used by the kernels and by the host code that sizes their
// launches.  It includes no HIP header, so that a host compiler takes it too
// (the cover tests run it).
#pragma once

#include <stddef.h>
#include <stdint.h>

#if defined(__HIP__)
#define WIDE_ORDER __host__ __device__ inline __attribute__((always_inline))
#else
#define WIDE_ORDER inline
#endif

namespace wide {

// Workgroup id -> tile id: each XCD (workgroups are dealt round-robin to the
// 8 XCDs) walks a contiguous range of tile ids.
WIDE_ORDER int xcd_remap(int id, int n) {
  const int q = n / 8, r = n % 8;
  const int xcd = id % 8, local = id / 8;
  return (xcd < r) ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
}

// ---- N axis, m-blocked -----------------------------------------------------------
// Each XCD takes an eighth of the `cols` column tiles and runs m-tile 0 of each
// of them, then m-tile 1, and so on; with `halves`, over one half of its columns
// and then the other (where a half has two groups, of ntpg column tiles, or more).
// The eighths are exact: a column is eight units, XCD x owns units [cols x,
// cols (x + 1)), and m-tile m of a column goes to the owner of its unit
// mblock_unit(m), which spreads any run of units over the m-tiles.  (Dealt in
// whole columns, 108 of them times 7 m-tiles gave four XCDs 98 tiles, two more
// than three rounds of their 32 CUs.)
// Bits of m % 8 reversed; bit r of mblock_below(f): unit(r) < f.
WIDE_ORDER int mblock_unit(int m) { return (m & 1) << 2 | (m & 2) | (m & 4) >> 2; }
WIDE_ORDER int mblock_below(int f) { return (int)(0x7f77575515110100ull >> (8 * f)) & 0xff; }
// Tiles of units [u0, u1).
WIDE_ORDER int mblock_count(int u0, int u1, int m_tiles) {
  const int r = m_tiles % 8, low = (1 << r) - 1;
  return m_tiles / 8 * (u1 - u0) + r * (u1 / 8 - u0 / 8) + __builtin_popcount(mblock_below(u1 % 8) & low) -
         __builtin_popcount(mblock_below(u0 % 8) & low);
}
// Workgroups per XCD, at least its tiles:
WIDE_ORDER int mblock_share(int cols, int m_tiles) { return m_tiles / 8 * cols + m_tiles % 8 * ((cols + 7) / 8); }
// Workgroup `local` of an XCD (m_tile = m_tiles: padding).
WIDE_ORDER void mblock_place(int cols, int m_tiles, int ntpg, bool halves, bool shift, int xcd, int local, int& col,
                             int& m_tile) {
  int u0 = cols * xcd, u1 = u0 + cols, l = local;
  if (halves && cols >= 32 * ntpg) {
    const int mid = (u0 + u1) / 16 * 8, n = mblock_count(u0, mid, m_tiles);
    if (l < n) {
      u1 = mid;
    } else {
      l -= n;
      u0 = mid;
    }
  }
  col = 0;
  m_tile = m_tiles;
  if (l >= mblock_count(u0, u1, m_tiles)) return;
  const int below0 = mblock_below(u0 % 8), below1 = mblock_below(u1 % 8);  // m-tiles (mod 8) of the cut columns:
  const int m8 = l / (u1 - u0), whole = u1 / 8 - u0 / 8;                   // not the first's, also the last's
  l -= m8 * (u1 - u0);
  int r = 0, n = whole + (below1 & 1) - (below0 & 1);
  while (l >= n) {
    l -= n;
    ++r;
    n = whole + (below1 >> r & 1) - (below0 >> r & 1);
  }
  m_tile = m8 * 8 + r;
  // Workgroups go to an XCD's four shader engines in turn.  In rows of an odd
  // number of columns a column's m-tiles then meet every engine; with `shift`, rows
  // of an even number start one column on in every m-tile (every second one where 4
  // does not divide it), so that theirs do too.  Else, with every other group off
  // for all tokens, the real tiles would all go to two of the engines (4096 x
  // 11008, groups of 128, 953 tokens: 235 us, 165 so; 2048 x 8192, groups of 256,
  // 1500 tokens 151 and 113).
  if (shift && !(n & 1)) l = (l + (n & 2 ? m_tile >> 1 : m_tile)) % n;
  col = u0 / 8 + (below0 >> r & 1) + l;
}

// ---- K axis, dense-masked (256 x 256 tiles, one workgroup a CU, 256 a round) -------
constexpr int kKdTile = 256, kKdStep = 64;
// Up to this many groups the rows go in mask-pattern order.
constexpr int kPatternMaxGroups = 8;

// Tiles [0, total): full rounds in XCD blocks where the column tiles allow it
// (round r covers the m-tiles [r mr, (r + 1) mr), mr = 256 / n_tiles, and XCD x
// a block of mr / 4 m-tiles by n_tiles / 2 column tiles of them), the rest m-major.
WIDE_ORDER void kd256_coords(int id, int n_tiles, int total, int& m_tile, int& n_tile) {
  const bool blocks = n_tiles % 2 == 0 && n_tiles <= 256 && 256 % n_tiles == 0 && (256 / n_tiles) % 4 == 0;
  const int rounds = blocks ? total / 256 : 0;
  if (id < rounds * 256) {
    const int xcd = id % 8, local = id / 8;  // workgroups are dealt round-robin to the 8 XCDs
    const int r = local / 32, q = local % 32;
    const int mr = 256 / n_tiles, bm = mr / 4, bn = n_tiles / 2;
    m_tile = r * mr + (xcd % 4) * bm + q % bm;
    n_tile = (xcd / 4) * bn + q / bm;
    return;
  }
  const int base = rounds * 256;
  const int tile = base + xcd_remap(id - base, total - base);  // m-major: n-tiles share the A panel
  m_tile = tile / n_tiles;
  n_tile = tile % n_tiles;
}

// The last, partial round: tiles [base, total) are each run by `split`
// workgroups (1: not split), token rows from m0 on; the chunks' partial sums
// take split * (M - m0) * N floats, at most `avail`.  At most as many chunks as
// fill the 256 CUs once, each at least kKdMinSteps steps deep; of that number and
// the powers of two below it (8 chunks give every XCD one slice of the operands)
// the one with the least estimated time, if that saves 1 us.
struct Kd256Tail {
  int base, split;
  int64_t m0;
};
constexpr int kKdMaxSplit = 16, kKdMinSteps = 4;
constexpr size_t kKd256PartMaxFloats = (size_t)256 * 256 * 256;  // at most 256 chunks of one tile's sums
WIDE_ORDER Kd256Tail kd256_tail(int64_t M, int N, int K, int ng, size_t avail) {
  const int n_tiles = N / kKdTile;
  const int64_t m_tiles = (M + kKdTile - 1) / kKdTile, total = m_tiles * n_tiles;
  Kd256Tail t{(int)total, 1, M};
  if (total == 0 || n_tiles > 256) return t;
  const int mr = 256 / n_tiles;  // m-tiles of a full round
  const int64_t mb = m_tiles / mr * mr, rem = total - mb * n_tiles, rows = M - mb * kKdTile;
  // (rows the mask-pattern order may move between a whole and a split tile
  // keep one summation order: there only launches of less than a round split)
  if (rem == 0 || (mb > 0 && ng > 1 && ng <= kPatternMaxGroups)) return t;
  int64_t split = 256 / rem;
  if (split > kKdMaxSplit) split = kKdMaxSplit;
  if (split > K / kKdStep / kKdMinSteps) split = K / kKdStep / kKdMinSteps;
  if (split > (int64_t)(avail / ((size_t)rows * N))) split = (int64_t)(avail / ((size_t)rows * N));
  // Measured (K 1024 to 8192, N 1024 to 4096, 200 to 3500 tokens): a whole tile
  // takes 0.97 us per step, and a cut one its share of that plus 0.5 us and, for
  // the partial sums written and read back, 0.06 us per chunk of 256 rows in the
  // launch.  Cut as often as the CUs allow, calls with little to share lost: K
  // 1024, N 2048, 2000 tokens at keep 0.5 33 us whole, 39 in four; K 1024, N 1024,
  // 5000 tokens 36 and 43.  In mask-pattern order a tile's union shrinks with the
  // tiles that share the patterns; keep 0.5 is assumed there (which steps a tile
  // skips is known on the device only; K 4096, N 4096, 2000 tokens, 4 groups, cut
  // in two: 55 -> 66 us at keep 0.25, 71 -> 71 at 0.5, 87 -> 77 at 0.75).
  float steps = (float)(K / kKdStep);
  if (ng > 1 && ng <= kPatternMaxGroups) {
    int bits = 0;  // of the pattern that stay the same over a tile
    while (bits < ng && (int64_t)2 << bits <= m_tiles) ++bits;
    steps *= 1.0f - 0.5f * (float)bits / (float)ng;
  }
  const float chunk_us = 0.06f * (float)(rows * n_tiles) / kKdTile;
  float best = 0.97f * steps - 1.0f;
  for (int64_t s = 2; s <= split; s = 2 * s <= split || s == split ? 2 * s : split) {
    const float us = 0.97f * steps / (float)s + 0.5f + chunk_us * (float)s;
    if (us < best) {
      best = us;
      t = Kd256Tail{(int)(mb * n_tiles), (int)s, mb * kKdTile};
    }
  }
  return t;
}
// Workgroup tail_base + id: chunk and tile.
WIDE_ORDER void kd256_chunk(int id, int m_tiles, int n_tiles, int tail_base, int split, int& chunk, int& m_tile,
                            int& n_tile) {
  const int rem = m_tiles * n_tiles - tail_base, mt = rem / n_tiles;
  const int j = xcd_remap(id, rem * split);
  chunk = j / rem;
  m_tile = tail_base / n_tiles + j % rem % mt;
  n_tile = j % rem / mt;
}
// The k steps [u0, u1) of chunk c.
WIDE_ORDER void kd256_steps(int K, int c, int split, int& u0, int& u1) {
  const int u = K / kKdStep;
  u0 = u * c / split;
  u1 = u * (c + 1) / split;
}

// ---- prefill attention --------------------------------------------------------------
// Place `rem` of a head block's n_seq * n_slots tiles: `block` sequences at a
// time, slot by slot from the last (longest key ranges first), the block's
// sequences in turn.
WIDE_ORDER void attn_place(int rem, int n_seq, int n_slots, int block, int& slot, int& b) {
  int b0 = 0, nb = n_seq;
  if (block < n_seq) {
    const int per = block * n_slots, i = rem / per;
    rem -= i * per;
    b0 = i * block;
    nb = block < n_seq - b0 ? block : n_seq - b0;
  }
  const int up = rem / nb;
  slot = n_slots - 1 - up;
  b = b0 + rem - up * nb;
}

}  // namespace wide
