// Large-tile prefill kernels (256 x 256 tiles, 4 waves, direct-to-LDS loads).
//
//   wide_mn256       N-axis masked projection (GEMM-MN): gate/up + SwiGLU
//                    (one tile = 256 sorted tokens x one 128-column slice
//                    of a group: 128 gate rows + 128 up rows), or plain
//                    Q/K/V (one tile = 256 tokens x 256 output columns).
//   wide_mn256_half  the same on half as many columns, for groups that narrow.
//   wide_mn256_fit   gate/up with few tiles: either width, chosen on the device.
//   wide_mn256_tail  adds the chunks of the Q/K/V tiles cut along k.
//   wide_kd256       K-axis masked projection, dense-masked schedule;
//   wide_kd256_finish  adds the chunks of its tiles cut along k.
//   wide_ks256       K-axis masked projection, scatter schedule (GEMM-K).
//
// Which tile a workgroup takes: tile_order.h, and mn256_coords below for the
// orders that follow the groups' counts.
//
// Semantics, skipping levels and the two K-axis schedules are those of the
// 128-tile kernels in gemm_mn.hip / gemm_k.hip (WIDE Section 3.1 equations
// (1)-(3); Section 3.3; Appendix B, Algorithms 2 and 3); only the tile engine
// differs (tile256.h).  Tiles whose 256 rows are all active take the
// all-active path (no per-fragment tests), as the paper does for full tiles
// of a sorted column.  BK is the ring's k depth, 64; BUF: operands through
// buffer views.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "tile256.h"

namespace wide {

using namespace t256;

namespace {
__device__ __attribute__((aligned(16))) uint16_t g_zero_blk[64];  // stays zero: never written

// Rings: three stages of A and two of B (160 KB, all of LDS), except the
// dense-masked K-axis kernel over more than 128 groups, which keeps 17 KB for
// its tile's mask bits and so runs two A stages.
using RingMN = Ring<3>;
// 128-wide N-axis tiles (NFN = 2): B stages are half as large, and four of
// them fit.
template <int NFN>
using RingN = std::conditional_t<NFN == 2, Ring<3, 4, 2>, RingMN>;
template <int NWR>
using RingKD = Ring<NWR == 0 ? 2 : 3>;

// Epilogue row map.  Output rows go back to token order through a per-row
// index (the reorder, or the pattern order); fetching it per output element
// put one dependent global load in front of every store.  Instead, thread
// r < 256 fetches tile row r's token (-1 past the end) before the k loop,
// and after it the map goes through the then idle ring LDS.
// `extra` (a row's mask bits, token-order regions) goes to map[BM + r].
__device__ __forceinline__ const int* stage_row_map(uint16_t* smem, int my_row, int extra = 0) {
  int* map = reinterpret_cast<int*>(smem);
  __syncthreads();  // every wave is done with the ring
  if (threadIdx.x < BM) {
    map[threadIdx.x] = my_row;
    map[BM + threadIdx.x] = extra;
  }
  __syncthreads();
  return map;
}

// Bit b of the result: byte b of the n (<= 32) mask bytes at mr is nonzero.
// Rows of ng bytes start 16-byte aligned when 16 divides ng (the mask itself
// is 16-byte aligned), 4-byte aligned when 4 does; the loads are as wide as
// that allows.
__device__ __forceinline__ uint32_t nz4(uint32_t w) {  // bit i: byte i of w != 0
  const uint32_t m = (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u;
  return ((m >> 7) & 1u) | ((m >> 14) & 2u) | ((m >> 21) & 4u) | ((m >> 28) & 8u);
}
__device__ __forceinline__ uint32_t mask_bits32(const uint8_t* mr, int n, int ng) {
  uint32_t bits = 0;
  if (n == 32 && ng % 16 == 0) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(mr);
    const u32x4 b = *reinterpret_cast<const u32x4*>(mr + 16);
    bits = nz4(a[0]) | nz4(a[1]) << 4 | nz4(a[2]) << 8 | nz4(a[3]) << 12 | nz4(b[0]) << 16 |
           nz4(b[1]) << 20 | nz4(b[2]) << 24 | nz4(b[3]) << 28;
  } else if (ng % 4 == 0) {  // n is a multiple of 4 too
    for (int b = 0; b < n; b += 4) bits |= nz4(*reinterpret_cast<const uint32_t*>(mr + b)) << b;
  } else {
    for (int b = 0; b < n; ++b) bits |= (uint32_t)(mr[b] != 0) << b;
  }
  return bits;
}

// Tiles of one region that each XCD runs (the region padded to a multiple of 8).
__host__ __device__ __forceinline__ int mn256_share(int tiles) { return (tiles + 7) / 8; }

// The k loop of one tile with the wave's live A fragments and A loads:
// `act` tile rows are active, always a prefix (rows past the active count, or
// past M, come last in a tile).
template <class Rg, int BL, class Koff, class LdA, class LdB>
__device__ __forceinline__ void run_tile(uint16_t* smem, int nsteps, Koff koff, LdA lda, LdB ldb,
                                         const int (&bb)[Rg::NFN], int64_t act, f32x16 (&acc)[4][Rg::NFN]) {
  const int p = (int)(act < 0 ? 0 : act > BM ? BM : act);
  const int w = wave_id(), wm = w >> 1;
  const int nl = min(4, max(0, (p - wm * 128 + 31) / 32));  // live A fragments of the wave
  const bool aon = 64 * w < p;                              // the wave's A load rows [64 w, 64 w + 64)
  // (nl, aon): (4|3, true) full or nearly; (2|1, true|false); (0, false) -- the
  // waves of the lower half of a tile with at most 128 active rows
  switch (nl) {
    case 4: mainloop<Rg, 4, true, BL>(smem, nsteps, koff, lda, ldb, bb, acc); break;
    case 3: mainloop<Rg, 3, true, BL>(smem, nsteps, koff, lda, ldb, bb, acc); break;
    case 2:
      if (aon) mainloop<Rg, 2, true, BL>(smem, nsteps, koff, lda, ldb, bb, acc);
      else mainloop<Rg, 2, false, BL>(smem, nsteps, koff, lda, ldb, bb, acc);
      break;
    case 1:
      if (aon) mainloop<Rg, 1, true, BL>(smem, nsteps, koff, lda, ldb, bb, acc);
      else mainloop<Rg, 1, false, BL>(smem, nsteps, koff, lda, ldb, bb, acc);
      break;
    default: mainloop<Rg, 0, false, BL>(smem, nsteps, koff, lda, ldb, bb, acc); break;
  }
}
}  // namespace

// Tile order inside an XCD's share of a region: group, then sorted m-tile,
// then column tile inside the group, so the tiles an XCD runs together share
// the group's weight panel in L2 (gate/up runs m-blocked instead, see
// mn256_mblocked).  A group wider than four column tiles (one group over a
// whole projection, the M-axis case) goes column tile first: each XCD then
// covers a slice of the weight once and re-reads the gathered rows, which
// fit the last-level cache, instead of streaming the whole weight once per
// m-tile.
//
// When an XCD's share is a whole number of groups ("ordered"), it runs the
// full tiles of its groups first, then their partial last m-tiles, then the
// empty ones, so its real tiles come first.
template <int BNO>
__device__ __forceinline__ bool mn256_ordered(const MN256Args& a, const MN256Region& R) {
  const int share = mn256_share(R.tiles), per_group = R.gw / BNO * a.m_tiles;
  return a.order && R.masked == kMN256Sorted && R.gw / BNO <= 4 && 8 * share == R.tiles &&
         share % per_group == 0;
}

// "m-blocked" (gate/up): each XCD takes an eighth of the column tiles and runs
// m-tile 0 of each of them, then m-tile 1, and so on, over one half of its
// columns and then the other.  The tiles that run together then gather rows
// from one stretch of tokens (a sorted m-tile of any group covers about the
// same token range) instead of one group's whole token list, so the gathered
// rows are mostly shared in L2 while each group's weight panel is re-read once
// per m-tile.  Measured on the Llama-3-8B gate/up at T = 8192 (topk, keep
// 0.5): traffic from beyond L2 down 37%, time down 2% against group by group;
// blocks of 4 or 8 m-tiles per group cut the traffic as much but ran 7-9%
// slower.  Halves (7 of the XCD's 14 groups at a time, so fewer weight panels
// per k step, and the first half's partial m-tiles run beside the second
// half's full ones) took another 2.5% off; pairs of groups did the same.  It
// also deals the real tiles in one run: workgroups go round-robin to an
// XCD's four shader engines, and real and empty tiles in turn (two m-tiles
// per group, one empty) sent all the real ones to two of them (Llama-7B
// gate/up, 300 tokens, 64-column tiles: 106 us, now 65).  The adaptive launch's
// 64-column tiles, at most one round, take no halves; those of 64-channel groups
// take them from eight m-tiles on (keep 0.25, 0.5 and 0.75, 14336 channels, 2000
// tokens: 391, 492 and 615 us without, 355, 464 and 586 with; 4096 tokens 680,
// 906 and 1127 against 651, 884 and 1111; 500 tokens 178 against 183 at keep 0.5).
template <int BNO>
__host__ __device__ __forceinline__ bool mn256_mblocked(const MN256Args& a, const MN256Region& R) {
  return a.mblock && R.masked == kMN256Sorted && (BNO == 64 || R.gw <= (BNO <= 128 ? 512 : 1024));
}

// Workgroups per XCD of a region.
template <int BNO>
__host__ __device__ __forceinline__ int mn256_region_share(const MN256Args& a, const MN256Region& R) {
  if (mn256_mblocked<BNO>(a, R)) return mblock_share(R.tiles / a.m_tiles, a.m_tiles);
  return mn256_share(R.tiles);
}

// FIT: the adaptive launch's narrow tiles, at most one round of real ones.
template <int BNO, bool FIT = false>
__device__ __forceinline__ void mn256_coords(const MN256Args& a, const MN256Region& R, int xcd, int local,
                                             int& g, int& m_tile, int& nt_in) {
  const int share = mn256_share(R.tiles);
  const int tile = xcd * share + local;
  const int ntpg = R.gw / BNO;  // tiles per group
  const int per_group = ntpg * a.m_tiles;
  if (mn256_mblocked<BNO>(a, R)) {
    int col;
    // (narrow tiles of the adaptive launch, one to a CU, keep their rows in place:
    // 4096 x 14336, every other group of 512 off, 373 tokens 104 us, shifted 139)
    mblock_place(R.tiles / a.m_tiles, a.m_tiles, ntpg, !FIT && (BNO != 64 || a.m_tiles >= 8), !FIT, xcd, local, col,
                 m_tile);
    g = col / ntpg;
    nt_in = col % ntpg;
    return;
  }
  if (mn256_ordered<BNO>(a, R)) {
    const int gps = share / per_group, gb = xcd * gps, gl = gb + gps - 1;
    int n_full = 0, n_part = 0;
    for (int i = gb; i <= gl; ++i) {
      const int c = a.cnt[i];
      n_full += c / BM;
      n_part += (c % BM) != 0;
    }
    int l = local;
    if (l < n_full * ntpg) {
      for (g = gb; g < gl; ++g) {
        const int f = a.cnt[g] / BM * ntpg;
        if (l < f) break;
        l -= f;
      }
      m_tile = l / ntpg;
      nt_in = l % ntpg;
    } else if ((l -= n_full * ntpg) < n_part * ntpg) {
      for (g = gb; g < gl; ++g) {
        const int f = (a.cnt[g] % BM) != 0 ? ntpg : 0;
        if (l < f) break;
        l -= f;
      }
      m_tile = a.cnt[g] / BM;
      nt_in = l;
    } else {
      l -= n_part * ntpg;
      for (g = gb; g < gl; ++g) {
        const int e = (a.m_tiles - (a.cnt[g] + BM - 1) / BM) * ntpg;
        if (l < e) break;
        l -= e;
      }
      m_tile = (a.cnt[g] + BM - 1) / BM + l / ntpg;
      nt_in = l % ntpg;
    }
  } else {
    if (ntpg > 4) {
      nt_in = (tile / a.m_tiles) % ntpg;
      m_tile = tile % a.m_tiles;
    } else {
      nt_in = tile % ntpg;
      m_tile = (tile / ntpg) % a.m_tiles;
    }
    g = tile / per_group;
  }
}

template <int BNO>
__host__ __device__ __forceinline__ int mn256_shares(const MN256Args& a) {
  int n = mn256_region_share<BNO>(a, a.reg[0]);
  if (a.n_regions > 1) n += mn256_region_share<BNO>(a, a.reg[1]);
  if (a.n_regions > 2) n += mn256_region_share<BNO>(a, a.reg[2]);
  return n;
}

// The XCD's last partial round.  An XCD's 32 CUs run its real tiles in
// rounds of 32; with T real tiles the last T % 32 would leave most CUs idle
// for a whole tile's time (measured: 15-20% of Q/K/V, 7% of gate/up).  With
// a.tail those n = T % 32 tiles are cut along k into split = 32 / n chunks,
// run by 32 extra workgroups per XCD that write fp32 partial tiles; a second
// kernel adds each tile's chunks in order and applies the epilogue.  Only
// for launches whose regions are dense or ordered (real tiles first in every
// share, so a tile's rank among the XCD's real tiles is known).
struct MN256Tail {
  int real[3], before[3];  // real tiles per region share; real tiles of earlier regions
  int base, n, split;      // first tail rank, tail tiles, chunks per tail tile
};

template <int BNO>
__device__ __forceinline__ int mn256_real(const MN256Args& a, const MN256Region& R, int xcd) {
  const int share = mn256_share(R.tiles);
  if (R.masked != kMN256Sorted) return max(0, min(share, R.tiles - xcd * share));
  const int ntpg = R.gw / BNO, gps = share / (ntpg * a.m_tiles), gb = xcd * gps;
  int n = 0;
  for (int i = 0; i < gps; ++i) n += (a.cnt[gb + i] + BM - 1) / BM;
  return n * ntpg;
}

template <int BNO>
__device__ __forceinline__ MN256Tail mn256_tail(const MN256Args& a, int xcd) {
  MN256Tail t;
  t.real[0] = mn256_real<BNO>(a, a.reg[0], xcd);
  t.real[1] = a.n_regions > 1 ? mn256_real<BNO>(a, a.reg[1], xcd) : 0;
  t.real[2] = a.n_regions > 2 ? mn256_real<BNO>(a, a.reg[2], xcd) : 0;
  t.before[0] = 0;
  t.before[1] = t.real[0];
  t.before[2] = t.real[0] + t.real[1];
  const int total = t.before[2] + t.real[2];
  t.base = total / kMN256TailJobs * kMN256TailJobs;
  t.n = total - t.base;
  // at most 8 chunks: each adds a 256 KB partial tile to write and read back
  t.split = t.n ? min(kMN256TailJobs / t.n, kMN256TailMaxSplit) : 0;
  if (!a.tail || t.split < 2) {  // nothing to gain: the tiles stay whole
    t.base = total;
    t.n = t.split = 0;
  }
  return t;
}

// Region and share-local index of tail tile k (rank base + k).
__device__ __forceinline__ void mn256_tail_tile(const MN256Tail& t, int k, int& ri, int& local) {
  const int rank = t.base + k;
  ri = rank < t.before[1] ? 0 : rank < t.before[2] ? 1 : 2;
  local = rank - (ri == 0 ? 0 : ri == 1 ? t.before[1] : t.before[2]);
}

// The k range of chunk c of n over K (in whole 64-wide units, so both ring
// depths cut at the same k): steps [s0, s0 + ns) of a BK-deep ring.
template <int BK>
__device__ __forceinline__ void mn256_chunk_steps(int K, int c, int n, int& s0, int& ns) {
  const int u = K / 64;
  const int u0 = (int)((int64_t)u * c / n), u1 = (int)((int64_t)u * (c + 1) / n);
  s0 = u0 * (64 / BK);
  ns = (u1 - u0) * (64 / BK);
}

// --------------------------------------------------------------------- GEMM-MN
// NFN = 2: tiles of 128 weight rows (64 gate/up columns or 128 plain ones), for
// narrow groups (wide_mn256_half) and few tiles (wide_mn256_fit).
// DOUBLE: the region's tiles are counted in 128-column ones (one region).
template <bool SWIGLU, int BK, bool BUF, int NFN, bool DOUBLE = false>
__device__ __forceinline__ void mn256_run(const MN256Args& a, uint16_t* smem) {
  static_assert(BK == t256::BK, "64-deep ring");
  using Rg = RingN<NFN>;
  constexpr int S = Rg::SLOTS, SB = Rg::BSLOTS;
  constexpr int BNO = (SWIGLU ? 32 : 64) * NFN;  // output columns per tile
  constexpr int WROWS = BNO;                     // rows of one weight panel
  const uint16_t* zero = g_zero_blk;

  // Workgroups are dealt round-robin to the 8 XCDs.  Each region's tiles
  // (padded to a multiple of 8) are cut into 8 contiguous shares and XCD x
  // runs share x of every region in turn: a masked region whose tail tiles
  // are mostly empty then loads the XCDs as evenly as the dense regions
  // beside it (one contiguous range per XCD over all regions left the XCDs
  // holding K and V with half again the work of the others).
  const int xcd = blockIdx.x % 8;
  int local = blockIdx.x / 8;
  int ri = 0, job = -1;   // region; tail job of a tail block
  int chunk = 0, nchunks = 1;
  if (const int shares = mn256_shares<BNO>(a); NFN == 4 && local >= shares) {  // one of the 32 tail blocks per XCD
    job = local - shares;
    const MN256Tail t = mn256_tail<BNO>(a, xcd);
    if (job >= t.n * t.split) return;
    chunk = job % t.split;
    nchunks = t.split;
    mn256_tail_tile(t, job / t.split, ri, local);
  } else {
    ri = 0;
    if (a.n_regions > 1 && local >= mn256_region_share<BNO>(a, a.reg[0])) {
      local -= mn256_region_share<BNO>(a, a.reg[0]);
      ri = 1;
      if (a.n_regions > 2 && local >= mn256_region_share<BNO>(a, a.reg[1])) {
        local -= mn256_region_share<BNO>(a, a.reg[1]);
        ri = 2;
      }
    }
    if (a.tail) {  // a tile of the XCD's last partial round is left to the tail blocks
      const MN256Tail t = mn256_tail<BNO>(a, xcd);
      const int real = ri == 0 ? t.real[0] : ri == 1 ? t.real[1] : t.real[2];  // no dynamic
      const int before = ri == 0 ? 0 : ri == 1 ? t.before[1] : t.before[2];   // indexing
      if (local < real && before + local >= t.base) return;
    }
  }
  MN256Region R = ri == 0 ? a.reg[0] : ri == 1 ? a.reg[1] : a.reg[2];
  if (DOUBLE) R.tiles *= 2;
  if (!mn256_mblocked<BNO>(a, R) && xcd * mn256_share(R.tiles) + local >= R.tiles) return;  // padding
  int g, nt_in, m_tile;
  mn256_coords<BNO, DOUBLE>(a, R, xcd, local, g, m_tile, nt_in);
  if (m_tile >= a.m_tiles) return;  // padding
  const int n0 = g * R.gw + nt_in * BNO;
  const int64_t M = a.M;
  const int K = a.K;
  const bool sorted = R.masked == kMN256Sorted;
  const int32_t* rows = sorted ? a.idx + (int64_t)g * M : nullptr;
  const int64_t cnt = sorted ? (int64_t)a.cnt[g] : M;
  const int64_t m0 = (int64_t)m_tile * BM;
  const int tid = threadIdx.x;

  // Token-order region: thread r < 256 holds row r's mask bits over the
  // tile's groups (bit i: group n0 / mask_G + i), for the epilogue.
  const bool tok_order = R.masked == kMN256TokenOrder;
  uint32_t rbits = 0;
  bool empty = m0 >= cnt;  // l = 0: the whole tile is inactive for group g
  if (tok_order) {
    const int gpt = BNO / a.mask_G;
    if (tid < BM && m0 + tid < M) {
      const uint8_t* mr = a.mask + (m0 + tid) * a.mask_ng + n0 / a.mask_G;
      for (int i = 0; i < gpt; ++i) rbits |= (uint32_t)(mr[i] != 0) << i;
    }
    // l = 0: no (row, group) of the tile is active.  (The flag lives in the
    // ring's LDS, not yet in use: a block-wide vote would take static LDS,
    // which the five-stage ring leaves none of.)
    int* flag = reinterpret_cast<int*>(smem);
    if (tid == 0) *flag = 0;
    __syncthreads();
    if (rbits) *flag = 1;
    __syncthreads();
    empty = *flag == 0;
    __syncthreads();  // before the ring's loads overwrite the flag
  }

  if (empty) {
    if (R.skip_zero) return;
    constexpr int CH = BNO / 8;
    int my_row = -1;
    if (tid < BM && m0 + tid < M) my_row = rows ? rows[m0 + tid] : (int)(m0 + tid);
    const int* map = stage_row_map(smem, my_row);
#pragma unroll 4
    for (int i = tid; i < BM * CH; i += NT) {
      const int t = map[i / CH];
      if (t >= 0) stg16(R.out + (int64_t)t * R.ldo + n0 + (i % CH) * 8, u32x4{0, 0, 0, 0});
    }
    return;
  }

  // Sources of the lane's load slots.  l = 1: rows past the active prefix
  // read zeros.  Under SwiGLU waves 0 and 1 load gate rows, 2 and 3 up rows.
  const uint16_t* wpanel = uniform_ptr((SWIGLU && wave_id() >= 2 ? R.w1 : R.w0) + (int64_t)n0 * K);
  const bufview_t va = buf_view(uniform_ptr(a.x), BUF ? (uint32_t)(M * K * 2) : 0u);
  const bufview_t vb = buf_view(wpanel, BUF ? (uint32_t)(WROWS * K * 2) : 0u);
  uint32_t aoff[S], boff[SB];
  const uint16_t* abase[S];
  const uint16_t* bbase[SB];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int rr = Rg::slot_row(j);
    const int c8 = Rg::slot_chunk(j) * 8;
    const int64_t p = m0 + rr;
    const int64_t arow = p < cnt ? (rows ? (int64_t)rows[p] : p) : -1;
    if (BUF) aoff[j] = arow >= 0 ? (uint32_t)((arow * K + c8) * 2) : kOffDead;
    else abase[j] = arow >= 0 ? a.x + arow * K + c8 : nullptr;
  }
#pragma unroll
  for (int j = 0; j < SB; ++j) {
    const int64_t brow = Rg::slot_row(j, SB) & (WROWS - 1);
    const int c8 = Rg::slot_chunk(j, SB) * 8;
    if (BUF) boff[j] = (uint32_t)((brow * K + c8) * 2);
    else bbase[j] = wpanel + brow * K + c8;
  }
  // B fragments of the wave: SwiGLU pairs gate column c (the tile's first half
  // of B rows) with up column c (the second half), so a wave takes 16 NFN gate
  // rows (the first NFN / 2 fragments) and the same up rows (the others)
  const int wn = wave_id() & 1;
  constexpr int BL = SWIGLU ? 1 : 0;
  int bb[NFN];
#pragma unroll
  for (int fn = 0; fn < NFN; ++fn) bb[fn] = wn * (SWIGLU ? 16 : 32) * NFN + bfrag_off<BL, NFN>(fn);

  f32x16 acc[4][NFN];
  zero_acc(acc);
  // A tail chunk runs its share of the k steps.  (Only Q/K/V launches have any,
  // but gate/up keeps the test: with s0 a constant the compiler's k loop ran
  // 10-20% slower.)
  int s0 = 0, ns = K / BK;
  if (job >= 0) mn256_chunk_steps<BK>(K, chunk, nchunks, s0, ns);
  auto koff = [&](int s) { return (s0 + s) * BK; };
  auto lda = [&](uint16_t* st, int k0, int j) {
    if (BUF) Rg::issue_buf(st, va, aoff[j], 2u * k0, j);
    else Rg::issue_ptr(st, abase[j] ? abase[j] + k0 : zero, j);
  };
  auto ldb = [&](uint16_t* st, int k0, int j) {
    if (BUF) Rg::issue_buf(st, vb, boff[j], 2u * k0, j, SB);
    else Rg::issue_ptr(st, bbase[j] + k0, j, SB);
  };
  int my_row = -1;
  if (job < 0 && tid < BM && m0 + tid < M) my_row = rows ? rows[m0 + tid] : (int)(m0 + tid);
  // l = 2: fragments wholly past the active prefix issue no MFMA
  run_tile<Rg, BL>(smem, ns, koff, lda, ldb, bb, cnt - m0, acc);
  const int col = acc_col();

  if (NFN == 4 && job >= 0) {  // tail chunk: fp32 partial tile [256 rows][256 B-tile rows]
    float* P = a.tail_ws + ((int64_t)xcd * kMN256TailJobs + job) * (BM * BN);
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = acc_row(fm, i);
        if (m0 + r >= cnt) continue;  // the finishing kernel does not read rows past the active ones
#pragma unroll
        for (int fn = 0; fn < NFN; ++fn) P[r * BN + bb[fn] + col] = acc[fm][fn][i];
      }
    return;
  }

  // Epilogue: rows back to token order; rows past cnt hold +0 accumulators.
  // A token-order region stores +0 where the row's group is inactive.  The
  // bf16 tile goes through the idle ring LDS (after the row map), rows
  // padded by 16 bytes, so that each lane then stores whole 16-byte pieces of
  // an output row: 8 times fewer store instructions than a 2-byte store per
  // accumulator, which is how the MFMA layout holds them (those stores cost
  // gate/up 3%; staged, gate/up is 1.5% faster).
  const int* map = stage_row_map(smem, my_row, (int)rbits);
  const int gsh = tok_order ? __builtin_ctz(a.mask_G) : 0;
  constexpr int NO = SWIGLU ? NFN / 2 : NFN;  // output fragments of the wave
  constexpr int PITCH = BNO + 8;      // bf16 per staged row
  static_assert(2 * BM * (int)sizeof(int) + BM * PITCH * 2 <= Rg::LDS, "row map and staged tile fit the ring");
  uint16_t* ot = smem + 2 * BM * (int)(sizeof(int) / sizeof(uint16_t));
#pragma unroll
  for (int fm = 0; fm < 4; ++fm) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = acc_row(fm, i);
      const int rb = tok_order ? map[BM + r] : 0;
#pragma unroll
      for (int fn = 0; fn < NO; ++fn) {
        const int c = bb[fn] + col;  // output column in the tile
        const bool on = !tok_order || ((rb >> (c >> gsh)) & 1);
        const float v = SWIGLU ? silu(acc[fm][fn][i]) * acc[fm][fn + NFN / 2][i] : acc[fm][fn][i];
        ot[r * PITCH + c] = f32_to_bf16_hw(on ? v : 0.f);
      }
    }
  }
  __syncthreads();
  constexpr int CPR = BNO / 8;  // 16-byte pieces per output row
#pragma unroll 4
  for (int q = tid; q < BM * CPR; q += NT) {
    const int r = q / CPR, c8 = q % CPR;
    const int t = map[r];
    if (t >= 0)
      stg16(R.out + (int64_t)t * R.ldo + n0 + c8 * 8, *reinterpret_cast<const u32x4*>(ot + r * PITCH + c8 * 8));
  }
}

template <bool SWIGLU, int BK, bool BUF>
__global__ __launch_bounds__(NT, 1) void wide_mn256(MN256Args a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  mn256_run<SWIGLU, BK, BUF, 4>(a, smem);
}

// Groups of half a tile: gate/up groups of 64 channels, Q groups of 128
// columns (K and V then run 128-wide too).  These ran on the 128 x 128 kernel
// of gemm_mn.hip (operands staged through registers, half the MFMAs per loaded
// byte).  Llama-3-8B widths, groups of 64: gate/up at 1000 tokens and keep 0.25
// 212 -> 110 us, at 4096 and 0.75 1131 -> 696; Q/K/V in groups of 128 at 777
// tokens 93 -> 55 us, at 8192 566 -> 365.
template <bool SWIGLU>
__global__ __launch_bounds__(NT, 1) void wide_mn256_half(MN256Args a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  mn256_run<SWIGLU, 64, true, 2>(a, smem);
}

// Gate/up with few tiles.  A tile of a short prompt is bound by streaming its
// weight panel through one CU (25-30 GB/s from beyond L2: the outstanding
// misses of a CU), so where the real 128-column tiles leave half of the CUs
// idle, twice as many 64-column ones (two B fragments per wave, four B
// stages) stream the same panels on twice the CUs; with more tiles than that
// they would only take a second round (450 tokens, all active: 101 us whole,
// 127 narrow).  How many tiles are real is known on the device only: every
// workgroup counts them.  Llama-3-8B widths, keep 0.5: 100 tokens 84 -> 59 us,
// 300 tokens 105 -> 71; d_model 1024, d_ff 4096, 1000 tokens 36 -> 23.
__global__ __launch_bounds__(NT, 1) void wide_mn256_fit(MN256Args a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const MN256Region& R = a.reg[0];
  bool narrow = true;  // (token-order regions: the host checks)
  if (R.masked == kMN256Sorted) {
    int* sum = reinterpret_cast<int*>(smem);
    if (threadIdx.x == 0) *sum = 0;
    __syncthreads();
    int n = 0;
    for (int g = threadIdx.x; g < R.ldo / R.gw; g += NT) n += (a.cnt[g] + BM - 1) / BM;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o);
    if (lane_id() == 0) atomicAdd(sum, n);
    __syncthreads();
    narrow = __builtin_amdgcn_readfirstlane(*sum) * (R.gw / 128) <= kMN256NarrowTiles;
    __syncthreads();  // before the ring's loads overwrite the sum
  }
  if (narrow) {
    mn256_run<true, 64, true, 2, true>(a, smem);
  } else if ((int)(blockIdx.x / 8) < mn256_shares<128>(a)) {
    mn256_run<true, 64, true, 4>(a, smem);
  }
}

// Finish the XCDs' tail tiles (Q/K/V): add each tile's chunks in order, then the
// mn256 epilogue (rows back to token order).  Workgroup
// (xcd, k, rb) takes kTailRows rows of tail tile k; each thread
// loads the chunks of its elements together (independent 16-byte loads) and adds
// them in chunk order.  Bound by the partial tiles' bytes per CU, so rows past
// the active ones are neither written nor read and a workgroup takes few rows
// (Llama-3-8B, 100 tokens: 20 us with 16 rows and 4-byte loads, now 12; 4 rows
// 14).
constexpr int kTailRows = 8;
constexpr int kTailTiles = kMN256TailJobs / 2;  // at most: two chunks each
__global__ __launch_bounds__(NT) void wide_mn256_tail(MN256Args a) {
  constexpr int PER = kTailRows * BN / NT / 4;  // runs of four columns per thread
  __shared__ int map[kTailRows];
  static_assert(kTailRows <= NT, "one thread per row for the row map");
  const int rb = blockIdx.x % (BM / kTailRows);
  const int k = (blockIdx.x / (BM / kTailRows)) % kTailTiles;
  const int xcd = blockIdx.x / (BM / kTailRows * kTailTiles);
  const MN256Tail t = mn256_tail<BN>(a, xcd);
  if (k >= t.n) return;
  int ri, local, g, m_tile, nt_in;
  mn256_tail_tile(t, k, ri, local);
  const MN256Region R = ri == 0 ? a.reg[0] : ri == 1 ? a.reg[1] : a.reg[2];
  mn256_coords<BN>(a, R, xcd, local, g, m_tile, nt_in);
  const int n0 = g * R.gw + nt_in * BN;
  const int32_t* rows = R.masked == kMN256Sorted ? a.idx + (int64_t)g * a.M : nullptr;
  const int64_t cnt = R.masked == kMN256Sorted ? (int64_t)a.cnt[g] : a.M;
  const int64_t p0 = (int64_t)m_tile * BM + rb * kTailRows;
  const int tid = threadIdx.x;
  if (tid < kTailRows) map[tid] = p0 + tid < a.M ? (rows ? rows[p0 + tid] : (int)(p0 + tid)) : -1;
  __syncthreads();
  const float* P = a.tail_ws + ((int64_t)xcd * kMN256TailJobs + k * t.split) * (BM * BN);
#pragma unroll
  for (int e = 0; e < PER; ++e) {  // four columns at a time
    const int i = (e * NT + tid) * 4;
    const int r = i / BN, c = i % BN;
    const int tok = map[r];
    if (tok < 0) continue;
    const bool live = p0 + r < cnt;  // past the active rows: +0, nothing was written
    const float* Pe = P + (rb * kTailRows + r) * BN + c;
    f32x4 v[kMN256TailMaxSplit];
#pragma unroll
    for (int q = 0; q < kMN256TailMaxSplit; ++q) {
      const bool on = live && q < t.split;
      v[q] = on ? *reinterpret_cast<const f32x4*>(Pe + (int64_t)q * (BM * BN)) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    f32x4 s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kMN256TailMaxSplit; ++q) s += v[q];  // chunk order
    // (token-order groups are at least 16 columns wide, so the four share one)
    const bool on = live && (R.masked != kMN256TokenOrder || a.mask[(int64_t)tok * a.mask_ng + (n0 + c) / a.mask_G] != 0);
    if (!on) s = f32x4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<uint2*>(R.out + (int64_t)tok * R.ldo + n0 + c) =
        uint2{pack_bf16x2_hw(s[0], s[1]), pack_bf16x2_hw(s[2], s[3])};
  }
}

// ----------------------------------------------------------- K-axis, dense-masked
// NWR: mask words (32 groups each) of the lane's slot rows held in registers
// for the whole k loop (1: up to 32 groups, 4: up to 128); 0 reads them from
// LDS at every step.
// Tile order of the dense-masked K axis.  One workgroup fits a CU, so the
// chip runs the tiles in rounds of 256.  When the column tiles divide a
// round (n_tiles even, 256 / n_tiles a multiple of 4), round r covers the
// m-tiles [r*mr, (r+1)*mr) (mr = 256 / n_tiles) times every column tile, and
// XCD x takes a block of mr/4 m-tiles x n_tiles/2 column tiles of it: a
// round's operands (mr row panels and all of W) then fit the last-level
// cache, and the tiles of one XCD share 12 k slices per step in its L2
// (Llama-3-8B down, 8192 x 4096 x 14336: 4-6% faster than walking the m-tiles
// of each XCD's contiguous range in turn, which needs 18 and, chip-wide,
// every row panel in each round).  Tiles past the last full round, and
// shapes the blocks do not fit, keep that m-major walk.
//
// The last round.  The tiles past the last full round (every tile, when the
// launch has fewer than 256) would leave CUs idle for a whole tile's time,
// and a lone tile is bound by one CU's memory latency: about 1.15 us per
// 64-deep step however few CUs are busy (32 tiles over K = 14336: 250 us).
// kd256_tail cuts those tiles along k into `split` chunks, one workgroup
// each, in as many chunks as pay for their partial sums, at most one round of
// workgroups; every chunk writes fp32 partial sums
// and wide_kd256_finish adds them in chunk order.  Chunks are fixed ranges of
// k, not shares of the tile's live groups, so a row's sum does not depend on
// which other rows share its tile.  Workgroups of one chunk and column tile
// (all row panels) sit next to each other on one XCD: its L2 reads that
// slice of the weights once, and with 8 chunks each XCD owns one slice of the
// activations too.  Llama-3-8B down, kernel plus finish: 300 tokens 253 ->
// 55 + 9 us, 1000 tokens 274 -> 105 + 14, 2048 tokens 284 -> 190 + 15; at
// 3000 tokens (192 of 256 tiles) a split would not fill the chip better.
// Mask tables of a dense-masked tile: the rows' mask bits, the groups some
// row uses (ascending), their union and count.  With NWR > 0 they live in the
// ring's LDS before its first load and move to registers (the ring then takes
// all of LDS); with NWR = 0 they sit past a ring of two A stages.
struct KdTables {
  uint32_t mbits[BM][kKd256MaxGroups / 32];
  uint16_t groups[kKd256MaxGroups];
  uint32_t uni[kKd256MaxGroups / 32];
  int n_live;
};
template <int NWR>
constexpr int kd256_lds() {
  return NWR == 0 ? RingKD<0>::LDS + (int)sizeof(KdTables) : RingKD<NWR>::LDS;
}
static_assert(kd256_lds<0>() <= LDS_MAX && (int)sizeof(KdTables) <= RingKD<4>::LDS, "tables fit");

// SPLIT: the launch has tiles cut along k (the chunk's step offset costs the
// uncut loop 0.9% where it is not needed).
template <int NWR, int BK, bool BUF, bool SPLIT>
__global__ __launch_bounds__(NT, 1) void wide_kd256(KArgs a) {
  static_assert(BK == t256::BK, "64-deep ring");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Rg = RingKD<NWR>;
  constexpr int S = Rg::SLOTS;
  KdTables& tb = *reinterpret_cast<KdTables*>(reinterpret_cast<char*>(smem) + (NWR == 0 ? Rg::LDS : 0));
  const uint16_t* zero = g_zero_blk;
  const int n_tiles = a.N / BN;
  int m_tile, n_tile, chunk = -1;
  if (!SPLIT || (int)blockIdx.x < a.tail_base) {
    kd256_coords(blockIdx.x, n_tiles, a.tail_base, m_tile, n_tile);
  } else {  // a chunk of a tile of the last round
    kd256_chunk(blockIdx.x - a.tail_base, (int)((a.M + BM - 1) / BM), n_tiles, a.tail_base, a.split, chunk, m_tile,
                n_tile);
  }
  const int64_t m0 = (int64_t)m_tile * BM;
  const int n0 = n_tile * BN;
  const int ng = a.K / a.G;
  const int nw = (ng + 31) / 32;
  const int tid = threadIdx.x;
  const int spg = a.G / BK;  // k steps per group
  // the workgroup's k steps [u0, u1) and the groups [g0, g1) they touch
  int u0 = 0, u1 = a.K / BK;
  if (SPLIT && chunk >= 0) kd256_steps(a.K, chunk, a.split, u0, u1);
  const int g0 = u0 / spg, g1 = (u1 + spg - 1) / spg;

  if (tid < nw) tb.uni[tid] = 0u;
  __syncthreads();
  // Tile row r is token m0 + r, or perm[m0 + r] when the rows are ordered by
  // mask pattern (rows that share groups then share the tile).
  auto token = [&](int64_t p) -> int64_t { return a.perm ? (int64_t)a.perm[p] : p; };
  for (int i = tid; i < BM * nw; i += NT) {
    const int r = i / nw, wd = i % nw;
    const int64_t p = m0 + r;
    const int64_t t = p < a.M ? token(p) : a.M;
    uint32_t bits = 0;
    // (words with no group of the workgroup's range are never used)
    if (t < a.M && wd * 32 < g1 && wd * 32 + 32 > g0)
      bits = mask_bits32(a.mask + t * ng + wd * 32, min(32, ng - wd * 32), ng);
    tb.mbits[r][wd] = bits;
    if (SPLIT && chunk >= 0) {  // only the range's groups count
      const int lo = max(g0 - wd * 32, 0), hi = min(g1 - wd * 32, 32);
      if (lo > 0) bits &= ~0u << min(lo, 31);
      if (hi < 32) bits &= hi > 0 ? ~0u >> (32 - hi) : 0u;
    }
    if (bits) atomicOr(&tb.uni[wd], bits);
  }
  __syncthreads();
  // groups some row of the tile uses, ascending: thread g places group g at
  // the count of union bits below it (no serial pass over the union)
  for (int gi = tid; gi < nw * 32; gi += NT) {
    const int wd = gi >> 5, b = gi & 31;
    int pos = __builtin_popcount(tb.uni[wd] & ((1u << b) - 1u));
    for (int i = 0; i < wd; ++i) pos += __builtin_popcount(tb.uni[i]);
    if ((tb.uni[wd] >> b) & 1u) tb.groups[pos] = (uint16_t)gi;
    if (gi == 0) {
      int n = 0;
      for (int i = 0; i < nw; ++i) n += __builtin_popcount(tb.uni[i]);
      tb.n_live = n;
    }
  }
  __syncthreads();
  // Steps run over the live groups; a chunk that starts or ends inside a
  // group takes that group's part only.
  const int n_live = __builtin_amdgcn_readfirstlane(tb.n_live);
  int sbeg = 0, nsteps = n_live * spg;
  if (SPLIT && chunk >= 0 && n_live > 0) {
    const int gf = __builtin_amdgcn_readfirstlane((int)tb.groups[0]);
    const int gl = __builtin_amdgcn_readfirstlane((int)tb.groups[n_live - 1]);
    sbeg = max(0, u0 - gf * spg);
    nsteps -= sbeg + max(0, (gl + 1) * spg - u1);
  }

  int srow[S];
  const uint16_t* wpanel = uniform_ptr(a.w + (int64_t)n0 * a.K);
  const bufview_t va = buf_view(uniform_ptr(a.a), BUF ? (uint32_t)(a.M * a.K * 2) : 0u);
  const bufview_t vb = buf_view(wpanel, BUF ? (uint32_t)(BN * a.K * 2) : 0u);
  uint32_t aoff[S], boff[S];
  const uint16_t* abase[S];
  const uint16_t* bbase[S];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int rr = Rg::slot_row(j);
    const int c8 = Rg::slot_chunk(j) * 8;
    const int64_t p = m0 + rr;
    const int64_t arow = p < a.M ? token(p) : -1;
    srow[j] = rr;
    if (BUF) {
      aoff[j] = arow >= 0 ? (uint32_t)((arow * a.K + c8) * 2) : kOffDead;
      boff[j] = (uint32_t)(((int64_t)rr * a.K + c8) * 2);
    } else {
      abase[j] = arow >= 0 ? a.a + arow * a.K + c8 : nullptr;
      bbase[j] = wpanel + (int64_t)rr * a.K + c8;
    }
  }
  const int lane = lane_id(), wn = wave_id() & 1;
  int bb[4];
#pragma unroll
  for (int fn = 0; fn < 4; ++fn) bb[fn] = wn * 128 + bfrag_off<0>(fn);

  f32x16 acc[4][4];
  zero_acc(acc);
  // Every step needs, per slot row, one bit of its mask row.  Reading them
  // from LDS at each step put several dependent LDS round trips in front of
  // the step's loads; with NWR > 0 the rows' mask words sit in registers,
  // inverted (rows past M hold zero words, all ones inverted, so their
  // blocks read as zeros), and so does the union's group list: lane l holds
  // groups l and 64 + l, and a step takes its group with a readlane.
  // (words past the row's last group are never selected: any value will do)
  uint64_t nlo[S], nhi[S];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    nlo[j] = nhi[j] = ~0ull;
    if (NWR >= 1) nlo[j] = ~(uint64_t)tb.mbits[srow[j]][0];
    if (NWR >= 4) {
      nlo[j] = ~((uint64_t)tb.mbits[srow[j]][0] | (uint64_t)tb.mbits[srow[j]][1] << 32);
      nhi[j] = ~((uint64_t)tb.mbits[srow[j]][2] | (uint64_t)tb.mbits[srow[j]][3] << 32);
    }
  }
  const int glo = NWR >= 1 ? tb.groups[lane] : 0;
  const int ghi = NWR >= 4 ? tb.groups[64 + lane] : 0;
  if (NWR > 0) __syncthreads();  // the ring's first loads overwrite the tables
  auto group = [&](int gi) -> int {  // gi-th group of the tile's union
    if (NWR == 1) return __builtin_amdgcn_readlane(glo, gi);
    if (NWR == 4) {  // both reads and a scalar select: no branch in the k loop
      const int lo = __builtin_amdgcn_readlane(glo, gi & 63), hi = __builtin_amdgcn_readlane(ghi, gi & 63);
      return gi < 64 ? lo : hi;
    }
    return __builtin_amdgcn_readfirstlane(tb.groups[gi]);  // one LDS word, the same for every lane
  };
  const int lg = __builtin_ctz(a.G), lsp = lg - 6;  // G is a power of two, at least BK
  auto koff = [&](int s) {
    if (SPLIT) s += sbeg;
    const int gi = s >> lsp;
    return group(gi) * a.G + (s & (spg - 1)) * BK;
  };
  // Inactive (t, g) blocks are never read.  Bit 31 of `dead` is set for
  // them: the inverted mask bit shifted up to bit 31 (one 64-bit shift by a
  // uniform amount) and merged into the row's view offset.  A row's offset
  // plus any step's k offset is a byte inside the view, below 2^31, so with
  // bit 31 added the sum is past the view and below 2^32 (no wrap).  Four
  // vector instructions per load where a compare and a select took six.
  auto lda = [&](uint16_t* st, int k0, int j) {
    const int gg = k0 >> lg;
    uint32_t dead;
    if (NWR == 0)
      dead = (tb.mbits[srow[j]][gg >> 5] >> (gg & 31)) & 1u ? 0u : kOffDead;
    else if (NWR == 1)
      dead = (uint32_t)nlo[j] << (31 - gg);
    else
      dead = (uint32_t)(((gg < 64 ? nlo[j] : nhi[j]) << (63 - (gg & 63))) >> 32);
    dead &= kOffDead;
    if (BUF) Rg::issue_buf(st, va, dead | aoff[j], 2u * k0, j);
    else Rg::issue_ptr(st, dead ? zero : abase[j] + k0, j);
  };
  auto ldb = [&](uint16_t* st, int k0, int j) {
    if (BUF) Rg::issue_buf(st, vb, boff[j], 2u * k0, j);
    else Rg::issue_ptr(st, bbase[j] + k0, j);
  };
  int my_row = -1;
  if (tid < BM && m0 + tid < a.M) my_row = (int)token(m0 + tid);
  run_tile<Rg, 0>(smem, nsteps, koff, lda, ldb, bb, a.M - m0, acc);

  const int col = acc_col();
  if (SPLIT && chunk >= 0) {  // fp32 partial sums, rows in tile order
    const int64_t p0 = (int64_t)(a.tail_base / n_tiles) * BM, rows = a.M - p0;
    float* P = a.part + ((int64_t)chunk * rows + (m0 - p0)) * a.N + n0 + col;
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = acc_row(fm, i);
        if (m0 + r >= a.M) continue;
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) P[(int64_t)r * a.N + bb[fn]] = acc[fm][fn][i];
      }
    return;
  }
  const int* map = stage_row_map(smem, my_row);
#pragma unroll
  for (int fm = 0; fm < 4; ++fm)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int t = map[acc_row(fm, i)];
      if (t < 0) continue;
      uint16_t* o = a.y + (int64_t)t * a.N + n0 + col;
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) o[bb[fn]] = f32_to_bf16_hw(acc[fm][fn][i]);
    }
}

// y rows [m0, M) (through the pattern order) = the chunks' partial sums added
// in chunk order; four columns per thread.
__global__ __launch_bounds__(NT) void wide_kd256_finish(const float* __restrict__ part, int split, int64_t m0,
                                                        int64_t rows, int N, const int32_t* __restrict__ perm,
                                                        uint16_t* __restrict__ y) {
  const int64_t n = rows * N, i = ((int64_t)blockIdx.x * NT + threadIdx.x) * 4;
  if (i >= n) return;
  f32x4 s = *reinterpret_cast<const f32x4*>(part + i);
#pragma unroll 8
  for (int q = 1; q < split; ++q) s += *reinterpret_cast<const f32x4*>(part + q * n + i);
  const int64_t p = m0 + i / N;
  const int64_t t = perm ? (int64_t)perm[p] : p;
  *reinterpret_cast<uint2*>(y + t * N + i % N) = uint2{pack_bf16x2_hw(s[0], s[1]), pack_bf16x2_hw(s[2], s[3])};
}

// -------------------------------------------------------------- K-axis, scatter
// One workgroup owns (sorted-position tile, 256 output columns, a run of
// a.pack K-groups) and runs the groups in turn, each with its own pipeline
// prologue and accumulator (Appendix B, Algorithm 3 and its outer loop that
// packs K-groups into one CTA).  When the column tiles divide among the 8
// XCDs, workgroup ids are dealt so that every workgroup adding into a column
// slab runs on the same XCD.
template <int BK, bool BUF>
__global__ __launch_bounds__(NT, 1) void wide_ks256(KArgs a) {
  static_assert(BK == t256::BK, "64-deep ring");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  using Rg = RingMN;
  constexpr int S = Rg::SLOTS;
  const uint16_t* zero = g_zero_blk;
  const int n_tiles = a.N / BN;
  const int m_tiles = (int)((a.M + BM - 1) / BM);
  const int ng = a.K / a.G;
  const int n_splits = (ng + a.pack - 1) / a.pack;
  int n_tile, m_tile, split;
  if (n_tiles % 8 == 0) {  // column slab of the workgroup's XCD (dispatch is round-robin over XCDs)
    const int xcd = blockIdx.x % 8, local = blockIdx.x / 8, per = n_tiles / 8;
    n_tile = xcd * per + local % per;
    m_tile = (local / per) % m_tiles;
    split = local / per / m_tiles;
  } else {
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    n_tile = tile % n_tiles;
    m_tile = (tile / n_tiles) % m_tiles;
    split = tile / (n_tiles * m_tiles);
  }
  if (split >= n_splits) return;
  const int g_end = min(ng, (split + 1) * a.pack);
  const int64_t m0 = (int64_t)m_tile * BM;
  const int n0 = n_tile * BN;
  const int wn = wave_id() & 1;
  int bb[4];
#pragma unroll
  for (int fn = 0; fn < 4; ++fn) bb[fn] = wn * 128 + bfrag_off<0>(fn);
  const int col = acc_col();
  const int* map = reinterpret_cast<const int*>(smem);
  const uint16_t* wpanel = uniform_ptr(a.w + (int64_t)n0 * a.K);
  const bufview_t va = buf_view(uniform_ptr(a.a), BUF ? (uint32_t)(a.M * a.K * 2) : 0u);
  const bufview_t vb = buf_view(wpanel, BUF ? (uint32_t)(BN * a.K * 2) : 0u);
  for (int g = split * a.pack; g < g_end; ++g) {
    const int64_t cnt = a.cnt[g];
    if (m0 >= cnt) continue;  // l = 0 for this group
    const int32_t* rows = a.idx + (int64_t)g * a.M;
    uint32_t aoff[S], boff[S];
    const uint16_t* abase[S];
    const uint16_t* bbase[S];
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int rr = Rg::slot_row(j);
      const int c8 = Rg::slot_chunk(j) * 8;
      const int64_t p = m0 + rr;
      const int64_t arow = p < cnt ? (int64_t)rows[p] : -1;  // l = 1
      if (BUF) {
        aoff[j] = arow >= 0 ? (uint32_t)((arow * a.K + c8) * 2) : kOffDead;
        boff[j] = (uint32_t)(((int64_t)rr * a.K + c8) * 2);
      } else {
        abase[j] = arow >= 0 ? a.a + arow * a.K + c8 : nullptr;
        bbase[j] = wpanel + (int64_t)rr * a.K + c8;
      }
    }
    f32x16 acc[4][4];
    zero_acc(acc);
    const int kbeg = g * a.G;
    auto koff = [&](int s) { return kbeg + s * BK; };
    auto lda = [&](uint16_t* st, int k0, int j) {
      if (BUF) Rg::issue_buf(st, va, aoff[j], 2u * k0, j);
      else Rg::issue_ptr(st, abase[j] ? abase[j] + k0 : zero, j);
    };
    auto ldb = [&](uint16_t* st, int k0, int j) {
      if (BUF) Rg::issue_buf(st, vb, boff[j], 2u * k0, j);
      else Rg::issue_ptr(st, bbase[j] + k0, j);
    };
    int my_row = -1;
    if ((int)threadIdx.x < BM && m0 + (int)threadIdx.x < cnt) my_row = rows[m0 + threadIdx.x];
    __syncthreads();  // the previous group's epilogue is done with the row map in the ring
    run_tile<Rg, 0>(smem, a.G / BK, koff, lda, ldb, bb, cnt - m0, acc);  // l = 2: dead fragments skipped
    stage_row_map(smem, my_row);
#pragma unroll
    for (int fm = 0; fm < 4; ++fm) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int t = map[acc_row(fm, i)];
        if (t < 0) continue;
        float* o = a.acc32 + (int64_t)t * a.N + n0 + col;
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) unsafeAtomicAdd(o + bb[fn], acc[fm][fn][i]);
      }
    }
  }
}

// ------------------------------------------------------------------ launchers
namespace {
template <class F>
hipError_t allow_big_lds(F* f, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(f),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// Raise the dynamic-LDS limit of one kernel instance once per process.
template <auto Kern, int Bytes>
hipError_t prepare() {
  static const hipError_t e = allow_big_lds(Kern, Bytes);
  return e;
}
}  // namespace

#define WIDE_RING_LAUNCH(NAME, KERN, LDSB, GRID, STREAM, ARGS)                                    \
  do {                                                                                            \
    hipError_t e_ = prepare<KERN, LDSB>();                                                        \
    if (e_ != hipSuccess) return e_;                                                              \
    WIDE_LAUNCH_NAMED(NAME "/bk64", (KERN), dim3(GRID), dim3(NT), LDSB, STREAM, ARGS);            \
  } while (0)

// Buffer-view sources when the token-row operand and a tile's weight panel
// (at most BN rows) each fit a view (2 GB); the same kernels on 64-bit
// addresses beyond.
bool views_fit(int64_t rows, int K) { return std::max<int64_t>(rows, BN) * (int64_t)K * 2 <= kBufViewMax; }

// Gate/up launches that wide_mn256_fit runs.  Sorted rows: 128-column tile
// slots (real or not) such that at least a quarter of the tokens active per
// group could fit kMN256NarrowTiles.  Token order: every tile is real.
static bool mn256_fit(const MN256Args& a) {
  const MN256Region& R = a.reg[0];
  return a.n_regions == 1 && views_fit(a.M, a.K) &&
         (R.masked == kMN256Sorted ? R.tiles <= 4 * kMN256NarrowTiles && R.gw % 128 == 0 && R.ldo % R.gw == 0
                                   : R.masked == kMN256TokenOrder && R.tiles <= kMN256NarrowTiles);
}

bool mn256_half_ok(int64_t M, int K) { return views_fit(M, K); }

hipError_t launch_mn256_half(const MN256Args& a, bool swiglu, hipStream_t s) {
  const int64_t total = 8 * (int64_t)(swiglu ? mn256_shares<64>(a) : mn256_shares<128>(a));
  if (total == 0) return hipSuccess;
  if (!views_fit(a.M, a.K) || a.tail) return hipErrorInvalidValue;
  if (swiglu)
    WIDE_RING_LAUNCH("wide_mn256_half<true>", (wide_mn256_half<true>), RingN<2>::LDS, (unsigned)total, s, a);
  else
    WIDE_RING_LAUNCH("wide_mn256_half<false>", (wide_mn256_half<false>), RingN<2>::LDS, (unsigned)total, s, a);
  return hipGetLastError();
}

hipError_t launch_mn256(const MN256Args& a, bool swiglu, hipStream_t s) {
  int64_t total = 0;
  for (int i = 0; i < a.n_regions; ++i) total += a.reg[i].tiles;
  if (total == 0) return hipSuccess;
  if (swiglu && a.tail) return hipErrorInvalidValue;  // Q/K/V only
  total = 8 * (int64_t)(swiglu ? mn256_shares<128>(a) : mn256_shares<256>(a));
  if (swiglu && mn256_fit(a)) {
    MN256Region r = a.reg[0];
    r.tiles *= 2;
    total = std::max(total, 8 * (int64_t)mn256_region_share<64>(a, r));
    WIDE_RING_LAUNCH("wide_mn256<true>", (wide_mn256_fit), std::max(RingN<2>::LDS, RingMN::LDS), (unsigned)total, s, a);
    return hipGetLastError();
  }
  if (a.tail) total += 8 * kMN256TailJobs;  // the tail blocks of every XCD, dispatched last
  const bool buf = views_fit(a.M, a.K);
  if (swiglu && buf)
    WIDE_RING_LAUNCH("wide_mn256<true>", (wide_mn256<true, 64, true>), RingMN::LDS, (unsigned)total, s, a);
  else if (swiglu)
    WIDE_RING_LAUNCH("wide_mn256<true>", (wide_mn256<true, 64, false>), RingMN::LDS, (unsigned)total, s, a);
  else if (buf)
    WIDE_RING_LAUNCH("wide_mn256<false>", (wide_mn256<false, 64, true>), RingMN::LDS, (unsigned)total, s, a);
  else
    WIDE_RING_LAUNCH("wide_mn256<false>", (wide_mn256<false, 64, false>), RingMN::LDS, (unsigned)total, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.tail) return e;
  WIDE_LAUNCH(wide_mn256_tail, dim3(8 * kTailTiles * (BM / kTailRows)), dim3(NT), 0, s, a);
  return hipGetLastError();
}

bool mn256_tail_ok(const MN256Args& a) {
  for (int i = 0; i < a.n_regions; ++i) {
    const MN256Region& R = a.reg[i];
    if (R.masked != kMN256Sorted) continue;  // dense and token-order regions: every tile is real
    const int share = mn256_share(R.tiles), per_group = R.gw / BN * a.m_tiles;
    if (!(a.order && !a.mblock && R.gw / BN <= 4 && 8 * share == R.tiles && share % per_group == 0))
      return false;
  }
  return true;
}

static_assert(kKdTile == BM && kKdTile == BN && kKdStep == BK, "tile_order.h");
size_t kd256_part_floats(int64_t M, int N, int K, int ng) {
  const Kd256Tail t = kd256_tail(M, N, K, ng, SIZE_MAX);
  return t.split > 1 ? (size_t)t.split * (size_t)(M - t.m0) * (size_t)N : 0;
}

hipError_t launch_kd256(const KArgs& args, hipStream_t s) {
  KArgs a = args;
  const int64_t m_tiles = (a.M + BM - 1) / BM;
  const int64_t tiles = m_tiles * (a.N / BN);
  if (tiles == 0) return hipSuccess;
  if (a.split < 2) {
    a.tail_base = (int)tiles;
    a.split = 1;
  }
  const int64_t total = a.tail_base + (tiles - a.tail_base) * a.split;
  if (a.K / a.G > kKd256MaxGroups) return hipErrorInvalidValue;
  const int ng = a.K / a.G;
  const bool buf = views_fit(a.M, a.K);
#define WIDE_KD(NWR, BUF)                                                                                            \
  do {                                                                                                               \
    if (a.split > 1)                                                                                                 \
      WIDE_RING_LAUNCH("wide_kd256<" #NWR ">", (wide_kd256<NWR, 64, BUF, true>), kd256_lds<NWR>(), (unsigned)total, s, \
                       a);                                                                                           \
    else                                                                                                             \
      WIDE_RING_LAUNCH("wide_kd256<" #NWR ">", (wide_kd256<NWR, 64, BUF, false>), kd256_lds<NWR>(), (unsigned)total, s, \
                       a);                                                                                           \
  } while (0)
  if (ng <= 32 && buf) WIDE_KD(1, true);
  else if (ng <= 32) WIDE_KD(1, false);
  else if (ng <= 128 && buf) WIDE_KD(4, true);
  else if (ng <= 128) WIDE_KD(4, false);
  else if (buf) WIDE_KD(0, true);
  else WIDE_KD(0, false);
#undef WIDE_KD
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.split < 2) return e;
  const int64_t p0 = (int64_t)(a.tail_base / (a.N / BN)) * BM, rows = a.M - p0;
  WIDE_LAUNCH(wide_kd256_finish, dim3((unsigned)((rows * a.N / 4 + NT - 1) / NT)), dim3(NT), 0, s, a.part, a.split,
              p0, rows, a.N, a.perm, a.y);
  return hipGetLastError();
}

hipError_t launch_ks256(const KArgs& a, hipStream_t s) {
  const int64_t m_tiles = (a.M + BM - 1) / BM;
  const int pack = a.pack > 0 ? a.pack : 1;
  const int64_t splits = (a.K / a.G + pack - 1) / pack;
  const int64_t total = splits * m_tiles * (a.N / BN);
  if (total == 0) return hipSuccess;
  if (views_fit(a.M, a.K))
    WIDE_RING_LAUNCH("wide_ks256", (wide_ks256<64, true>), RingMN::LDS, (unsigned)total, s, a);
  else
    WIDE_RING_LAUNCH("wide_ks256", (wide_ks256<64, false>), RingMN::LDS, (unsigned)total, s, a);
  return hipGetLastError();
}

}  // namespace wide
