// fp32 masked projections on the fp32 matrix cores (no reduced precision).
//
// The fp32 data path keeps every value in fp32 end to end.
//   f32_nproj  out[t, n] = x_t . w[n] for active (t, group of n), else +0
//              (optionally the SwiGLU pair: silu(x_t . w0[n]) * (x_t . w1[n]));
//              a tile whose tokens are all inactive in its groups exits after
//              writing +0.  (WIDE Section 3.1, equations (1) and (3).)
//   f32_kproj  y[t, n] = sum over active groups g of t of
//              sum_{k in g} a[t, k] w[n, k]; inactive (t, g) blocks are not
//              read.  (Section 3.1 equations (2)-(3), the GEMM-K sum of
//              Appendix B.)
//
// A workgroup owns a tile of 16*F tokens x 16*F columns (F 1 or 2) and its 8
// waves share the reduction: each takes a contiguous run of the 16-deep k
// chunks, loads them straight into MFMA operands (lane l: row l % 16, four
// consecutive k from 4 * (l / 16); MFMA e of a chunk multiplies element e of
// the four, the same k on both sides) several chunks ahead, and the waves'
// partial tiles are added in LDS in wave order.  These calls are small (a
// 128-token, 512 x 1536 FFN is 0.3 GFLOP), so what bounds them is latency:
// the wave split shortens the serial chain by 8, nothing in the k loop waits
// on a barrier, and F is 2 only where enough tiles of 32 remain (frags()).  Against the
// vector-ALU kernels this replaces (16 x 16 tiles staged through LDS, one
// serial k loop per workgroup): 128 tokens, d_model 512, d_ff 1536 in groups
// of 64, gate/up 45 -> 14 us, down 75 -> 10 us; 512 tokens, 1024 x 2048:
// 240 -> 69 and 168 -> 33 us.
#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "tile256.h"

namespace wide {

namespace {

constexpr int T = 16, KC = 16, NW = 8, NT = NW * kWave;

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Workgroup id -> tile id: each XCD (workgroups are dealt round-robin to the
// 8 XCDs) walks a contiguous range of tiles, so the tiles of one column run
// share its weight rows in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int id, int n) {
  const int q = n / 8, r = n % 8;
  const int xcd = id % 8, local = id / 8;
  return (xcd < r) ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
}

// Wave w's run [c0, c1) of n chunks.
__device__ __forceinline__ void wave_run(int n, int& c0, int& c1) {
  const int w = wave_id();
  c0 = (int)((int64_t)n * w / NW);
  c1 = (int)((int64_t)n * (w + 1) / NW);
}

// The lane's 16 bytes of row r of a tile whose rows start at `base`, K floats
// apart: k from `k`, or zeros.
__device__ __forceinline__ u32x4 row_ld(const float* base, int K, int r, int k, bool on) {
  return on ? ldg16(base + (int64_t)r * K + k) : u32x4{0, 0, 0, 0};
}

// acc[v][i][j] += A fragment i x B fragment j of weight v over chunks
// [c0, c1), D chunks in flight.  lda(c, i), ldw(v, c, j): the lane's 16 bytes
// of A fragment i, and of B fragment j of weight v, at chunk c (lda is called
// once per chunk, in order).
template <int NV, int F, int D, class LdA, class LdW>
__device__ __forceinline__ void k_loop(int c0, int c1, LdA lda, LdW ldw, f32x4 (&acc)[NV][F][F]) {
  struct Regs {
    u32x4 a[F], w[NV][F];
  };
  auto load = [&](int c, Regs& r) {
#pragma unroll
    for (int i = 0; i < F; ++i) r.a[i] = lda(c, i);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int j = 0; j < F; ++j) r.w[v][j] = ldw(v, c, j);
  };
  auto mma = [&](const Regs& r) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j)
            acc[v][i][j] = mfma_f32(__uint_as_float(r.a[i][e]), __uint_as_float(r.w[v][j][e]), acc[v][i][j]);
  };
  Regs rr[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (c0 + d < c1) load(c0 + d, rr[d]);
  for (int c = c0; c < c1; c += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (c + d < c1) {
        mma(rr[d]);
        if (c + d + D < c1) load(c + d + D, rr[d]);
      }
    }
  }
}

// The 8 waves' partial tiles added in wave order; out(row, col, sums) runs
// for every element of the tile.
template <int NV, int F, class Out>
__device__ __forceinline__ void reduce_tile(f32x4 (*red)[NW][kWave], const f32x4 (&acc)[NV][F][F], Out out) {
  const int w = wave_id(), lane = lane_id();
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) red[(v * F + i) * F + j][w][lane] = acc[v][i][j];
  __syncthreads();
  // Thread -> (fragment, accumulator element i, lane): 16 lanes share a row.
  for (int q = threadIdx.x; q < F * F * 4 * kWave; q += NT) {
    const int f = q / (4 * kWave), l = q % kWave, e = (q / kWave) % 4;
    float s[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      s[v] = 0.f;
#pragma unroll
      for (int p = 0; p < NW; ++p) s[v] += red[v * F * F + f][p][l][e];
    }
    out(f / F * T + (l >> 4) * 4 + e, f % F * T + (l & 15), s);
  }
}

}  // namespace

// BUF: 32 rows of either operand fit a buffer view (under 2^31 bytes) and a
// lane keeps 32-bit byte offsets; rows of 2^24 floats or more take 64-bit
// addresses.
template <bool SWIGLU, int F, bool BUF>
__global__ __launch_bounds__(NT) void wide_f32_nproj(F32NArgs a) {
  constexpr int NV = SWIGLU ? 2 : 1, TM = T * F;
  __shared__ f32x4 red[NV * F * F][NW][kWave];
  __shared__ uint8_t s_on[TM][F];  // row r runs the group of column fragment j
  __shared__ int any;
  const int m_tiles = (int)((a.M + TM - 1) / TM);
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t t0 = (int64_t)(tile % m_tiles) * TM;
  const int n0 = tile / m_tiles * TM;
  const int rows = (int)min((int64_t)TM, a.M - t0), cols = min(TM, a.N - n0);
  const int tid = threadIdx.x;
  if (tid == 0) any = a.mask == nullptr;
  __syncthreads();
  if (a.mask && tid < TM * F) {
    const int r = tid / F, j = tid % F;
    // (a fragment of 16 columns lies inside one group)
    const bool on = r < rows && j * T < cols && a.mask[(t0 + r) * a.n_groups + (n0 + j * T) / a.G] != 0;
    s_on[r][j] = on;
    if (on) any = 1;
  }
  __syncthreads();
  if (!any) {
    for (int q = tid; q < rows * cols; q += NT) a.out[(t0 + q / cols) * a.ldo + n0 + q % cols] = 0.f;
    return;
  }
  const uint32_t rb = (uint32_t)a.K * 4u;
  const float *xt = a.x + t0 * a.K, *wt[NV];
  wt[0] = a.w0 + (int64_t)n0 * a.K;
  if (SWIGLU) wt[NV - 1] = a.w1 + (int64_t)n0 * a.K;
  const bufview_t av = buf_view(xt, BUF ? (uint32_t)rows * rb : 0u);
  bufview_t wv[NV];
  wv[0] = buf_view(wt[0], BUF ? (uint32_t)cols * rb : 0u);
  if (SWIGLU) wv[NV - 1] = buf_view(wt[NV - 1], BUF ? (uint32_t)cols * rb : 0u);
  f32x4 acc[NV][F][F];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) acc[v][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int c0, c1;
  wave_run(a.K / KC, c0, c1);
  const int l16 = lane_id() & 15, k4 = lane_id() / 16 * 4;
  const uint32_t off = (uint32_t)l16 * rb + k4 * 4;  // within a fragment's chunk, both operands
  k_loop<NV, F, 4>(
      c0, c1,
      [&](int c, int i) {
        if constexpr (BUF) return buf_ld16(av, off + (uint32_t)i * T * rb + (uint32_t)c * (KC * 4));
        else return row_ld(xt, a.K, i * T + l16, c * KC + k4, i * T + l16 < rows);
      },
      [&](int v, int c, int j) {
        if constexpr (BUF) return buf_ld16s(wv[v], off, (uint32_t)j * T * rb + (uint32_t)c * (KC * 4));
        else return row_ld(wt[v], a.K, j * T + l16, c * KC + k4, j * T + l16 < cols);
      },
      acc);
  reduce_tile<NV, F>(red, acc, [&](int r, int c, const float (&s)[NV]) {
    if (r >= rows || c >= cols) return;
    const bool on = !a.mask || s_on[r][c / T];
    a.out[(t0 + r) * a.ldo + n0 + c] = on ? (SWIGLU ? silu(s[0]) * s[NV - 1] : s[0]) : 0.f;
  });
}

template <int F, bool BUF>
__global__ __launch_bounds__(NT) void wide_f32_kproj(F32KArgs a) {
  constexpr int TM = T * F, MAXG = 4096;
  __shared__ f32x4 red[F * F][NW][kWave];
  __shared__ uint64_t s_bits[TM][MAXG / 64];  // bit g: row r runs group g
  const int m_tiles = (int)((a.M + TM - 1) / TM);
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t t0 = (int64_t)(tile % m_tiles) * TM;
  const int n0 = tile / m_tiles * TM;
  const int rows = (int)min((int64_t)TM, a.M - t0), cols = min(TM, a.N - n0);
  const int w = wave_id(), lane = lane_id(), ng = a.n_groups;
  for (int s = 0; s * 64 < ng; ++s) {
    uint8_t m[TM / NW];
#pragma unroll
    for (int i = 0; i < TM / NW; ++i) {  // independent loads
      const int r = i * NW + w, g = s * 64 + lane;
      m[i] = a.mask[(t0 + min(r, rows - 1)) * ng + min(g, ng - 1)];
    }
#pragma unroll
    for (int i = 0; i < TM / NW; ++i) {
      const int r = i * NW + w;
      const uint64_t b = __ballot(m[i] != 0 && r < rows && s * 64 + lane < ng);
      if (lane == 0) s_bits[r][s] = b;
    }
  }
  __syncthreads();
  const uint32_t rb = (uint32_t)a.K * 4u;
  const float *at = a.a + t0 * a.K, *wt = a.w + (int64_t)n0 * a.K;
  const bufview_t av = buf_view(at, BUF ? (uint32_t)rows * rb : 0u), wv = buf_view(wt, BUF ? (uint32_t)cols * rb : 0u);
  f32x4 acc[1][F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[0][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int c0, c1;
  wave_run(a.K / KC, c0, c1);
  const int l16 = lane & 15, k4 = lane / 16 * 4;
  const uint32_t off = (uint32_t)l16 * rb + k4 * 4;  // within a fragment's chunk, both operands
  // a chunk lies inside one group; the chunks are asked for in order
  int g = c0 * KC / a.G, left = (g + 1) * a.G - c0 * KC;
  k_loop<1, F, 4>(
      c0, c1,
      [&](int c, int i) {
        const bool on = (s_bits[i * T + l16][g >> 6] >> (g & 63)) & 1u;
        if (i == F - 1 && (left -= KC) == 0) {
          ++g;
          left = a.G;
        }
        if constexpr (BUF) return buf_ld16(av, on ? off + (uint32_t)i * T * rb + (uint32_t)c * (KC * 4) : kOffNone);
        else return row_ld(at, a.K, i * T + l16, c * KC + k4, on);  // (rows past the tile's have no bit set)
      },
      [&](int, int c, int j) {
        if constexpr (BUF) return buf_ld16s(wv, off, (uint32_t)j * T * rb + (uint32_t)c * (KC * 4));
        else return row_ld(wt, a.K, j * T + l16, c * KC + k4, j * T + l16 < cols);
      },
      acc);
  reduce_tile<1, F>(red, acc, [&](int r, int c, const float (&s)[1]) {
    if (r < rows && c < cols) a.y[(t0 + r) * a.N + n0 + c] = s[0];
  });
}

namespace {
// 32 x 32 tiles read half the operand bytes per product of 16 x 16 ones but
// leave fewer workgroups: taken where they give every CU one, for gate/up
// (two products per tile) every second CU.  At 192 tiles of 32 (128 tokens, 512 x
// 1536) gate/up ran 14.0 us with them and 15.7 without; at 128 tiles (256
// tokens, 512 outputs) down ran 12.8 and 11.0 us.
int64_t tiles(int64_t M, int N, int tm) { return (M + tm - 1) / tm * ((N + tm - 1) / tm); }
int frags(int64_t M, int N, bool pair) { return tiles(M, N, 2 * T) >= (pair ? 128 : 256) ? 2 : 1; }
// Rows of which 32 do not fit a buffer view.
bool long_rows(int K) { return (int64_t)2 * T * K * 4 > t256::kBufViewMax; }
}  // namespace

hipError_t launch_f32_nproj(const F32NArgs& a, bool swiglu, hipStream_t s) {
  const bool lr = long_rows(a.K);
  const int f = lr ? 1 : frags(a.M, a.N, swiglu);
  const int64_t total = tiles(a.M, a.N, f * T);
  if (total == 0) return hipSuccess;
  const dim3 grid((unsigned)total), block(NT);
  if (swiglu && lr)
    WIDE_LAUNCH((wide_f32_nproj<true, 1, false>), grid, block, 0, s, a);
  else if (swiglu && f == 2)
    WIDE_LAUNCH((wide_f32_nproj<true, 2, true>), grid, block, 0, s, a);
  else if (swiglu)
    WIDE_LAUNCH((wide_f32_nproj<true, 1, true>), grid, block, 0, s, a);
  else if (lr)
    WIDE_LAUNCH((wide_f32_nproj<false, 1, false>), grid, block, 0, s, a);
  else if (f == 2)
    WIDE_LAUNCH((wide_f32_nproj<false, 2, true>), grid, block, 0, s, a);
  else
    WIDE_LAUNCH((wide_f32_nproj<false, 1, true>), grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_f32_kproj(const F32KArgs& a, hipStream_t s) {
  const bool lr = long_rows(a.K);
  const int f = lr ? 1 : frags(a.M, a.N, false);
  const int64_t total = tiles(a.M, a.N, f * T);
  if (total == 0) return hipSuccess;
  const dim3 grid((unsigned)total), block(NT);
  if (lr)
    WIDE_LAUNCH((wide_f32_kproj<1, false>), grid, block, 0, s, a);
  else if (f == 2)
    WIDE_LAUNCH((wide_f32_kproj<2, true>), grid, block, 0, s, a);
  else
    WIDE_LAUNCH((wide_f32_kproj<1, true>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace wide
