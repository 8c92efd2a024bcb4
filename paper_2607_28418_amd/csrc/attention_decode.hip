// Head-group masked attention at decode on gfx950 (WIDE Section 3.1,
// equations (1)-(2); Appendix B: for decoding the reorder is bypassed, the
// routing is checked per block, and the online softmax is split over the
// keys; Appendix C on GQA packing).
//
// One query token per sequence attends to the sequence's cached keys
// [0, kv_len).  Decode attention is bound by reading the KV cache, so the
// point of the mask is to read less of it.  The work is cut into segments,
// runs of keys of one (sequence, KV head) pair, that pack every query head of
// that KV head (GQA packing); a pair none of whose heads' groups is active for
// the token is not read (l = 0), so an inactive KV head of a token costs no HBM
// traffic.  Small calls cut every pair into equal chunks, one wave each, and an
// inactive pair's waves return at once; large ones list the active units first
// (the workgroup's waves meet at barriers there) and give every wave an equal
// run of them, which may cross from one pair into the next (list_units).
//
// Past the listing each wave runs alone, streaming its segments in 16-key units
// straight into registers with three units in flight
// (the bytes in flight per CU, not the arithmetic, set the rate here):
//   scores  S^T[16 keys][16 heads] = K Q^T: four v_mfma_f32_16x16x32_bf16,
//           K rows as the A operand (16 bytes of a row per lane), the packed
//           heads' q as the B operand (columns past the heads are zero);
//   softmax online per head column, in fp32;
//   P.V     on the vector ALUs in fp32: lane = (one of 4 keys of each group
//           of 4, 8 of the 128 dims); the probabilities and rescale factors
//           pass through a per-wave LDS scratch.
// Per (segment, head) the wave leaves (max, sum, unnormalised o) in the
// workspace; a second kernel merges a pair's segments (and writes +0 for
// inactive heads).
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "tile256.h"

namespace wide {
namespace {

constexpr int kHd = 128;
constexpr int kDT = 256;    // threads per workgroup: 4 independent waves
constexpr int kU = 16;      // keys per unit
constexpr int kDepth = 3;   // units in flight per wave

// Lanes of one wave exchange values through LDS: the fences tell the
// compiler that other lanes read what this lane wrote (and the reverse), so
// it neither forwards stale values nor moves accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct Unit {
  u32x4 k[4];  // lane: key row lane%16, dims 32s + 8*(lane/16) .. +8
  u32x4 v[4];  // lane: key 4i + lane/16, dims 8*(lane%16) .. +8
};

// Active query heads of (sequence b, KV head hkv): bit i = head hkv*qpk + i.
__device__ __forceinline__ uint32_t active_heads(const AttnDecArgs& a, int b, int hkv) {
  const uint8_t* mrow = a.mask + (int64_t)b * a.ng;
  uint32_t act = 0;
  for (int i = 0; i < a.qpk; ++i)
    if (mrow[(hkv * a.qpk + i) / a.hpg]) act |= 1u << i;
  return act;
}
__device__ __forceinline__ int seq_len(const AttnDecArgs& a, int b) {
  return a.kv_len ? min(a.kv_len[b], a.L) : a.L;
}

// Balanced split.  What a token reads depends on the mask and on its
// sequence's length, both known on the device only, so cutting every
// (sequence, KV head) pair into equal chunks leaves some CUs with several
// times the work of others.  Here every workgroup first lists the pairs'
// 16-key units (0 for a pair no head of which is active) as a prefix sum in
// LDS; with U units in all, wave i of a.waves (one round of resident waves)
// takes units [i q, (i + 1) q), q = max(ceil(U / waves), kMinUnits), which may
// cross from one pair into the next.  Each (wave, pair) segment leaves one
// partial result, in slot i + (active pairs before the pair); workgroup 0
// writes every pair's first slot and segment count for the merge.
// Ragged caches, 32 sequences of up to 8192 keys, half the KV heads active:
// kernel 91 -> 69 us; nothing ragged, all heads active: 201 -> 197.
constexpr int kMinUnits = 4;  // 64 keys

constexpr uint64_t kUnitBits = (1ull << 40) - 1;  // of a prefix: units; above them: active pairs

__device__ __forceinline__ void list_units(const AttnDecArgs& a, uint64_t* s_pre, uint64_t* s_sum) {
  const int tid = threadIdx.x, w = wave_id(), lane = lane_id();
  const int P = a.B * a.n_kv, per = (P + kDT - 1) / kDT;
  const int p0 = min(P, tid * per), p1 = min(P, p0 + per);
  uint64_t sum = 0;  // active pairs << 40 | units
  for (int p = p0; p < p1; ++p) {
    const int b = p / a.n_kv, h0 = (p - b * a.n_kv) * a.qpk;
    const uint8_t* mrow = a.mask + (int64_t)b * a.ng;
    const int g0 = h0 / a.hpg, g1 = (h0 + a.qpk - 1) / a.hpg;
    const int len = max(seq_len(a, b), 0);
    uint32_t on = mrow[g0];
    for (int g = g0 + 1; g <= g1; ++g) on |= mrow[g];
    const int n = on ? (len + kU - 1) / kU : 0;
    s_pre[p] = n;
    sum += (uint64_t)(n > 0) << 40 | (uint32_t)n;
  }
  uint64_t x = sum;  // inclusive scan over the wave, then over the waves
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint64_t y = __shfl_up((unsigned long long)x, d);
    if (lane >= d) x += y;
  }
  if (lane == kWave - 1) s_sum[w] = x;
  __syncthreads();
  uint64_t run = x - sum, all = 0;
#pragma unroll
  for (int i = 0; i < kDT / kWave; ++i) {
    if (i < w) run += s_sum[i];
    all += s_sum[i];
  }
  const int units = (int)(all & kUnitBits), q = max((units + a.waves - 1) / a.waves, kMinUnits);
  for (int p = p0; p < p1; ++p) {
    const int n = (int)s_pre[p], u = (int)(run & kUnitBits), rank = (int)(run >> 40);
    s_pre[p] = run;
    if (blockIdx.x == 0) {
      a.table[2 * p] = u / q + rank;
      a.table[2 * p + 1] = n > 0 ? (u + n - 1) / q - u / q + 1 : 0;
    }
    run += (uint64_t)(n > 0) << 40 | (uint32_t)n;
  }
  if (tid == 0) {
    s_pre[P] = all;
    s_sum[kDT / kWave] = (uint64_t)q;
  }
  __syncthreads();
}

// HMAX: the most query heads per KV head this instance serves (qpk <= HMAX);
// BAL: balanced split, else equal chunks.
template <int HMAX, bool BAL>
__global__ __launch_bounds__(kDT, HMAX <= 8 ? 2 : 1) void wide_attn_decode(AttnDecArgs a) {
  constexpr int HB = HMAX < 4 ? HMAX : 4;  // head columns per LDS read group
  __shared__ __attribute__((aligned(16))) float s_p[4][kU][16];  // per wave: p[key][head]
  __shared__ __attribute__((aligned(16))) float s_al[4][16];     // per wave: rescale per head
  extern __shared__ uint64_t s_pre[];  // balanced: units and active pairs before each pair
  __shared__ uint64_t s_sum[kDT / kWave + 1];
  const int w = wave_id(), lane = lane_id();
  int p, slot, j_begin, j_end, u_end = 0, wave = 0, rank = 0;
  auto pre = [&](int i) { return (int)(s_pre[i] & kUnitBits); };
  if constexpr (BAL) {
    list_units(a, s_pre, s_sum);
    const int P = a.B * a.n_kv, q = __builtin_amdgcn_readfirstlane((int)s_sum[kDT / kWave]);
    const int units = pre(P), nwg = (int)(((int64_t)units + 4 * q - 1) / (4 * q));
    if ((int)blockIdx.x >= nwg) return;
    // Workgroups with work take their waves' runs in order, neighbours on
    // different XCDs.  In a head-major cache whose sequences all have the same
    // length, a multiple of 1024 keys, that left an XCD always the same part of
    // every pair (32 x 8192 keys, every other KV head off: 116 us), so long
    // runs there go to each XCD in one piece (107; 113 in equal chunks, dealt
    // the same way).  Other lengths, and 16 sequences of 4096 (8 units a wave),
    // ran up to 4% slower that way, the token-major layout up to 8%.
    const bool by_xcd = a.head_major && !a.kv_len && a.L % 1024 == 0 && q >= 16;
    wave = (by_xcd ? xcd_remap(blockIdx.x, nwg) : (int)blockIdx.x) * 4 + w;
    const int64_t u0 = (int64_t)wave * q;
    if (u0 >= units) return;
    u_end = (int)min(u0 + q, (int64_t)units);
    // the pair of unit u0, the last one with at most u0 units before it: 64
    // candidates per step, one per lane
    int lo = 0, n = P;
    while (n > 1) {
      const int st = (n + kWave - 1) / kWave, i = lo + lane * st;
      const uint64_t le = __ballot(lane * st < n && pre(min(i, P)) <= (int)u0);
      const int k = 63 - __builtin_clzll(le);  // (lane 0's candidate always qualifies)
      n = min(st, n - k * st);
      lo += k * st;
    }
    p = __builtin_amdgcn_readfirstlane(lo);
    rank = __builtin_amdgcn_readfirstlane((int)(s_pre[p] >> 40));
    j_begin = (int)(u0 - pre(p)) * kU;
  } else {
    // Work items in (sequence, KV head, chunk) order, four per workgroup; each
    // XCD (workgroups are dealt round-robin to the 8 XCDs) takes a contiguous
    // range of them, i.e. whole sequences, so masks that switch whole KV heads
    // off still leave every XCD the same share of the work.
    const int64_t item = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * 4 + w;
    if (item >= (int64_t)a.B * a.n_kv * a.n_chunks) return;
    slot = (int)item;
    p = (int)(item / a.n_chunks);
    j_begin = (int)(item % a.n_chunks) * a.chunk;
  }
  for (;; ++p) {  // the wave's segments
    // Nothing of an inactive pair is loaded: where few heads are active, waves
    // cross long runs of them.  (An active one follows: units are left.)
    if (BAL)
      while (pre(p + 1) == pre(p)) ++p;
    const int b = p / a.n_kv, hkv = p - b * a.n_kv;
    const int len = seq_len(a, b);
    const uint32_t act = active_heads(a, b, hkv);
    if (BAL) {
      j_end = min(len, (u_end - pre(p)) * kU);
      slot = wave + rank;
    } else {
      j_end = min(len, j_begin + a.chunk);
      if (act == 0 || j_begin >= j_end) return;  // l = 0: no cache read for this item
    }

    const int l16 = lane & 15, g4 = lane >> 4;
    // B operand: column = head l16 (zero unless an active packed head), dims 32s + 8*g4
    u32x4 qf[4];
    {
      const bool qa = l16 < a.qpk && ((act >> l16) & 1u);
      const uint16_t* qp = a.q + (int64_t)b * a.n_q * kHd + (int64_t)(hkv * a.qpk + (qa ? l16 : 0)) * kHd + 8 * g4;
#pragma unroll
      for (int s = 0; s < 4; ++s) qf[s] = qa ? ldg16(qp + 32 * s) : u32x4{0, 0, 0, 0};
    }
    // token-major cache: row (b, key) holds all KV heads; head-major: the
    // (b, KV head) cache is one contiguous [L][128] block
    const int64_t ldk = a.head_major ? kHd : (int64_t)a.n_kv * kHd;
    const int64_t cache0 = a.head_major ? ((int64_t)b * a.n_kv + hkv) * a.L * kHd
                                        : (int64_t)b * a.L * ldk + hkv * kHd;
    auto load = [&](int j0, Unit& u) {  // rows past kv_len re-read the last key (finite, p = 0)
      const uint16_t* kp = a.k + cache0 + (int64_t)min(j0 + l16, len - 1) * ldk + 8 * g4;
#pragma unroll
      for (int s = 0; s < 4; ++s) u.k[s] = ldg16(kp + 32 * s);
#pragma unroll
      for (int i = 0; i < 4; ++i) u.v[i] = ldg16(a.v + cache0 + (int64_t)min(j0 + 4 * i + g4, len - 1) * ldk + 8 * l16);
    };

    float m = -INFINITY, zl = 0.0f;  // running max of head column l16; this lane's share of its sum
    float acc[HMAX][8];
#pragma unroll
    for (int h = 0; h < HMAX; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
    const float sc = a.scale_log2;

    auto process = [&](int j0, const Unit& U) {
      f32x4 S = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < 4; ++s) S = mfma16(U.k[s], qf[s], S);  // lane: keys 4*g4 + r, head l16
      float sv[4], mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sv[r] = j0 + 4 * g4 + r < j_end ? S[r] * sc : -INFINITY;
        mx = fmaxf(mx, sv[r]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mnew = fmaxf(m, mx);  // finite: the unit has a key before j_end
      const float alpha = __builtin_amdgcn_exp2f(m - mnew);
      m = mnew;
      float ps = 0.0f, pr[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pr[r] = __builtin_amdgcn_exp2f(sv[r] - mnew);
        ps += pr[r];
      }
      zl = zl * alpha + ps;
      wave_lds_sync();  // the previous unit's reads of the scratch are done
#pragma unroll
      for (int r = 0; r < 4; ++r) s_p[w][4 * g4 + r][l16] = pr[r];
      if (g4 == 0) s_al[w][l16] = alpha;
      wave_lds_sync();  // this unit's values are visible to every lane of the wave
      // Up to four head columns, every column up to HMAX is carried, active or
      // not (an inactive or padding column has a zero query: finite scores,
      // discarded at the end), so the unit's arithmetic is straight-line code
      // (3-5% faster at Llama-3-8B's four heads per KV head); wider instances
      // test each head (the registers would not hold more).
#pragma unroll
      for (int h4 = 0; h4 < HMAX; h4 += HB) {
        float al[HB];  // (element reads through float: the writes above are float)
#pragma unroll
        for (int t = 0; t < HB; ++t) al[t] = s_al[w][h4 + t];
#pragma unroll
        for (int h = h4; h < h4 + HB; ++h)
          if (HMAX <= 4 || ((act >> h) & 1u))
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[h][e] *= al[h - h4];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float vf[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vf[2 * e] = __uint_as_float(U.v[i][e] << 16);
          vf[2 * e + 1] = __uint_as_float(U.v[i][e] & 0xffff0000u);
        }
#pragma unroll
        for (int h4 = 0; h4 < HMAX; h4 += HB) {
          float p4[HB];
#pragma unroll
          for (int t = 0; t < HB; ++t) p4[t] = s_p[w][4 * i + g4][h4 + t];
#pragma unroll
          for (int h = h4; h < h4 + HB; ++h)
            if (HMAX <= 4 || ((act >> h) & 1u))
#pragma unroll
              for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(p4[h - h4], vf[e], acc[h][e]);
        }
      }
    };

    // Full groups of kDepth units run branch-free, so the compiler can wait
    // for exactly the unit about to be used (the two younger ones stay in
    // flight); prefetches past the last unit re-read it (from L2) instead of
    // branching.  The last 0-2 units are processed after the loop.
    const int nunits = (j_end - j_begin + kU - 1) / kU;
    const int last = nunits - 1;
    Unit buf[kDepth];
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(j_begin + min(d, last) * kU, buf[d]);
    const int nfull = nunits / kDepth;
    for (int g = 0; g < nfull; ++g) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        process(j_begin + (g * kDepth + d) * kU, buf[d]);
        load(j_begin + min((g + 1) * kDepth + d, last) * kU, buf[d]);
      }
    }
#pragma unroll
    for (int d = 0; d < kDepth - 1; ++d)
      if (nfull * kDepth + d < nunits) process(j_begin + (nfull * kDepth + d) * kU, buf[d]);

    // partials: (max, sum, o[128]) per (token, head, chunk)
    float z = zl + __shfl_xor(zl, 16);
    z += __shfl_xor(z, 32);
#pragma unroll
    for (int h = 0; h < HMAX; ++h) {
      if (!((act >> h) & 1u)) continue;
      float o8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {  // add the four key groups
        float v = acc[h][e];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        o8[e] = v;
      }
      float* part = a.part + ((int64_t)slot * a.qpk + h) * (kHd + 2);
      if (lane == h) {
        part[0] = m;
        part[1] = z;
      }
      if (g4 == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) part[2 + 8 * l16 + e] = o8[e];
      }
    }
    if (!BAL || u_end <= pre(p + 1)) break;
    j_begin = 0;
    ++rank;
  }
}

// Merge of the chunks: WPH (1 or 4) waves per (token, query head).  Every wave
// finds the maximum over the chunks (lanes take 64 at a time); wave w of a head
// then adds chunks w, w + WPH, ..., four loads together, lane = two dims, each
// chunk's weight coming out of its lane by readlane, and four waves' sums
// meet in LDS.  One wave per head serves few chunks (a barrier costs more than it saves:
// 2048 heads of one chunk 6.2 us, 7.2 with four); one sequence of 8192 keys (128 chunks a
// head) takes 15 us with four, and took 39 with one wave and one load at a time.  With more
// than 2048 heads of short pairs one wave each fills the chip (5312 heads of up to 14 chunks
// 7.9 us, 13.7 with four).
template <int WPH>
__global__ __launch_bounds__(kDT) void wide_attn_decode_merge(AttnDecArgs a) {
  __shared__ float s_o[4][kHd + 1];
  const int gh = WPH == 4 ? blockIdx.x : blockIdx.x * 4 + wave_id();
  if (gh >= a.B * a.n_q) return;
  const int b = gh / a.n_q, h = gh - b * a.n_q;
  const int w = WPH == 4 ? wave_id() : 0, lane = lane_id();
  uint16_t* orow = a.o + (int64_t)b * a.n_q * kHd + (int64_t)h * kHd + 2 * lane;
  const int len = a.kv_len ? min(a.kv_len[b], a.L) : a.L;
  if (!a.mask[(int64_t)b * a.ng + h / a.hpg] || len <= 0) {  // inactive head: +0
    if (w == 0) *reinterpret_cast<uint32_t*>(orow) = 0u;
    return;
  }
  const int p = b * a.n_kv + h / a.qpk;
  const int nc = a.table ? a.table[2 * p + 1] : (len + a.chunk - 1) / a.chunk;
  const int64_t slot = a.table ? a.table[2 * p] : (int64_t)p * a.n_chunks;
  const int ld = a.qpk * (kHd + 2);  // floats from one chunk's partial to the next (nc * ld fits 31 bits)
  const float* part = a.part + slot * ld + (h % a.qpk) * (kHd + 2);
  float mx = -INFINITY;
  for (int c0 = 0; c0 < nc; c0 += kWave)
    if (c0 + lane < nc) mx = fmaxf(mx, part[(c0 + lane) * ld]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  float z = 0.0f, o0 = 0.0f, o1 = 0.0f;
  for (int c0 = 0; c0 < nc; c0 += kWave) {
    const int c = c0 + lane;
    float f = 0.0f;
    if (c < nc) {
      f = __builtin_amdgcn_exp2f(part[c * ld] - mx);
      if (lane % WPH == w) z = fmaf(f, part[c * ld + 1], z);
    }
    const int cnt = min(kWave, nc - c0);
    for (int j0 = w; j0 < cnt; j0 += 4 * WPH) {
      float2 v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)  // four chunks' loads together (past the end: the last one's again)
        v[t] = *reinterpret_cast<const float2*>(part + min(c0 + j0 + WPH * t, nc - 1) * ld + 2 + 2 * lane);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (j0 + WPH * t >= cnt) break;
        const float fj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), j0 + WPH * t));
        o0 = fmaf(fj, v[t].x, o0);
        o1 = fmaf(fj, v[t].y, o1);
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) z += __shfl_xor(z, o);
  if constexpr (WPH == 4) {
    s_o[w][2 * lane] = o0;
    s_o[w][2 * lane + 1] = o1;
    if (lane == 0) s_o[w][kHd] = z;
    __syncthreads();
    if (w != 0) return;
    o0 = o1 = z = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o0 += s_o[i][2 * lane];
      o1 += s_o[i][2 * lane + 1];
      z += s_o[i][kHd];
    }
  }
  const float inv = 1.0f / z;
  *reinterpret_cast<uint32_t*>(orow) = pack_bf16x2_hw(o0 * inv, o1 * inv);
}

}  // namespace

int attn_decode_chunk(int B, int n_kv, int L) {
  int ch = 2048;  // keys per work item (wave): enough items to fill the chip
  while (ch > 64 && (int64_t)B * n_kv * ((L + ch - 1) / ch) < 4096) ch /= 2;
  return ch;
}

// Waves of the balanced split (0: equal chunks stay): one round of resident
// waves, two workgroups a CU.  It pays from
// about 16 units (256 keys) per wave on; below, listing the units costs more
// (2-4 us) than an even split saves: 64 sequences of up to 1000 keys 30 us
// balanced and 28 in chunks, 32 of up to 4096 (head groups of one head) 59 and
// 67.  Short sequences leave a wave several small segments with a start each, and
// many more waves of equal chunks hide that better: 250 of up to 300 keys 43 us
// balanced, 36 in chunks, 128 of up to 600 39 and 33; from 900 keys on 4-20% less
// balanced.  A table of kAttnDecMaxPairs pairs and its segments fit the equal
// chunks' workspace (at least 4096 partials here).
int attn_decode_waves(int64_t B, int n_kv, int L) {
  const int64_t pairs = B * n_kv, units = pairs * ((L + kU - 1) / kU);
  return pairs <= kAttnDecMaxPairs && L >= 768 && units >= 32768 && units <= 0x7fffffff ? kAttnDecWaves : 0;
}

hipError_t launch_attention_decode(AttnDecArgs a, hipStream_t s) {
  if (a.B == 0) return hipSuccess;
  const int64_t items = a.table ? a.waves : (int64_t)a.B * a.n_kv * a.n_chunks;
  const dim3 grid((unsigned)((items + 3) / 4));
  const int lds = a.table ? (a.B * a.n_kv + 1) * (int)sizeof(uint64_t) : 0;
#define WIDE_DEC(H)                                                                                         \
  do {                                                                                                      \
    if (a.table) WIDE_LAUNCH_NAMED("wide_attn_decode", (wide_attn_decode<H, true>), grid, dim3(kDT), lds, s, a); \
    else WIDE_LAUNCH_NAMED("wide_attn_decode", (wide_attn_decode<H, false>), grid, dim3(kDT), 0, s, a);     \
  } while (0)
  if (a.qpk == 1) WIDE_DEC(1);
  else if (a.qpk == 2) WIDE_DEC(2);
  else if (a.qpk <= 4) WIDE_DEC(4);
  else if (a.qpk <= 8) WIDE_DEC(8);
  else WIDE_DEC(16);
#undef WIDE_DEC
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int heads = a.B * a.n_q;
  const bool wide_merge = a.n_chunks > (heads <= 1024 ? 4 : 8) &&
                          (heads <= 2048 || (a.table && a.waves >= 4 * a.B * a.n_kv));
  const dim3 mg((unsigned)(wide_merge ? heads : (heads + 3) / 4));
  if (wide_merge)
    WIDE_LAUNCH_NAMED("wide_attn_decode_merge", wide_attn_decode_merge<4>, mg, dim3(kDT), 0, s, a);
  else
    WIDE_LAUNCH_NAMED("wide_attn_decode_merge", wide_attn_decode_merge<1>, mg, dim3(kDT), 0, s, a);
  return hipGetLastError();
}

}  // namespace wide
