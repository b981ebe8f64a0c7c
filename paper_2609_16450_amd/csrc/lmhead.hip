// Fused LM head + softmax statistics for gfx950.
//
// z = W h is formed tile by tile with bf16 MFMA (fp32 accumulation) and folded straight into
// per-(row, vocabulary tile) partials (max, sum of exponentials, entropy moment, argmax); the
// logits never leave registers.  A second kernel merges the partials of each row in a fixed
// order and emits kappa = 1/s, H = ln s - t/s, the argmax and the max logit.
//
// Orientation: the MFMA "row" dimension is the vocabulary and the "column" dimension is the
// block position, so every lane owns one position and reduces the logits it holds in
// registers before a single cross-half exchange.
#include <type_traits>

#include "attn_small.hpp"
#include "eb_common.hpp"
#include "eb_internal.hpp"
#include "tile_loads.hpp"

namespace eb {
namespace {

// ---------------------------------------------------------------------------------------
// Streaming kernel for few block positions (n_rows <= 16 * NT).
//
// With a handful of positions the product is a bandwidth-bound pass over W.  One workgroup per
// compute unit owns a contiguous slice of vocabulary rows.  Each of its 16 waves (8 for slices
// above 768 rows) streams its share of the slice from HBM straight into MFMA A-operand
// registers, keeping kDepth k-steps of loads in flight; h, the B operand shared by all waves,
// goes through a double-buffered LDS chunk.  Every W byte is read once, by one lane, with no
// LDS round trip, in whole or half cache lines per load (kLines).  Bound by HBM: 32 positions of a
// 126464 x 4096 head take 178 us (5.8 TB/s) where W lies well in memory, against 184 us with half
// lines and 32-column steps, 64 positions 181 against 188 us (195 to 222 against 202 to 228 us at
// other allocations); of a 152064 x 3584 head 187 against 202 us and 199 against 215 us.
// (Loading h per wave straight into registers instead, with no LDS and no
// barrier, measured 237 us against 203 us at 32 positions: the per-wave h traffic from L2 costs
// more than the shared chunks.)
// ---------------------------------------------------------------------------------------
#ifndef EB_STREAM_GROUPS
#define EB_STREAM_GROUPS 256
#endif
constexpr int kStreamGroups = EB_STREAM_GROUPS;  // workgroups (256: one per compute unit)

// The streaming kernel uses 16x16x32 MFMA tiles (mfma16; 32x32x16 tiles measured 4.65 TB/s at best
// against 5.4).  A lane of the A operand holds 8 k-values of row l % 16.
//  * Half lines: a k-step is 32 columns, loaded straight into that layout, 16 rows x 64 bytes per
//    load.
//  * Whole lines (kLines): a k-step is 64 columns of a 16-row tile in two loads of 8 rows x 128
//    bytes: lane l loads 16-byte chunk line_chunk(l) of row l % 8 (v0) and of row 8 + l % 8 (v1).
//    line_to_frag exchanges v0 and v1 between lanes l and l ^ 8, after which lane l holds row l %
//    16 in both, chunk l / 16 in the first and 4 + l / 16 in the second: the A operands of the
//    MFMAs of the step's first and last 32 columns.
// Either way a logit is summed in the order of its columns, as in the tile kernel, so a position's
// logits do not depend on how many positions the call has.
__device__ __forceinline__ int line_chunk(int lane) { return (lane >> 4) + 4 * ((lane >> 3) & 1); }
__device__ __forceinline__ void line_to_frag(const u32x4& v0, const u32x4& v1, bf16x8& first,
                                             bf16x8& last) {
  constexpr int kRor8 = 0x128;  // DPP row_ror:8: from the lane 8 away in the row of 16
  u32x4 f, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[i] = __builtin_amdgcn_update_dpp(v0[i], v1[i], kRor8, 0xf, 0xc, false);  // lanes 8..15
    l[i] = __builtin_amdgcn_update_dpp(v1[i], v0[i], kRor8, 0xf, 0x3, false);  // lanes 0..7
  }
  first = __builtin_bit_cast(bf16x8, f);
  last = __builtin_bit_cast(bf16x8, l);
}

// Second-largest logit (with multiplicity) of the union of two sets whose largest values are
// m_a, m_b and second-largest m2_a, m2_b.  Exact and order-free, so every merge order gives
// the same bits.  kNegBig stands for "none".
__device__ __forceinline__ float top2_merge(float m_a, float m2_a, float m_b, float m2_b) {
  return fmaxf(fminf(m_a, m_b), fmaxf(m2_a, m2_b));
}

// top2_merge of a lane's (m, m2) with the lane `mask` away.
__device__ __forceinline__ float top2_shfl_merge(float m, float m2, int mask) {
  return top2_merge(m, m2, __shfl_xor(m, mask), __shfl_xor(m2, mask));
}

// Statistics of column l % 16 of position tile nt of a wave's natural-order 16x16 accumulator
// tiles, whose rows are vocabulary entries wb + 16 tm + 4 (l / 16) + r below we: per lane, then
// merged over the column's four lanes in a canonical order.  With kTop2, m2 is the second-largest
// logit (kNegBig if none).  With kAnyLogit, logits of -inf (and NaN) add nothing, instead of the
// NaN that 0 * -inf makes of t; no other result changes.
template <int TM, int NT, bool kTop2, bool kAnyLogit = false>
__device__ __forceinline__ Partial wave_column_stats(const f32x4 (&acc)[TM][NT], int nt, int wb,
                                                     int we, int lane, float& m2) {
  const int grp = lane >> 4;
  float m = kNegBig;
  m2 = kNegBig;
  int32_t idx = kNoIndex;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int v = wb + tm * 16 + 4 * grp + r;
      const float z = acc[tm][nt][r];
      if (kTop2 && v < we) m2 = __builtin_amdgcn_fmed3f(m, m2, z);
      if (v < we && z > m) {
        m = z;
        idx = v;
      }
    }
  float s = 0.f, t = 0.f;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int v = wb + tm * 16 + 4 * grp + r;
      if (v < we) {
        float y = (acc[tm][nt][r] - m) * kLog2e;
        if (kAnyLogit) y = fmaxf(y, -1.0e30f);
        const float e = fast_exp2(y);
        s += e;
        t = fmaf(e, y, t);
      }
    }
  Partial p{m, s, t, idx};
  if (kTop2) m2 = top2_shfl_merge(p.m, m2, 16);
  p = partial_xor_merge(p, 16, lane);
  if (kTop2) m2 = top2_shfl_merge(p.m, m2, 32);
  return partial_xor_merge(p, 32, lane);
}

// kTop2: also track the second-largest logit of each (row, slice) into part2.
// kWaves waves per workgroup, shares of at most 8 NL vocabulary rows per wave (NL whole-line loads
// per k-step), NT 16-position tiles.
// kAttnD != 0: workgroups n_slices and up run the small block attention (head dimension kAttnD)
// on unit blockIdx.x - n_slices of ap; the dispatcher starts them as the slices finish.
template <int kWaves, int NL, int NT, int kDepth, bool kTop2, int kAttnD, bool kLines>
__global__ __launch_bounds__(kWaves * 64) void lmhead_stream16_kernel(
    const uint16_t* __restrict__ h, const uint16_t* __restrict__ w, int n_rows, int hidden,
    int vocab, int rows_per_wg, Partial* __restrict__ part, float* __restrict__ part2,
    int n_slices, AttnParams ap) {
  static_assert(kAttnD == 0 || kWaves * 64 == kSmallThreads, "attention role shape");
  if constexpr (kAttnD != 0) {
    if (static_cast<int>(blockIdx.x) >= n_slices) {  // whole workgroup
      attn_small_role<kAttnD, kSmallThreads>(ap, static_cast<int>(blockIdx.x) - n_slices, 0);
      return;
    }
  }
  constexpr int TM = (NL + 1) / 2;     // 16-row tiles; the last one may lack its upper rows
  constexpr int kCols = kLines ? 64 : 32;   // columns per k-step
  constexpr int kLoads = kLines ? NL : TM;  // loads per k-step
  constexpr int KC = 1024 / NT;        // h columns per LDS chunk
  constexpr int kPitch = KC + 8;       // LDS row pitch (bf16)
  constexpr int kSpc = KC / kCols;     // k-steps per chunk
  constexpr int kHRows = NT * 16;
  constexpr int kHChunks16 = kHRows * KC / 8;
  constexpr int kThreads = kWaves * 64;
  constexpr int kHPer = kHChunks16 / kThreads;
  static_assert(kHChunks16 % kThreads == 0, "h chunk splits evenly");
  static_assert(kSpc % kDepth == 0, "chunk boundary falls on a group boundary");
  __shared__ __attribute__((aligned(16))) uint16_t hs[2][kHRows * kPitch];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 4, l16 = lane & 15;
  const int wg = blockIdx.x;
  const int vb = wg * rows_per_wg;
  const int ve = min(vocab, vb + rows_per_wg);
  const int rw = (rows_per_wg + kWaves - 1) / kWaves;
  const int wb = vb + wave * rw;
  const int we = min(ve, wb + rw);

  // Unconditional loads with clamped addresses: rows 8 i + l % 8 of the wave's share, or 16 i +
  // l % 16.
  const int wlast = max(min(we, vocab) - 1, 0);
  const uint16_t* wp[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int row = min(wb + (kLines ? i * 8 + (lane & 7) : i * 16 + l16), wlast);
    wp[i] = w + static_cast<size_t>(row) * hidden + 8 * (kLines ? line_chunk(lane) : grp);
  }
  const int nsteps = hidden / kCols;
  const int nsteps_p = (nsteps + kDepth - 1) / kDepth * kDepth;
  const int nchunks = (hidden + KC - 1) / KC;

  // Every workgroup walks the hidden dimension from column 0.  (With starts turned by workgroup the
  // worst of nine allocations of W, at 32 positions or one, took 188 us instead of 205-233 us, but
  // a logit's sum then depended on its vocabulary slice: equal rows of W got unequal logits, and
  // neither the lowest id nor a gap of 0 on a shared maximum held any more.)
  u32x4 buf[kDepth][kLoads];
  auto issue = [&](int j, int step) {
    const int st = min(step, nsteps - 1);
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      buf[j][i] = *reinterpret_cast<const u32x4*>(wp[i] + kCols * st);
  };
  u32x4 hreg[kHPer];
  auto load_h = [&](int c) {
#pragma unroll
    for (int i = 0; i < kHPer; ++i) {
      const int idx = tid + i * kThreads;
      const int row = min(idx / (KC / 8), n_rows - 1);
      const int col = min(c * KC + (idx % (KC / 8)) * 8, hidden - 8);
      hreg[i] = *reinterpret_cast<const u32x4*>(h + static_cast<size_t>(row) * hidden + col);
    }
  };
  auto store_h = [&](int b, int c) {
#pragma unroll
    for (int i = 0; i < kHPer; ++i) {
      const int idx = tid + i * kThreads;
      const int row = idx / (KC / 8), col = (idx % (KC / 8)) * 8;
      const bool ok = c * KC + col < hidden;
      *reinterpret_cast<u32x4*>(&hs[b][row * kPitch + col]) = ok ? hreg[i] : u32x4{0u, 0u, 0u, 0u};
    }
  };

  f32x4 acc[TM][NT];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[a][b] = f32x4{};

#pragma unroll
  for (int j = 0; j < kDepth; ++j) issue(j, j);
  load_h(0);
  store_h(0, 0);
  __syncthreads();
  if (nchunks > 1) load_h(1);

  auto consume = [&](int g, int j) {
    constexpr int kMfmas = kCols / 32;  // MFMAs per tile and k-step
    const uint16_t* hb = hs[(g / kSpc) & 1] + (g % kSpc) * kCols + 8 * grp + kCols * j;
    bf16x8 a[TM][kMfmas];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {  // (upper rows that are not there repeat the lower ones)
      if constexpr (kLines)
        line_to_frag(buf[j][2 * tm], buf[j][min(2 * tm + 1, NL - 1)], a[tm][0], a[tm][1]);
      else
        a[tm][0] = __builtin_bit_cast(bf16x8, buf[j][tm]);
    }
#pragma unroll
    for (int i = 0; i < kMfmas; ++i) {
      auto frag = [&](int nt) {
        return *reinterpret_cast<const bf16x8*>(hb + (nt * 16 + l16) * kPitch + 32 * i);
      };
      if constexpr (kLines) {  // (all NT fragments together spill: 1 to 3% at 152064 x 3584)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 b = frag(nt);
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) acc[tm][nt] = mfma16(a[tm][i], b, acc[tm][nt]);
        }
      } else {
        bf16x8 b[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b[nt] = frag(nt);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = mfma16(a[tm][i], b[nt], acc[tm][nt]);
      }
    }
  };
  auto chunk_boundary = [&](int g) {
    if (g > 0 && g % kSpc == 0) {
      const int c = g / kSpc;
      store_h(c & 1, c);
      __syncthreads();
      if (c + 1 < nchunks) load_h(c + 1);
    }
  };

  for (int g = 0; g < nsteps_p - kDepth; g += kDepth) {
    chunk_boundary(g);
#pragma unroll
    for (int j = 0; j < kDepth; ++j) {
      consume(g, j);
      issue(j, g + kDepth + j);
    }
  }
  chunk_boundary(nsteps_p - kDepth);
#pragma unroll
  for (int j = 0; j < kDepth; ++j) consume(nsteps_p - kDepth, j);

  __syncthreads();
  Partial* red = reinterpret_cast<Partial*>(&hs[0][0]);  // [kWaves][kHRows]
  float* red2 = reinterpret_cast<float*>(red + kWaves * kHRows);
  static_assert(kWaves * kHRows * (sizeof(Partial) + 4) <= sizeof(hs), "reduction fits");
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float m2 = kNegBig;
    const Partial p = wave_column_stats<TM, NT, kTop2>(acc, nt, wb, we, lane, m2);
    if (lane < 16) {
      red[wave * kHRows + nt * 16 + l16] = p;
      if (kTop2) red2[wave * kHRows + nt * 16 + l16] = m2;
    }
  }
  __syncthreads();
  if (tid < kHRows && tid < n_rows) {
    Partial p = red[tid];
    float m2 = kTop2 ? red2[tid] : kNegBig;
#pragma unroll
    for (int k = 1; k < kWaves; ++k) {
      const Partial q = red[k * kHRows + tid];
      if (kTop2) m2 = top2_merge(p.m, m2, q.m, red2[k * kHRows + tid]);
      p = partial_merge(p, q);
    }
    part[static_cast<size_t>(tid) * n_slices + wg] = p;
    if (kTop2) part2[static_cast<size_t>(tid) * n_slices + wg] = m2;
  }
}

constexpr int kStreamShape = 16;  // rows (and positions) per MFMA tile
constexpr int kStreamLoad = 8;    // rows per load
// 16 waves per workgroup while each wave's share of the slice fits in kStreamMaxTm16 row tiles
// (at 1024 threads a lane has 128 VGPRs; four tiles with two or more position tiles spill), else
// 8 waves, which leaves 256 VGPRs per lane for up to 8 row tiles (16 waves with depth 8 measured
// 186 us against 195 us for 8 waves with depth 2 at 32 positions of a 126464 x 4096 head).
constexpr int kStreamMaxTm16 = 3;
constexpr int kStreamMaxTm8 = 8;

struct StreamPlan {
  int groups, rows_per_wg, waves, tm;  // tm: MFMA row tiles per wave
  int nl;                              // 8-row loads per wave
};

StreamPlan stream_plan(int vocab) {
  const int groups = min(kStreamGroups, (vocab + 31) / 32);
  const int rows = (vocab + groups - 1) / groups;
  auto plan = [&](int waves) {
    const int rw = (rows + waves - 1) / waves;
    return StreamPlan{groups, rows, waves, (rw + kStreamShape - 1) / kStreamShape,
                      (rw + kStreamLoad - 1) / kStreamLoad};
  };
  return plan(16).tm <= kStreamMaxTm16 ? plan(16) : plan(8);
}

constexpr int kStreamMaxRows = 64;  // n_rows handled by the streaming kernel

bool use_stream(int n_rows, int vocab) {
  if (n_rows > kStreamMaxRows) return false;
  const StreamPlan pl = stream_plan(vocab);
  if (pl.waves == 16) return true;
  if (n_rows > 2 * kStreamShape) return pl.tm <= 6;  // register budget with four position tiles
  return pl.tm <= kStreamMaxTm8;
}

// Block attention queued behind the slices of a streaming launch (attn_d 0: none).
struct HostedAttn {
  AttnParams p;
  int units, attn_d;
};

// Whole lines or half lines per load.  Half lines make the shorter k-step, so the loop runs closer
// to its loads; whole lines make half the requests.  With three or more 8-row shares per wave what
// decides is whether W fits the 256 MB cache in front of HBM, where a program that calls the head
// again and again finds it: whole lines take 2 to 5% longer up to 260 MB (100000 x 1024: 37.3 ->
// 38.9 us for one position, 41.2 -> 43.0 us for 64) and 2 to 8% less above 300 MB (126464 x 4096:
// 193.7 -> 183.1 us, 195.4 -> 189.0 us).  With two, half lines are never behind (65536 x 2048: 42.8
// against 48.6 us for one position; x 4096: 110.7 against 112.9 us).  With one, whole lines read 8
// rows instead of 16 (8192 x 2048: 16.5 -> 13.9 us), except that with four position tiles there is
// nothing to gain (24000 x 4096, 64 positions: 45.4 -> 48.7 us).
constexpr size_t kStreamLineBytes = 280u << 20;
enum StreamForm { kHalfLines, kWholeLines, kBySize };
template <int kWaves, int NL, int NT>
constexpr StreamForm kStreamForm = kWaves == 8 || (NL == 1 && NT <= 2) ? kWholeLines
                                   : NL <= 2                           ? kHalfLines
                                                                       : kBySize;

template <int kWaves, int NL, int NT, bool kTop2, int kAttnD, bool kLines>
hipError_t launch_stream_form(int n_rows, int hidden, int vocab, const StreamPlan& pl,
                              const void* h, const void* w, Partial* part, float* part2,
                              hipStream_t s, const HostedAttn& ha) {
  // 16 waves: up to 16 W registers in flight per lane (16 bytes each; 8 with four position tiles,
  // where more spill and 4 measured 182 against 177 us; five and six shares spill 3 to 5 registers
  // all the same), at most 256 columns, a power of two that divides the per-chunk step count.  8
  // waves: one k-step (more measured no faster).
  constexpr int kLoads = kLines ? NL : (NL + 1) / 2, kMax = kLines ? 4 : 8;
  constexpr int D = kWaves == 8 ? 1 : (NT >= 4 ? 8 : 16) / kLoads;
  constexpr int Dp = D >= kMax ? kMax : (D >= 4 ? 4 : (D >= 2 ? 2 : 1));
  const int extra = kAttnD != 0 ? ha.units : 0;
  hipLaunchKernelGGL((lmhead_stream16_kernel<kWaves, NL, NT, Dp, kTop2, kAttnD, kLines>),
                     dim3(pl.groups + extra), dim3(kWaves * 64), 0, s,
                     static_cast<const uint16_t*>(h), static_cast<const uint16_t*>(w), n_rows,
                     hidden, vocab, pl.rows_per_wg, part, part2, pl.groups, ha.p);
  return hipGetLastError();
}

template <int kWaves, int NL, int NT, bool kTop2, int kAttnD = 0>
hipError_t launch_stream_nl(int n_rows, int hidden, int vocab, const StreamPlan& pl,
                            const void* h, const void* w, Partial* part, float* part2,
                            hipStream_t s, const HostedAttn& ha) {
  constexpr StreamForm form = kStreamForm<kWaves, NL, NT>;
  auto go = [&](auto lines) {
    return launch_stream_form<kWaves, NL, NT, kTop2, kAttnD, lines.value>(
        n_rows, hidden, vocab, pl, h, w, part, part2, s, ha);
  };
  if constexpr (form == kBySize) {
    if (static_cast<size_t>(vocab) * hidden * 2 <= kStreamLineBytes) return go(std::false_type{});
  }
  return go(std::bool_constant<form != kHalfLines>{});
}

// 16 waves, NL 8-row loads: the variant for the hosted attention's head dimension.
template <int NL, int NT, bool kTop2>
hipError_t launch_stream16(int n_rows, int hidden, int vocab, const StreamPlan& pl,
                           const void* h, const void* w, Partial* part, float* part2,
                           hipStream_t s, const HostedAttn& ha) {
  if constexpr (!kTop2) {
    if (ha.attn_d == 128)
      return launch_stream_nl<16, NL, NT, false, 128>(n_rows, hidden, vocab, pl, h, w, part,
                                                      part2, s, ha);
    if (ha.attn_d == 64)
      return launch_stream_nl<16, NL, NT, false, 64>(n_rows, hidden, vocab, pl, h, w, part,
                                                     part2, s, ha);
  }
  if (ha.attn_d != 0) return hipErrorInvalidValue;  // excluded by lmhead_hosts_attn
  return launch_stream_nl<16, NL, NT, kTop2>(n_rows, hidden, vocab, pl, h, w, part, part2, s,
                                             ha);
}

// NT: 16-position tiles covering n_rows.
template <int NT, bool kTop2>
hipError_t launch_stream(int n_rows, int hidden, int vocab, const void* h, const void* w,
                         Partial* part, float* part2, hipStream_t s, const HostedAttn& ha) {
  const StreamPlan pl = stream_plan(vocab);
  auto go16 = [&](auto nl) {
    return launch_stream16<nl.value, NT, kTop2>(n_rows, hidden, vocab, pl, h, w, part, part2, s,
                                                ha);
  };
  if (pl.waves == 16) {
    switch (pl.nl) {
      case 1: return go16(std::integral_constant<int, 1>{});
      case 2: return go16(std::integral_constant<int, 2>{});
      case 3: return go16(std::integral_constant<int, 3>{});
      case 4: return go16(std::integral_constant<int, 4>{});
      case 5: return go16(std::integral_constant<int, 5>{});
      case 6: return go16(std::integral_constant<int, 6>{});
      default: return hipErrorInvalidValue;  // excluded by stream_plan
    }
  }
  if (ha.attn_d != 0) return hipErrorInvalidValue;  // excluded by lmhead_hosts_attn
  // More than 48 tiles of rows per workgroup: the 8-wave shape has 7 or 8 tiles per wave.
  if constexpr (NT < 4) {
    if (pl.tm == 7)
      return launch_stream_nl<8, 14, NT, kTop2>(n_rows, hidden, vocab, pl, h, w, part, part2, s,
                                                ha);
    if (pl.tm == 8)
      return launch_stream_nl<8, 16, NT, kTop2>(n_rows, hidden, vocab, pl, h, w, part, part2, s,
                                                ha);
  }
  return hipErrorInvalidValue;  // excluded by use_stream
}

template <bool kTop2>
hipError_t launch_stream_rows(int n_rows, int hidden, int vocab, const void* h, const void* w,
                              Partial* part, float* part2, hipStream_t s,
                              const HostedAttn& ha = HostedAttn{}) {
  if (n_rows <= 16)
    return launch_stream<1, kTop2>(n_rows, hidden, vocab, h, w, part, part2, s, ha);
  if (n_rows <= 32)
    return launch_stream<2, kTop2>(n_rows, hidden, vocab, h, w, part, part2, s, ha);
  if (n_rows <= 64)
    return launch_stream<4, kTop2>(n_rows, hidden, vocab, h, w, part, part2, s, ha);
  return hipErrorInvalidValue;  // excluded by use_stream
}

// ---------------------------------------------------------------------------------------
// Large-batch kernel: tiles of 256 vocabulary rows x up to 256 positions.
//
// Both operands go HBM/L2 -> LDS by buffer loads straight into LDS (lane l of a wave writes its
// 16 bytes to LDS base + 16 l), in stages of BK = 64 hidden columns; no staging registers and no
// LDS store instructions.  LDS rows are 128 bytes without padding, their eight 16-byte chunks
// permuted by row so that the 16-row MFMA operand reads (rows in the order rho of tile_run) are
// free of bank conflicts.  Four waves form a 2 x 2 grid of sub-tiles of 16x16x32 MFMA blocks.
//
// Tile order is XCD-aware: the launch sequence takes vocabulary tiles in bands of kBand, each
// band swept position tile by position tile, and is cut into one contiguous segment per XCD
// (lmhead_tile_kernel), so the workgroups an XCD runs at once work on neighbouring tiles that
// share a few W and h tiles in its L2.
// ---------------------------------------------------------------------------------------
constexpr int kXcds = 8;
constexpr int kBand = 4;
constexpr int kTileBM = 256;     // vocabulary rows per tile
constexpr int kTileBK = 64;      // hidden columns per ring stage
constexpr int kTileGroups = 256; // persistent workgroups (one per compute unit)

int tile_vtiles(int vocab) { return (vocab + kTileBM - 1) / kTileBM; }

// 16x16x32 MFMA with its accumulator tied to the same AGPRs as input and output.  Written as asm:
// with the builtin, the compiler picks the untied form for this size and moves the accumulators
// through other registers around every MFMA of a 64-accumulator loop (hundreds of copies per
// step, seen in the ISA).
__device__ __forceinline__ void mfma16_tied(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// The compiler does not see that the asm above is an MFMA, so it inserts none of the wait states
// between an MFMA and other instructions touching its accumulators.  Every accumulator passes
// through an empty asm that "writes" it, which no access of it can cross, and s_nops supply the
// wait states: acc_fence_in after the accumulators are written and before the first MFMA reads
// them, acc_fence_out after the last MFMA and before anything reads its results.
template <int TM, int TN>
__device__ __forceinline__ void acc_fence_in(f32x4 (&acc)[TM][TN]) {
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) asm volatile("" : "+a"(acc[a][b]));
  asm volatile("s_nop 7");
}
template <int TM, int TN>
__device__ __forceinline__ void acc_fence_out(f32x4 (&acc)[TM][TN]) {
  asm volatile("s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7");
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) asm volatile("" : "+a"(acc[a][b]));
}

// Reductions over the four lanes l % 16 + 16 q (q < 4) of a column, in registers: the gfx950
// swaps v_permlane16_swap / v_permlane32_swap hand every lane the values of the lower and upper
// lane of its pair (l & ~16 and l | 16, then l & ~32 and l | 32), which are combined as
// lower op upper, so both lanes of a pair evaluate the same expression and end with the same
// bits.
__device__ __forceinline__ void lane_pair16(float x, float& lo, float& hi) {
  const auto r =
      __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}
__device__ __forceinline__ void lane_pair32(float x, float& lo, float& hi) {
  const auto r =
      __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_max(float m) {
  float lo, hi;
  lane_pair16(m, lo, hi);
  m = fmaxf(lo, hi);
  lane_pair32(m, lo, hi);
  return fmaxf(lo, hi);
}
__device__ __forceinline__ void pair_sum_min(float& s, float& t, int32_t& idx) {
  float lo, hi, lo2, hi2, lo3, hi3;
  lane_pair16(s, lo, hi);
  lane_pair16(t, lo2, hi2);
  lane_pair16(__int_as_float(idx), lo3, hi3);
  s = lo + hi;
  t = lo2 + hi2;
  idx = min(__float_as_int(lo3), __float_as_int(hi3));
  lane_pair32(s, lo, hi);
  lane_pair32(t, lo2, hi2);
  lane_pair32(__int_as_float(idx), lo3, hi3);
  s = lo + hi;
  t = lo2 + hi2;
  idx = min(__float_as_int(lo3), __float_as_int(hi3));
}

// Statistics of one column of a wave's 16x16x32 accumulator tile: lane l holds, for column block
// tn, vocabulary rows vbase + 16 tm + 4 r (tm < TM, r < 4; vbase includes the lane's l / 16) of
// one column, and the four lanes l % 16 + 16 q together hold the column's 16 TM rows (the rows
// of a 16-row block reach the MFMA in the order the fragment reads use, see tile_run).  A max pass
// in four chains (by r), the column maximum M over the four lanes (pair_max), one exponential pass
// against M, then the four lanes' sums added pairwise in registers (pair_sum_min): identical bits
// on all four lanes.  Each chain walks its rows in decreasing order, so its last z == M is its
// lowest row; the argmax is kept as the block index tm, a constant of the unrolled code.  kFull
// (every row inside the vocabulary) drops the per-row bounds test.  With kTop2, m2 returns the
// column's second-largest logit (kNegBig if none).
template <int TM, int TN, bool kTop2, bool kFull>
__device__ __forceinline__ Partial column_stats16(const f32x4 (&acc)[TM][TN], int tn, int vbase,
                                                  int vocab, float* m2) {
  float mc[4] = {kNegBig, kNegBig, kNegBig, kNegBig};
  float mc2[4] = {kNegBig, kNegBig, kNegBig, kNegBig};
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (kFull || vbase + tm * 16 + 4 * r < vocab) {
        const float z = acc[tm][tn][r];
        // with mc >= mc2, the new second-largest is the median of (mc, mc2, z): one v_med3
        if (kTop2) mc2[r] = __builtin_amdgcn_fmed3f(mc[r], mc2[r], z);
        mc[r] = fmaxf(mc[r], z);
      }
    }
  const float m = fmaxf(fmaxf(mc[0], mc[1]), fmaxf(mc[2], mc[3]));
  if (kTop2) {
    float x = top2_merge(fmaxf(mc[0], mc[1]), top2_merge(mc[0], mc2[0], mc[1], mc2[1]),
                         fmaxf(mc[2], mc[3]), top2_merge(mc[2], mc2[2], mc[3], mc2[3]));
    x = top2_shfl_merge(m, x, 16);
    *m2 = top2_shfl_merge(fmaxf(m, __shfl_xor(m, 16)), x, 32);
  }
  float M = pair_max(m);
  constexpr int kNoK = TM;  // "not seen"
  float sc[4] = {0.f, 0.f, 0.f, 0.f}, tc[4] = {0.f, 0.f, 0.f, 0.f};
  int32_t kc[4] = {kNoK, kNoK, kNoK, kNoK};
#pragma unroll
  for (int tm = TM - 1; tm >= 0; --tm)
#pragma unroll
    for (int r = 3; r >= 0; --r) {
      const float z = acc[tm][tn][r];
      if (kFull) {
        const float y = (z - M) * kLog2e;
        const float e = fast_exp2(y);
        sc[r] += e;
        tc[r] = fmaf(e, y, tc[r]);
        kc[r] = z == M ? tm : kc[r];
      } else {
        // rows past the vocabulary contribute e = 0 and y = 0 (with no valid row in the
        // column, M = kNegBig, where z - M would overflow and 0 * inf would poison t)
        const bool ok = vbase + tm * 16 + 4 * r < vocab;
        const float y = ok ? (z - M) * kLog2e : 0.f;
        const float e = ok ? fast_exp2(y) : 0.f;
        sc[r] += e;
        tc[r] = fmaf(e, y, tc[r]);
        kc[r] = (ok && z == M) ? tm : kc[r];
      }
    }
  int32_t ob = kNoIndex;
#pragma unroll
  for (int c = 0; c < 4; ++c) ob = min(ob, kc[c] == kNoK ? kNoIndex : 16 * kc[c] + 4 * c);
  int32_t idx = ob == kNoIndex ? kNoIndex : vbase + ob;
  float s = (sc[0] + sc[1]) + (sc[2] + sc[3]), t = (tc[0] + tc[1]) + (tc[2] + tc[3]);
  pair_sum_min(s, t, idx);
  return Partial{M, s, t, idx};
}

// column_stats16 with the bounds test only where the tile reaches past the vocabulary.
template <int TM, int TN, bool kTop2>
__device__ __forceinline__ Partial column_stats16(const f32x4 (&acc)[TM][TN], int tn, int vbase,
                                                  int vocab, bool full, float* m2) {
  return full ? column_stats16<TM, TN, kTop2, true>(acc, tn, vbase, vocab, m2)
              : column_stats16<TM, TN, kTop2, false>(acc, tn, vbase, vocab, m2);
}

// Tile (vt, rt) of position s of the launch sequence: bands of kBand vocabulary tiles (the last
// band may be narrower), each band swept position tile by position tile (vocabulary tiles of the
// band innermost).  Every s in [0, n_vtiles * n_rtiles) is a tile.
__device__ __forceinline__ void band_tile(int s, int n_vtiles, int n_rtiles, int& vt, int& rt) {
  const int per_band = kBand * n_rtiles;
  const int band = s / per_band;
  const int tt = s - band * per_band;
  const int nv = min(kBand, n_vtiles - band * kBand);
  vt = band * kBand + tt % nv;
  rt = tt / nv;
}

// Persistent form of the large-batch kernel: kTileGroups workgroups, one per compute unit, each
// computing a sequence of tiles of 256 vocabulary rows x BN = 32 TN block positions.  The launch
// sequence is cut into 8 contiguous segments, one per XCD (workgroup g runs on XCD g % 8 and
// takes every 32nd tile of its XCD's segment), so each XCD gets the same number of tiles and
// its 32 resident workgroups share a few W and h tiles in its L2.  With fewer tiles than
// workgroups, workgroup g computes tile g.
//
// Per tile: 4 waves form a 2 x 2 grid of 128 x 16 TN sub-tiles, each 8 x TN blocks of 16x16x32
// bf16 MFMAs (32 TN accumulator registers per lane).  A stage is 64 hidden columns, two MFMA k
// steps a and b; per step a wave reads 8 + TN fragments (1 KB each) from LDS into one of two
// register sets and issues 8 TN MFMAs from the other.  W stages go round three LDS slots, h
// stages round two, 160 KB at TN = 8:
//   step a of stage s: MFMAs of (s, a); reads the fragments of (s, b); loads W of stage s + 2 into
//                      the slot that stage s - 1 left;
//   barrier:           stage s + 1 has landed, and every wave's reads of stage s are done;
//   step b of stage s: MFMAs of (s, b); reads the fragments of (s + 1, a); loads h of stage s + 2
//                      into the slot that stage s left.
// W, which comes from HBM, thus has three steps to land, h, which mostly comes from L2, two.
// (Two slots for both: 870 us against 806 us for 1024 positions of a 126464 x 4096 head; a third
// slot for h where it fits, TN <= 5, is no faster.)  The slots go on across tiles: the last two
// stages of a tile load the next tile's first two and read its stage 0, so its operands arrive
// while this tile finishes and runs its epilogue.  Measured against 32x32x16 blocks (the
// same tiles): 16x16x32 MFMAs sustain a higher clock under the chip's power limit.
//
// Every wave loads a quarter of W (8 instructions of 1 KB per stage) and of h (TN).
constexpr int kTileTM = kTileBM / 32;  // 16-row blocks per wave

template <int TN>
struct TileShape {
  static constexpr int BM = kTileBM, BN = 32 * TN, BK = kTileBK;
  static constexpr int kRowB = BK * 2;  // 128 bytes per LDS row
  static constexpr int kWSlot = BM * kRowB, kHSlot = BN * kRowB;
  static constexpr int kH0 = 3 * kWSlot;  // the two h slots follow the three W slots
  static constexpr int kLdsBytes = kH0 + 2 * kHSlot;
};

template <int TN, bool kTop2>
__device__ __forceinline__ void tile_run(uint8_t* smem, const uint16_t* __restrict__ h,
                                         const uint16_t* __restrict__ w, int n_rows, int hidden,
                                         int vocab, int n_vtiles, int n_rtiles,
                                         Partial* __restrict__ part, float* __restrict__ part2,
                                         int s0, int step, int s_end, int wave) {
  using Shape = TileShape<TN>;
  constexpr int BM = Shape::BM, BN = Shape::BN, BK = Shape::BK, kRowB = Shape::kRowB;
  constexpr int kWSlot = Shape::kWSlot, kHSlot = Shape::kHSlot, kH0 = Shape::kH0;
  constexpr int WM = 2, TM = kTileTM;
  constexpr int kWaveM = 16 * TM, kWaveN = 16 * TN;
  constexpr int kReads = TM + TN, kMfmas = TM * TN;
  constexpr int kWInst = TM, kHInst = TN;  // 1 KB load instructions of this wave per stage
  static_assert(BK == 64, "two 16x16x32 k steps per stage");
  static_assert(Shape::kLdsBytes <= 160 * 1024, "slots fit in LDS");
  static_assert(WM * BN * (sizeof(Partial) + 4) <= kWSlot, "reduction fits in a W slot");

  const int lane = threadIdx.x & 63;
  const int wm = wave % WM, wn = wave / WM;
  const int q4 = lane >> 4, l16 = lane & 15;
  const int ns = hidden / BK;  // stages per tile, >= 1
  const bool chain = ns >= 2;  // the last stages of a tile load the next tile's first two

  // Load instruction i of this wave covers rows 8 q .. 8 q + 7 of W, q = wave kWInst + i, or of h,
  // q = wave kHInst + i: eight lanes read 128 contiguous bytes of a row, a whole cache line in one
  // L2 request. (16 rows x 64 bytes per instruction make twice the requests, and the L2 request
  // rate then bounds the kernel.)  The loads are buffer loads into LDS, whose range ends with the
  // operand's last row, so rows past the end read as zero without a clamp; tile_loads.hpp has the
  // addresses. The resource of a 16-row group is scalar arithmetic on the tile's base; the vector
  // offset is the same for every second instruction.  (Global loads into LDS would count on the
  // LDS-read counter as well, and the compiler then waits for every outstanding fragment read
  // before each use of one.)
  const int wq0 = wave * kWInst, hq0 = wave * kHInst;
  const uint32_t row_bytes = static_cast<uint32_t>(hidden) * 2;
  uint32_t wvoff[2], hvoff[2];  // by the parity of i
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    wvoff[i] = tile_load_voff((wq0 + i) & 1, lane, row_bytes);
    hvoff[i] = tile_load_voff((hq0 + i) & 1, lane, row_bytes);
  }
  struct Src {
    const uint8_t *w, *h;
    int w_rows, h_rows;  // of the tile inside the operands, > 0
  };
  auto source = [&](int vt_, int rt_) {
    return Src{reinterpret_cast<const uint8_t*>(w + static_cast<size_t>(vt_) * BM * hidden),
               reinterpret_cast<const uint8_t*>(h + static_cast<size_t>(rt_) * BN * hidden),
               min(vocab - vt_ * BM, BM), min(n_rows - rt_ * BN, BN)};
  };
  // Load instruction i of W or of h of stage `stage` of the tile at p, into the slot at `slot`.
  auto load = [&](const uint8_t* base, int rows, int q, uint32_t voff, int stage, int slot) {
    const int row0 = tile_load_row0(q, rows);
    buffer_load_to_lds(make_rsrc(base + static_cast<uint32_t>(row0) * row_bytes,
                                 tile_load_range(row0, rows, row_bytes)),
                       smem + slot + q * 1024, voff, stage * (BK * 2));
  };
  auto load_w = [&](const Src& p, int stage, int slot, int i) {
    load(p.w, p.w_rows, wq0 + i, wvoff[i & 1], stage, slot);
  };
  auto load_h = [&](const Src& p, int stage, int slot, int i) {
    load(p.h, p.h_rows, hq0 + i, hvoff[i & 1], stage, slot);
  };
  // Fragment f of k step `half` of a stage (f < TM: W block f of this wave, else h block f - TM):
  // lane l reads row rho(l % 16) = 4 (l % 4) + (l % 16) / 4 of the 16-row block, 16-byte chunk
  // 4 half + l / 16 (k = 32 half + 8 (l / 16) .. + 7).  The MFMA then sees the block's rows
  // permuted by rho, on both operands: accumulator register r of lane l holds vocabulary row
  // 16 tm + rho(4 (l / 16) + r) = 16 tm + 4 r + l / 16 of the wave's W rows, for position
  // tn * 16 + rho(l % 16) of its h rows.
  const int rho = 4 * (l16 & 3) + (l16 >> 2);
  auto frag = [&](int wslot, int hslot, int half, int f) {
    const int r = f < TM ? wm * kWaveM + f * 16 + rho : wn * kWaveN + (f - TM) * 16 + rho;
    return *reinterpret_cast<const bf16x8*>(smem + (f < TM ? wslot : hslot) + r * kRowB +
                                            16 * ((4 * half + q4) ^ tile_swizzle(r)));
  };

  // LDS offsets of the slots of the current stage and of the next ones, turned once per stage.
  int w0 = 0, w1 = kWSlot, w2 = 2 * kWSlot;
  int h0 = kH0, h1 = kH0 + kHSlot;
  f32x4 acc[TM][TN];
  int s = s0, vt, rt;
  band_tile(s, n_vtiles, n_rtiles, vt, rt);
  Src src = source(vt, rt), nsrc = src;
  // Stages 0 and 1 of a tile, then the fragments of (0, a).
  bf16x8 xa[TM], xb[TN], ya[TM], yb[TN];
  auto start = [&]() {
    auto stage = [&](int st, int wslot, int hslot) {
#pragma unroll
      for (int i = 0; i < kWInst; ++i) load_w(src, st, wslot, i);
#pragma unroll
      for (int i = 0; i < kHInst; ++i) load_h(src, st, hslot, i);
    };
    stage(0, w0, h0);
    stage(min(1, ns - 1), w1, h1);
    wait_vm_lds_and_barrier<kWInst + kHInst>();  // stage 0 has landed
#pragma unroll
    for (int f = 0; f < TM; ++f) xa[f] = frag(w0, h0, 0, f);
#pragma unroll
    for (int f = 0; f < TN; ++f) xb[f] = frag(w0, h0, 0, TM + f);
  };
  start();
  for (;;) {
    const int nxt = s + step;
    const bool next = nxt < s_end;
    int nvt = 0, nrt = 0;
    if (next) {
      band_tile(nxt, n_vtiles, n_rtiles, nvt, nrt);
      nsrc = source(nvt, nrt);
    }
    const bool pre = next && chain;

    // One k step: the MFMAs from (ca, cb), the fragments of k step `half` of the stage in slots
    // wslot / hslot into (na, nb), and the n_loads calls load_one(l); loads and fragment reads
    // spread over the first three quarters of the MFMAs.
    auto body = [&](int wslot, int hslot, int half, int n_loads, auto load_one,
                    const bf16x8 (&ca)[TM], const bf16x8 (&cb)[TN], bf16x8 (&na)[TM],
                    bf16x8 (&nb)[TN]) {
      auto load_at = [&](int l) { return (6 * l + 1) * kMfmas / (8 * n_loads); };
      auto read_at = [](int f) { return (6 * (f / 2) + 3 + 2 * (f & 1)) * kMfmas / (4 * kReads); };
      int l = 0, f = 0;  // constants of the unrolled code
#pragma unroll
      for (int i = 0; i < kMfmas; ++i) {
        mfma16_tied(acc[i / TN][i % TN], ca[i / TN], cb[i % TN]);
        if (l < n_loads && load_at(l) <= i) load_one(l++);
        if (f < kReads && read_at(f) <= i) {
          if (f < TM)
            na[f] = frag(wslot, hslot, half, f);
          else
            nb[f - TM] = frag(wslot, hslot, half, f);
          ++f;
        }
      }
      static_assert(kWInst <= kMfmas * 7 / 8 && kHInst <= kMfmas * 7 / 8,
                    "every load finds its MFMA");
    };
    // One stage; stage `stage` of p is loaded on the way.
    auto run_stage = [&](const Src& p, int stage) {
      body(w0, h0, 1, kWInst, [&](int l) { load_w(p, stage, w2, l); }, xa, xb, ya, yb);
      // the next stage has landed: all but the W loads just issued
      wait_vm_lds_and_barrier<kWInst>();
      body(w1, h1, 0, kHInst, [&](int l) { load_h(p, stage, h0, l); }, ya, yb, xa, xb);
      const int w_left = w0, h_left = h0;
      w0 = w1;
      w1 = w2;
      w2 = w_left;
      h0 = h1;
      h1 = h_left;
    };
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{};
    acc_fence_in(acc);  // the zeros are in place before the first MFMA reads them
    // The last two stages load the next tile's first two (or, without a next tile or with one
    // stage per tile, this tile's last stage again, never read).
    int st = 0;
    for (; st + 2 < ns; ++st) run_stage(src, st + 2);
    const Src tsrc{pre ? nsrc.w : src.w, pre ? nsrc.h : src.h, pre ? nsrc.w_rows : src.w_rows,
                   pre ? nsrc.h_rows : src.h_rows};
    for (; st < ns; ++st) run_stage(tsrc, pre ? st + 2 - ns : ns - 1);
    if (!pre) wait_vm_lds_and_barrier<0>();  // no DMA in flight
    acc_fence_out(acc);  // every MFMA has written its accumulator before the epilogue reads it

    // Column statistics; the two halves of the vocabulary rows meet through the W slot that the
    // last stage left, which is loaded again only in step a of the next tile's first stage.
    Partial* red = reinterpret_cast<Partial*>(smem + w2);  // [WM][BN]
    float* red2 = reinterpret_cast<float*>(red + WM * BN);
    const bool full = vt * BM + BM <= vocab;
    const int vbase = vt * BM + wm * kWaveM + q4;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      float m2 = kNegBig;
      const Partial p = column_stats16<TM, TN, kTop2>(acc, tn, vbase, vocab, full, &m2);
      if (lane < 16) {
        red[wm * BN + wn * kWaveN + tn * 16 + rho] = p;
        if (kTop2) red2[wm * BN + wn * kWaveN + tn * 16 + rho] = m2;
      }
    }
    __syncthreads();
    const int c = threadIdx.x;  // one column per thread
    if (c < BN) {
      const Partial p = red[c], o = red[BN + c];
      const int row = rt * BN + c;
      if (row < n_rows) {
        part[static_cast<size_t>(row) * n_vtiles + vt] = partial_merge(p, o);
        if (kTop2)
          part2[static_cast<size_t>(row) * n_vtiles + vt] =
              top2_merge(p.m, red2[c], o.m, red2[BN + c]);
      }
    }
    if (!next) break;
    s = nxt;
    vt = nvt;
    rt = nrt;
    src = nsrc;
    __syncthreads();  // every wave is done with the reduction's slot (and, without pre, the ring)
    if (!pre) start();
  }
}

template <int TN, bool kTop2>
__global__ __launch_bounds__(256, 1) void lmhead_tile_kernel(
    const uint16_t* __restrict__ h, const uint16_t* __restrict__ w, int n_rows, int hidden,
    int vocab, int n_vtiles, int n_rtiles, Partial* __restrict__ part,
    float* __restrict__ part2) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[TileShape<TN>::kLdsBytes];

  // this workgroup's tiles: s0, s0 + step, ... below s_end
  const int n_tiles = n_vtiles * n_rtiles;
  const int g = blockIdx.x, groups = gridDim.x;
  int s0 = g, step = groups, s_end = n_tiles;
  if (groups == kTileGroups) {
    const int x = g % kXcds;
    s_end = static_cast<int>(static_cast<long long>(n_tiles) * (x + 1) / kXcds);
    s0 = static_cast<int>(static_cast<long long>(n_tiles) * x / kXcds) + g / kXcds;
    step = kTileGroups / kXcds;
  }
  if (s0 >= s_end) return;  // whole workgroup

  // the wave index is the same on every lane: taken as a scalar, so the LDS destinations of the
  // loads (M0) are scalar arithmetic
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  tile_run<TN, kTop2>(smem, h, w, n_rows, hidden, vocab, n_vtiles, n_rtiles, part, part2, s0, step,
                      s_end, wave);
}

// Tile kernel of the large-batch path: 4 waves, one workgroup per compute unit.  1000 positions of a
// 126464 x 4096 head take 768 us, against 900 us with stages of 32 columns (64 contiguous bytes per
// row and load: twice the L2 requests), 2048 positions of 126464 x 2048 811 against 949 us.  With two
// waves loading W and two loading h, and the body once per role, it was 781 and 827 us.
// Measured and dropped (with 32x32x16 blocks): 8 waves of 128 x 64 (10.55 ms), 256 x 128 tiles
// with a ring of 3 at two workgroups per compute unit (11.8 ms), stages reaching LDS through
// registers (9.65 ms), 384 x 256 tiles (384 accumulators per lane: the compiler spills).
template <int TN, bool kTop2>
hipError_t launch_tile_tn(int n_rows, int hidden, int vocab, const void* h, const void* w,
                          Partial* part, float* part2, hipStream_t s) {
  const int n_vtiles = tile_vtiles(vocab);
  const int n_rtiles = (n_rows + 32 * TN - 1) / (32 * TN);
  const int n_tiles = n_vtiles * n_rtiles;
  const int groups = n_tiles >= kTileGroups ? kTileGroups : n_tiles;
  hipLaunchKernelGGL((lmhead_tile_kernel<TN, kTop2>), dim3(groups), dim3(256), 0, s,
                     static_cast<const uint16_t*>(h), static_cast<const uint16_t*>(w), n_rows,
                     hidden, vocab, n_vtiles, n_rtiles, part, part2);
  return hipGetLastError();
}

// Width of the position tiles in 32 positions: the one whose rounds of kTileGroups tiles cost
// least, a tile of 32 TN positions counting TN + 3.  Per round of tiles (126464 x 4096, 384 to
// 512 positions) TN = 3 .. 8 take 59, 66, 77, 87, 98 and 107 us: MFMAs and h loads go with TN,
// the rest (W's loads, LDS traffic and latency) counts as three.  Up to 160 positions the tiles
// are bound by W from HBM and the narrowest that covers them is the best as well (128 positions:
// 183 us at TN = 4, 209 us at TN = 8).  On equal cost the wider tile, which reads less from L2.
// Results do not depend on the width: a column's statistics are formed per vocabulary tile.
int tile_width(int n_rows, int vocab) {
  const long n_vtiles = tile_vtiles(vocab);
  int best = 0;
  long best_cost = 0;
  for (int tn = 8; tn >= 3; --tn) {
    const long n_tiles = n_vtiles * ((n_rows + 32 * tn - 1) / (32 * tn));
    const long cost = (n_tiles + kTileGroups - 1) / kTileGroups * (tn + 3);
    if (best == 0 || cost < best_cost) {
      best = tn;
      best_cost = cost;
    }
  }
  return best;
}

template <bool kTop2>
hipError_t launch_tile(int n_rows, int hidden, int vocab, const void* h, const void* w,
                       Partial* part, float* part2, hipStream_t s) {
  auto go = [&](auto tn) {
    return launch_tile_tn<tn.value, kTop2>(n_rows, hidden, vocab, h, w, part, part2, s);
  };
  switch (tile_width(n_rows, vocab)) {
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    default: return go(std::integral_constant<int, 8>{});
  }
}

// ---------------------------------------------------------------------------------------
// fp32 kernel: one workgroup of four wavefronts per slice of vocabulary rows and 32 positions, on
// 16x16x4 fp32 MFMAs (fp32 multiply-adds).  Lane l loads 16 bytes, columns 16 j + 4 (l / 16) .. +3
// of row l % 16, of W and of h straight into the operand registers: element e of them is the k-slot
// of MFMA e, so four lanes read 64 contiguous bytes of a row and nothing passes through LDS.
// Slices have 256 rows, or 64 where 256 would leave compute units without work (f32_slice_rows).
// 32 positions of a 2048 x 256 head: 8.4 us, against 37 us for a thread per (row, vocabulary
// entry) walking its row of W alone.
// ---------------------------------------------------------------------------------------
constexpr int kF32SliceRows = 256;
constexpr int kF32SmallSliceRows = 64;
constexpr int kF32Waves = 4;
constexpr int kF32NT = 2;  // 16-position tiles per workgroup

// Rows per slice.  Slices of 64 rows make four times the workgroups and partials: only where
// 256-row slices would give fewer workgroups than compute units, so the partials stay few.  That is
// up to f32_small_slice_rows position rows.
int f32_small_slice_rows(int vocab) {
  const int slices = (vocab + kF32SliceRows - 1) / kF32SliceRows;
  return 255 / slices * 16 * kF32NT;
}
int f32_slice_rows(int n_rows, int vocab) {
  return n_rows <= f32_small_slice_rows(vocab) ? kF32SmallSliceRows : kF32SliceRows;
}

// Four floats of row `row` from column `col`; columns from `n` on are zero.
__device__ __forceinline__ f32x4 load4_f32(const float* __restrict__ row, int col, int n) {
  if (col + 4 <= n) return *reinterpret_cast<const f32x4u*>(row + col);
  f32x4 x;
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = col + e < n ? row[col + e] : 0.f;
  return x;
}

template <int TM, bool kTop2>
__global__ __launch_bounds__(kF32Waves * 64) void lmhead_f32_kernel(
    const float* __restrict__ h, const float* __restrict__ w, int n_rows, int hidden, int vocab,
    int n_slices, Partial* __restrict__ part, float* __restrict__ part2) {
  constexpr int NT = kF32NT, kRows = 16 * NT;
  __shared__ Partial red[kF32Waves][kRows];
  __shared__ float red2[kF32Waves][kRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 4, l16 = lane & 15;
  const int slice = blockIdx.x, row0 = blockIdx.y * kRows;
  const int wb = (slice * kF32Waves + wave) * 16 * TM;  // this wave's vocabulary rows
  const int we = min(vocab, wb + 16 * TM);
  // rows past the end repeat a valid one; their logits are left out below
  const float* wp[TM];
  const float* hp[NT];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
    wp[tm] = w + static_cast<size_t>(min(wb + 16 * tm + l16, vocab - 1)) * hidden;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    hp[nt] = h + static_cast<size_t>(min(row0 + 16 * nt + l16, n_rows - 1)) * hidden;
  f32x4 acc[TM][NT];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = f32x4{};
  auto step = [&](const f32x4 (&a)[TM], const f32x4 (&b)[NT]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = mfma16_f32(a[tm][e], b[nt][e], acc[tm][nt]);
  };
  f32x4 a[TM], b[NT];
  // whole 16-column steps, four at a time with their loads in flight together
  constexpr int kAhead = 4;
  const int whole = hidden / (16 * kAhead) * (16 * kAhead);
  for (int k = 0; k < whole; k += 16 * kAhead) {
    f32x4 aa[kAhead][TM], bb[kAhead][NT];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int col = k + 16 * j + 4 * grp;
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) aa[j][tm] = *reinterpret_cast<const f32x4u*>(wp[tm] + col);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) bb[j][nt] = *reinterpret_cast<const f32x4u*>(hp[nt] + col);
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) step(aa[j], bb[j]);
  }
  for (int k = whole; k < hidden; k += 16) {
    const int col = k + 4 * grp;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) a[tm] = load4_f32(wp[tm], col, hidden);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) b[nt] = load4_f32(hp[nt], col, hidden);
    step(a, b);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float m2 = kNegBig;
    const Partial p = wave_column_stats<TM, NT, kTop2, true>(acc, nt, wb, we, lane, m2);
    if (lane < 16) {
      red[wave][nt * 16 + l16] = p;
      if (kTop2) red2[wave][nt * 16 + l16] = m2;
    }
  }
  __syncthreads();
  if (tid < kRows && row0 + tid < n_rows) {
    Partial p = red[0][tid];
    float m2 = kTop2 ? red2[0][tid] : kNegBig;
#pragma unroll
    for (int k = 1; k < kF32Waves; ++k) {
      const Partial q = red[k][tid];
      if (kTop2) m2 = top2_merge(p.m, m2, q.m, red2[k][tid]);
      p = partial_merge(p, q);
    }
    const size_t at = static_cast<size_t>(row0 + tid) * n_slices + slice;
    part[at] = p;
    if (kTop2) part2[at] = m2;
  }
}

template <bool kTop2>
hipError_t launch_f32(int n_rows, int hidden, int vocab, int n_slices, const void* h,
                      const void* w, Partial* part, float* part2, hipStream_t s) {
  const dim3 grid(n_slices, (n_rows + 16 * kF32NT - 1) / (16 * kF32NT));
  const float* hp = static_cast<const float*>(h);
  const float* wp = static_cast<const float*>(w);
  if (f32_slice_rows(n_rows, vocab) == kF32SliceRows)
    hipLaunchKernelGGL((lmhead_f32_kernel<kF32SliceRows / 64, kTop2>), grid,
                       dim3(kF32Waves * 64), 0, s, hp, wp, n_rows, hidden, vocab, n_slices, part,
                       part2);
  else
    hipLaunchKernelGGL((lmhead_f32_kernel<kF32SmallSliceRows / 64, kTop2>), grid,
                       dim3(kF32Waves * 64), 0, s, hp, wp, n_rows, hidden, vocab, n_slices, part,
                       part2);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// combine: one wavefront per row, fixed merge order (lane-strided, then butterfly)
// ---------------------------------------------------------------------------------------
template <bool kTop2>
__global__ __launch_bounds__(256) void lmhead_combine_kernel(const Partial* __restrict__ part,
                                                             const float* __restrict__ part2,
                                                             int n_rows, int n_slices,
                                                             float* __restrict__ conf,
                                                             float* __restrict__ entropy,
                                                             int32_t* __restrict__ argmax,
                                                             float* __restrict__ max_logit,
                                                             float* __restrict__ top2_gap) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;  // uniform per wavefront
  const Partial* pr = part + static_cast<size_t>(row) * n_slices;
  const Partial p = wave_merge(pr, n_slices, lane);
  float m2 = kNegBig;
  if (kTop2) {
    // (max, second max) over the slices: lane-strided, then a butterfly; exact in any order
    float m = kNegBig;
    const float* p2 = part2 + static_cast<size_t>(row) * n_slices;
    for (int j = lane; j < n_slices; j += 64) {
      const float mj = pr[j].m;
      m2 = top2_merge(m, m2, mj, p2[j]);
      m = fmaxf(m, mj);
    }
    for (int mask = 32; mask >= 1; mask >>= 1) {
      m2 = top2_shfl_merge(m, m2, mask);
      m = fmaxf(m, __shfl_xor(m, mask));
    }
  }
  if (lane == 0) {
    write_row_stats(p, row, conf, entropy, argmax, max_logit);
    // p_(1) - p_(2) = (1 - e^(z2 - m)) / s; 0 when the maximum is shared (z2 = m)
    if (kTop2) top2_gap[row] = (1.0f - fast_exp2((m2 - p.m) * kLog2e)) * (1.0f / p.s);
  }
}

}  // namespace

int lmhead_num_slices(bool bf16, int n_rows, int vocab) {
  if (bf16 && use_stream(n_rows, vocab)) return stream_plan(vocab).groups;
  if (bf16) return tile_vtiles(vocab);
  const int rows = f32_slice_rows(n_rows, vocab);
  return (vocab + rows - 1) / rows;
}

// Workspace: partials [n_rows, n_slices] (16 B each), then with top2 the second-largest logits
// [n_rows, n_slices] (4 B each) from the next 256-byte boundary.
static size_t lmhead_part_bytes(bool bf16, int n_rows, int vocab) {
  const size_t b = static_cast<size_t>(n_rows) * lmhead_num_slices(bf16, n_rows, vocab) *
                   sizeof(Partial);
  return (b + 255) / 256 * 256;
}

size_t lmhead_ws_bytes(bool bf16, int n_rows, int vocab, bool top2) {
  auto bytes = [&](int rows) {
    size_t b = lmhead_part_bytes(bf16, rows, vocab);
    if (top2) b += static_cast<size_t>(rows) * lmhead_num_slices(bf16, rows, vocab) * 4;
    return b;
  };
  // fp32: also enough for every smaller row count, whose slices may be four times as many, so that
  // a workspace made for the largest call serves the others
  return bf16 ? bytes(n_rows)
              : max(bytes(n_rows), bytes(min(n_rows, f32_small_slice_rows(vocab))));
}

hipError_t lmhead_partials(bool bf16, int n_rows, int hidden, int vocab, const void* h,
                           const void* w, void* ws, bool top2, hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  Partial* part = static_cast<Partial*>(ws);
  float* part2 = top2 ? reinterpret_cast<float*>(static_cast<char*>(ws) +
                                                 lmhead_part_bytes(bf16, n_rows, vocab))
                      : nullptr;
  if (!bf16) {
    const int n_slices = lmhead_num_slices(false, n_rows, vocab);
    return top2 ? launch_f32<true>(n_rows, hidden, vocab, n_slices, h, w, part, part2, s)
                : launch_f32<false>(n_rows, hidden, vocab, n_slices, h, w, part, part2, s);
  }
  if (use_stream(n_rows, vocab))
    return top2 ? launch_stream_rows<true>(n_rows, hidden, vocab, h, w, part, part2, s)
                : launch_stream_rows<false>(n_rows, hidden, vocab, h, w, part, part2, s);
  return top2 ? launch_tile<true>(n_rows, hidden, vocab, h, w, part, part2, s)
              : launch_tile<false>(n_rows, hidden, vocab, h, w, part, part2, s);
}

bool lmhead_hosts_attn(bool bf16, int n_rows, int vocab, const AttnArgs& a) {
  return bf16 && n_rows > 0 && use_stream(n_rows, vocab) && stream_plan(vocab).waves == 16 &&
         attn_small_ok(bf16, a);
}

hipError_t lmhead_partials_attn(int n_rows, int hidden, int vocab, const void* h, const void* w,
                                void* ws, const AttnArgs& a, void* attn_ws, hipStream_t s) {
  const SplitPlan sp = split_plan(a.batch, a.max_block, attn_max_keys(a), a.hq, a.hkv);
  const HostedAttn ha{attn_params(a, sp, attn_ws), attn_small_units(a, sp), a.head_dim};
  return launch_stream_rows<false>(n_rows, hidden, vocab, h, w, static_cast<Partial*>(ws),
                                   nullptr, s, ha);
}

hipError_t lmhead_combine(bool bf16, int n_rows, int vocab, const void* ws, float* conf,
                          float* entropy, int32_t* argmax, float* max_logit, float* top2_gap,
                          hipStream_t s) {
  if (n_rows == 0) return hipSuccess;
  const int n_slices = lmhead_num_slices(bf16, n_rows, vocab);
  const Partial* part = static_cast<const Partial*>(ws);
  const dim3 grid((n_rows + 3) / 4);
  if (top2_gap) {
    const float* part2 = reinterpret_cast<const float*>(static_cast<const char*>(ws) +
                                                        lmhead_part_bytes(bf16, n_rows, vocab));
    hipLaunchKernelGGL(lmhead_combine_kernel<true>, grid, dim3(256), 0, s, part, part2, n_rows,
                       n_slices, conf, entropy, argmax, max_logit, top2_gap);
  } else {
    hipLaunchKernelGGL(lmhead_combine_kernel<false>, grid, dim3(256), 0, s, part, nullptr,
                       n_rows, n_slices, conf, entropy, argmax, max_logit, nullptr);
  }
  return hipGetLastError();
}

}  // namespace eb
