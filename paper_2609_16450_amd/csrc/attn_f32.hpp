// Block attention in fp32, shared by the attention kernel and the fp32 step.
#pragma once

#include <cfloat>

#include "eb_common.hpp"
#include "eb_internal.hpp"

namespace eb {
namespace {

// fp32 attention, as the role of a workgroup: a kernel of its own (attn_f32_kernel) or, in a small
// step, the last workgroups of the epilogue launch, which saves the step a launch.  One workgroup
// of kWaves wavefronts per (sequence, K/V head, 16 query rows), where the query rows are the
// (position, head-in-group) pairs.  Wave v takes the 16-key chunks v, v + kWaves, ... of the
// sequence's keys with an online softmax of its own, and the waves' partial results are merged
// through LDS.  Scores are formed transposed, S^T = K Q^T, by 16x16x4 fp32 MFMAs (fp32
// multiply-adds): lane l owns query l % 16 and holds keys 4 (l / 16) + r of the chunk, which are
// exactly the k-slots of the B operand of O^T = V^T P^T, one register r per MFMA.  Contraction
// indices are permuted so that K and Q arrive by 16-byte loads; K and V come straight from global
// memory (each element is used once per workgroup).  Bound by latency at the sizes this path
// serves: 32 rows x 4 heads x 64 over 128 keys take 6.3 us, where a wavefront per (row, head) that
// walked the keys one by one took 61 us.
struct AttnParamsF32 {
  const int32_t* cu_block;
  const int32_t* cu_prefix;
  int hq, hkv, group, tiles;
  float scale;
  const float* q;
  const float* k_blk;
  const float* v_blk;
  const float* k_pre;
  const float* v_pre;
  float* out;
  const int32_t* cu_suffix;  // nullptr: no suffix segment
  const float* k_suf;
  const float* v_suf;
};

constexpr int kF32Waves = 8;  // waves over the keys in a small step, and of launch_attn_f32
constexpr int kF32Rows = 16;  // query rows per workgroup
constexpr int kF32Keys = 16;  // keys per chunk

// Workgroups of the role, one per (tile of query rows, K/V head, sequence), and its parameters.
inline long attn_f32_tiles(const AttnArgs& a) {
  return (static_cast<long>(a.max_block) * (a.hq / a.hkv) + kF32Rows - 1) / kF32Rows;
}
inline long attn_f32_groups(const AttnArgs& a) { return attn_f32_tiles(a) * a.hkv * a.batch; }
// Too few rows and keys for MFMA tiles (see launch_attn_f32).
inline bool attn_f32_few(const AttnArgs& a) {
  return static_cast<long>(a.max_block) * (a.hq / a.hkv) * attn_max_keys(a) <= 8;
}
inline AttnParamsF32 attn_params_f32(const AttnArgs& a) {
  auto f = [](const void* x) { return static_cast<const float*>(x); };
  return AttnParamsF32{a.cu_block, a.cu_prefix, a.hq, a.hkv, a.hq / a.hkv,
                       static_cast<int>(attn_f32_tiles(a)), a.scale, f(a.q), f(a.k_blk),
                       f(a.v_blk), f(a.k_pre), f(a.v_pre), static_cast<float*>(a.out),
                       a.cu_suffix, f(a.k_suf), f(a.v_suf)};
}

// Role of the workgroup of tile `tile`, K/V head g and sequence b.  Every thread of the workgroup
// calls it; waves past kWaves only help with the final merge, so the results do not depend on the
// workgroup's size.  Nor do they depend on kWaves as long as no wave has a second chunk: a wave
// without keys adds exact zeros.
template <int D, int kThreads, int kWaves>
__device__ __forceinline__ void attn_f32_role(const AttnParamsF32& p, int tile, int g, int b) {
  constexpr int kChunks = D / 16;  // 16-column chunks of the head dimension
  constexpr int kPitch = D + 4;    // LDS row pitch of a partial O
  __shared__ __attribute__((aligned(16))) float s_o[kWaves][kF32Rows * kPitch];
  __shared__ float s_m[kWaves][kF32Rows], s_l[kWaves][kF32Rows];
  const int row0 = tile * kF32Rows;
  const int bbeg = p.cu_block[b];
  const int len = p.cu_block[b + 1] - bbeg;
  const int G = p.group;
  const int n_rows = len * G;
  if (row0 >= n_rows) return;  // whole workgroup
  const int pbeg = p.cu_prefix[b];
  const int plen = p.cu_prefix[b + 1] - pbeg;
  const int sbeg = p.cu_suffix ? p.cu_suffix[b] : 0;
  const int slen = p.cu_suffix ? p.cu_suffix[b + 1] - sbeg : 0;
  const int n_keys = plen + len + slen;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 4, l16 = lane & 15;

  // element offset of query row i of this workgroup (rows past the end repeat the last one)
  auto row_off = [&](int i) {
    const int r = min(row0 + i, n_rows - 1);
    return (static_cast<size_t>(bbeg + r / G) * p.hq + g * G + r % G) * D;
  };
  // key j of the sequence: prefix rows, then block rows, then suffix rows (an unordered set)
  auto key_src = [&](int j, const float* pre, const float* blk, const float* suf) -> const float* {
    if (j < plen) return pre + (static_cast<size_t>(pbeg + j) * p.hkv + g) * D;
    if (j < plen + len) return blk + (static_cast<size_t>(bbeg + j - plen) * p.hkv + g) * D;
    return suf + (static_cast<size_t>(sbeg + j - plen - len) * p.hkv + g) * D;
  };

  // MFMA e of chunk c contracts over d = 16 c + 4 (l / 16) + e.
  if (wave < kWaves) {
    f32x4u qf[kChunks];
    const float* q = p.q + row_off(l16) + 4 * grp;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) qf[c] = *reinterpret_cast<const f32x4u*>(q + 16 * c);
    f32x4 o[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) o[c] = f32x4{};
    // from the lowest finite value on: a chunk whose scores are all -inf then has weights of zero
    float m_run = -FLT_MAX, l_run = 0.f;
    for (int k0 = wave * kF32Keys; k0 < n_keys; k0 += kWaves * kF32Keys) {
      // keys past the end are loaded from the last, valid one; their scores are set to -inf
      const float* kp = key_src(min(k0 + l16, n_keys - 1), p.k_pre, p.k_blk, p.k_suf) + 4 * grp;
      f32x4u kf[kChunks];
#pragma unroll
      for (int c = 0; c < kChunks; ++c) kf[c] = *reinterpret_cast<const f32x4u*>(kp + 16 * c);
      float vf[4][kChunks];  // V of key k0 + 4 grp + r at d = 16 c + l16
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* vp = key_src(min(k0 + 4 * grp + r, n_keys - 1), p.v_pre, p.v_blk, p.v_suf);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) vf[r][c] = vp[16 * c + l16];
      }
      if (k0 + kF32Keys > n_keys) {  // no V past the end: its weight of zero times infinity is NaN
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < kChunks; ++c)
            vf[r][c] = k0 + 4 * grp + r < n_keys ? vf[r][c] : 0.f;
      }
      f32x4 acc[2] = {f32x4{}, f32x4{}};
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e & 1] = mfma16_f32(kf[c][e], qf[c][e], acc[e & 1]);
      float sc[4], mloc = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[r] = k0 + 4 * grp + r < n_keys ? (acc[0][r] + acc[1][r]) * p.scale : -INFINITY;
        mloc = fmaxf(mloc, sc[r]);
      }
      mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
      const float m_new = fmaxf(m_run, mloc);
      const float alpha = expf(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < kChunks; ++c) o[c] *= alpha;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = expf(sc[r] - m_new);
        l_run += e;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) o[c] = mfma16_f32(vf[r][c], e, o[c]);
      }
    }
    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    if (grp == 0) {
      s_m[wave][l16] = m_run;
      s_l[wave][l16] = l_tot;
    }
    // register r of o[c]: d = 16 c + 4 (l / 16) + r of query l % 16
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      *reinterpret_cast<f32x4*>(&s_o[wave][l16 * kPitch + 16 * c + 4 * grp]) = o[c];
  }
  __syncthreads();
  // merge in wave order; a wave without keys has l = 0 and o = 0
  for (int i = tid; i < kF32Rows * D; i += kThreads) {
    const int r = i / D, d = i % D;
    if (row0 + r >= n_rows) break;
    float m = s_m[0][r];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) m = fmaxf(m, s_m[v][r]);
    float l = 0.f, x = 0.f;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      const float f = expf(s_m[v][r] - m);
      l = fmaf(f, s_l[v][r], l);
      x = fmaf(f, s_o[v][r * kPitch + d], x);
    }
    p.out[row_off(r) + d] = x / l;
  }
}

}  // namespace
}  // namespace eb
