// Block-attention pieces shared by the attention kernels and the fused step epilogue: the bf16
// kernel parameters, the key-split plan, and the merge of one (block row, query head)'s splits.
#pragma once

#include "eb_common.hpp"
#include "eb_internal.hpp"

namespace eb {
namespace {

constexpr int kAttnRowsPerWg = 128;  // query rows (position, head-in-group) per workgroup
constexpr int kAttnKeys = 64;        // keys per LDS stage
// The key split aims at this many workgroups, two per compute unit, however few stages that leaves
// a range.  Half as many where a range would have under 8 stages is up to a tenth faster (15.5
// against 16.7 us with 8 sequences, 16 heads x 64, up to 1500 keys), but the largest probability of
// a row within a range is the one that bf16 holds exactly, so fewer ranges are a larger error:
// 0.00218 against 0.00215 of the result's 2-norm, measured against 64 bits.
constexpr int kAttnTargetWgs = 512;

struct AttnParams {
  const int32_t* cu_block;
  const int32_t* cu_prefix;
  int hq, hkv, group;
  float scale_log2;  // scale * log2(e)
  const uint16_t* q;
  const uint16_t* k_blk;
  const uint16_t* v_blk;
  const uint16_t* k_pre;
  const uint16_t* v_pre;
  uint16_t* out;
  // optional cached suffix segment (dual cache): rows cu_suffix[b] .. cu_suffix[b+1]-1 of
  // k_suf / v_suf are further keys of sequence b; cu_suffix == nullptr: none
  const int32_t* cu_suffix;
  const uint16_t* k_suf;
  const uint16_t* v_suf;
  // key split: keys of a sequence are cut into ranges of kps keys, one workgroup per range;
  // with nsplit > 1 the workgroups write unnormalised partials that attn_merge_kernel (or the
  // fused step epilogue) combines
  int nsplit, kps;
  float* o_part;  // [T * hq * nsplit, D]
  float* m_part;  // [T * hq * nsplit]  running max (log2 units)
  float* l_part;  // [T * hq * nsplit]  sum of 2^(s - m)
};

struct SplitPlan {
  int nsplit, kps;
};

// Key-split plan: enough workgroups to fill the chip, in whole 64-key stages.  max_keys is the
// largest number of keys of a sequence (prefix + block + suffix).
inline SplitPlan split_plan(int batch, int max_block, int max_keys, int hq, int hkv) {
  const int group = hq / hkv;
  const long row_tiles =
      (static_cast<long>(max_block) * group + kAttnRowsPerWg - 1) / kAttnRowsPerWg;
  const long base = row_tiles * hkv * batch;
  const int stages = (max_keys + kAttnKeys - 1) / kAttnKeys;
  int nsplit = static_cast<int>((kAttnTargetWgs + base - 1) / base);
  nsplit = max(1, min(nsplit, stages));
  const int stages_per = (stages + nsplit - 1) / nsplit;
  const int kps = stages_per * kAttnKeys;
  nsplit = (stages * kAttnKeys + kps - 1) / kps;
  return SplitPlan{nsplit, kps};
}

// Parameters of a bf16 launch under plan sp; with a split the partials live in ws as
// o [T * hq * nsplit, D], then m and l [T * hq * nsplit] each.
inline AttnParams attn_params(const AttnArgs& a, const SplitPlan& sp, void* ws) {
  const size_t n_part = static_cast<size_t>(a.total_block) * a.hq * sp.nsplit;
  float* o_part = sp.nsplit > 1 ? static_cast<float*>(ws) : nullptr;
  float* m_part = sp.nsplit > 1 ? o_part + n_part * a.head_dim : nullptr;
  float* l_part = sp.nsplit > 1 ? m_part + n_part : nullptr;
  return AttnParams{a.cu_block, a.cu_prefix, a.hq, a.hkv, a.hq / a.hkv, a.scale * kLog2e,
                    static_cast<const uint16_t*>(a.q), static_cast<const uint16_t*>(a.k_blk),
                    static_cast<const uint16_t*>(a.v_blk), static_cast<const uint16_t*>(a.k_pre),
                    static_cast<const uint16_t*>(a.v_pre), static_cast<uint16_t*>(a.out),
                    a.cu_suffix, static_cast<const uint16_t*>(a.k_suf),
                    static_cast<const uint16_t*>(a.v_suf), sp.nsplit, sp.kps, o_part, m_part,
                    l_part};
}

// Combine the key-split partials of pair rh = row * hq + head (one wavefront, lane = lane id):
// splits merged in index order (max, rescale, sum), output rounded to bf16.  kGroup splits are
// loaded together.  Bound by latency: the first group's loads do not wait for the search of the
// row's sequence, whose number of key ranges only decides which of them count (the others are
// slots of the workspace that no workgroup wrote), and the search is one load per 64 sequences.
// 380 rows x 16 heads x 64 in 7 ranges: 4.1 us, against 7.9 us with a binary search first, the
// maxima next and always 16 ranges loaded last.
template <int D, int kGroup = 16>
__device__ __forceinline__ void attn_merge_pair(const AttnParams& p, int rh, int batch, int lane) {
  constexpr int kPer = D / 64;  // values per lane
  const size_t base = static_cast<size_t>(rh) * p.nsplit;
  float mk[kGroup], lk[kGroup], ok[kGroup][kPer];
  auto load = [&](int k0) {
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      const size_t k = base + min(k0 + j, p.nsplit - 1);
      mk[j] = p.m_part[k];
      lk[j] = p.l_part[k];
#pragma unroll
      for (int e = 0; e < kPer; ++e) ok[j][e] = p.o_part[k * D + lane * kPer + e];
    }
  };
  load(0);
  const int row = rh / p.hq;
  // sequence of this row: the number of sequences that end at or before it (64 at a time)
  int b = 0;
  for (int b0 = 0; b0 < batch; b0 += 64) {
    const bool before = b0 + lane < batch && p.cu_block[b0 + lane + 1] <= row;
    const int n = __popcll(__ballot(before));
    b += n;
    if (n < 64) break;
  }
  const int n_keys = (p.cu_prefix[b + 1] - p.cu_prefix[b]) + (p.cu_block[b + 1] - p.cu_block[b]) +
                     (p.cu_suffix ? p.cu_suffix[b + 1] - p.cu_suffix[b] : 0);
  const int nvalid = min(p.nsplit, (n_keys + p.kps - 1) / p.kps);
  float M = -INFINITY;
#pragma unroll
  for (int j = 0; j < kGroup; ++j)
    if (j < nvalid) M = fmaxf(M, mk[j]);
  // the later groups' maxima, a lane each (fmaxf is exact, so the order does not matter)
  if (nvalid > kGroup) {
    for (int k = kGroup + lane; k < nvalid; k += 64) M = fmaxf(M, p.m_part[base + k]);
    for (int mask = 32; mask >= 1; mask >>= 1) M = fmaxf(M, __shfl_xor(M, mask));
  }
  float acc[kPer] = {};
  float L = 0.f;
  for (int k0 = 0; k0 < nvalid; k0 += kGroup) {
    if (k0 > 0) load(k0);
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      if (k0 + j >= nvalid) continue;
      const float f = fast_exp2(mk[j] - M);
      L = fmaf(f, lk[j], L);
#pragma unroll
      for (int e = 0; e < kPer; ++e) acc[e] = fmaf(f, ok[j][e], acc[e]);
    }
  }
  const float inv = 1.0f / L;
  uint16_t* dst = p.out + static_cast<size_t>(rh) * D + lane * kPer;
#pragma unroll
  for (int e = 0; e < kPer; ++e) dst[e] = f32_to_bf16_bits_rne(acc[e] * inv);
}

}  // namespace
}  // namespace eb
