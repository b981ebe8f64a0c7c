// Segmented unmask with the anti-stall fallback (the block step is in unmask_block.hpp), one
// workgroup per block, and the LPS feature rows of each block.
#include "eb_common.hpp"
#include "eb_internal.hpp"
#include "unmask_block.hpp"

namespace eb {
namespace {

constexpr int kThreads = kUnmaskThreads;

template <Rule R>
__global__ __launch_bounds__(kThreads) void unmask_kernel(
    const int32_t* __restrict__ cu_block, const float* __restrict__ conf,
    const int32_t* __restrict__ argmax, const float* __restrict__ tau, RuleArgs ra,
    uint8_t* __restrict__ masked, int32_t* __restrict__ tokens, uint8_t* __restrict__ unmask,
    int32_t* __restrict__ n_commit, uint8_t* __restrict__ resolved) {
  unmask_block<R>(blockIdx.x, cu_block, conf, argmax, tau, ra, masked, tokens, unmask, n_commit,
                  resolved);
}

// Budgeted block step (Eq. prelim-update with a budget m), one workgroup per block: a masked row
// passes when conf >= tau_b or fewer than m masked rows of the block rank above it (larger conf, or
// equal conf and a lower row); the fallback and the commit are those of unmask_block.
//
// Each row's rank is counted once, by four lanes that share the block's rows four at a time from
// LDS (an unmasked row is a NaN there, which compares with nothing).  Bound by latency, as the
// counts of a block of 256 rows are 65536 compares: 64 blocks of 16 to 256 rows take 9.1 us, where
// one thread per row counting twice took 52 us.  Blocks of more than kRankTile rows are staged
// tile by tile.
constexpr int kRankLanes = 4;    // lanes that count one row's rank
constexpr int kRankTile = 2048;  // rows of a block staged at once

template <int kTopmThreads>  // 64, 256, 512 or 1024
__global__ __launch_bounds__(kTopmThreads) void unmask_topm_kernel(
    const int32_t* __restrict__ cu_block, const float* __restrict__ conf,
    const int32_t* __restrict__ argmax, const float* __restrict__ tau, int budget,
    uint8_t* __restrict__ masked, int32_t* __restrict__ tokens, uint8_t* __restrict__ unmask,
    int32_t* __restrict__ n_commit, uint8_t* __restrict__ resolved) {
  constexpr int kWaves = kTopmThreads / 64;
  constexpr int kRankRows = kTopmThreads / kRankLanes;  // rows per round
  __shared__ __attribute__((aligned(16))) float s_key[kRankTile];
  __shared__ int s_masked[kWaves], s_pass[kWaves];
  __shared__ Best s_best[kWaves];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int beg = cu_block[b], len = cu_block[b + 1] - beg;
  const float tb = tau[b];
  // rows t0 .. t0 + kRankTile - 1 of the block into LDS, NaN past the end
  auto stage = [&](int t0) {
    for (int j = tid; j < kRankTile && j < ((len - t0 + 3) & ~3); j += kTopmThreads)
      s_key[j] = t0 + j < len && masked[beg + t0 + j] ? conf[beg + t0 + j] : NAN;
  };
  const bool one_tile = len <= kRankTile;
  if (one_tile) stage(0);

  int n_masked = 0;
  Best best{-INFINITY, kNoIndex};
  for (int i = beg + tid; i < beg + len; i += kTopmThreads) {
    if (masked[i]) {
      const float c = conf[i];
      ++n_masked;
      if (c > best.c) best = Best{c, i};  // rows ascend per thread: strict > keeps the lowest
    }
  }
  for (int mask = 32; mask >= 1; mask >>= 1) {
    n_masked += __shfl_xor(n_masked, mask);
    Best o{__shfl_xor(best.c, mask), __shfl_xor(best.i, mask)};
    best = best_of(best, o);
  }
  if (lane == 0) {
    s_masked[wave] = n_masked;
    s_best[wave] = best;
  }
  __syncthreads();
  n_masked = 0;
  best = Best{-INFINITY, kNoIndex};
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    n_masked += s_masked[k];
    best = best_of(best, s_best[k]);
  }

  // Decide every row, kRankRows per round, without touching the mask flags: lane 0 of a row's four
  // writes `unmask` and remembers the decision of the first 32 rounds.
  const bool all = budget >= n_masked;      // every masked row is within the budget
  const bool ranked = budget > 0 && !all;
  const int part = tid & (kRankLanes - 1), own = tid / kRankLanes;
  uint32_t took = 0;
  int n_pass = 0;
  for (int r0 = 0, round = 0; r0 < len; r0 += kRankRows, ++round) {
    const int i = r0 + own;
    const bool mine = i < len;
    const float c = mine ? conf[beg + i] : 0.f;
    const bool mk = mine && masked[beg + i];
    int rank = 0;
    if (ranked) {
      for (int t0 = 0; t0 < len; t0 += kRankTile) {
        if (!one_tile) {
          __syncthreads();
          stage(t0);
          __syncthreads();
        }
        const int tn = min(kRankTile, len - t0);
        for (int j = 4 * part; j < tn; j += 4 * kRankLanes) {
          const f32x4 k = *reinterpret_cast<const f32x4*>(s_key + j);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            rank += (k[e] > c || (k[e] == c && t0 + j + e < i)) ? 1 : 0;
        }
      }
      rank += __shfl_xor(rank, 1);
      rank += __shfl_xor(rank, 2);
    }
    const bool take = mk && (c >= tb || all || (ranked && rank < budget));
    if (part == 0) {
      n_pass += take ? 1 : 0;
      if (mine) unmask[beg + i] = take ? 1 : 0;
      if (round < 32) took |= static_cast<uint32_t>(take) << round;
    }
  }
  for (int mask = 32; mask >= 1; mask >>= 1) n_pass += __shfl_xor(n_pass, mask);
  if (lane == 0) s_pass[wave] = n_pass;
  __syncthreads();  // every decision is made before any mask flag changes
  n_pass = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) n_pass += s_pass[k];
  if (n_pass > 0) {
    if (part == 0)
      for (int r0 = 0, round = 0; r0 < len; r0 += kRankRows, ++round) {
        const int i = beg + r0 + own;
        if (i >= beg + len) break;
        if (round < 32 ? (took >> round) & 1 : unmask[i] != 0) {
          tokens[i] = argmax[i];
          masked[i] = 0;
        }
      }
  } else if (part == 0) {  // fallback: the best masked row, if any
    for (int i = beg + own; i < beg + len; i += kRankRows)
      if (i == best.i) {
        unmask[i] = 1;
        tokens[i] = argmax[i];
        masked[i] = 0;
      }
  }
  if (tid == 0) {
    const int commits = n_pass > 0 ? n_pass : (n_masked > 0 ? 1 : 0);
    n_commit[b] = commits;
    resolved[b] = (n_masked - commits == 0) ? 1 : 0;
  }
}

// LPS router inputs (Sec. 5.2, Alg. 5), one workgroup per block: the block's mask ratio rho
// before this step's commit, then per row feat = (kappa, H * inv_ln_v, Delta, rho) and the
// intra-block position pos = (p_i - p_first) / len, where p is the row's sequence position
// (seq_pos) or, without seq_pos, its packed row index.
__global__ __launch_bounds__(kThreads) void lps_features_kernel(
    const int32_t* __restrict__ cu_block, float inv_ln_v, const float* __restrict__ conf,
    const float* __restrict__ entropy, const float* __restrict__ gap,
    const uint8_t* __restrict__ masked, const int32_t* __restrict__ seq_pos,
    float* __restrict__ feat, float* __restrict__ pos, float* __restrict__ mask_ratio) {
  __shared__ int s_cnt[kThreads / 64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int beg = cu_block[b], end = cu_block[b + 1], len = end - beg;
  int cnt = 0;
  for (int i = beg + tid; i < end; i += kThreads) cnt += masked[i] ? 1 : 0;
  for (int mask = 32; mask >= 1; mask >>= 1) cnt += __shfl_xor(cnt, mask);
  if (lane == 0) s_cnt[wave] = cnt;
  __syncthreads();
  cnt = 0;
  for (int k = 0; k < kThreads / 64; ++k) cnt += s_cnt[k];
  const float rho = len > 0 ? static_cast<float>(cnt) / static_cast<float>(len) : 0.f;
  if (tid == 0 && mask_ratio) mask_ratio[b] = rho;
  const int first = (seq_pos && len > 0) ? seq_pos[beg] : beg;
  for (int i = beg + tid; i < end; i += kThreads) {
    *reinterpret_cast<f32x4*>(feat + 4 * static_cast<size_t>(i)) =
        f32x4{conf[i], entropy[i] * inv_ln_v, gap[i], rho};
    const int p = seq_pos ? seq_pos[i] : i;
    pos[i] = static_cast<float>(p - first) / static_cast<float>(len);
  }
}

}  // namespace

hipError_t unmask_select(int batch, int max_block, const int32_t* cu_block, const float* conf,
                         const int32_t* argmax, const float* tau, uint8_t* masked,
                         int32_t* tokens, uint8_t* unmask, int32_t* n_commit, uint8_t* resolved,
                         hipStream_t s) {
  (void)max_block;
  const RuleArgs ra{nullptr, 0.f};
  hipLaunchKernelGGL(unmask_kernel<kThreshold>, dim3(batch), dim3(kThreads), 0, s, cu_block,
                     conf, argmax, tau, ra, masked, tokens, unmask, n_commit, resolved);
  return hipGetLastError();
}

hipError_t unmask_select_lps(int batch, const int32_t* cu_block, const float* conf,
                             const int32_t* argmax, const float* tau, const float* p_psi,
                             float tau_psi, uint8_t* masked, int32_t* tokens, uint8_t* unmask,
                             int32_t* n_commit, uint8_t* resolved, hipStream_t s) {
  const RuleArgs ra{p_psi, tau_psi};
  hipLaunchKernelGGL(unmask_kernel<kUnion>, dim3(batch), dim3(kThreads), 0, s, cu_block, conf,
                     argmax, tau, ra, masked, tokens, unmask, n_commit, resolved);
  return hipGetLastError();
}

hipError_t unmask_select_topm(int batch, int max_block, const int32_t* cu_block, const float* conf,
                              const int32_t* argmax, const float* tau, int m, uint8_t* masked,
                              int32_t* tokens, uint8_t* unmask, int32_t* n_commit,
                              uint8_t* resolved, hipStream_t s) {
  if (m == 0)  // no row is within the budget: the threshold rule
    return unmask_select(batch, max_block, cu_block, conf, argmax, tau, masked, tokens, unmask,
                         n_commit, resolved, s);
  // The fewest threads that rank a whole block in one round, up to 1024: a barrier costs less with
  // fewer waves, and small workgroups share a compute unit.  With the copy that refills the mask
  // flags, 32768 blocks of one row take 25 us with 64 threads, 290 us with 1024; 64 blocks of 16,
  // 64 and 128 rows 6.3, 7.4 and 8.5 us with one round of 64, 256 and 512 threads, 7.6, 8.4 and 9.1
  // us with 1024, and with two rounds 7.6 (32 rows by 64 threads) and 10.5 us (128 by 256).
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(threads), 0, s, cu_block, conf, argmax, tau, m,
                       masked, tokens, unmask, n_commit, resolved);
    return hipGetLastError();
  };
  if (max_block <= 64 / kRankLanes) return go(unmask_topm_kernel<64>, 64);
  if (max_block <= 256 / kRankLanes) return go(unmask_topm_kernel<256>, 256);
  if (max_block <= 512 / kRankLanes) return go(unmask_topm_kernel<512>, 512);
  return go(unmask_topm_kernel<1024>, 1024);
}

hipError_t lps_features(int batch, const int32_t* cu_block, int vocab, const float* conf,
                        const float* entropy, const float* gap, const uint8_t* masked,
                        const int32_t* seq_pos, float* feat, float* pos, float* mask_ratio,
                        hipStream_t s) {
  const float inv_ln_v = static_cast<float>(1.0 / log(static_cast<double>(vocab)));
  hipLaunchKernelGGL(lps_features_kernel, dim3(batch), dim3(kThreads), 0, s, cu_block, inv_ln_v,
                     conf, entropy, gap, masked, seq_pos, feat, pos, mask_ratio);
  return hipGetLastError();
}

}  // namespace eb
