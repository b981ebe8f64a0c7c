// One block step of the unmask rules, shared by the unmask kernels and the fused step epilogue.
//
// For block b: masked rows passing the accept rule are committed; if none passes and a row is
// still masked, the masked row of largest conf (lowest row on ties) is committed.  A commit
// writes the top-1 token and clears the mask flag.
#pragma once

#include "eb_common.hpp"

namespace eb {
namespace {

constexpr int kUnmaskThreads = 256;  // threads of a workgroup running unmask_block

struct Best {
  float c;
  int32_t i;
};

// Larger conf wins; equal conf -> lower row.  Symmetric, so both butterfly lanes agree.
__device__ __forceinline__ Best best_of(Best a, Best b) {
  if (a.c > b.c) return a;
  if (b.c > a.c) return b;
  return a.i <= b.i ? a : b;
}

// Accept rules of one block step:
//   kThreshold: conf >= tau_b (Eq. prelim-update, threshold branch);
//   kUnion:     conf >= tau_b or p_psi > tau_psi (Alg. 5, union accept rule).
// (The rule with a budget m is unmask_topm_kernel.)  Masked rows only.  When no masked row passes,
// the masked row of largest conf (lowest row on ties) is committed (Alg. 5, anti-stall fallback).
enum Rule { kThreshold = 0, kUnion = 1 };

struct RuleArgs {
  const float* p_psi;
  float tau_psi;
};

// Block step of a block of at most 64 rows by one wavefront (the commit, fallback and tie-break
// of unmask_block): lane l holds row `row` (valid when `mine`), its mask flag m, its conf c, its
// top-1 token x, and whether it passes the accept rule.
__device__ __forceinline__ void unmask_wave(int b, int row, bool mine, bool m, float c, int32_t x,
                                            bool pass, uint8_t* __restrict__ masked,
                                            int32_t* __restrict__ tokens,
                                            uint8_t* __restrict__ unmask,
                                            int32_t* __restrict__ n_commit,
                                            uint8_t* __restrict__ resolved, int lane) {
  const bool mk = mine && m;
  int n_masked = mk ? 1 : 0;
  int n_pass = (mk && pass) ? 1 : 0;
  Best best = mk ? Best{c, row} : Best{-INFINITY, kNoIndex};
  for (int mask = 32; mask >= 1; mask >>= 1) {
    n_masked += __shfl_xor(n_masked, mask);
    n_pass += __shfl_xor(n_pass, mask);
    Best o{__shfl_xor(best.c, mask), __shfl_xor(best.i, mask)};
    best = best_of(best, o);
  }
  const bool use_rule = n_pass > 0;
  if (mine) {
    const bool take = mk && (use_rule ? pass : row == best.i);
    unmask[row] = take ? 1 : 0;
    if (take) {
      tokens[row] = x;
      masked[row] = 0;
    }
  }
  if (lane == 0) {
    const int commits = use_rule ? n_pass : (n_masked > 0 ? 1 : 0);
    n_commit[b] = commits;
    resolved[b] = (n_masked - commits == 0) ? 1 : 0;
  }
}

// Step of block b by one workgroup of kThreads threads under rule R.
template <Rule R, int kThreads = kUnmaskThreads>
__device__ __forceinline__ void unmask_block(
    int b, const int32_t* __restrict__ cu_block, const float* __restrict__ conf,
    const int32_t* __restrict__ argmax, const float* __restrict__ tau, RuleArgs ra,
    uint8_t* __restrict__ masked,
    int32_t* __restrict__ tokens, uint8_t* __restrict__ unmask, int32_t* __restrict__ n_commit,
    uint8_t* __restrict__ resolved) {
  __shared__ int s_pass[kThreads / 64], s_masked[kThreads / 64];
  __shared__ Best s_best[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int beg = cu_block[b], end = cu_block[b + 1];
  const float tb = tau[b];

  if (end - beg <= 64) {  // one wavefront: no reduction across waves, no barrier
    if (wave == 0) {
      const int i = beg + lane;
      const bool mine = i < end;
      const bool m = mine && masked[i];
      const float c = mine ? conf[i] : 0.f;
      const int32_t x = mine ? argmax[i] : 0;
      bool pass = c >= tb;
      if constexpr (R == kUnion) pass = pass || (mine && ra.p_psi[i] > ra.tau_psi);
      unmask_wave(b, i, mine, m, c, x, pass, masked, tokens, unmask, n_commit, resolved, lane);
    }
    return;
  }
  // One pass counts the masked rows, finds the best masked row and counts the rows passing
  // the rule.  Each thread then decides and commits its own rows: the rule reads no other
  // row's mask flag, so a row is committed as soon as it is decided.
  int n_masked = 0, n_pass = 0;
  Best best{-INFINITY, kNoIndex};
  for (int i = beg + tid; i < end; i += kThreads) {
    if (masked[i]) {
      const float c = conf[i];
      ++n_masked;
      if (c > best.c) best = Best{c, i};  // rows ascend per thread: strict > keeps the lowest
      bool ok = c >= tb;
      if constexpr (R == kUnion) ok = ok || ra.p_psi[i] > ra.tau_psi;
      n_pass += ok ? 1 : 0;
    }
  }
  for (int mask = 32; mask >= 1; mask >>= 1) {
    n_masked += __shfl_xor(n_masked, mask);
    n_pass += __shfl_xor(n_pass, mask);
    Best o{__shfl_xor(best.c, mask), __shfl_xor(best.i, mask)};
    best = best_of(best, o);
  }
  if (lane == 0) {
    s_masked[wave] = n_masked;
    s_pass[wave] = n_pass;
    s_best[wave] = best;
  }
  __syncthreads();
  n_masked = 0;
  n_pass = 0;
  best = Best{-INFINITY, kNoIndex};
  for (int k = 0; k < kThreads / 64; ++k) {
    n_masked += s_masked[k];
    n_pass += s_pass[k];
    best = best_of(best, s_best[k]);
  }
  const bool use_rule = n_pass > 0;
  for (int i = beg + tid; i < end; i += kThreads) {
    bool take = false;
    if (masked[i]) {
      if (use_rule) {
        take = conf[i] >= tb;
        if constexpr (R == kUnion) take = take || ra.p_psi[i] > ra.tau_psi;
      } else {
        take = i == best.i;
      }
    }
    unmask[i] = take ? 1 : 0;
    if (take) {
      tokens[i] = argmax[i];
      masked[i] = 0;
    }
  }
  if (tid == 0) {
    const int commits = use_rule ? n_pass : (n_masked > 0 ? 1 : 0);
    n_commit[b] = commits;
    resolved[b] = (n_masked - commits == 0) ? 1 : 0;
  }
}

}  // namespace
}  // namespace eb
