// kern_rollout.hip -- priority vectors of MCTS rollouts (DIP, arXiv
// 2504.14145, Sec. 5.1).
//
// A rollout completes a search-tree node's class prefix at random and hands
// the sequence to the interleaving as priorities: the class at position i of
// n gets priority n - i, and every group takes its class's priority.  Rollout
// i of draw d shuffles the classes not in the prefix (ascending order to
// start) with Durstenfeld's Fisher-Yates; for j = m-1 down to 1 the swap
// partner k in [0, j] is (hi32(u) * (j + 1)) >> 32, u the next output of
// SplitMix64 (Steele, Lea and Flood, OOPSLA 2014) started from
// mix(mix(seed + (d + 1) G) + (i + 1) G), G = 0x9E3779B97F4A7C15.
// SplitMix64's states are start + i G, so every swap partner can be drawn
// independently; only the swaps themselves are a serial chain.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace dipsim {

namespace {

constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// A block handles B consecutive rollouts (rows), a wave per row in turn: row
// r belongs to leaf r / per_leaf, whose template is its class prefix followed
// by the other classes ascending, and is that leaf's rollout r % per_leaf,
// drawn with the leaf's draw number.  The lanes draw the row's swap partners,
// then one lane a row swaps (neighbouring rows lie an odd number of words
// apart, so that lanes at equal positions meet different banks), then the
// lanes fill the class-priority table over the partners and write the row.
//
// Bound by the swaps, one LDS round trip each.  A thread a row that drew as it
// swapped, its block writing the rows with as many threads as it held rows,
// took 131 us for 1,024 rollouts of 384 classes and 520 groups, and 65 us for
// 16,384 of 128 classes and 200 groups; this takes 34 and 27.
constexpr int kRolloutThreads = 256;

__global__ __launch_bounds__(kRolloutThreads) void rollout_prio_kernel(RolloutArgs a, int32_t B) {
  extern __shared__ __align__(16) uint32_t sh[];
  const int32_t n = a.n_classes;
  const int64_t first = int64_t(blockIdx.x) * B;
  const int32_t rows = int32_t(a.n - first < B ? a.n - first : B);
  const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  auto seq_of = [&](int32_t rr) { return reinterpret_cast<uint16_t *>(sh + int64_t(rr) * (n | 1)); };
  for (int32_t rr = wave; rr < rows; rr += n_waves) {
    const int64_t leaf = (first + rr) / a.per_leaf, ri = (first + rr) % a.per_leaf;
    const int32_t dep = a.depths[leaf], m = n - dep;
    const int32_t *tmpl = a.seqs + leaf * n;
    const uint64_t draw = a.draw + uint64_t(leaf);
    const uint64_t st = mix(mix(a.seed + (draw + 1) * kGolden) + uint64_t(ri + 1) * kGolden);
    uint16_t *seq = seq_of(rr), *partner = seq + n;
    for (int32_t j = lane; j < m; j += 64) {
      seq[j] = uint16_t(tmpl[dep + j]);
      const uint64_t u = mix(st + uint64_t(m - j) * kGolden);
      partner[j] = uint16_t(((u >> 32) * uint64_t(j + 1)) >> 32);
    }
  }
  __syncthreads();
  if (int32_t(threadIdx.x) < rows) {
    const int64_t leaf = (first + threadIdx.x) / a.per_leaf;
    const int32_t m = n - a.depths[leaf];
    uint16_t *seq = seq_of(threadIdx.x);
    const uint16_t *partner = seq + n;
    uint32_t k = m > 1 ? partner[m - 1] : 0u;
    for (int32_t j = m - 1; j >= 1; --j) {
      const uint32_t k1 = partner[j - 1];       // (partner 0 is drawn, and not used)
      const uint16_t x = seq[j], y = seq[k];
      seq[j] = y;
      seq[k] = x;
      k = k1;
    }
  }
  __syncthreads();
  for (int32_t rr = wave; rr < rows; rr += n_waves) {
    const int64_t leaf = (first + rr) / a.per_leaf;
    const int32_t dep = a.depths[leaf];
    const int32_t *tmpl = a.seqs + leaf * n;
    uint16_t *seq = seq_of(rr), *prio_of = seq + n;
    for (int32_t k = lane; k < n; k += 64)
      prio_of[k < dep ? tmpl[k] : int32_t(seq[k - dep])] = uint16_t(n - k);
  }
  __syncthreads();
  for (int32_t rr = wave; rr < rows; rr += n_waves) {
    const uint16_t *prio_of = seq_of(rr) + n;
    int32_t *out = a.out_prio + (first + rr) * a.G;
    for (int32_t g = lane; g < a.G; g += 64) out[g] = prio_of[a.group_class[g]];
  }
}

}  // namespace

hipError_t launch_rollout_prio(hipStream_t s, const RolloutArgs &a) {
  // rows per block: a power of two up to 64 whose tables fit 64 KiB, a block
  // for every CU and SIMD pair first (512 blocks), but a row for each wave
  const int64_t per = int64_t(a.n_classes | 1) * 4;
  int B = 64;
  while (B > 4 && (a.n + B - 1) / B < 512) B /= 2;
  while (B > 1 && B * per > 65536) B /= 2;
  if (B * per > 65536) return hipErrorInvalidValue;
  const int64_t blocks = (a.n + B - 1) / B;
  hipLaunchKernelGGL(rollout_prio_kernel, dim3(unsigned(blocks)), dim3(kRolloutThreads),
                     size_t(B * per), s, a, B);
  return hipGetLastError();
}

}  // namespace dipsim
