// kern_selcheck.hip -- candidate schedules under a per-layer memory selection
// (DIP, arXiv 2504.14145, Sec. 5.3), ahead of their re-timed simulation.
//
// With a selection an op's cost and activation depend on its candidate: the
// backward of a stage pair runs the chosen candidate's extra time, and the
// pair holds the candidate's memory.  A block per schedule, its waves
// splitting the ranks; for each of its ranks a wave walks the order 64 ops at
// a time: the op's pair, the pair's choice, the choice's time and memory.  It
// checks that the section is a permutation (a bitmap in LDS) and every choice
// exists, writes each op's extra cost where the simulation kernel reads it in
// order, and keeps the rank's peak memory (a wave scan a step) and the sum of
// its extra costs (left in out_bub, from which the simulation takes it).
//
// Bound: the latency of the four dependent lookups, hidden by up to 32 waves a
// CU; 0.45 ns per schedule and rank of up to 64 ops.  It replaced the general
// kernel's walk of the whole DAG, which looked all of this up in every round of
// every op, but for candidates of few ops, whose ranks leave most of a wave's
// lanes idle here and take few rounds there.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dip_sim.h"
#include "dev_util.h"
#include "internal.h"

namespace dipsim {

namespace {

// inclusive prefix sum over the 64 lanes: within rows of 16, then the rows
// before a lane's own
__device__ __forceinline__ int32_t wave_scan(int32_t v, int lane) {
#pragma unroll
  for (int s = 1; s < 16; s <<= 1) {
    const int32_t y = __shfl_up(v, s, 16);
    if ((lane & 15) >= s) v += y;
  }
  const int32_t r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
                r2 = __builtin_amdgcn_readlane(v, 47);
  const int row = lane >> 4;
  return v + (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
}

extern __shared__ uint32_t sc_bits[];   // [waves][bm_words]

__global__ __launch_bounds__(256) void selcheck_kernel(SelCheckArgs a) {
  __shared__ uint32_t verdict;           // bit 0: invalid, bit 1: over a cap
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave, nw = blockDim.x / kWave;
  const int64_t cand = blockIdx.x;
  if (threadIdx.x == 0) verdict = 0;
  if (cand == 0 && a.retry_count && threadIdx.x < kRetryCounters) a.retry_count[threadIdx.x] = 0;
  __syncthreads();
  uint32_t *bm = sc_bits + wave * a.bm_words;
  const int16_t *row = a.orders + cand * a.stride;
  const uint8_t *choice = a.choice + cand * a.n_pairs;
  int32_t *xrow = a.xcost + cand * a.stride;
  bool bad = false, over = false;
  for (int r = wave; r < a.P; r += nw) {
    const int rb = a.rank_off[r], nr = a.rank_off[r + 1] - rb, pb = a.pair_off[r];
    for (int i = lane; i < a.bm_words; i += kWave) bm[i] = 0;
    wave_lds_order();
    int32_t run = 0, peak = 0, sum = 0;
    for (int p0 = 0; p0 < nr; p0 += kWave) {
      const int p = p0 + lane;
      int32_t d = 0, x = 0;
      if (p < nr) {
        const int lid = row[rb + p];
        bool ok = uint32_t(lid) < uint32_t(nr);
        if (ok) {
          const uint32_t bit = 1u << (lid & 31);
          ok = (atomicOr(bm + (lid >> 5), bit) & bit) == 0;
          const uint32_t w = uint32_t(a.lid_pair[rb + lid]);
          const int64_t pr = int64_t(pb + int(w & 0x7fffffffu)) * kMemoptMaxCands;
          const uint32_t c = choice[pb + int(w & 0x7fffffffu)];
          if (c >= uint32_t(kMemoptMaxCands) || (c > 0 && a.cand_key[pr + c - 1] == kMemoptNoMove)) {
            ok = false;
          } else {
            const int32_t m = a.cand_mem[pr + c];
            d = (w >> 31) ? -m : m;
            if (w >> 31) x = int32_t(a.cand_time[pr + c] - a.cand_time[pr]);
          }
        }
        bad = bad || !ok;
        xrow[rb + p] = x;
      }
      const int32_t s = run + wave_scan(d, lane);
      peak = max(peak, p < nr ? s : 0);
      run = __builtin_amdgcn_readlane(s, kWave - 1);
      sum += x;
    }
    wave_lds_order();
    peak = int32_t(wave_max_u32(uint32_t(peak)));      // (at least 0)
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) sum += __shfl_xor(sum, s);
    const int32_t cap = a.cap[r];
    over = over || (cap >= 0 && peak > cap);
    if (lane == 0) {
      a.out_peak[cand * a.P + r] = peak;
      a.out_bub[cand * a.P + r] = sum;
    }
  }
  if (__any(bad) && lane == 0) atomicOr(&verdict, 1u);
  if (over && lane == 0) atomicOr(&verdict, 2u);
  __syncthreads();
  const uint32_t v = verdict;
  if (v & 1u) {
    for (int r = threadIdx.x; r < a.P; r += blockDim.x) {
      a.out_peak[cand * a.P + r] = -1;
      a.out_bub[cand * a.P + r] = -1;
    }
    if (threadIdx.x == 0) a.out_ms[cand] = -1;
  }
  if (threadIdx.x == 0)
    a.out_flags[cand] = (v & 1u) ? uint8_t(DIP_FLAG_INVALID) : uint8_t((v & 2u) ? DIP_FLAG_CAP : 0u);
}

}  // namespace

hipError_t launch_selcheck(int waves, hipStream_t s, const SelCheckArgs &a) {
  selcheck_kernel<<<dim3(unsigned(a.n_cand)), dim3(unsigned(waves * kWave)),
                    size_t(waves) * size_t(a.bm_words) * 4, s>>>(a);
  return hipGetLastError();
}

}  // namespace dipsim
