// kern_memopt.hip -- per-layer memory optimisation (DIP, arXiv 2504.14145,
// Sec. 5.3) of many candidate schedules at once.
//
// For every (candidate schedule, rank), each stage pair of the rank takes one
// of its memory candidates (time ascending, memory strictly descending) so
// that the live memory at every forward start stays within the rank's cap,
// with the least total time (Sec. 5.3's ILP, solved to within 5 %):
//   1. the greedy warm start: all pairs on their fastest candidate; while the
//      most loaded checkpoint (lowest index among equal loads) is over the
//      cap, move the live pair with the least added time per freed memory
//      unit (dt_a * dm_b < dt_b * dm_a, lowest pair index on ties) to its
//      next candidate; give up when no live pair can move;
//   2. an improvement pass: pairs in index order each go back to the fastest
//      candidate that keeps every checkpoint it is live at within the cap,
//      until a pass changes nothing;
//   3. a depth-first branch and bound from there, pairs in the order of their
//      forward starts, candidates fastest first: a placement whose own
//      checkpoint exceeds the cap is dropped, a node whose placed time plus
//      the unplaced pairs' fastest times, times 1.05, reaches the incumbent
//      is cut with its slower siblings, and a complete placement below the
//      incumbent replaces it.  A finished search proves the incumbent within
//      5 % of the optimum (status 1); after bb_nodes placements examined, or
//      on ranks of more than 512 pairs (no search), status 3;
//   4. when the search stopped early, a certificate from the Lagrangian
//      relaxation of the checkpoint constraints (the dual side of the ILP's
//      LP bound), by exact integer subgradient steps: status 1 once 1.05
//      times the bound reaches the incumbent.
// Pair i is live at pair k's forward start when its forward comes no later
// and its backward no earlier in the rank's order.
//
// The comparison of moves depends on the candidates only, not on the
// schedule, so the host ranks every move of a rank once (exact 128-bit cross
// products) and hands each a 32-bit key: the least key is the greedy's
// choice.  Two kernels:
//   memopt_group_kernel a group of 16 or 64 lanes per (schedule, rank), lane
//                       j owning pairs j, j + G, ...; a block holds schedules
//                       of one rank and shares that rank's tables in LDS.
//                       The pairs are numbered once in forward order, where
//                       a pair is live at a run of checkpoints: loads are
//                       prefix sums of differences, "live there" is one
//                       subtraction and one comparison, and in the search
//                       the load at a depth is the one above it plus the
//                       placed pair less those whose run ends (a list per
//                       checkpoint), so that a visit of a depth tries all
//                       its candidates at once, a lane each.  The search is
//                       left out where its bound already cuts every first
//                       placement (the fastest times alone reach it).
//                       Bound by vector instructions where problems are
//                       many: 16 lanes, since the state of up to 96 pairs
//                       fits six registers a lane and the steps' fixed cost
//                       (three reductions a move) serves four problems.
//                       Few or large problems are bound by the LDS round
//                       trips of their serial steps: 64 lanes.  32,768
//                       schedules of 8 ranks (32 to 68 pairs): 2.5 ms, 10.1
//                       with a wave per problem, its loads summed over all
//                       pairs, its search a candidate at a time and its
//                       tables in device memory; 1,024 rollouts of 16 ranks
//                       (128 and 196 pairs): 1.23 ms, 2.34.
//   memopt_kernel       a thread per (schedule, rank), for ranks of more
//                       than 512 pairs (steps 1 and 2); its state sits in
//                       LDS, element-major across the block.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dev_util.h"
#include "internal.h"

namespace dipsim {

namespace {

// the Lagrangian certificate: subgradient steps, fraction bits of the
// multipliers (at most), and the magnitude every value stays below
constexpr int kMemoptLagrIters = 200;
constexpr int kMemoptLagrF = 20;
constexpr int kMemoptLagrLimitBits = 60;
constexpr int kMemoptLagrHalve = 24;   // steps between halvings of the step size

// bits of a non-negative value (0 for 0)
__device__ __forceinline__ int bits64(int64_t x) { return x ? 64 - __clzll(x) : 0; }

// min / max of one value over the 64 lanes of a wave, read out of lane 63:
// the row reduction of dpp_row, then the row broadcasts (lane 15 of each row
// into the next row, lane 31 into rows 2 and 3), rows outside the mask
// keeping their value (the identity as the old value)
template <bool MAX>
__device__ __forceinline__ uint32_t wave_reduce63(uint32_t v) {
  auto op = [](uint32_t x, uint32_t y) { return MAX ? max(x, y) : min(x, y); };
  constexpr int kId = MAX ? 0 : -1;
  v = op(v, dpp_row<0xb1>(v));    // quad_perm [1,0,3,2]
  v = op(v, dpp_row<0x4e>(v));    // quad_perm [2,3,0,1]
  v = op(v, dpp_row<0x141>(v));   // row_half_mirror
  v = op(v, dpp_row<0x140>(v));   // row_mirror
  v = op(v, uint32_t(__builtin_amdgcn_update_dpp(kId, int(v), 0x142, 0xa, 0xf, false)));  // row_bcast:15
  v = op(v, uint32_t(__builtin_amdgcn_update_dpp(kId, int(v), 0x143, 0xc, 0xf, false)));  // row_bcast:31
  return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}

__device__ __forceinline__ void write_out(const MemoptArgs &a, int64_t o, int64_t t, int32_t pk,
                                          uint8_t st) {
  a.out_time[o] = t;
  a.out_peak[o] = pk;
  a.out_status[o] = st;
}

// ---------------------------------------------------------------- thread per problem

__global__ __launch_bounds__(256) void memopt_kernel(MemoptArgs a) {
  extern __shared__ __align__(16) unsigned char sh[];
  const int64_t id = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (id >= a.n_cand * a.P) return;
  const int64_t c = id / a.P;
  const int r = int(id % a.P);
  const int32_t np = a.pair_off[r + 1] - a.pair_off[r];
  const int32_t pbase = a.pair_off[r];
  // element-major arrays, [element][thread], so that the lanes of a wave
  // touch consecutive words
  const int T = blockDim.x, t = threadIdx.x;
  const int64_t m = a.max_pairs;
  int32_t *load_ = reinterpret_cast<int32_t *>(sh) + t;
  uint16_t *pf_ = reinterpret_cast<uint16_t *>(sh + 4 * m * T) + t;
  uint16_t *pb_ = pf_ + m * T;
  uint8_t *cur_ = reinterpret_cast<uint8_t *>(sh + 8 * m * T) + t;
#define load(i) load_[int64_t(i) * T]
#define pf(i) pf_[int64_t(i) * T]
#define pb(i) pb_[int64_t(i) * T]
#define cur(i) cur_[int64_t(i) * T]
  for (int32_t i = 0; i < np; ++i) {
    pf(i) = 0xffffu;
    pb(i) = 0xffffu;
    cur(i) = 0;
  }
  // positions of each pair's forward and backward in the rank's order
  const int32_t base = a.rank_off[r], nr = a.rank_off[r + 1] - base;
  const int16_t *row = a.orders + c * a.stride + base;
  bool valid = true;
  for (int32_t p = 0; p < nr; ++p) {
    const int32_t lid = row[p];
    if (lid < 0 || lid >= nr) {
      valid = false;
      break;
    }
    const uint32_t w = uint32_t(a.lid_pair[base + lid]);
    uint16_t *slot = ((w >> 31) ? pb_ : pf_) + int64_t(w & 0x7fffffffu) * T;
    if (*slot != 0xffffu) {
      valid = false;
      break;
    }
    *slot = uint16_t(p);
  }
  const int64_t o = c * a.P + r;
  if (!valid) {
    write_out(a, o, -1, -1, 2);
    return;
  }
  const int64_t *ct = a.cand_time + int64_t(pbase) * kMemoptMaxCands;
  const int32_t *cm = a.cand_mem + int64_t(pbase) * kMemoptMaxCands;
  const uint32_t *mk = a.move_key + int64_t(pbase) * kMemoptMaxCands;
  const int32_t *md = a.move_dm + int64_t(pbase) * kMemoptMaxCands;
  for (int32_t k = 0; k < np; ++k) {
    int32_t s = 0;
    for (int32_t i = 0; i < np; ++i)
      if (pf(i) <= pf(k) && pf(k) <= pb(i)) s += cm[i * kMemoptMaxCands];
    load(k) = s;
  }
  const int32_t cap = a.cap[r];
  bool ok = true;
  if (cap >= 0) {
    for (;;) {
      int32_t kk = 0;
      for (int32_t k = 1; k < np; ++k)
        if (load(k) > load(kk)) kk = k;
      if (np == 0 || load(kk) <= cap) break;
      uint32_t best = kMemoptNoMove;
      for (int32_t i = 0; i < np; ++i)
        if (pf(i) <= pf(kk) && pf(kk) <= pb(i)) best = min(best, mk[i * kMemoptMaxCands + cur(i)]);
      if (best == kMemoptNoMove) {
        ok = false;
        break;
      }
      const int32_t bi = int32_t(best & ((1u << kMemoptPairBits) - 1));
      const int32_t dm = md[bi * kMemoptMaxCands + cur(bi)];
      cur(bi) += 1;
      for (int32_t k = 0; k < np; ++k)
        if (pf(bi) <= pf(k) && pf(k) <= pb(bi)) load(k) -= dm;
    }
  }
  uint8_t status = ok ? 1 : 0;
  if (ok && cap >= 0 && np > 0) {
    // step 2; no search on ranks this large
    for (bool changed = true; changed;) {
      changed = false;
      for (int32_t i = 0; i < np; ++i) {
        int32_t top = INT32_MIN;
        for (int32_t k = 0; k < np; ++k)
          if (pf(i) <= pf(k) && pf(k) <= pb(i)) top = max(top, load(k));
        const int32_t ci = cur(i);
        const int32_t mc = cm[i * kMemoptMaxCands + ci];
        for (int32_t j = 0; j < ci; ++j) {
          const int32_t add = cm[i * kMemoptMaxCands + j] - mc;
          if (int64_t(top) + add <= int64_t(cap)) {
            for (int32_t k = 0; k < np; ++k)
              if (pf(i) <= pf(k) && pf(k) <= pb(i)) load(k) += add;
            cur(i) = uint8_t(j);
            changed = true;
            break;
          }
        }
      }
    }
    status = 3;
  }
  int64_t total = 0;
  int32_t peak = 0;
  for (int32_t i = 0; i < np; ++i) {
    total += ct[i * kMemoptMaxCands + cur(i)];
    peak = max(peak, load(i));
    if (a.out_choice) a.out_choice[c * a.n_pairs + pbase + i] = cur(i);
  }
  write_out(a, o, total, peak, status);
}
#undef load
#undef pf
#undef pb
#undef cur

// ---------------------------------------------------------------- lane group per problem

// Reductions over the G lanes of a group (16: one row of the wave, 64: the
// wave), the result in every lane.  A group's lanes are all active or none.
template <int G>
struct group_ops {
  static __device__ __forceinline__ uint32_t dpp16(uint32_t v, bool is_max) {
    auto op = [&](uint32_t x, uint32_t y) { return is_max ? max(x, y) : min(x, y); };
    v = op(v, dpp_row<0xb1>(v));    // quad_perm [1,0,3,2]
    v = op(v, dpp_row<0x4e>(v));    // quad_perm [2,3,0,1]
    v = op(v, dpp_row<0x141>(v));   // row_half_mirror
    v = op(v, dpp_row<0x140>(v));   // row_mirror
    return v;
  }
  static __device__ __forceinline__ uint32_t max32(uint32_t v) {
    return G == 64 ? wave_reduce63<true>(v) : dpp16(v, true);
  }
  static __device__ __forceinline__ uint32_t min32(uint32_t v) {
    return G == 64 ? wave_reduce63<false>(v) : dpp16(v, false);
  }
  template <int CTRL>
  static __device__ __forceinline__ int64_t dpp64(int64_t v) {
    return int64_t((uint64_t(dpp_row<CTRL>(uint32_t(uint64_t(v) >> 32))) << 32) |
                   dpp_row<CTRL>(uint32_t(v)));
  }
  static __device__ __forceinline__ int64_t read64(int64_t v, int l) {
    return int64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), l))) |
           (int64_t(__builtin_amdgcn_readlane(int(v >> 32), l)) << 32);
  }
  template <class Op>
  static __device__ __forceinline__ int64_t all64(int64_t v, Op op) {
    v = op(v, dpp64<0xb1>(v));      // quad_perm [1,0,3,2]
    v = op(v, dpp64<0x4e>(v));      // quad_perm [2,3,0,1]
    v = op(v, dpp64<0x141>(v));     // row_half_mirror
    v = op(v, dpp64<0x140>(v));     // row_mirror
    if (G == 64) v = op(op(read64(v, 0), read64(v, 16)), op(read64(v, 32), read64(v, 48)));
    return v;
  }
  static __device__ __forceinline__ int64_t sum64(int64_t v) {
    return all64(v, [](int64_t x, int64_t y) { return x + y; });
  }
  static __device__ __forceinline__ int64_t max64(int64_t v) {
    return all64(v, [](int64_t x, int64_t y) { return max(x, y); });
  }
  // lanes of the group where p holds
  static __device__ __forceinline__ uint64_t ballot(bool p, int lane) {
    const uint64_t b = __ballot(p);
    if (G == 64) return b;
    const uint32_t w = (lane & 32) ? uint32_t(b >> 32) : uint32_t(b);
    return (w >> (lane & 16)) & 0xffffu;
  }
  // inclusive prefix sum; zeros come in at a row's start
  static __device__ __forceinline__ int32_t scan32(int32_t v, int lane) {
    v += int32_t(dpp_row<0x111>(uint32_t(v)));   // row_shr:1
    v += int32_t(dpp_row<0x112>(uint32_t(v)));
    v += int32_t(dpp_row<0x114>(uint32_t(v)));
    v += int32_t(dpp_row<0x118>(uint32_t(v)));
    if (G == 64) {
      const int32_t r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
                    r2 = __builtin_amdgcn_readlane(v, 47);
      v += lane < 16 ? 0 : lane < 32 ? r0 : lane < 48 ? r0 + r1 : r0 + r1 + r2;
    }
    return v;
  }
  // the value of the group's last lane
  static __device__ __forceinline__ int32_t last32(int32_t v, int lane) {
    return G == 64 ? __builtin_amdgcn_readlane(v, 63) : __shfl(v, lane | 15);
  }
  static __device__ __forceinline__ int64_t last64(int64_t v, int lane) {
    return int64_t(uint32_t(last32(int32_t(uint32_t(v)), lane))) |
           (int64_t(last32(int32_t(v >> 32), lane)) << 32);
  }
  static __device__ __forceinline__ int64_t scan64(int64_t v, int lane) {
    v += dpp64<0x111>(v);
    v += dpp64<0x112>(v);
    v += dpp64<0x114>(v);
    v += dpp64<0x118>(v);
    if (G == 64) {
      const int64_t r0 = read64(v, 15), r1 = read64(v, 31), r2 = read64(v, 47);
      v += lane < 16 ? 0 : lane < 32 ? r0 : lane < 48 ? r0 + r1 : r0 + r1 + r2;
    }
    return v;
  }
};

// 105 x >= 100 y for y >= 0: x >= y - y / 21
__device__ __forceinline__ int64_t gap_bound(int64_t y) { return y - int64_t(uint64_t(y) / 21); }

// LDS bytes of the tables a block shares (per pair of the rank: candidates'
// times, memories and move keys, the two ends' op entries, candidate count)
// and of one problem's arrays
__host__ __device__ constexpr int64_t group_table_bytes(int64_t mp) {
  return (mp * (kMemoptMaxCands * 16 + 5) + 7) / 8 * 8;
}
__host__ __device__ constexpr int64_t group_problem_bytes(int64_t mp) {
  return (18 * mp + 16 + 7) / 8 * 8;
}

template <int G, int PPL>
__global__ __launch_bounds__(512) void memopt_group_kernel(MemoptArgs a) {
  extern __shared__ __align__(16) unsigned char sh[];
  using R = group_ops<G>;
  constexpr int C = kMemoptMaxCands;
  const int lane = threadIdx.x & 63;
  const int gl = lane & (G - 1);
  const int gb = threadIdx.x / G;
  const int r = blockIdx.y;
  const int64_t c = int64_t(blockIdx.x) * (blockDim.x / G) + gb;
  const int32_t pbase = a.pair_off[r];
  const int32_t np = a.pair_off[r + 1] - pbase;
  const int64_t mp = a.max_pairs;
  const int nq = (np + G - 1) / G;
  // shared tables
  int64_t *tt = reinterpret_cast<int64_t *>(sh);
  int32_t *tm = reinterpret_cast<int32_t *>(sh + 8 * C * mp);
  uint32_t *tk = reinterpret_cast<uint32_t *>(sh + 12 * C * mp);
  uint16_t *tw = reinterpret_cast<uint16_t *>(sh + 16 * C * mp);
  uint8_t *tn = sh + (16 * C + 4) * mp;
  const int32_t base = a.rank_off[r], nr = a.rank_off[r + 1] - base;
  {
    const int64_t *gt = a.cand_time + int64_t(pbase) * C;
    const int32_t *gm = a.cand_mem + int64_t(pbase) * C;
    const uint32_t *gk = a.move_key + int64_t(pbase) * C;
    for (int32_t x = threadIdx.x; x < np * C; x += blockDim.x) {
      tt[x] = gt[x];
      tm[x] = gm[x];
      tk[x] = gk[x];
    }
    for (int32_t x = threadIdx.x; x < nr; x += blockDim.x) {
      const uint32_t w = uint32_t(a.lid_pair[base + x]);
      tw[x] = uint16_t((w & 0x7fffu) | (w >> 31 << 15));
    }
    for (int32_t i = threadIdx.x; i < np; i += blockDim.x) {
      int32_t n = 1;
      while (n < C && gk[i * C + n - 1] != kMemoptNoMove) ++n;
      tn[i] = uint8_t(n);
    }
  }
  __syncthreads();
  if (c >= a.n_cand) return;                        // whole groups, after the last barrier
  // this problem's arrays: 13 bytes a pair that the steps use in turn, then
  // each pair's first checkpoint (in forward order), how many it is live at,
  // and its choice
  unsigned char *ws = sh + group_table_bytes(mp) + gb * group_problem_bytes(mp);
  uint16_t *plo = reinterpret_cast<uint16_t *>(ws + 13 * mp + 12 + (mp & 1));
  uint16_t *pln = plo + mp;
  uint8_t *cur = reinterpret_cast<uint8_t *>(pln + mp);
  int32_t *acc = reinterpret_cast<int32_t *>(ws);   // [np + 1]

  // ---- forward order of the pairs and the checkpoints each is live at
  for (int32_t i = gl; i < np; i += G) {
    plo[i] = 0xffffu;
    pln[i] = 0xffffu;
    cur[i] = 0;
  }
  for (int32_t d = gl; d <= np; d += G) acc[d] = 0;
  wave_lds_order();
  const int16_t *row = a.orders + c * a.stride + base;
  bool bad = false;
  int32_t nf = 0;                                   // forwards so far
  for (int32_t p0 = 0; p0 < nr; p0 += 4 * G) {
    int32_t lid[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t p = p0 + u * G + gl;
      lid[u] = p < nr ? int32_t(row[p]) : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u * G >= nr) break;
      const bool in = lid[u] >= 0 && lid[u] < nr;
      bad |= p0 + u * G + gl < nr && !in;
      const uint32_t w = in ? tw[lid[u]] : 0u;
      const bool fwd = in && !(w >> 15);
      const uint64_t m = R::ballot(fwd, lane);
      const int32_t before = nf + __popcll(m & ((uint64_t(1) << gl) - 1));
      if (in) (fwd ? plo : pln)[w & 0x7fffu] = uint16_t(before);
      nf += __popcll(m);
    }
  }
  wave_lds_order();
  // own pairs: forward-order index (with the pair's index above it), length
  // of the live range (0: its backward comes first), key of its next move
  uint32_t P[PPL], key[PPL];
  uint16_t ln[PPL];
  int32_t load[PPL];
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    P[q] = 0xffffffffu;
    ln[q] = 0;
    key[q] = kMemoptNoMove;
    load[q] = 0;
    const int32_t i = gl + G * q;
    if (i < np) {
      const uint32_t x = plo[i], y = pln[i];
      // every rank op is one end of one pair, so with all nr ids in range a
      // repeated id leaves some end unfilled
      if (x == 0xffffu || y == 0xffffu) bad = true;
      P[q] = uint32_t(i) << 16 | x;
      ln[q] = uint16_t(y > x ? y - x : 0);
      key[q] = tk[i * C];
    }
  }
  const int64_t o = c * a.P + r;
  if (R::ballot(bad, lane)) {
    if (gl == 0) write_out(a, o, -1, -1, 2);
    return;
  }
  // loads under the fastest candidates: sums of differences over the
  // checkpoints in forward order
  auto scan_loads = [&]() {
    int32_t run = 0, top = 0;
    for (int32_t q = 0; q < nq; ++q) {
      const int32_t d = gl + G * q;
      const int32_t v = R::scan32(d < np ? acc[d] : 0, lane) + run;
      if (d < np) acc[d] = v;
      top = max(top, v);
      run = R::last32(v, lane);
    }
    return top;
  };
#pragma unroll
  for (int q = 0; q < PPL; ++q) {
    const int32_t i = gl + G * q;
    if (i < np) {
      pln[i] = ln[q];
      if (ln[q]) {
        const int32_t x = P[q] & 0xffffu;
        atomicAdd(acc + x, tm[i * C]);
        atomicAdd(acc + x + ln[q], -tm[i * C]);
      }
    }
  }
  wave_lds_order();
  (void)scan_loads();
  wave_lds_order();
#pragma unroll
  for (int q = 0; q < PPL; ++q)
    if (gl + G * q < np) load[q] = acc[P[q] & 0xffffu];
  // checkpoint of slot q within the range of a pair
  auto covers = [](uint32_t at, uint32_t lo, uint32_t len) {
    return uint16_t(at - lo) < uint16_t(len);
  };

  // ---- step 1: the greedy warm start
  const int32_t cap = a.cap[r];
  bool ok = true, moved = false;
  if (cap >= 0 && np > 0) {
    for (;;) {
      // most loaded checkpoint, lowest pair index among equal loads
      int32_t bl = -1;
      uint32_t bp = 0xffffffffu;
#pragma unroll
      for (int q = 0; q < PPL; ++q)
        if (q < nq) {
          bp = load[q] > bl ? P[q] : bp;
          bl = max(bl, load[q]);
        }
      const uint32_t top = R::max32(uint32_t(bl));
      if (int32_t(top) <= cap) break;
      const uint32_t dk = R::min32(uint32_t(bl) == top ? bp : 0xffffffffu);
      // best move among the pairs live there
      uint32_t m = kMemoptNoMove;
#pragma unroll
      for (int q = 0; q < PPL; ++q)
        if (q < nq) m = min(m, covers(dk, P[q], ln[q]) ? key[q] : kMemoptNoMove);
      m = R::min32(m);
      if (m == kMemoptNoMove) {
        ok = false;
        break;
      }
      moved = true;
      // every checkpoint the moved pair is live at drops; the pair steps on
      // (every lane of the group writes the same choice)
      const uint32_t bi = m & ((1u << kMemoptPairBits) - 1);
      const uint32_t ci = cur[bi], x = bi * C + ci;
      const int32_t dm = tm[x] - tm[x + 1];
      const uint32_t nkey = tk[x + 1];
      const uint32_t slo = plo[bi], sln = pln[bi];
      cur[bi] = uint8_t(ci + 1);
#pragma unroll
      for (int q = 0; q < PPL; ++q)
        if (q < nq) {
          load[q] -= covers(P[q], slo, sln) ? dm : 0;
          key[q] = bi == uint32_t(gl + G * q) ? nkey : key[q];
        }
    }
  }
  wave_lds_order();
  uint8_t status = ok ? 1 : 0;
  if (ok && moved) {
    // ---- step 2: back to faster candidates where every checkpoint allows
    for (bool changed = true; changed;) {
      changed = false;
      for (int32_t q0 = 0; q0 < nq; ++q0) {
        const int32_t own = gl + G * q0;
        uint64_t todo = R::ballot(own < np && cur[own < np ? own : 0] > 0, lane);
        while (todo) {
          const int32_t i = G * q0 + __builtin_ctzll(todo);
          todo &= todo - 1;
          const uint32_t slo = plo[i], sln = pln[i];
          int32_t mx = 0;
#pragma unroll
          for (int q = 0; q < PPL; ++q)
            if (q < nq) mx = covers(P[q], slo, sln) ? max(mx, load[q]) : mx;
          const uint32_t top = R::max32(uint32_t(mx));
          const int32_t ci = cur[i];
          const int32_t mc = tm[i * C + ci], mj = tm[i * C + (gl & (C - 1))];
          // (a pair whose backward comes before its forward is live nowhere)
          const uint64_t fit = R::ballot(
              gl < ci && (sln == 0 || uint32_t(mj) <= uint32_t(cap) - top + uint32_t(mc)), lane);
          if (fit) {
            const int32_t nj = __builtin_ctzll(fit);
            const int32_t add = tm[i * C + nj] - mc;
#pragma unroll
            for (int q = 0; q < PPL; ++q)
              if (q < nq) load[q] += covers(P[q], slo, sln) ? add : 0;
            cur[i] = uint8_t(nj);
            changed = true;
          }
        }
      }
      wave_lds_order();
    }
  }
  int32_t peak = 0;
#pragma unroll
  for (int q = 0; q < PPL; ++q) peak = max(peak, load[q]);
  peak = int32_t(R::max32(uint32_t(peak)));
  // the incumbent's time, and the least any choice takes
  int64_t inc = 0, fastest = 0;
  for (int32_t i = gl; i < np; i += G) {
    inc += tt[i * C + cur[i]];
    fastest += tt[i * C];
  }
  inc = R::sum64(inc);
  if (ok && moved) {
    // ---- step 3: branch and bound, pairs by forward position
    fastest = R::sum64(fastest);
    int64_t cut = gap_bound(inc);
    bool proven = true;
    // every placement of the first pair is dropped or cut when the fastest
    // times alone reach the bound (its candidates fit any sensible budget)
    if (fastest < cut || a.bb_nodes < C) {
      // by forward order: the pair; the pairs whose live range ends before
      // the checkpoint (a list); by pair: the list's next, the candidate and
      // the live memory of the current placement
      int32_t *head = reinterpret_cast<int32_t *>(ws);          // [np + 1]
      int32_t *pmem = head + mp + 1;                            // [np]
      uint16_t *ord = reinterpret_cast<uint16_t *>(pmem + mp);  // [np]
      uint16_t *nxt = ord + mp;                                 // [np]
      uint8_t *chp = reinterpret_cast<uint8_t *>(nxt + mp);     // [np]
      for (int32_t d = gl; d <= np; d += G) head[d] = -1;
      wave_lds_order();
      for (int32_t i = gl; i < np; i += G) {
        ord[plo[i]] = uint16_t(i);
        if (pln[i]) nxt[i] = uint16_t(atomicExch(head + plo[i] + pln[i], i));
      }
      wave_lds_order();
      bool better = false;
      uint32_t seen = 0;
      int32_t d = 0, c0 = 0;          // depth, first candidate to try there
      int32_t held = 0;               // load of the placed pairs at depth d's checkpoint
      int64_t f = 0, rest = fastest;  // placed time; fastest time of depths d and on
      for (;;) {
        const int32_t i = ord[d];
        const int32_t n = tn[i];
        const int32_t mj = pln[i] ? tm[i * C + (gl & (C - 1))] : 0;
        const int64_t t0 = tt[i * C];
        const uint64_t fit = R::ballot(gl >= c0 && gl < n && mj <= cap - held, lane);
        const int32_t cc = fit ? __builtin_ctzll(fit) : n - 1;
        seen += uint32_t(cc + 1 - c0);   // placements looked at (none when c0 == n)
        if (seen > uint32_t(a.bb_nodes)) {
          proven = false;
          break;
        }
        bool back = !fit;
        if (fit) {
          const int64_t ft = f + tt[i * C + cc];
          if (ft + rest - t0 >= cut) {
            back = true;                 // cut, with the slower ones
          } else {
            const int32_t pm = pln[i] ? tm[i * C + cc] : 0;
            chp[i] = uint8_t(cc);
            pmem[i] = pm;
            if (d == np - 1) {           // every pair placed, below the incumbent
              inc = ft;
              cut = gap_bound(inc);
              better = true;
              wave_lds_order();
              for (int32_t k = gl; k < np; k += G) cur[k] = chp[k];
              wave_lds_order();
              c0 = cc + 1;
            } else {
              f = ft;
              rest -= t0;
              held += pm;
              ++d;
              c0 = 0;
              for (int32_t k = head[d]; k != -1;) {
                held -= pmem[k];
                const int32_t k1 = nxt[k];
                k = k1 == 0xffff ? -1 : k1;
              }
            }
          }
        }
        if (back) {
          if (d == 0) break;
          for (int32_t k = head[d]; k != -1;) {
            held += pmem[k];
            const int32_t k1 = nxt[k];
            k = k1 == 0xffff ? -1 : k1;
          }
          --d;
          const int32_t k = ord[d], ck = chp[k];
          held -= pmem[k];
          f -= tt[k * C + ck];
          rest += tt[k * C];
          c0 = ck + 1;
        }
      }
      status = proven ? 1 : 3;
      if (better) {                      // the new choice's loads
        wave_lds_order();
        for (int32_t k = gl; k <= np; k += G) acc[k] = 0;
        wave_lds_order();
        for (int32_t k = gl; k < np; k += G)
          if (pln[k]) {
            const int32_t m = tm[k * C + cur[k]];
            atomicAdd(acc + plo[k], m);
            atomicAdd(acc + plo[k] + pln[k], -m);
          }
        wave_lds_order();
        peak = int32_t(R::max32(uint32_t(scan_loads())));
      }
      if (!proven) {
        // ---- step 4: the Lagrangian certificate.  Multipliers l_k >= 0
        // (units of 2^-F time per memory unit), one per checkpoint k (pair
        // k's forward start).  Each step: a pair's price is the sum of the
        // multipliers of the checkpoints it is live at; it takes its cheapest
        // candidate under t * 2^F + m * price (the first on ties); the bound
        // (times 2^F) is the sum of those values less cap * sum_k l_k, and
        // proves the incumbent once 1.05 times it reaches the incumbent;
        // otherwise each multiplier moves by g_k * step / 2^b, b the bits of
        // max |g| (the magnitude shifted down, the sign kept; kept in [0,
        // lmax]), g_k being the memory of the taken candidates live at
        // checkpoint k less the cap, step = s0 / 2^(t / 24).  F = min(20, 60 -
        // bits(np * tmax)), lmax = 2^60 / 2^bits(np^2 * max(1, mmax, cap)) and
        // s0 = half the largest (dt << F) / 2^(bits(dm) - 1) over the moves
        // from each pair's fastest candidate (at least 1, at most lmax) keep
        // every value below 2^61, with no division.  A pair is live at a run
        // of checkpoints in forward order, so both sums are differences of
        // prefix sums over them.  Integer arithmetic: the same values as any
        // other order of summation.
        int64_t tmx = 0, mmx = 0, s0 = 0;
        for (int32_t i = gl; i < np; i += G) {          // candidates ascend in time
          tmx = max(tmx, tt[i * C + tn[i] - 1]);
          mmx = max(mmx, int64_t(tm[i * C]));
        }
        tmx = R::max64(tmx);
        mmx = R::max64(mmx);
        const int F = min(kMemoptLagrF, kMemoptLagrLimitBits - bits64(int64_t(np) * max(tmx, int64_t(1))));
        const int lb = bits64(int64_t(np) * np * max(max(int64_t(1), mmx), int64_t(cap)));
        const int64_t lmax = lb <= kMemoptLagrLimitBits ? int64_t(1) << (kMemoptLagrLimitBits - lb) : 0;
        if (F >= 0 && lmax > 0) {
          for (int32_t i = gl; i < np; i += G)
            for (int32_t j = 1; j < tn[i]; ++j)
              s0 = max(s0, ((tt[i * C + j] - tt[i * C]) << F) >>
                               (bits64(int64_t(tm[i * C]) - tm[i * C + j]) - 1));
          s0 = min(lmax, max(int64_t(1), R::max64(s0) >> 1));
          const int64_t goal = gap_bound(inc << F);
          // prefix sums of the multipliers (multiplier d is ps[d + 1] - ps[d])
          // and memory differences, [np + 1] each
          int64_t *ps = reinterpret_cast<int64_t *>(ws);
          int32_t *dif = reinterpret_cast<int32_t *>(ps + (mp + 1));
          wave_lds_order();
          for (int32_t d = gl; d <= np; d += G) {
            ps[d] = 0;
            dif[d] = 0;
          }
          for (int t = 0; t < kMemoptLagrIters; ++t) {
            wave_lds_order();
            int64_t part = 0;
            for (int32_t i = gl; i < np; i += G) {
              const int32_t lo = plo[i], len = pln[i];
              const int64_t price = ps[lo + len] - ps[lo];
              int64_t bv = (tt[i * C] << F) + int64_t(tm[i * C]) * price;
              int32_t bm = tm[i * C];
              const int32_t n = tn[i];
              for (int32_t j = 1; j < n; ++j) {
                const int32_t m = tm[i * C + j];
                const int64_t v = (tt[i * C + j] << F) + int64_t(m) * price;
                if (v < bv) {
                  bv = v;
                  bm = m;
                }
              }
              part += bv;
              if (len) {
                atomicAdd(dif + lo, bm);
                atomicAdd(dif + lo + len, -bm);
              }
            }
            if (R::sum64(part) - int64_t(cap) * ps[np] >= goal) {
              status = 1;
              break;
            }
            wave_lds_order();
            // the memory live at every checkpoint, written over its differences
            // (32 bits hold it: the fastest candidates' memories of a rank do)
            uint32_t gabs = 0;
            int32_t run = 0;
            for (int32_t q = 0; q < nq; ++q) {
              const int32_t d = gl + G * q;
              const int32_t v = R::scan32(d < np ? dif[d] : 0, lane) + run;
              run = R::last32(v, lane);
              if (d < np) {
                dif[d] = v;
                gabs = max(gabs, uint32_t(abs(v - cap)));
              }
            }
            const int sft = bits64(R::max32(gabs));
            if (sft == 0) break;
            // the multipliers' move and their new prefix sums; the
            // differences cleared
            const int64_t step = s0 >> (t / kMemoptLagrHalve);
            int64_t carry = 0, old = 0;      // new and old prefix sum at the chunk's start
            for (int32_t q = 0; q < nq; ++q) {
              const int32_t d = gl + G * q;
              int64_t lam = 0, at = 0;
              if (d < np) {
                at = ps[d + 1];
                lam = at - (gl == 0 ? old : ps[d]);
                const int64_t g = dif[d] - cap;
                const int64_t mv = ((g < 0 ? -g : g) * step) >> sft;
                lam = min(lmax, max(int64_t(0), lam + (g < 0 ? -mv : mv)));
              }
              old = R::last64(at, lane);
              const int64_t v = R::scan64(lam, lane) + carry;
              carry = R::last64(v, lane);
              wave_lds_order();
              if (d < np) ps[d + 1] = v;
              if (d <= np) dif[d] = 0;
            }
            if (nq * G == np && gl == 0) dif[np] = 0;
          }
        }
      }
    }
  }
  if (a.out_choice)
    for (int32_t i = gl; i < np; i += G) a.out_choice[c * a.n_pairs + pbase + i] = cur[i];
  if (gl == 0) write_out(a, o, inc, peak, status);
}

}  // namespace

int64_t memopt_group_lds(int32_t max_pairs, int groups_per_block) {
  return group_table_bytes(max_pairs) + groups_per_block * group_problem_bytes(max_pairs);
}

const void *memopt_group_ptr(int lanes, int32_t max_pairs) {
  auto ptr = [](void (*k)(MemoptArgs)) { return reinterpret_cast<const void *>(k); };
  const int n = (max_pairs + lanes - 1) / lanes;
  if (lanes == 16)
    return n <= 2   ? ptr(memopt_group_kernel<16, 2>)
           : n <= 4 ? ptr(memopt_group_kernel<16, 4>)
           : n <= 6 ? ptr(memopt_group_kernel<16, 6>)
                    : nullptr;
  return n <= 1   ? ptr(memopt_group_kernel<64, 1>)
         : n <= 2 ? ptr(memopt_group_kernel<64, 2>)
         : n <= 4 ? ptr(memopt_group_kernel<64, 4>)
         : n <= 8 ? ptr(memopt_group_kernel<64, 8>)
                  : nullptr;
}

hipError_t launch_memopt_group(int lanes, int waves_per_block, hipStream_t s, const MemoptArgs &a) {
  const void *k = memopt_group_ptr(lanes, a.max_pairs);
  if (!k) return hipErrorInvalidValue;
  const int per = waves_per_block * 64 / lanes;
  const dim3 grid{unsigned((a.n_cand + per - 1) / per), unsigned(a.P)};
  MemoptArgs arg = a;
  void *args[] = {&arg};
  return hipLaunchKernel(k, grid, dim3(unsigned(64 * waves_per_block)), args,
                         size_t(memopt_group_lds(a.max_pairs, per)), s);
}

hipError_t launch_memopt(int threads_per_block, hipStream_t s, const MemoptArgs &a) {
  const int64_t n = a.n_cand * a.P;
  const int64_t blocks = (n + threads_per_block - 1) / threads_per_block;
  const size_t lds = size_t(threads_per_block) * size_t(a.bytes_per_thread);
  hipLaunchKernelGGL(memopt_kernel, dim3(unsigned(blocks)), dim3(unsigned(threads_per_block)), lds,
                     s, a);
  return hipGetLastError();
}

}  // namespace dipsim
