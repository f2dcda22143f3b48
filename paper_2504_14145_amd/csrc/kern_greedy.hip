// kern_greedy.hip -- dual-queue stage interleaving (DIP, arXiv 2504.14145,
// Sec. 5.2) of many candidate priority vectors at once.
//
// Per candidate the kernel builds each rank's stage order the way Sec. 5.2's
// greedy does, and the timeline that comes with it:
//   * a stage is queued on its rank once all its predecessors are scheduled,
//     with t_start = max over them of end + comm (0 without predecessors);
//   * a rank can next start at t_min = max(t_last, smallest queued t_start);
//     if both a forward and a backward were queued before t_last, it takes the
//     kind opposite to its last stage (1F1B); otherwise it takes any stage
//     that can start at t_min; within that set the highest priority wins
//     (priority, then group index, then rank-local id);
//   * a forward that would raise the rank's live activation above its cap
//     disables the forward queue for that decision (Sec. 5.2's memory rule);
//   * the rank with the smallest t_min (lowest index on ties) commits its
//     choice; when every rank is held back by its cap, the cap is lifted for
//     one decision.
//
// Several decisions per round.  Let E be the least end time over the ranks'
// current choices.  No stage can be delivered to any rank before E: the next
// commits are these choices, or later stages of their ranks, which start no
// earlier.  So every rank whose t_min lies below E keeps its choice whatever
// the others do first, and all of them commit in the same round; the rank of
// the least t_min always does.  On the workloads that is 1.8 to 6.2 commits a
// round (34,896 stages of 16 ranks in 19,258 rounds, 5,184 in 832; 11 on 64
// equal ranks), with the sequential greedy's result.
//
// Mapping: lane = rank; a group of 2^GWL lanes per candidate.  GWL is the
// rank count's power of two (64 >> GWL candidates side by side in a wave), or
// 6: a wave per candidate, whose branches are then uniform, for batches too
// small to fill the SIMDs otherwise (the launch chooses).
//
// A rank's queue, per kind, by overall priority rank q (0 best):
//   S     a bitmap in LDS with a register mask of its non-zero words and its
//         first member in a register.  All members have t_start < t_last
//         (ts < t_last), or all have t_start == ts >= t_last: runs of equal
//         times, such as the zero-cost stages of empty pieces, cost one bit
//         a stage;
//   ring  the stages that start later than S (or at t_last beside an
//         earlier S), sorted by (t_start, q): the first in a register, the
//         next few in LDS, the rest in device memory (one region per
//         resident candidate slot, as large as the rank's stage count, so it
//         never fills).  97 % of the time a ring is empty or holds one stage.
// With (start, q) as one 64-bit number, a kind's best stage is the lesser of
// (max(ts, t_last), first of S) and the ring's first entry, and the rank's
// choice the lesser of its two kinds, unless the kinds alternate.
// A committing lane changes its own queue only.  What its stage completes
// goes to the target ranks as messages, one per sender and pass.  In a wave
// of one candidate a lane permute moves them from the senders' registers into
// the targets' (one at a time where two are for one rank, and where all 64
// lanes are ranks); in a wave of several, the sender writes its message into
// its slot in LDS and sets its bit in the target's mask, and each target
// takes its messages in turn.
//
// What bounds it: latency and issue of a round's serial chain (choice,
// record, reduction, commit, messages); bandwidth is a few percent.  At one
// wave a SIMD a round takes about 3,300 cycles (16 ranks, 1,024 candidates of
// 34,896 stages), 1,400 of them waiting.  So the usual round is kept short and
// straight: what few rounds need (a choice out of a ring, joins, a second
// successor, arrivals into a ring in use) stands behind wave-wide tests and
// out of line, and a wave's messages move by one lane permute instead of two
// lane reads each.  That took 1,024 vectors on 16 x 4 lanes from 29.3 to 27.9
// ms, 2,001 on 32 ranks from 4.81 to 4.43, 65,536 on 8 from 2.89 to 2.83.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dip_sim.h"
#include "dev_util.h"
#include "internal.h"

namespace dipsim {

namespace {

constexpr uint32_t kNone = 0xffffu;        // no priority rank
constexpr uint32_t kNever = 0xffffffffu;   // no time
constexpr uint64_t kNoEntry = ~uint64_t(0);

// one lane's value through a DPP move, `id` where no lane feeds it (every
// lane is fed here; with the operation's identity the move and the operation
// become one instruction)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t id, uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(id), int(v), CTRL, 0xf, 0xf, false));
}

// min / max over aligned runs of 2^WL lanes: quad permutations, then the
// half-row and row mirrors (each lane meets the other half), then shuffles
template <int WL, bool MAX>
__device__ __forceinline__ uint32_t run_reduce(uint32_t v) {
  constexpr uint32_t id = MAX ? 0u : 0xffffffffu;
  auto op = [](uint32_t x, uint32_t y) { return MAX ? max(x, y) : min(x, y); };
  if constexpr (WL >= 1) v = op(v, dpp<0xb1>(id, v));    // quad_perm [1,0,3,2]
  if constexpr (WL >= 2) v = op(v, dpp<0x4e>(id, v));    // quad_perm [2,3,0,1]
  if constexpr (WL >= 3) v = op(v, dpp<0x141>(id, v));   // row_half_mirror
  if constexpr (WL >= 4) v = op(v, dpp<0x140>(id, v));   // row_mirror
  if constexpr (WL >= 5) v = op(v, uint32_t(__shfl_xor(int(v), 16)));
  if constexpr (WL >= 6) v = op(v, uint32_t(__shfl_xor(int(v), 32)));
  return v;
}

// the same over a candidate's 2^GWL lanes, whose ranks are the first 2^RWL
template <int RWL, int GWL, bool MAX>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v) {
  if constexpr (GWL == 6 && RWL >= 4) {
    // rows of 16 lanes, then their results as uniform values
    v = run_reduce<4, MAX>(v);
    uint32_t u = uint32_t(__builtin_amdgcn_readlane(int(v), 0));
#pragma unroll
    for (int i = 1; i < (1 << (RWL - 4)); ++i) {
      const uint32_t x = uint32_t(__builtin_amdgcn_readlane(int(v), 16 * i));
      u = MAX ? max(u, x) : min(u, x);
    }
    return u;
  }
  v = run_reduce<RWL, MAX>(v);
  if constexpr (GWL == 6) v = uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
  return v;
}

// bits of this lane's group in a wave-wide mask, lowest rank at bit 0
template <int GWL>
__device__ __forceinline__ uint64_t group_bits(uint64_t m, int grp) {
  if constexpr (GWL == 6) return m;
  constexpr uint64_t low = (uint64_t(1) << ((1 << GWL) & 63)) - 1;
  return (m >> (grp << GWL)) & low;
}

// a loaded value is waited for here
__device__ __forceinline__ void arrived(uint4 &v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

// LDS accesses below are to the lane's own words unless said otherwise.
struct RingMeta {
  uint32_t h, n;       // head and count of the entries in LDS
  uint32_t gh, gn;     // and in device memory
};

// One rank's queues.  What every round needs lies in registers, by kind;
// the rings beyond their first entries are touched in few rounds.
struct Queues {
  uint32_t first[2];   // S's first member, kNone if empty
  uint32_t ts[2];      // its members' t_start when that is >= t_last; kNever if empty
  uint64_t nz[2];      // its non-zero words
  uint64_t fr[2];      // the ring's first entry (t_start << 32 | q), or kNoEntry
  uint64_t *bits;      // [2][nwd] S, by priority rank
  uint64_t *ring;      // [2][kl] the ring's next entries
  RingMeta *meta;      // [2]
  uint64_t *dev;       // [2][kg] the ring's tail
  uint32_t nwd, kl, kg;

  template <class T>
  static __device__ __forceinline__ T get(const T (&v)[2], uint32_t kind) {
    return kind ? v[1] : v[0];
  }
  template <class T>
  static __device__ __forceinline__ void put(T (&v)[2], uint32_t kind, T x) {
    v[0] = kind ? v[0] : x;
    v[1] = kind ? x : v[1];
  }
  __device__ __forceinline__ uint64_t *words(uint32_t kind) const {
    return bits + (kind ? nwd : 0u);
  }
  // the kind's best stage as start << 32 | q, all ones if none is queued
  __device__ __forceinline__ uint64_t best(int kind, uint32_t t_last) const {
    const uint32_t t = max(ts[kind], t_last);
    const uint64_t s = (uint64_t(t) << 32) | first[kind];
    const uint64_t x = fr[kind] < s ? fr[kind] : s;
    return x;
  }
  // (t, q) into S, which it joins
  __device__ __forceinline__ void join(uint32_t kind, uint32_t t, uint32_t q) {
    const uint32_t k = q >> 6;
    atomicOr(reinterpret_cast<unsigned long long *>(words(kind) + k),
             static_cast<unsigned long long>(uint64_t(1) << (q & 63u)));
    put(nz, kind, get(nz, kind) | (uint64_t(1) << k));
    const uint32_t s = get(ts, kind);
    put(ts, kind, s == kNever ? t : s);
    put(first, kind, min(get(first, kind), q));
  }
  // S's first member leaves
  __device__ __forceinline__ void drop_first(uint32_t kind) {
    uint64_t *b = words(kind);
    uint32_t k = get(first, kind) >> 6;
    uint64_t w = b[k];
    w &= w - 1;
    b[k] = w;
    uint32_t f = k * 64u + uint32_t(__builtin_ctzll(w));
    if (w == 0) {
      const uint64_t z = get(nz, kind) & (get(nz, kind) - 1);
      put(nz, kind, z);
      f = kNone;
      if (z == 0) {
        put(ts, kind, kNever);
      } else {
        k = uint32_t(__builtin_ctzll(z));
        f = k * 64u + uint32_t(__builtin_ctzll(b[k]));
      }
    }
    put(first, kind, f);
  }
  __device__ __forceinline__ uint32_t wrap(uint32_t x) const { return x >= kg ? x - kg : x; }
  // x into the sorted ring; true if an entry went to device memory
  __device__ bool ring_insert(uint32_t kind, uint64_t x) {
    const uint64_t f = get(fr, kind);
    if (x < f) {
      put(fr, kind, x);
      if (f == kNoEntry) return false;
      x = f;
    }
    uint64_t *l = ring + (kind ? kl : 0u), *g = dev + (kind ? kg : 0u);
    RingMeta m = meta[kind];
    const uint32_t mask = kl - 1u;
    bool spilled = false;
    if (m.gn > 0 || m.n >= kl) {
      // (entries in device memory only ever follow a non-empty LDS part)
      spilled = true;
      const uint64_t back = l[(m.h + m.n - 1u) & mask];
      if (back <= x) {
        uint32_t i = m.gn;
        for (; i > 0; --i) {
          const uint64_t p = g[wrap(m.gh + i - 1u)];
          if (p <= x) break;
          g[wrap(m.gh + i)] = p;
        }
        g[wrap(m.gh + i)] = x;
        meta[kind].gn = m.gn + 1u;
        return true;
      }
      // the last entry in LDS makes room
      m.gh = m.gh == 0 ? kg - 1u : m.gh - 1u;
      g[m.gh] = back;
      ++m.gn;
      --m.n;
    }
    uint32_t i = m.n;
    for (; i > 0; --i) {
      const uint64_t p = l[(m.h + i - 1u) & mask];
      if (p <= x) break;
      l[(m.h + i) & mask] = p;
    }
    l[(m.h + i) & mask] = x;
    ++m.n;
    meta[kind] = m;
    return spilled;
  }
  __device__ void ring_pop(uint32_t kind) {
    RingMeta m = meta[kind];
    if (m.n == 0) {
      put(fr, kind, kNoEntry);
      return;
    }
    uint64_t *l = ring + (kind ? kl : 0u), *g = dev + (kind ? kg : 0u);
    const uint32_t mask = kl - 1u;
    put(fr, kind, l[m.h & mask]);
    m.h = (m.h + 1u) & mask;
    --m.n;
    if (m.n == 0)
      for (; m.n < kl && m.gn > 0; ++m.n, --m.gn) {
        l[(m.h + m.n) & mask] = g[m.gh];
        m.gh = wrap(m.gh + 1u);
      }
    meta[kind] = m;
  }
  // whether a stage at t joins S: S is empty, or both lie before t_last, or
  // it starts with S's run
  __device__ __forceinline__ bool joins(uint32_t kind, uint32_t t, uint32_t t_last) const {
    const uint32_t s = get(ts, kind);
    return max(s, t) < t_last || t == s || s == kNever;
  }
  // a stage that does not join S arrives; true if an entry went to device memory
  __device__ bool arrive_late(uint32_t kind, uint32_t t, uint32_t q, uint32_t t_last) {
    const uint32_t s = get(ts, kind);
    if (s < t_last || t > s) return ring_insert(kind, (uint64_t(t) << 32) | q);
    // S is a run of later stages: they go to the ring, the new one takes S
    bool spilled = false;
    do {
      spilled |= ring_insert(kind, (uint64_t(s) << 32) | get(first, kind));
      drop_first(kind);
    } while (get(first, kind) != kNone);
    join(kind, t, q);
    return spilled;
  }
  // ring entries that now belong to S
  __device__ void pull(uint32_t kind, uint32_t t_last) {
    for (;;) {
      const uint64_t f = get(fr, kind);
      if (f == kNoEntry || !joins(kind, uint32_t(f >> 32), t_last)) break;
      join(kind, uint32_t(f >> 32), uint32_t(f) & 0xffffu);
      ring_pop(kind);
    }
  }
};

}  // namespace

template <int RWL, int GWL>
__global__ __launch_bounds__(64, 4) void greedy_kernel(GreedyArgs a) {
  constexpr int RW = 1 << RWL;
  constexpr int GL = 1 << GWL;
  constexpr int GW = kWave >> GWL;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x;
  const int grp = lane >> GWL;
  const int r = lane & (GL - 1);
  const int G = a.G, P = a.P;
  const int rk = r < P ? r : 0;

  unsigned char *cb = lds + int64_t(grp) * a.cand_bytes;
  int32_t *prio = reinterpret_cast<int32_t *>(cb);               // set-up only ...
  // ... then the bitmaps, rings, messages and joins
  uint64_t *msg = reinterpret_cast<uint64_t *>(cb + a.off_msg);       // [RW] one per sender
  uint64_t *mask = msg + RW;                                          // [RW] senders per target
  uint16_t *qof = reinterpret_cast<uint16_t *>(cb + a.off_qof);       // group -> priority rank
  uint16_t *gof = reinterpret_cast<uint16_t *>(cb + a.off_gof);       // priority rank -> group
  const int64_t slot0 = int64_t(blockIdx.x) * GW + grp;
  uint32_t *jtab = reinterpret_cast<uint32_t *>(cb + a.off_join);     // {latest, arrived}
  uint32_t *jdev = a.joins_dev + slot0 * 2 * a.J;                     // in their place
  Queues qu;
  qu.nwd = uint32_t(a.nwd);
  qu.kl = uint32_t(a.kl);
  qu.kg = uint32_t(a.kg);
  qu.bits = reinterpret_cast<uint64_t *>(cb) + int64_t(rk) * (2 * a.nwd + 1);
  qu.ring = reinterpret_cast<uint64_t *>(cb + a.off_ring) + int64_t(rk) * (2 * a.kl + 1);
  qu.meta = reinterpret_cast<RingMeta *>(cb + a.off_meta) + 2 * rk;
  qu.dev = a.dring + (slot0 * P + rk) * 2 * int64_t(a.kg);

  const int64_t n_slots = int64_t(gridDim.x) * GW;
  for (int64_t cand = slot0;; cand += n_slots) {
    const bool has = cand < a.n_cand;
    if (!__any(has)) break;
    const bool real = has && r < P;

    // ---- set-up: priority ranks of the groups (priority, then index)
    const int Gp = (G + 3) & ~3;
    if (has) {
      const int32_t *pv = a.prio + cand * G;
      for (int g = r; g < Gp; g += GL) prio[g] = g < G ? pv[g] : INT32_MIN;
    }
    wave_sync();
    if (has) {
      // B groups of this lane against every group in turn; a group of lower
      // index wins a tie
      constexpr int B = 4;
      const int4 *p4 = reinterpret_cast<const int4 *>(prio);
      for (int g0 = 0; g0 < G; g0 += B * GL) {
        int32_t p[B];
        uint32_t n[B];
#pragma unroll
        for (int t = 0; t < B; ++t) {
          const int g = g0 + t * GL + r;
          p[t] = g < G ? prio[g] : INT32_MAX;
          n[t] = 0;
        }
        for (int h = 0; h < g0; h += 4) {
          const int4 x = p4[h >> 2];
#pragma unroll
          for (int t = 0; t < B; ++t)
            n[t] += uint32_t(x.x >= p[t]) + uint32_t(x.y >= p[t]) + uint32_t(x.z >= p[t]) +
                    uint32_t(x.w >= p[t]);
        }
#pragma unroll
        for (int s = 0; s < B; ++s) {
          const int hb = g0 + s * GL;
          for (int h = hb; h < min(hb + GL, Gp); h += 4) {
            const int4 x = p4[h >> 2];
            const int32_t xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int t = 0; t < B; ++t) {
                if (s < t)
                  n[t] += uint32_t(xs[e] >= p[t]);
                else if (s > t)
                  n[t] += uint32_t(xs[e] > p[t]);
                else
                  n[t] += uint32_t(xs[e] > p[t] || (xs[e] == p[t] && h + e - hb < r));
              }
          }
        }
        for (int h = g0 + B * GL; h < Gp; h += 4) {
          const int4 x = p4[h >> 2];
#pragma unroll
          for (int t = 0; t < B; ++t)
            n[t] += uint32_t(x.x > p[t]) + uint32_t(x.y > p[t]) + uint32_t(x.z > p[t]) +
                    uint32_t(x.w > p[t]);
        }
#pragma unroll
        for (int t = 0; t < B; ++t) {
          const int g = g0 + t * GL + r;
          if (g < G) {
            qof[g] = uint16_t(n[t]);
            gof[n[t]] = uint16_t(g);
          }
        }
      }
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      qu.first[k] = kNone;
      qu.ts[k] = kNever;
      qu.nz[k] = 0;
      qu.fr[k] = kNoEntry;
    }
    if (has) {
      if (a.joins_dev)
        for (int j = r; j < 2 * a.J; j += GL) jdev[j] = 0;
      else
        for (int j = r; j < 2 * a.J; j += GL) jtab[j] = 0;
    }
    if (r < RW) mask[r] = 0;         // (also of a group without a candidate)
    if (real) {
      for (int i = 0; i < 2 * a.nwd; ++i) qu.bits[i] = 0;
      qu.meta[0] = qu.meta[1] = RingMeta{0u, 0u, 0u, 0u};
      // the stages without predecessors: t_start 0
      const int32_t *src_list = a.src + P + 1;
      for (int s = a.src[r]; s < a.src[r + 1]; ++s) {
        const uint32_t g = uint32_t(src_list[s]);
        qu.join(g >> 16, 0u, qof[g & 0xffffu]);
      }
    }
    if (a.joins_dev) __threadfence();
    wave_sync();

    uint32_t t_last = 0, last_kind = 0, n_emit = 0;
    uint32_t rec_q = kNone;
    int4 q0 = make_int4(0, 0, 0, 0), q1 = q0;
    int32_t live = 0, peak = 0;
    bool spilled = false, stuck = false, bad = false;
    const int32_t capr = real ? a.cap[r] : -1;
    int16_t *const row = a.out_orders + (real ? cand * a.stride + a.rank_off[r] : 0);
    const uint32_t n_own = real ? uint32_t(a.rank_off[r + 1] - a.rank_off[r]) : 0u;
    int32_t left = has ? a.n_stages : 0;      // stages of the candidate to commit
    if constexpr (GWL == 6) left = __builtin_amdgcn_readfirstlane(left);

    while (GWL == 6 ? left > 0 : bool(__any(left > 0))) {
      // ---- 1. this rank's choice (lanes without a rank, and candidates that
      // are done, have empty queues)
      const uint64_t bF = qu.best(0, t_last), bB = qu.best(1, t_last);
      const bool alt = max(qu.ts[0], qu.ts[1]) < t_last;            // 1F1B
      uint32_t kind = alt ? (last_kind ^ 1u) : (bF < bB ? 0u : 1u);
      uint64_t c = kind ? bB : bF;
      uint32_t tau = uint32_t(c >> 32), q = uint32_t(c) & 0xffffu;
      // its record {cost, act, local id | successors << 16, second
      // successor's index}, {first successor}, kept while the choice stays
      // the same
      auto fetch = [&]() {
        const uint32_t at = (uint32_t(gof[q]) * uint32_t(P) + uint32_t(r)) * 32u;
        const int4 *rp =
            reinterpret_cast<const int4 *>(reinterpret_cast<const unsigned char *>(a.rec) + at);
        q0 = rp[0];
        q1 = rp[1];
        rec_q = q;
      };
      if (q != rec_q && q != kNone) fetch();
      uint32_t key = tau, tau_e = tau;
      if (a.has_cap) {
        if (q != kNone && kind == 0 && capr >= 0 && live + q0.y > capr) {
          // the forward queue is disabled: the best backward, if there is one
          kind = 1;
          c = bB;
          key = tau = uint32_t(c >> 32);
          q = uint32_t(c) & 0xffffu;
          if (q != kNone) fetch();
        }
      }

      // ---- 2. who commits: every rank whose start lies before the least
      // end, else the first rank of the least start (a stage without cost)
      const uint32_t end = tau + uint32_t(q0.x);
      const uint32_t e_min = group_reduce<RWL, GWL, false>(q != kNone ? end : kNever);
      bool com = key < e_min;
      uint64_t coms = group_bits<GWL>(__ballot(com), grp);
      if (GWL == 6 ? coms == 0 : bool(__any(left > 0 && coms == 0))) {
        const bool none = left > 0 && coms == 0;
        uint32_t m = group_reduce<RWL, GWL, false>(key);
        // every rank held back by its cap: the cap is lifted for one decision
        const bool lift = none && m == kNever;
        if (__any(lift)) {
          const uint32_t m2 = group_reduce<RWL, GWL, false>(tau_e);
          if (lift) {
            m = m2;
            key = tau_e;
          }
        }
        if (none && m == kNever) {              // only a cyclic data graph gets here
          stuck = true;
          left = 0;
        }
        const uint64_t mine = group_bits<GWL>(__ballot(none && m != kNever && key == m), grp);
        const bool win = mine != 0 && r == int(__builtin_ctzll(mine));
        if (win && lift) {
          // the first choice again
          kind = bF < bB ? 0u : 1u;
          if (alt) kind = last_kind ^ 1u;
          c = kind ? bB : bF;
          tau = uint32_t(c >> 32);
          q = uint32_t(c) & 0xffffu;
          fetch();
        }
        com = com || win;
        if (none) coms = group_bits<GWL>(__ballot(win), grp);
        if constexpr (GWL == 6) {
          left = __builtin_amdgcn_readfirstlane(left);
          if (coms == 0) break;
        }
      }
      left -= int32_t(__builtin_popcountll(coms));

      // The rest of the record is waited for here, before the commit's order
      // store: loads and stores share one counter, so a later wait for it
      // would wait for that store too.  The first successor's priority rank
      // is looked up at once, beside the commit's own LDS accesses.
      uint4 e = make_uint4(uint32_t(q1.x), uint32_t(q1.y), uint32_t(q1.z), uint32_t(q1.w));
      arrived(e);
      uint32_t eq = qof[e.x & 0xffffu];

      // ---- 3. commits: each lane's own queue, order and memory
      uint32_t ns = 0, t_end = 0;
      bool from_ring = false;
      if (com) {
        t_end = tau + uint32_t(q0.x);
        t_last = t_end;
        last_kind = kind;
        if (uint32_t(Queues::get(qu.fr, kind)) != q) {
          qu.drop_first(kind);
        } else {
          from_ring = true;
        }
        live += kind ? -q0.y : q0.y;
        peak = kind ? peak : max(peak, live);
        if (n_emit < n_own) {
          if (a.out_orders) row[n_emit] = int16_t(q0.z & 0xffff);
        } else {
          bad = true;     // more commits than stages: never with consistent tables
        }
        ++n_emit;
        ns = uint32_t(q0.z) >> 16;
        rec_q = kNone;
      }
      if (__builtin_expect(__any(from_ring), 0)) {
        if (from_ring) qu.ring_pop(kind);
      }
      const bool queued = com && (qu.fr[0] & qu.fr[1]) != kNoEntry;
      if (__builtin_expect(__any(queued), 0)) {
        if (queued) {
          qu.pull(0u, t_last);
          qu.pull(1u, t_last);
        }
      }

      // ---- 4. the stages these commits complete join their ranks' queues:
      // pass s sends every committed stage's successor s
      for (uint32_t s = 0; __any(s < ns); ++s) {
        bool send = s < ns;
        if (__builtin_expect(s > 0, 0)) {
          if (send) {
            const int4 x = a.succ[q0.w + int32_t(s) - 1];
            e = make_uint4(uint32_t(x.x), uint32_t(x.y), uint32_t(x.z), uint32_t(x.w));
            arrived(e);
            eq = qof[e.x & 0xffffu];
          }
        }
        const uint32_t w = (e.x & 0xffff0000u) | eq;    // priority rank, kind, target rank
        uint32_t t = t_end + e.y;
        const bool join = send && int32_t(e.z) >= 0;
        if (__builtin_expect(__any(join), 0)) {
          if (join) {
            // (every lane's maximum lands before any lane's count: the lanes
            // take each of the two steps together)
            if (a.joins_dev) {
              uint32_t *jb = jdev + 2 * int64_t(e.z);
              atomicMax(jb, t);
              __threadfence();
              send = atomicAdd(jb + 1, 1u) + 1u >= e.w;
              if (send) t = atomicMax(jb, 0u);
            } else {
              uint32_t *jb = jtab + 2 * int64_t(e.z);
              atomicMax(jb, t);
              wave_lds_order();
              send = atomicAdd(jb + 1, 1u) + 1u >= e.w;
              if (send) t = jb[0];
            }
          }
        }
        // a stage arrives at the lanes of `in`: word w (priority rank, kind),
        // start t
        auto deliver = [&](bool in, uint32_t aw, uint32_t at) {
          const uint32_t ak = (aw >> 16) & 1u, aq = aw & 0xffffu;
          const bool now = qu.joins(ak, at, t_last);
          if (in && now) qu.join(ak, at, aq);
          const bool late = in && !now;
          if (__any(late)) {
            // most rings are empty
            const uint32_t ts = Queues::get(qu.ts, ak);
            const bool first =
                late && Queues::get(qu.fr, ak) == kNoEntry && (ts < t_last || at > ts);
            if (first) Queues::put(qu.fr, ak, (uint64_t(at) << 32) | aq);
            const bool rest = late && !first;
            if (__builtin_expect(__any(rest), 0)) {
              if (rest) spilled |= qu.arrive_late(ak, at, aq, t_last);
            }
          }
        };
        if constexpr (GWL == 6) {
          uint64_t todo = __ballot(send);
          if (todo) {
            uint64_t to = 0;
            uint32_t aw = 0, at = 0;
            if constexpr (RWL < 6) {
              // every message into its target's lane at once; lanes without
              // one write to the last lane, which is no rank.  Of two for one
              // rank only one lands, and the lanes that got one are fewer.
              const int lane_at = send ? int((w >> 17) & 63u) * 4 : 63 * 4;
              aw = uint32_t(__builtin_amdgcn_ds_permute(lane_at, int(w | 0x80000000u)));
              at = uint32_t(__builtin_amdgcn_ds_permute(lane_at, int(t)));
              to = __ballot(lane != 63 && int32_t(aw) < 0);
              if (__builtin_popcountll(to) == __builtin_popcountll(todo)) todo = 0;
            }
            do {
              if (__builtin_expect(todo != 0, RWL == 6)) {
                // one by one, up to a second message for a rank
                to = 0;
                do {
                  const int i = __builtin_ctzll(todo);
                  const uint32_t sw = uint32_t(__builtin_amdgcn_readlane(int(w), i));
                  const uint32_t st = uint32_t(__builtin_amdgcn_readlane(int(t), i));
                  const uint32_t tr = (sw >> 17) & 63u;
                  if ((to >> tr) & 1u) break;
                  todo &= todo - 1;
                  to |= uint64_t(1) << tr;
                  aw = uint32_t(lane) == tr ? sw : aw;
                  at = uint32_t(lane) == tr ? st : at;
                } while (todo);
              }
              deliver(__builtin_amdgcn_inverse_ballot_w64(to), aw, at);
            } while (todo);
          }
        } else {
          if (send) {
            msg[r] = (uint64_t(t) << 32) | w;
            atomicOr(reinterpret_cast<unsigned long long *>(mask + ((w >> 17) & 63u)),
                     static_cast<unsigned long long>(uint64_t(1) << r));
          }
          wave_lds_order();
          uint64_t from = mask[r];
          if (from) mask[r] = 0;
          while (__any(from != 0)) {
            const bool in = from != 0;
            const uint64_t x = msg[in ? __builtin_ctzll(from) : 0];
            from &= from - 1;
            deliver(in, uint32_t(x), uint32_t(x >> 32));
          }
          wave_lds_order();
        }
      }
    }

    // ---- outputs
    const uint32_t T = group_reduce<RWL, GWL, true>(real ? t_last : 0u);
    const uint64_t wcap = __ballot(real && capr >= 0 && peak > capr);
    const uint64_t wspill = __ballot(spilled);
    const uint64_t wbad = __ballot(bad);
    const bool gcap = group_bits<GWL>(wcap, grp) != 0;
    const bool gbad = group_bits<GWL>(wbad, grp) != 0;
    if (has) {
      if (real) {
        a.out_bub[cand * P + r] = stuck || gbad ? -1 : int32_t(T) - a.busy[r];
        a.out_peak[cand * P + r] = gbad ? -1 : peak;
      }
      if (r == 0) {
        a.out_ms[cand] = stuck || gbad ? -1 : int32_t(T);
        a.out_flags[cand] = gbad ? uint8_t(DIP_FLAG_INVALID)
                                 : uint8_t((stuck ? DIP_FLAG_DEADLOCK : 0u) | (gcap ? DIP_FLAG_CAP : 0u));
        if (a.spill_count && group_bits<GWL>(wspill, grp) != 0) atomicAdd(a.spill_count, 1u);
      }
    }
    wave_sync();
  }
}

__global__ void zero_words_kernel(uint32_t *p, int n) {
  if (int(threadIdx.x) < n) p[threadIdx.x] = 0u;
}

hipError_t launch_zero_words(uint32_t *p, int n, hipStream_t s) {
  zero_words_kernel<<<1, 64, 0, s>>>(p, n);
  return hipGetLastError();
}

const void *greedy_kernel_ptr(int rwl, bool wide) {
  switch (rwl) {
    case 2:
      return wide ? reinterpret_cast<const void *>(&greedy_kernel<2, 6>)
                  : reinterpret_cast<const void *>(&greedy_kernel<2, 2>);
    case 3:
      return wide ? reinterpret_cast<const void *>(&greedy_kernel<3, 6>)
                  : reinterpret_cast<const void *>(&greedy_kernel<3, 3>);
    case 4:
      return wide ? reinterpret_cast<const void *>(&greedy_kernel<4, 6>)
                  : reinterpret_cast<const void *>(&greedy_kernel<4, 4>);
    case 5:
      return wide ? reinterpret_cast<const void *>(&greedy_kernel<5, 6>)
                  : reinterpret_cast<const void *>(&greedy_kernel<5, 5>);
    case 6: return reinterpret_cast<const void *>(&greedy_kernel<6, 6>);
    default: return nullptr;
  }
}

hipError_t launch_greedy(int rwl, bool wide, int blocks, size_t lds, hipStream_t s,
                         const GreedyArgs &a) {
  const void *k = greedy_kernel_ptr(rwl, wide);
  if (!k) return hipErrorInvalidValue;
  void *args[] = {const_cast<GreedyArgs *>(&a)};
  return hipLaunchKernel(k, dim3(unsigned(blocks)), dim3(kWave), args, lds, s);
}

}  // namespace dipsim
