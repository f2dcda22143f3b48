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
// the least t_min always does.  On the workloads that is 2 to 5 commits a
// round (11 on 64 equal ranks), with the sequential greedy's result.
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
// A committing lane changes its own queue only.  What its stage completes
// goes to the target ranks as messages, one per sender and pass: the sender
// writes {t_start, q, kind} into its slot and sets its bit in the target's
// mask; each target takes its messages in turn.
//
// What bounds it: latency and vector issue of a round's serial chain (choice,
// record, reductions, commit, messages); bandwidth is a few percent.
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

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xf, 0xf, false));
}

// min / max over aligned runs of 2^WL lanes: quad permutations, then the
// half-row and row mirrors (each lane meets the other half), then shuffles
template <int WL, bool MAX>
__device__ __forceinline__ uint32_t run_reduce(uint32_t v) {
  auto op = [](uint32_t x, uint32_t y) { return MAX ? max(x, y) : min(x, y); };
  if constexpr (WL >= 1) v = op(v, dpp<0xb1>(v));    // quad_perm [1,0,3,2]
  if constexpr (WL >= 2) v = op(v, dpp<0x4e>(v));    // quad_perm [2,3,0,1]
  if constexpr (WL >= 3) v = op(v, dpp<0x141>(v));   // row_half_mirror
  if constexpr (WL >= 4) v = op(v, dpp<0x140>(v));   // row_mirror
  if constexpr (WL >= 5) v = op(v, uint32_t(__shfl_xor(int(v), 16)));
  if constexpr (WL >= 6) v = op(v, uint32_t(__shfl_xor(int(v), 32)));
  return v;
}

// the same over a candidate's 2^GWL lanes, whose ranks are the first 2^RWL
template <int RWL, int GWL, bool MAX>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v) {
  v = run_reduce<RWL, MAX>(v);
  if constexpr (GWL == 6 && RWL < 6) v = uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
  return v;
}

// bits of this lane's group in a wave-wide mask, lowest rank at bit 0
template <int GWL>
__device__ __forceinline__ uint64_t group_bits(uint64_t m, int grp) {
  if constexpr (GWL == 6) return m;
  constexpr uint64_t low = (uint64_t(1) << ((1 << GWL) & 63)) - 1;
  return (m >> (grp << GWL)) & low;
}

// Where a rank's rings lie beyond their first entry: KL entries (a power of
// two) a kind in LDS, KG entries a kind in device memory.
struct RingMem {
  uint64_t *lds, *dev;
  uint32_t kl, kg;
};

// One kind's queue of one rank (registers of its lane).
struct Queue {
  uint64_t *bits;      // S, by priority rank
  uint64_t nz;         // its non-zero words
  uint32_t first;      // its first member, kNone if empty
  uint32_t ts;         // the members' t_start when that is >= t_last
  uint64_t fr;         // the ring's first entry (t_start << 32 | q), or kNoEntry
  uint32_t h, n;       // head and count of its entries in LDS
  uint32_t gh, gn;     // and in device memory
  RingMem m;

  __device__ __forceinline__ void clear(uint64_t *b, const RingMem &mem) {
    bits = b;
    m = mem;
    nz = 0;
    first = kNone;
    ts = 0;
    fr = kNoEntry;
    h = n = gh = gn = 0;
  }
  __device__ __forceinline__ void set(uint32_t q) {
    const uint32_t k = q >> 6;
    bits[k] |= uint64_t(1) << (q & 63u);
    nz |= uint64_t(1) << k;
    first = min(first, q);
  }
  // takes the first member out
  __device__ __forceinline__ void drop_first() {
    uint32_t k = first >> 6;
    uint64_t w = bits[k];
    w &= w - 1;
    bits[k] = w;
    if (w == 0) {
      nz &= nz - 1;
      if (nz == 0) {
        first = kNone;
        return;
      }
      k = uint32_t(__builtin_ctzll(nz));
      w = bits[k];
    }
    first = k * 64u + uint32_t(__builtin_ctzll(w));
  }
  __device__ __forceinline__ uint32_t dev_at(uint32_t i) const {
    const uint32_t x = gh + i;
    return x >= m.kg ? x - m.kg : x;
  }
  // x into the sorted ring; true if an entry went to device memory
  __device__ __forceinline__ bool ring_insert(uint64_t x) {
    if (x < fr) {
      const uint64_t y = fr;
      fr = x;
      if (y == kNoEntry) return false;
      x = y;
    }
    const uint32_t mask = m.kl - 1u;
    bool spilled = false;
    if (gn > 0 || n >= m.kl) {
      // (entries in device memory only ever follow a non-empty LDS part)
      spilled = true;
      const uint64_t back = m.lds[(h + n - 1u) & mask];
      if (back <= x) {
        uint32_t i = gn;
        for (; i > 0; --i) {
          const uint64_t p = m.dev[dev_at(i - 1u)];
          if (p <= x) break;
          m.dev[dev_at(i)] = p;
        }
        m.dev[dev_at(i)] = x;
        ++gn;
        return true;
      }
      // the last entry in LDS makes room
      gh = gh == 0 ? m.kg - 1u : gh - 1u;
      m.dev[gh] = back;
      ++gn;
      --n;
    }
    uint32_t i = n;
    for (; i > 0; --i) {
      const uint64_t p = m.lds[(h + i - 1u) & mask];
      if (p <= x) break;
      m.lds[(h + i) & mask] = p;
    }
    m.lds[(h + i) & mask] = x;
    ++n;
    return spilled;
  }
  __device__ __forceinline__ void ring_pop() {
    if (n == 0) {
      fr = kNoEntry;
      return;
    }
    const uint32_t mask = m.kl - 1u;
    fr = m.lds[h & mask];
    h = (h + 1u) & mask;
    --n;
    if (n == 0 && gn > 0) {
      for (; n < m.kl && gn > 0; ++n, --gn) {
        m.lds[(h + n) & mask] = m.dev[gh];
        gh = dev_at(1u);
      }
    }
  }
  // whether a stage at t joins S: S is empty, or both lie before t_last, or
  // it starts with S's run
  __device__ __forceinline__ bool joins(uint32_t t, uint32_t t_last) const {
    return first == kNone || (ts < t_last && t < t_last) || t == ts;
  }
  __device__ __forceinline__ void join(uint32_t t, uint32_t q) {
    if (first == kNone) ts = t;
    set(q);
  }
  // a stage arrives; true if an entry went to device memory
  __device__ __forceinline__ bool arrive(uint32_t t, uint32_t q, uint32_t t_last) {
    if (joins(t, t_last)) {
      join(t, q);
      return false;
    }
    if (ts < t_last || t > ts) return ring_insert((uint64_t(t) << 32) | q);
    // S is a run of later stages: they go to the ring, the new one takes S
    bool spilled = false;
    do {
      spilled |= ring_insert((uint64_t(ts) << 32) | first);
      drop_first();
    } while (first != kNone);
    ts = t;
    set(q);
    return spilled;
  }
  // ring entries that now belong to S
  __device__ __forceinline__ void pull(uint32_t t_last) {
    while (fr != kNoEntry && joins(uint32_t(fr >> 32), t_last)) {
      join(uint32_t(fr >> 32), uint32_t(fr) & 0xffffu);
      ring_pop();
    }
  }
  __device__ __forceinline__ uint32_t least() const { return first == kNone ? kNever : ts; }
};

// One rank's choice: start time, priority rank, kind (0 forward, 1 backward)
// and whether it is the kind's first ring entry.
struct Choice {
  uint32_t tau, q, kind;
  bool ring;
};

}  // namespace

template <int RWL, int GWL>
__global__ __launch_bounds__(64) void greedy_kernel(GreedyArgs a) {
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
  uint64_t *bits0 = reinterpret_cast<uint64_t *>(cb) + int64_t(rk) * (2 * a.nwd + 1);
  uint64_t *ring0 = reinterpret_cast<uint64_t *>(cb + a.off_ring) + int64_t(rk) * (2 * a.kl + 1);
  uint64_t *msg = reinterpret_cast<uint64_t *>(cb + a.off_msg);       // [RW] one per sender
  uint64_t *mask = msg + RW;                                          // [RW] senders per target
  uint16_t *qof = reinterpret_cast<uint16_t *>(cb + a.off_qof);       // group -> priority rank
  uint16_t *gof = reinterpret_cast<uint16_t *>(cb + a.off_gof);       // priority rank -> group
  const int64_t slot0 = int64_t(blockIdx.x) * GW + grp;
  uint32_t *jtab = reinterpret_cast<uint32_t *>(cb + a.off_join);     // {latest, arrived}
  uint32_t *jdev = a.joins_dev + slot0 * 2 * a.J;                     // in their place
  uint64_t *dev0 = a.dring + (slot0 * P + rk) * 2 * int64_t(a.kg);
  const RingMem memF{ring0, dev0, uint32_t(a.kl), uint32_t(a.kg)};
  const RingMem memB{ring0 + a.kl, dev0 + a.kg, uint32_t(a.kl), uint32_t(a.kg)};

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
    Queue qF, qB;
    qF.clear(bits0, memF);
    qB.clear(bits0 + a.nwd, memB);
    if (has) {
      if (a.joins_dev)
        for (int j = r; j < 2 * a.J; j += GL) jdev[j] = 0;
      else
        for (int j = r; j < 2 * a.J; j += GL) jtab[j] = 0;
      if (r < RW) mask[r] = 0;
    }
    if (real) {
      for (int i = 0; i < 2 * a.nwd; ++i) bits0[i] = 0;
      // the stages without predecessors: t_start 0
      const int32_t *src_list = a.src + P + 1;
      for (int s = a.src[r]; s < a.src[r + 1]; ++s) {
        const int g = src_list[s];
        if (g >> 16)
          qB.join(0u, qof[g & 0xffff]);
        else
          qF.join(0u, qof[g]);
      }
    }
    if (a.joins_dev) __threadfence();
    wave_sync();

    uint32_t t_last = 0, last_kind = 0, n_emit = 0;
    uint32_t rec_key = kNever;
    int4 q0 = make_int4(0, 0, 0, 0), q1 = q0;
    int32_t live = 0, peak = 0;
    bool spilled = false, stuck = false, bad = false;
    const int32_t capr = real ? a.cap[r] : -1;
    const int64_t row = real ? cand * a.stride + a.rank_off[r] : 0;
    const uint32_t n_own = real ? uint32_t(a.rank_off[r + 1] - a.rank_off[r]) : 0u;
    int32_t left = has ? a.n_stages : 0;      // stages of the candidate to commit

    while (__any(left > 0)) {
      // ---- 1. this rank's choice
      // the best stage of each kind able to start at tau: S's first, or the
      // ring's first when it starts at tau too (beside an S before t_last)
      const uint32_t tB = qB.least();
      auto decide = [&](bool fw) {
        Choice c;
        const uint32_t tF = fw ? qF.least() : kNever;
        const uint32_t tmin = min(tF, tB);
        c.tau = max(t_last, tmin);
        uint32_t bF = tF <= c.tau && fw ? qF.first : kNone;
        uint32_t bB = tB <= c.tau ? qB.first : kNone;
        const bool inF = fw && uint32_t(qF.fr >> 32) == c.tau && (uint32_t(qF.fr) & 0xffffu) < bF;
        const bool inB = uint32_t(qB.fr >> 32) == c.tau && (uint32_t(qB.fr) & 0xffffu) < bB;
        if (inF) bF = uint32_t(qF.fr) & 0xffffu;
        if (inB) bB = uint32_t(qB.fr) & 0xffffu;
        const bool alt = tF < t_last && tB < t_last;               // 1F1B
        c.kind = alt ? (last_kind ^ 1u) : (bF < bB ? 0u : 1u);
        c.q = tmin == kNever ? kNone : (c.kind ? bB : bF);
        c.ring = c.kind ? inB : inF;
        return c;
      };
      // the record of a choice: {cost, act, local id | successors << 16,
      // second successor's index}, {first successor}; kept while the choice
      // stays the same
      auto fetch = [&](const Choice &c) {
        if (c.q != rec_key) {
          const int4 *rp = a.rec + (int64_t(gof[c.q]) * P + r) * 2;
          q0 = rp[0];
          q1 = rp[1];
          rec_key = c.q;
        }
      };
      Choice ce = decide(true);
      const bool act = left > 0 && r < P;
      if (!act) ce.q = kNone;
      Choice cd = ce;
      if (ce.q != kNone) {
        fetch(ce);
        if (a.has_cap && ce.kind == 0 && capr >= 0 && live + q0.y > capr) {
          cd = decide(false);                   // forward queue disabled
          if (cd.q != kNone) fetch(cd);
        }
      }

      // ---- 2. who commits: the rank of the least t_min, and every rank
      // whose t_min lies before the least end
      uint32_t key = cd.q != kNone ? cd.tau : kNever;
      const uint32_t end = cd.tau + uint32_t(q0.x);
      uint32_t m = group_reduce<RWL, GWL, false>(key);
      const uint32_t e_min = group_reduce<RWL, GWL, false>(cd.q != kNone ? end : kNever);
      bool forced = false;
      if (__any(left > 0 && m == kNever)) {
        const uint32_t key_e = ce.q != kNone ? ce.tau : kNever;
        const uint32_t m2 = group_reduce<RWL, GWL, false>(key_e);
        if (m == kNever) {
          forced = true;
          m = m2;
          key = key_e;
        }
      }
      if (left > 0 && m == kNever) {            // only a cyclic data graph gets here
        stuck = true;
        left = 0;
      }
      const uint64_t mine = group_bits<GWL>(__ballot(act && m != kNever && key == m), grp);
      const bool win = mine != 0 && r == int(__builtin_ctzll(mine));
      const bool com = win || (!forced && key < e_min);
      const uint64_t coms = group_bits<GWL>(__ballot(com), grp);
      left -= int32_t(__builtin_popcountll(coms));

      // ---- 3. commits: each lane's own queue, order and memory
      uint32_t ns = 0, t_end = 0;
      if (com) {
        Choice c = cd;
        if (forced) {
          c = ce;
          fetch(c);
        }
        t_end = c.tau + uint32_t(q0.x);
        t_last = t_end;
        last_kind = c.kind;
        if (c.kind) {
          if (c.ring)
            qB.ring_pop();
          else
            qB.drop_first();
        } else {
          if (c.ring)
            qF.ring_pop();
          else
            qF.drop_first();
        }
        qF.pull(t_last);
        qB.pull(t_last);
        live += c.kind ? -q0.y : q0.y;
        if (c.kind == 0) peak = max(peak, live);
        if (n_emit < n_own) {
          if (a.out_orders) a.out_orders[row + n_emit] = int16_t(q0.z & 0xffff);
        } else {
          bad = true;     // more commits than stages: never with consistent tables
        }
        ++n_emit;
        ns = uint32_t(q0.z) >> 16;
        rec_key = kNever;
      }

      // ---- 4. the stages these commits complete join their ranks' queues:
      // pass s sends every committed stage's successor s
      for (uint32_t s = 0; __any(s < ns); ++s) {
        bool send = s < ns;
        if (send) {
          const int4 e = s == 0 ? q1 : a.succ[q0.w + int32_t(s) - 1];
          uint32_t t = t_end + uint32_t(e.y);
          if (e.z >= 0) {
            // (every lane's maximum lands before any lane's count: the lanes
            // take each of the two steps together)
            if (a.joins_dev) {
              uint32_t *jb = jdev + 2 * e.z;
              atomicMax(jb, t);
              __threadfence();
              send = atomicAdd(jb + 1, 1u) + 1u >= uint32_t(e.w);
              if (send) t = atomicMax(jb, 0u);
            } else {
              uint32_t *jb = jtab + 2 * e.z;
              atomicMax(jb, t);
              wave_lds_order();
              send = atomicAdd(jb + 1, 1u) + 1u >= uint32_t(e.w);
              if (send) t = jb[0];
            }
          }
          if (send) {
            const uint32_t w = uint32_t(e.x);
            const uint32_t tr = (w >> 17) & 63u, tk = (w >> 16) & 1u;
            msg[r] = (uint64_t(t) << 32) | (tk << 16) | qof[w & 0xffffu];
            atomicOr(reinterpret_cast<unsigned long long *>(mask + tr),
                     static_cast<unsigned long long>(uint64_t(1) << r));
          }
        }
        wave_lds_order();
        uint64_t from = 0;
        if (act) {
          from = mask[r];
          if (from) mask[r] = 0;
        }
        while (__any(from != 0)) {
          if (from) {
            const uint64_t x = msg[__builtin_ctzll(from)];
            from &= from - 1;
            const uint32_t t = uint32_t(x >> 32), q = uint32_t(x) & 0xffffu;
            if (uint32_t(x) & 0x10000u)
              spilled |= qB.arrive(t, q, t_last);
            else
              spilled |= qF.arrive(t, q, t_last);
          }
        }
        wave_lds_order();
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
