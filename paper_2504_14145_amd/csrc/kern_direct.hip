// kern_direct.hip -- timing simulation of candidate schedules with every end
// time of a candidate in LDS.
//
// The same simulation, records, order rings and verdicts as the simulation
// kernel (kern_sim.hip): a group of PW lanes per candidate, lane r playing
// rank r, one op of every rank looked at a round.  There, end times travel
// through small pools that a consumer searches and that can fill; here an op
// writes its end time to its own word of a table of N words, and a consumer
// reads its predecessor's word: no tags, no reader counts, no back-pressure,
// so nothing is ever left to a later pass, and a round takes about two thirds
// of the time (64 candidates: 8 ranks 72 -> 56 us, 16 x 2 lanes 207 -> 150, 32
// ranks 329 -> 242).  The table costs 4 N bytes a candidate, so this kernel is
// for batches whose candidates are all resident at once, and for the few that
// filled the pools (list mode, a resident group taking several in turn); the
// pools hold many more candidates of many ops (65,536 on 16 x 2 lanes: 1.2 ms
// against 9.3 here).
//
// Records are those of the simulation kernel but for the edge word, which
// holds the predecessor's global index relative to the op's own, so that its
// address is one addition.
#include "dip_sim.h"
#include "dev_util.h"
#include "internal.h"
#include "lds_util.h"

namespace dipsim {
namespace {

constexpr uint32_t kNotRun = 0xffffffffu;

// SEL: the re-timed simulation of a memory selection, where every op has an
// extra cost of its own in its candidate; they are staged as the ids are.
template <int PWL, bool PAGED, bool SEL>
__global__ __launch_bounds__(1024) void direct_kernel(DirectArgs a) {
  constexpr int PW = 1 << PWL;
  constexpr int G = kWave / PW;
  constexpr uint32_t kRingBytes = uint32_t(sim_ring_bytes(SEL));

  if (a.list && *a.list_count == 0) return;
  // the tables into LDS, once per block
  for (int i = threadIdx.x; i < a.tab_vec; i += blockDim.x)
    *reinterpret_cast<uint4 *>(s_lds + 16u * uint32_t(i)) = a.tab[i];
  __syncthreads();

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int grp = lane >> PWL;
  const int r = lane & (PW - 1);
  const bool on = r < a.P;
  const int gbit = grp << PWL;
  const int64_t n_slots = int64_t(gridDim.x) * a.wpb * G;
  const uint32_t gbase = uint32_t(a.tab_vec) * 16u + uint32_t(wave * G + grp) * a.group_bytes;
  const uint32_t rr = on ? uint32_t(r) : 0u;
  const uint32_t my_ring = gbase + a.off_ring + rr * kRingBytes;
  int rb = 0, nr = 0, busy_r = 0, recb = 0;
  if (on) {
    const int4 li = reinterpret_cast<const int4 *>(a.lane_info)[r];
    rb = li.x;
    nr = li.y;
    busy_r = li.z;
    recb = li.w;
  }
  // absolute row positions: past this lane's section, its last block
  const uint32_t a_end = uint32_t(rb + nr);
  const uint32_t blk_last = uint32_t(rb + max(nr - 1, 0)) / uint32_t(kSimBlockIds);
  const uint32_t pmap_lane = lds_abs(a.off_pmap + 2u * uint32_t(recb));
  const uint32_t my_ends = gbase + 4u * uint32_t(rb);     // end time of local id 0

  // the record of local id `id` of this lane's rank
  auto rec_of = [&](uint32_t id) -> uint2 {
    uint32_t first;   // record index of the page's first op, or of the rank's
    if constexpr (PAGED) {
      first = lds16_at(shl_add<1>(id >> 4, pmap_lane)) | (id & 15u);
    } else {
      first = uint32_t(recb) + id;
    }
    return lds64(first << 3);
  };
  const uint32_t my_ring_abs = lds_abs(my_ring);
  auto ring_id = [&](uint32_t pos) { return lds16_at(shl_add<1>(pos & 15u, my_ring_abs)); };
  // (SEL) the ring's extra costs: block b at kSimRingBytes + 32 (b & 1)
  auto ring_x = [&](uint32_t pos) -> uint32_t {
    if constexpr (SEL) return lds32(my_ring + uint32_t(kSimRingBytes) + 4u * (pos & 15u));
    return 0u;
  };

  // candidates: 0 .. n_cand - 1, or those of the list
  const int64_t n_todo = a.list ? int64_t(*a.list_count) : a.n_cand;
  auto cand_at = [&](int64_t i) { return a.list ? a.list[i] : i; };
  // slot of this group: neighbouring candidates in different blocks, then in
  // different waves, so that few candidates spread over the CUs
  int64_t k = (int64_t(grp) * a.wpb + wave) * gridDim.x + blockIdx.x;

  // per-lane state
  int64_t cand = 0;
  bool has = false;        // the group holds a candidate
  uint8_t fl = 0;          // the check kernel's flags for it
  uint32_t apos1 = 0;      // absolute row position of the op after the current one
  uint32_t tfree = 0, acc = 0;
  uint32_t mya = 0, cur0 = 0;   // current op: its end time's address, record word 0
  uint32_t ce = 0, xi = 0;      // its current edge word; index of its next extra edge
  uint32_t lb = 0;         // next absolute order block to load
  uint4 blk{};             // a loaded block waiting to be stored
  uint4 xb0{}, xb1{};      // (SEL) its extra costs
  uint32_t curx = 0;       // (SEL) the current op's extra cost
  const int16_t *row = a.orders;
  const int32_t *xrow = a.xcost;
  auto load_x = [&](uint32_t b) {
    if constexpr (SEL) {
      const uint4 *q = reinterpret_cast<const uint4 *>(xrow + int64_t(b) * kSimBlockIds);
      xb0 = q[0];
      xb1 = q[1];
    }
  };
  auto store_x = [&](uint32_t b) {
    if constexpr (SEL) {
      const uint32_t at = my_ring + uint32_t(kSimRingBytes) + (b & 1u) * 32u;
      store_block(at, xb0);
      store_block(at + 16u, xb1);
    }
  };

  // wave-uniform lane masks
  uint64_t m_live = 0;     // lanes running an op sequence
  uint64_t m_npend = 0;    // live lanes whose current op waits for no edge
  uint64_t m_blk = 0;      // lanes holding a loaded block for the ring

  auto set_current = [&](uint32_t id, uint2 c) {
    mya = my_ends + 4u * id;
    cur0 = c.x;
    ce = c.y;
    xi = c.y + 1u;
    if (c.x >= (kSimHasPred | kSimMulti)) ce = lds32(a.off_extra + 4u * c.y);   // several predecessors
  };

  // The lanes of one group call this together (a group without a candidate
  // keeps its lanes out of m_live).
  auto start_candidate = [&]() {
    // (candidates whose verdict the check kernel already settled: not a
    // permutation, or an op ordered before its own-rank predecessor)
    while (k < n_todo && (a.out_flags[cand_at(k)] & (DIP_FLAG_INVALID | DIP_FLAG_DEADLOCK)))
      k += n_slots;
    has = k < n_todo;
    if (!has) return;
    for (uint32_t i = uint32_t(r); i < a.end_vec; i += PW)
      *reinterpret_cast<uint4 *>(s_lds + gbase + 16u * i) = make_uint4(kNotRun, kNotRun, kNotRun, kNotRun);
    cand = cand_at(k);
    fl = a.out_flags[cand];
    tfree = 0;
    acc = 0;
    if (!on || nr == 0) return;
    row = a.orders + cand * a.stride;
    // the first two blocks of the section into the ring
    const uint32_t b0 = uint32_t(rb) / uint32_t(kSimBlockIds);
    const uint32_t bn = min(b0 + 1u, blk_last);
    if constexpr (SEL) xrow = a.xcost + cand * a.stride;
    for (uint32_t b = b0; b <= bn; ++b) {
      store_block(my_ring + (b & 1u) * 16u, load_block(row, b));
      load_x(b);
      store_x(b);
    }
    lb = bn + 1u;
    apos1 = uint32_t(rb) + 1u;
    const uint32_t id0 = ring_id(uint32_t(rb));
    set_current(id0, rec_of(id0));
    curx = ring_x(uint32_t(rb));
  };

  start_candidate();
  {
    const bool live = has && on && nr > 0;
    m_live = ballot(live);
    m_npend = m_live & ballot(int32_t(cur0) >= 0);
  }
  uint64_t g_has = any_in_group<PWL>(ballot(has));

  uint32_t rnd = 0;
  while (g_has) {
    // ---- order blocks: loaded every 4 rounds, stored 3 rounds later
    const uint32_t phase = rnd & 3u;
    if (phase == 3u && m_blk) {
      if (lane_in(m_blk)) {
        store_block(my_ring + (lb & 1u) * 16u, blk);
        store_x(lb);
        ++lb;
      }
      m_blk = 0;
    }

    // ---- reads: the predecessor's end time, the next id and its record
    const uint32_t pe = lds32(mya + 4u * uint32_t(int32_t(ce << 15) >> 15));
    const uint32_t idn = ring_id(apos1);
    const uint2 nrec = rec_of(idn);
    const uint32_t nx = ring_x(apos1);

    const uint64_t m_found = ballot(int32_t(pe) >= 0) & m_live & ~m_npend;
    const bool found = lane_in(m_found);
    const uint32_t acc_n = found ? max(acc, pe + ((ce >> 17) & 0x7ffu)) : acc;
    const uint64_t m_last = ballot(int32_t(ce) < 0);
    const uint64_t m_fire = (m_found & m_last) | m_npend;
    const bool fire = lane_in(m_fire);
    const uint32_t en = max(tfree, acc_n) + (cur0 & kSimCostMax) + (SEL ? curx : 0u);

    // ---- writes and register state
    const uint64_t m_fin = m_fire & ballot(apos1 == a_end);
    const uint64_t m_adv = m_fire & ~m_fin;
    if (fire) {
      st32(mya, en);
      tfree = en;
    }
    acc = fire ? 0u : acc_n;
    if (lane_in(m_found & ~m_last)) {   // the op's next predecessor edge
      ce = lds32(a.off_extra + 4u * xi);
      ++xi;
    }
    if (lane_in(m_adv)) {   // the next op becomes current
      set_current(idn, nrec);
      if constexpr (SEL) curx = nx;
      ++apos1;
    }
    m_npend = m_adv & ballot(int32_t(cur0) >= 0);
    m_live &= ~m_fin;

    // ---- order blocks: every 4 rounds, a lane in the later of its two
    // blocks loads the one after it
    if (phase == 0u) {
      const uint32_t next_blk = (apos1 + uint32_t(kSimBlockIds) - 1u) / uint32_t(kSimBlockIds);
      const bool load = lane_in(m_live) && lb <= min(next_blk, blk_last);
      m_blk = ballot(load);
      if (load) {
        blk = load_block(row, lb);
        load_x(lb);
      }
    }

    // ---- verdicts, every 8 rounds (a group that finished or stalled waits
    // for the next check; its state does not change meanwhile): all lanes ran
    // their whole order, or none fired an op or read an end time -- nothing
    // but a later end time could change that, so the orders deadlock
    ++rnd;
    if ((rnd & 7u) != 0u) continue;
    const uint64_t g_run = any_in_group<PWL>(m_live);
    const uint64_t g_done = g_has & ~g_run;
    const uint64_t g_stall = g_run & ~any_in_group<PWL>(m_fire | m_found);
    const uint64_t ev = g_done | g_stall;
    if (ev == 0) continue;

    const uint64_t m_ev = any_lane_of_group<PWL>(ev);
    if (lane_in(m_ev)) {
      const bool stalled = (g_stall >> gbit) & 1;
      uint32_t T = on ? tfree : 0u;
#pragma unroll
      for (int off = 1; off < PW; off <<= 1) T = max(T, uint32_t(__shfl_xor(int(T), off, kWave)));
      if (has && on) {
        int32_t busy = busy_r;
        if constexpr (SEL) busy += a.out_bub[cand * a.P + r];
        a.out_bub[cand * a.P + r] = stalled ? -1 : int32_t(T) - busy;
        if (r == 0) {
          a.out_ms[cand] = stalled ? -1 : int32_t(T);
          if (stalled) a.out_flags[cand] = uint8_t(fl | DIP_FLAG_DEADLOCK);
        }
      }
      k += n_slots;
      start_candidate();
    }
    // the restarted groups' lanes: live and edge state from their new records
    const bool live_new = has && on && nr > 0;
    m_live = (m_live & ~m_ev) | (m_ev & ballot(live_new));
    m_npend = (m_npend & ~m_ev) | (m_ev & m_live & ballot(int32_t(cur0) >= 0));
    m_blk &= ~m_ev;
    g_has = any_in_group<PWL>(ballot(has));
  }
}

template <bool PAGED, bool SEL>
const void *ptr_of(int pwl) {
  switch (pwl) {
    case 0: return reinterpret_cast<const void *>(direct_kernel<0, PAGED, SEL>);
    case 1: return reinterpret_cast<const void *>(direct_kernel<1, PAGED, SEL>);
    case 2: return reinterpret_cast<const void *>(direct_kernel<2, PAGED, SEL>);
    case 3: return reinterpret_cast<const void *>(direct_kernel<3, PAGED, SEL>);
    case 4: return reinterpret_cast<const void *>(direct_kernel<4, PAGED, SEL>);
    case 5: return reinterpret_cast<const void *>(direct_kernel<5, PAGED, SEL>);
    default: return reinterpret_cast<const void *>(direct_kernel<6, PAGED, SEL>);
  }
}

}  // namespace

const void *direct_kernel_ptr(int pwl, bool paged, bool sel) {
  if (paged) return sel ? ptr_of<true, true>(pwl) : ptr_of<true, false>(pwl);
  return sel ? ptr_of<false, true>(pwl) : ptr_of<false, false>(pwl);
}

hipError_t launch_direct(int pwl, bool paged, bool sel, int blocks, int wpb, size_t lds,
                         hipStream_t s, const DirectArgs &a) {
  void *args[] = {const_cast<DirectArgs *>(&a)};
  return hipLaunchKernel(direct_kernel_ptr(pwl, paged, sel), dim3(unsigned(blocks)),
                         dim3(unsigned(wpb * kWave)), args, lds, s);
}

}  // namespace dipsim
