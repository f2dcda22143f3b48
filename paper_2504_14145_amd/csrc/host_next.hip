// host_next.hip -- entry points beyond the simulation: the dual-queue greedy
// interleaving (Sec. 5.2), MCTS rollouts scored on the GPU (Sec. 5.1) and the
// per-layer memory selection with the re-timed evaluate (Sec. 5.3).
#include "host_state.h"

using namespace dipsim;
using namespace dipsim_host;

namespace dipsim_host {

// The inbox sizes a grouping accepts: rings of K stages per rank and kind,
// with the per-group tables and join accumulators, for a whole wave's
// candidates within a block's LDS.  (The launches keep K / 2 of them in LDS
// and go on in device memory, so they always fit; dip_sim_set_greedy_inbox
// and the growth below stay within this bound.)
bool greedy_inbox_fits(const dip_sim *h, int64_t K, int pwl) {
  const int64_t G = h->gr_G, P = h->P, J = h->gr_J;
  const int64_t lanes = int64_t(1) << pwl;
  const int64_t off_join = P * (2 * K + 1) * 8 + 8 * lanes;
  const int64_t head = align16(std::max<int64_t>(4 * G, off_join + 8 * J));
  const int64_t ebits = h->gr_nw >= 32 ? lanes * 16 * int64_t(h->gr_nw) : 0;
  const int64_t cand = head + 3 * align16(2 * G) + ebits;
  return align16(2 * G) + int64_t(kWave >> pwl) * cand <= h->lds_block_max;
}

// LDS plan of a greedy launch: per candidate the bitmaps, rings, messages and
// join accumulators overlay the priorities, which only the set-up reads; then
// group -> priority rank and back.
static bool greedy_layout(const dip_sim *h, int kl, bool wide, bool joins_dev,
                          dip_sim::GrLaunch *L) {
  const int64_t G = h->gr_G, P = h->P, J = h->gr_J;
  const int64_t nwd = (G + 63) / 64;
  L->kl = kl;
  L->joins_dev = joins_dev;
  const int64_t ring = P * (2 * nwd + 1) * 8;
  const int64_t meta = align16(ring + P * (2 * int64_t(kl) + 1) * 8);
  const int64_t msg = meta + P * 32;
  const int64_t join = msg + (int64_t(16) << h->gr_rwl);
  const int64_t head =
      align16(std::max<int64_t>(4 * ((G + 3) & ~int64_t(3)), join + (joins_dev ? 0 : 8 * J)));
  const int64_t tab = align16(2 * G);
  L->off_ring = int32_t(ring);
  L->off_meta = int32_t(meta);
  L->off_msg = int32_t(msg);
  L->off_join = int32_t(join);
  L->off_qof = int32_t(head);
  L->off_gof = int32_t(head + tab);
  L->cand_bytes = int32_t(head + 2 * tab);
  L->lds = (wide ? 1 : int64_t(kWave >> h->gr_rwl)) * int64_t(L->cand_bytes);
  L->blocks_per_cu = 0;
  if (L->lds > h->lds_block_max) return false;
  const void *k = greedy_kernel_ptr(h->gr_rwl, wide);
  int bpc = 0;
  if (!k || (L->lds > 65536 && hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   int(L->lds)) != hipSuccess) ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc, k, kWave, size_t(L->lds)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  L->blocks_per_cu = bpc;
  return bpc > 0;
}

// Both launch shapes for the current inbox size: K / 2 ring entries in LDS
// (with the first one in a register and a run of equal times beside the
// ring, as many stages again), 4 where most candidates spill anyway.  Fewer
// where they do not fit, and then the join accumulators in device memory.
bool greedy_plan(dip_sim *h) {
  const int want = h->gr_direct ? 4 : std::max(1, h->gr_K / 2);
  for (int wide = 0; wide < 2; ++wide) {
    dip_sim::GrLaunch &L = wide ? h->gr_wide : h->gr_dense;
    bool ok = false;
    for (int jd = 0; jd < 2 && !ok; ++jd)
      for (int kl = want; kl >= 1 && !ok; kl /= 2) ok = greedy_layout(h, kl, wide != 0, jd != 0, &L);
    if (!ok) L.blocks_per_cu = 0;
  }
  return h->gr_dense.blocks_per_cu > 0 || h->gr_wide.blocks_per_cu > 0;
}

// Resident candidate slots of a launch shape: what the CUs hold, within 1 GiB
// of rings.
static int64_t greedy_slots(const dip_sim *h, bool wide) {
  const dip_sim::GrLaunch &L = wide ? h->gr_wide : h->gr_dense;
  const int64_t gw = wide ? 1 : kWave >> h->gr_rwl;
  const int64_t per = h->P * 2 * int64_t(h->gr_kg) * 8 * gw;
  const int64_t blocks = std::max<int64_t>(
      1, std::min<int64_t>(int64_t(h->n_cu) * L.blocks_per_cu, (int64_t(1) << 30) / per));
  return L.blocks_per_cu > 0 ? blocks * gw : 0;
}

// Device memory of the rings (and joins) for the resident candidates of either
// shape, fewer of them where memory is short (down to a wave's).  Allocated
// with the grouping and kept with it: no call allocates, and a shape that holds
// more candidates (smaller inboxes) stays within these slots.
static int alloc_greedy_slots(dip_sim *h) {
  const int64_t gw = kWave >> h->gr_rwl;
  const int64_t per = h->P * 2 * int64_t(h->gr_kg) * 8;
  const bool joins = h->gr_dense.joins_dev || h->gr_wide.joins_dev;
  const int64_t jper = joins ? int64_t(h->gr_J) * 8 : 0;
  for (int64_t slots = std::max(greedy_slots(h, true), greedy_slots(h, false));; slots /= 2) {
    slots = std::max(slots, gw);
    const hipError_t e = hipMalloc(&h->d_gr_ring, size_t(slots * per));
    const hipError_t e2 = e == hipSuccess && jper ? hipMalloc(&h->d_gr_joins, size_t(slots * jper)) : e;
    if (e2 == hipSuccess) {
      h->gr_slots = slots;
      h->gr_mem_bytes = slots * (per + jper);
      return DIP_OK;
    }
    (void)hipGetLastError();
    if (e == hipSuccess) (void)hipFree(h->d_gr_ring);
    h->d_gr_ring = nullptr;
    h->d_gr_joins = nullptr;
    if (slots == gw) {
      g_last_hip = e2;
      return DIP_E_HIP;
    }
  }
}

}  // namespace dipsim_host

extern "C" {

int dip_sim_configure_greedy(dip_sim *h, int32_t n_groups, const int32_t *op_group) {
  if (!h || !op_group || n_groups < 1 || n_groups > 65535) return DIP_E_INVAL;
  const int32_t N = h->N, P = h->P;
  // every group holds stages of one kind, at most one per rank
  std::vector<int8_t> gk(n_groups, -1);
  std::vector<int32_t> at(int64_t(n_groups) * P, -1);
  for (int32_t g = 0; g < N; ++g) {
    const int32_t q = op_group[g];
    if (q < 0 || q >= n_groups) return DIP_E_TOPO;
    if (gk[q] >= 0 && gk[q] != int8_t(h->kind[g])) return DIP_E_TOPO;
    gk[q] = int8_t(h->kind[g]);
    int32_t &slot = at[int64_t(q) * P + h->rank_of[g]];
    if (slot >= 0) return DIP_E_TOPO;
    slot = g;
  }
  // the data edges must be acyclic (Kahn)
  std::vector<int32_t> succ_ptr(N + 1, 0), succ_op(std::max(h->E, 1)), succ_edge(std::max(h->E, 1));
  for (int32_t e = 0; e < h->E; ++e) ++succ_ptr[h->pred_op[e] + 1];
  for (int32_t g = 0; g < N; ++g) succ_ptr[g + 1] += succ_ptr[g];
  {
    std::vector<int32_t> fill(succ_ptr.begin(), succ_ptr.end() - 1);
    for (int32_t g = 0; g < N; ++g)
      for (int32_t e = h->pred_ptr[g]; e < h->pred_ptr[g + 1]; ++e) {
        const int32_t k = fill[h->pred_op[e]]++;
        succ_op[k] = g;
        succ_edge[k] = e;
      }
    std::vector<int32_t> left(N), stack;
    for (int32_t g = 0; g < N; ++g) {
      left[g] = h->pred_ptr[g + 1] - h->pred_ptr[g];
      if (left[g] == 0) stack.push_back(g);
    }
    int32_t seen = 0;
    while (!stack.empty()) {
      const int32_t g = stack.back();
      stack.pop_back();
      ++seen;
      for (int32_t k = succ_ptr[g]; k < succ_ptr[g + 1]; ++k)
        if (--left[succ_op[k]] == 0) stack.push_back(succ_op[k]);
    }
    if (seen != N) return DIP_E_TOPO;
  }
  int32_t GF = 0;
  for (int32_t q = 0; q < n_groups; ++q) GF += gk[q] == 1 ? 0 : 1;
  const int32_t wmax = (std::max(GF, n_groups - GF) + 63) / 64;
  int nw = 1;
  while (nw < wmax) nw *= 2;
  if (nw > 32) return DIP_E_UNSUPPORTED;

  (void)hipDeviceSynchronize();   // no call may still read the old tables
  release_rollouts(h);             // the classes belong to the old grouping
  release_greedy(h);
  h->gr_G = n_groups;
  h->gr_nw = nw;
  h->gr_ig.assign(op_group, op_group + N);
  h->gr_op = at;
  h->gr_join.assign(N, -1);
  h->gr_J = 0;
  for (int32_t g = 0; g < N; ++g)
    if (h->pred_ptr[g + 1] - h->pred_ptr[g] >= 2) h->gr_join[g] = h->gr_J++;
  h->gr_succ_ptr = succ_ptr;
  h->gr_succ_op = succ_op;
  h->gr_succ_edge = succ_edge;
  h->gr_n_extra = 0;
  for (int32_t g = 0; g < N; ++g) h->gr_n_extra += std::max(succ_ptr[g + 1] - succ_ptr[g] - 1, 0);
  std::vector<int32_t> src(P + 1, 0), src_list;
  for (int32_t r = 0; r < P; ++r) {
    for (int32_t g = h->rank_off[r]; g < h->rank_off[r + 1]; ++g)
      if (h->pred_ptr[g + 1] == h->pred_ptr[g])
        src_list.push_back(h->gr_ig[g] | (int32_t(h->kind[g]) << 16));
    src[r + 1] = int32_t(src_list.size());
  }
  src.insert(src.end(), src_list.begin(), src_list.end());
  // inboxes of 8 stages per kind to start with
  h->gr_rwl = std::max(2, h->pwl);
  h->gr_K = 8;
  h->gr_K_fixed = false;
  h->gr_direct = false;
  if (!greedy_inbox_fits(h, h->gr_K, h->gr_rwl) || !greedy_plan(h)) return DIP_E_UNSUPPORTED;
  // a stage joins its rank's ring of its kind once
  int32_t most = 1;
  {
    std::vector<int32_t> per(2 * int64_t(P), 0);
    for (int32_t g = 0; g < N; ++g) most = std::max(most, ++per[2 * h->rank_of[g] + h->kind[g]]);
  }
  h->gr_kg = most;
  // whether a whole rank's inboxes would fit in LDS (the rings in device memory
  // are then seldom used)
  int kr = 1;
  while (kr < most) kr *= 2;
  h->gr_lds_whole = false;
  for (int w = h->gr_rwl; w <= 6 && !h->gr_lds_whole; ++w)
    h->gr_lds_whole = greedy_inbox_fits(h, kr, w);

  auto fail = [&](hipError_t e) {
    g_last_hip = e;
    release_greedy(h);
    return int(DIP_E_HIP);
  };
  hipError_t e;
  const int64_t rec_bytes = int64_t(n_groups) * P * 32;
  const int64_t ext_bytes = int64_t(std::max(h->gr_n_extra, 1)) * 16;
  if ((e = hipMalloc(&h->d_gr_src, src.size() * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_gr_rec, size_t(rec_bytes))) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_gr_succ, size_t(ext_bytes))) != hipSuccess) return fail(e);
  if ((e = hipHostMalloc(reinterpret_cast<void **>(&h->h_gr_stage), size_t(rec_bytes + ext_bytes),
                         hipHostMallocDefault)) != hipSuccess)
    return fail(e);
  if ((e = hipMemcpy(h->d_gr_src, src.data(), src.size() * 4, hipMemcpyHostToDevice)) != hipSuccess)
    return fail(e);
  if ((e = hipMalloc(&h->d_gr_spills, 16)) != hipSuccess) return fail(e);
  if ((e = launch_zero_words(h->d_gr_spills, 1, nullptr)) != hipSuccess) return fail(e);
  if ((e = hipStreamSynchronize(nullptr)) != hipSuccess) return fail(e);
  if ((e = hipHostMalloc(reinterpret_cast<void **>(&h->h_gr_seen), 16, hipHostMallocDefault)) != hipSuccess)
    return fail(e);
  if ((e = hipEventCreateWithFlags(&h->gr_seen_ev, hipEventDisableTiming)) != hipSuccess) return fail(e);
  if (alloc_greedy_slots(h) != DIP_OK) return fail(g_last_hip);
  h->gr_ok = true;
  h->gr_costs_ok = false;
  return DIP_OK;
}

int dip_sim_greedy(dip_sim *h, const dip_costs *costs, const int32_t *prio, int64_t n_cand,
                   int16_t *out_orders, int32_t *out_makespan, int32_t *out_bubble,
                   int32_t *out_peakmem, uint8_t *out_flags, void *stream_) {
  if (!h || n_cand < 0) return DIP_E_INVAL;
  if (!h->gr_ok) return DIP_E_STATE;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (costs) {
    int rc = upload_costs(h, costs, stream);
    if (rc != DIP_OK) return rc;
  }
  if (!h->gr_costs_ok) return DIP_E_STATE;
  if (n_cand == 0) return DIP_OK;
  if (n_cand > INT32_MAX) return DIP_E_INVAL;
  if (!prio || !out_makespan || !out_bubble || !out_peakmem || !out_flags) return DIP_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(prio) | reinterpret_cast<uintptr_t>(out_makespan) |
       reinterpret_cast<uintptr_t>(out_bubble) | reinterpret_cast<uintptr_t>(out_peakmem)) & 3)
    return DIP_E_INVAL;
  if (reinterpret_cast<uintptr_t>(out_orders) & 1) return DIP_E_INVAL;
  if (h->gr_seen_pending && hipEventQuery(h->gr_seen_ev) == hipSuccess) {
    // earlier calls' spill count: more than 1/64 of their candidates doubles
    // the inboxes while they fit; more than half of them at the largest size
    // gives the LDS back and leaves the rings to device memory
    h->gr_seen_pending = false;
    const int64_t seen = int64_t(uint32_t(*h->h_gr_seen - h->gr_seen_last));
    h->gr_seen_last = *h->h_gr_seen;
    if (!h->gr_K_fixed && !h->gr_direct && seen * 64 > h->gr_seen_n) {
      // (below two waves a SIMD a larger ring is not worth its waves: 2,001
      // candidates on 32 ranks took 5.9 ms with 4 entries in LDS and all
      // waves resident, 10.7 ms with 8 in two rounds of waves)
      const dip_sim::GrLaunch dense = h->gr_dense, wide = h->gr_wide;
      bool grown = false;
      if (h->gr_K < 256 && greedy_inbox_fits(h, 2 * h->gr_K, h->gr_rwl)) {
        h->gr_K *= 2;
        grown = greedy_plan(h) &&
                h->gr_dense.blocks_per_cu >= std::min(dense.blocks_per_cu, 8) &&
                h->gr_wide.blocks_per_cu >= std::min(wide.blocks_per_cu, 8);
        if (!grown) {
          h->gr_K /= 2;
          h->gr_dense = dense;
          h->gr_wide = wide;
        }
      }
      if (!grown && seen * 2 > h->gr_seen_n) {
        h->gr_direct = true;
        (void)greedy_plan(h);
      }
    }
  }
  // a wave per candidate while every one is resident at once and the SIMDs
  // hold at most two waves each; else 64 >> rwl candidates a wave
  const int64_t slots_w = std::min(greedy_slots(h, true), h->gr_slots);
  const int64_t slots_d = std::min(greedy_slots(h, false), h->gr_slots);
  const bool wide = slots_d == 0 || (n_cand <= slots_w && n_cand <= 8 * int64_t(h->n_cu));
  const dip_sim::GrLaunch &L = wide ? h->gr_wide : h->gr_dense;
  const int64_t gw = wide ? 1 : kWave >> h->gr_rwl;
  const int64_t blocks = std::min<int64_t>((n_cand + gw - 1) / gw, (wide ? slots_w : slots_d) / gw);
  (void)hipGetLastError();
  h->prof_n = 0;
  auto mark = [&](int i) -> hipError_t {
    if (!h->profile) return hipSuccess;
    h->prof_n = i + 1;
    return hipEventRecord(h->prof_ev[i], stream);
  };
  (void)hipGetLastError();
  GreedyArgs a{};
  a.prio = prio;
  a.n_cand = n_cand;
  a.out_orders = out_orders;
  a.stride = h->stride;
  a.out_ms = out_makespan;
  a.out_bub = out_bubble;
  a.out_peak = out_peakmem;
  a.out_flags = out_flags;
  a.rec = h->d_gr_rec;
  a.succ = h->d_gr_succ;
  a.src = h->d_gr_src;
  a.rank_off = h->d_rank_off;
  a.busy = h->d_busy;
  a.cap = h->d_cap;
  a.P = h->P;
  a.G = h->gr_G;
  a.J = h->gr_J;
  a.n_stages = h->N;
  a.has_cap = 0;
  for (int r = 0; r < h->P; ++r) a.has_cap |= h->cap[r] >= 0 ? 1 : 0;
  a.nwd = (h->gr_G + 63) / 64;
  a.kl = L.kl;
  a.kg = h->gr_kg;
  a.cand_bytes = L.cand_bytes;
  a.off_ring = L.off_ring;
  a.off_meta = L.off_meta;
  a.off_msg = L.off_msg;
  a.off_join = L.off_join;
  a.off_qof = L.off_qof;
  a.off_gof = L.off_gof;
  a.dring = h->d_gr_ring;
  a.joins_dev = L.joins_dev ? h->d_gr_joins : nullptr;
  a.spill_count = h->gr_K_fixed || h->gr_direct ? nullptr : h->d_gr_spills;
  DIP_HIP(mark(0));
  DIP_HIP(launch_greedy(h->gr_rwl, wide, int(blocks), size_t(L.lds), stream, a));
  DIP_HIP(mark(1));
  if (a.spill_count) {
    h->gr_unseen_n += n_cand;
    if (!h->gr_seen_pending) {
      DIP_HIP(hipMemcpyAsync(h->h_gr_seen, h->d_gr_spills, 4, hipMemcpyDeviceToHost, stream));
      DIP_HIP(hipEventRecord(h->gr_seen_ev, stream));
      h->gr_seen_pending = true;
      h->gr_seen_n = h->gr_unseen_n;
      h->gr_unseen_n = 0;
    }
  }
  return DIP_OK;
}

int dip_sim_set_greedy_inbox(dip_sim *h, int32_t k) {
  if (!h || k < 0 || k > 256 || (k & (k - 1)) != 0) return DIP_E_INVAL;
  if (!h->gr_ok) return DIP_E_STATE;
  const int kk = k ? k : 8;
  if (!greedy_inbox_fits(h, kk, h->gr_rwl)) return DIP_E_UNSUPPORTED;
  h->gr_K = kk;
  h->gr_K_fixed = k != 0;
  h->gr_direct = false;
  return greedy_plan(h) ? DIP_OK : DIP_E_UNSUPPORTED;
}

int dip_sim_configure_rollouts(dip_sim *h, int32_t n_classes, const int32_t *group_class) {
  if (!h || !group_class || n_classes < 1) return DIP_E_INVAL;
  if (!h->gr_ok) return DIP_E_STATE;
  if (n_classes > 8192) return DIP_E_UNSUPPORTED;   // a rollout's tables in 64 KiB of LDS
  const int32_t G = h->gr_G;
  std::vector<int32_t> cls(group_class, group_class + G);
  std::vector<char> used(n_classes, 0);
  for (int32_t g = 0; g < G; ++g) {
    if (cls[g] < 0 || cls[g] >= n_classes) return DIP_E_TOPO;
    used[cls[g]] = 1;
  }
  (void)hipDeviceSynchronize();
  release_rollouts(h);
  auto fail = [&](hipError_t e) {
    g_last_hip = e;
    release_rollouts(h);
    return int(DIP_E_HIP);
  };
  hipError_t e;
  if ((e = hipMalloc(&h->d_rl_class, size_t(G) * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_rl_seq, size_t(n_classes + 1) * 4)) != hipSuccess) return fail(e);
  if ((e = hipHostMalloc(reinterpret_cast<void **>(&h->h_rl_seq), size_t(n_classes + 1) * 4,
                         hipHostMallocDefault)) != hipSuccess)
    return fail(e);
  h->rl_leaf_cap = 1;
  if ((e = hipEventCreateWithFlags(&h->rl_seq_ev, hipEventDisableTiming)) != hipSuccess) return fail(e);
  if ((e = hipMemcpy(h->d_rl_class, cls.data(), size_t(G) * 4, hipMemcpyHostToDevice)) != hipSuccess)
    return fail(e);
  h->rl_class = cls;
  h->rl_n = n_classes;
  h->rl_ok = true;
  return DIP_OK;
}

int dip_sim_rollouts_batch(dip_sim *h, int32_t n_leaves, const int32_t *depths,
                           const int32_t *prefixes, int64_t per_leaf, uint64_t seed,
                           uint64_t draw_base, int32_t *out_prio, int32_t *out_makespan,
                           uint8_t *out_flags, uint64_t *inout_keys, void *stream_) {
  if (!h || n_leaves < 1 || n_leaves > 65535 || per_leaf < 0 || !depths) return DIP_E_INVAL;
  if (!h->rl_ok || !h->gr_ok) return DIP_E_STATE;
  if (!h->gr_costs_ok) return DIP_E_STATE;
  const int32_t n = h->rl_n;
  // every prefix: distinct classes in range
  int64_t total = 0;
  for (int32_t l = 0; l < n_leaves; ++l) {
    if (depths[l] < 0 || depths[l] > n) return DIP_E_INVAL;
    total += depths[l];
  }
  if (total > 0 && !prefixes) return DIP_E_INVAL;
  {
    std::vector<int32_t> seen(n, -1);
    int64_t k = 0;
    for (int32_t l = 0; l < n_leaves; ++l)
      for (int32_t d = 0; d < depths[l]; ++d, ++k) {
        const int32_t c = prefixes[k];
        if (c < 0 || c >= n || seen[c] == l) return DIP_E_INVAL;
        seen[c] = l;
      }
  }
  if (per_leaf == 0) return DIP_OK;
  if (per_leaf > INT32_MAX / n_leaves || !out_prio || !out_makespan || !out_flags || !inout_keys)
    return DIP_E_INVAL;
  if (reinterpret_cast<uintptr_t>(inout_keys) & 7) return DIP_E_INVAL;
  const int64_t rows = per_leaf * n_leaves;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (h->rl_cap < rows) {
    if (h->d_rl_bub) (void)hipFree(h->d_rl_bub);
    if (h->d_rl_peak) (void)hipFree(h->d_rl_peak);
    h->d_rl_bub = h->d_rl_peak = nullptr;
    h->rl_cap = 0;
    DIP_HIP(hipMalloc(&h->d_rl_bub, size_t(rows) * h->P * 4));
    DIP_HIP(hipMalloc(&h->d_rl_peak, size_t(rows) * h->P * 4));
    h->rl_cap = rows;
  }
  // per leaf its prefix, then the other classes ascending; then the depths;
  // through pinned staging
  if (h->rl_seq_pending) {
    DIP_HIP(hipEventSynchronize(h->rl_seq_ev));
    h->rl_seq_pending = false;
  }
  const size_t words = size_t(n_leaves) * size_t(n + 1);
  if (h->rl_leaf_cap < n_leaves) {
    DIP_HIP(hipDeviceSynchronize());              // no launch may still read the old buffer
    if (h->d_rl_seq) (void)hipFree(h->d_rl_seq);
    if (h->h_rl_seq) (void)hipHostFree(h->h_rl_seq);
    h->d_rl_seq = h->h_rl_seq = nullptr;
    h->rl_leaf_cap = 0;
    DIP_HIP(hipMalloc(&h->d_rl_seq, words * 4));
    DIP_HIP(hipHostMalloc(reinterpret_cast<void **>(&h->h_rl_seq), words * 4, hipHostMallocDefault));
    h->rl_leaf_cap = n_leaves;
  }
  {
    std::vector<char> on(n);
    int64_t k = 0;
    for (int32_t l = 0; l < n_leaves; ++l) {
      int32_t *row = h->h_rl_seq + int64_t(l) * n;
      std::fill(on.begin(), on.end(), 0);
      int32_t w = 0;
      for (int32_t d = 0; d < depths[l]; ++d, ++k) {
        row[w++] = prefixes[k];
        on[prefixes[k]] = 1;
      }
      for (int32_t c = 0; c < n; ++c)
        if (!on[c]) row[w++] = c;
      h->h_rl_seq[int64_t(n_leaves) * n + l] = depths[l];
    }
  }
  DIP_HIP(hipMemcpyAsync(h->d_rl_seq, h->h_rl_seq, words * 4, hipMemcpyHostToDevice, stream));
  DIP_HIP(hipEventRecord(h->rl_seq_ev, stream));
  h->rl_seq_pending = true;
  RolloutArgs a{};
  a.n = rows;
  a.per_leaf = per_leaf;
  a.out_prio = out_prio;
  a.seqs = h->d_rl_seq;
  a.depths = h->d_rl_seq + int64_t(n_leaves) * n;
  a.group_class = h->d_rl_class;
  a.seed = seed;
  a.draw = draw_base;
  a.n_classes = n;
  a.G = h->gr_G;
  DIP_HIP(launch_rollout_prio(stream, a));
  int rc;
  if (!h->mo_ok) {
    rc = dip_sim_greedy(h, nullptr, out_prio, rows, nullptr, out_makespan, h->d_rl_bub,
                        h->d_rl_peak, out_flags, stream_);
    if (rc != DIP_OK) return rc;
  } else {
    // Sec. 5.1's score: the interleaved schedule after the per-layer memory
    // optimisation, re-timed with its selection (a rank whose cap cannot be
    // met keeps a selection over the cap, which the re-timed run flags)
    if (h->rl_mo_cap < rows) {
      DIP_HIP(hipDeviceSynchronize());
      release_rollout_memopt(h);
      DIP_HIP(hipMalloc(&h->d_rl_orders, size_t(rows) * size_t(h->stride) * 2));
      DIP_HIP(hipMalloc(&h->d_rl_mo_time, size_t(rows) * h->P * 8));
      DIP_HIP(hipMalloc(&h->d_rl_mo_peak, size_t(rows) * h->P * 4));
      DIP_HIP(hipMalloc(&h->d_rl_mo_status, size_t(rows) * h->P));
      DIP_HIP(hipMalloc(&h->d_rl_choice, size_t(rows) * std::max(h->mo_n_pairs, 1)));
      h->rl_mo_cap = rows;
    }
    rc = dip_sim_greedy(h, nullptr, out_prio, rows, h->d_rl_orders, out_makespan, h->d_rl_bub,
                        h->d_rl_peak, out_flags, stream_);
    if (rc != DIP_OK) return rc;
    rc = dip_sim_memopt(h, h->d_rl_orders, rows, h->d_rl_mo_time, h->d_rl_mo_peak,
                        h->d_rl_mo_status, h->d_rl_choice, stream_);
    if (rc != DIP_OK) return rc;
    rc = dip_sim_evaluate_selected(h, h->d_rl_orders, h->d_rl_choice, rows, out_makespan,
                                   h->d_rl_bub, h->d_rl_peak, out_flags, stream_);
    if (rc != DIP_OK) return rc;
  }
  // the best unflagged rollout of each leaf, indexed within the leaf
  const int64_t want = (per_leaf + 255) / 256;
  const int blocks = int(std::max<int64_t>(1, std::min<int64_t>(want, int64_t(h->n_cu) * 8 / n_leaves)));
  DIP_HIP(launch_argmin(blocks, stream, out_makespan, out_flags, rows, per_leaf, n_leaves, 0,
                        reinterpret_cast<unsigned long long *>(inout_keys)));
  return DIP_OK;
}

int dip_sim_rollouts(dip_sim *h, const int32_t *prefix, int32_t depth, int64_t n_rollouts,
                     uint64_t seed, uint64_t draw, int32_t *out_prio, int32_t *out_makespan,
                     uint8_t *out_flags, uint64_t *inout_best_key, void *stream_) {
  if (!h || n_rollouts < 0 || depth < 0) return DIP_E_INVAL;
  return dip_sim_rollouts_batch(h, 1, &depth, prefix, n_rollouts, seed, draw, out_prio,
                                out_makespan, out_flags, inout_best_key, stream_);
}

// Launch shapes of the memory selection, for groups of 16 and of 64 lanes:
// the waves per block that leave the most problems resident on a CU (the
// rank's tables are shared by a block, so more waves take less LDS each).
static void plan_memopt(dip_sim *h) {
  const int32_t mp = std::max(h->mo_max_pairs, 1);
  for (int g = 0; g < 2; ++g) {
    const int lanes = g ? 64 : 16;
    const void *k = memopt_group_ptr(lanes, mp);
    int best = 0;
    h->mo_waves[g] = 0;
    for (int w = 1; k && w <= 8; w *= 2) {
      const int64_t lds = memopt_group_lds(mp, w * 64 / lanes);
      int nb = 0;
      if (lds > h->lds_block_max) break;
      if ((lds > 65536 && hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                              int(h->lds_block_max)) != hipSuccess) ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, w * kWave, size_t(lds)) != hipSuccess) {
        (void)hipGetLastError();
        break;
      }
      if (nb * w >= best && nb > 0) {
        best = nb * w;
        h->mo_waves[g] = w;
      }
    }
    h->mo_slots[g] = int64_t(best) * (kWave / lanes) * h->n_cu;
  }
}

// The re-timed simulation's working rows: extra costs and two retry lists for
// up to 131,072 schedules within a GiB of extra costs, which is several
// resident generations (a larger batch goes through them in steps; with a
// quarter of that, 4,000 schedules of 34,896 ops took 8.3 ms instead of 4.4,
// 100,000 of 680 ops 1.41 instead of 1.25).  Less where the memory is short;
// without any, the general kernel runs.
static void alloc_selected(dip_sim *h) {
  int64_t rows = std::max<int64_t>(
      1, std::min<int64_t>(131072, (int64_t(1) << 30) / (4 * h->stride)));
  for (;; rows /= 2) {
    if (hipMalloc(&h->d_sel_x, size_t(rows) * size_t(h->stride) * 4) == hipSuccess &&
        hipMalloc(&h->d_sel_list, size_t(rows) * 16) == hipSuccess &&
        hipMalloc(&h->d_sel_count, kRetryCounters * 4) == hipSuccess &&
        // (it orders streams of one device: no system-wide fence, 1 us a call)
        hipEventCreateWithFlags(&h->sel_ev, hipEventDisableTiming | hipEventDisableSystemFence) ==
            hipSuccess) {
      h->sel_rows = rows;
      return;
    }
    (void)hipGetLastError();
    release_selected(h);
    if (rows < 64) return;
  }
}

int dip_sim_configure_memopt(dip_sim *h, const int32_t *slot_layers, const int64_t *layer_time,
                             const int64_t *layer_mem, int32_t n_strategies, int32_t n_candidates,
                             int32_t bb_nodes) {
  if (!h || !slot_layers || n_strategies < 1 || n_candidates < 2 ||
      n_candidates > kMemoptMaxCands || bb_nodes < 0)
    return DIP_E_INVAL;
  const int32_t P = h->P, N = h->N, ns = h->n_slots;
  // every slot: one forward and one backward on one rank
  std::vector<int32_t> f_of(ns, -1), b_of(ns, -1);
  for (int32_t g = 0; g < N; ++g) {
    int32_t &x = h->kind[g] ? b_of[h->op_slot[g]] : f_of[h->op_slot[g]];
    if (x >= 0) return DIP_E_TOPO;
    x = g;
  }
  for (int32_t q = 0; q < ns; ++q)
    if (f_of[q] < 0 || b_of[q] < 0 || h->rank_of[f_of[q]] != h->rank_of[b_of[q]]) return DIP_E_TOPO;
  if (slot_layers[0] != 0) return DIP_E_INVAL;
  for (int32_t q = 0; q < ns; ++q)
    if (slot_layers[q + 1] < slot_layers[q]) return DIP_E_INVAL;
  if (slot_layers[ns] > 0 && (!layer_time || !layer_mem)) return DIP_E_INVAL;
  // candidates per slot: exact Pareto front of the layers' choices, then the
  // fastest, the leanest and one knapsack answer per bucket edge
  struct Pt {
    int64_t t, m;
  };
  std::vector<std::vector<Pt>> cand(ns);
  for (int32_t q = 0; q < ns; ++q) {
    std::vector<Pt> front{{0, 0}}, pts;
    for (int32_t l = slot_layers[q]; l < slot_layers[q + 1]; ++l) {
      pts.clear();
      for (const Pt &p : front)
        for (int32_t k = 0; k < n_strategies; ++k) {
          const int64_t t = layer_time[int64_t(l) * n_strategies + k];
          const int64_t m = layer_mem[int64_t(l) * n_strategies + k];
          if (t < 0 || m < 0) return DIP_E_RANGE;
          pts.push_back({p.t + t, p.m + m});
        }
      std::sort(pts.begin(), pts.end(),
                [](const Pt &x, const Pt &y) { return x.m != y.m ? x.m < y.m : x.t < y.t; });
      front.clear();
      for (const Pt &p : pts)
        if (front.empty() || (p.t < front.back().t && p.m != front.back().m)) front.push_back(p);
      if (front.size() > (size_t(1) << 20)) return DIP_E_UNSUPPORTED;
    }
    std::vector<Pt> pick{front.back(), front.front()};
    const int64_t lo = front.front().m, hi = front.back().m;
    for (int32_t k = 1; k + 1 < n_candidates; ++k) {
      const int64_t edge = lo + ((hi - lo) * k) / (n_candidates - 2);
      size_t j = 0;
      while (j + 1 < front.size() && front[j + 1].m <= edge) ++j;
      pick.push_back(front[j]);
    }
    std::sort(pick.begin(), pick.end(),
              [](const Pt &x, const Pt &y) { return x.t != y.t ? x.t < y.t : x.m < y.m; });
    std::vector<Pt> uniq;
    for (const Pt &p : pick)
      if (uniq.empty() || uniq.back().t != p.t || uniq.back().m != p.m) uniq.push_back(p);
    for (const Pt &p : uniq)
      if (p.m > INT32_MAX || p.t > (int64_t(1) << 40)) return DIP_E_RANGE;
    cand[q] = uniq;
  }
  // pairs per rank in slot order; each op's pair index and kind
  std::vector<int32_t> pair_off(P + 1, 0), lid_pair(N, 0), slot_pair(ns, 0), pair_b;
  std::vector<int64_t> pair_extra;
  std::vector<int32_t> mem, mdm;
  std::vector<int64_t> tim;
  std::vector<uint32_t> mkey;
  int32_t max_pairs = 0;
  struct Move {
    int64_t dt, dm;
    int32_t at;                  // index into the rank's [pair][candidate] slice
  };
  std::vector<Move> moves;
  for (int32_t r = 0; r < P; ++r) {
    int32_t i = 0;
    const size_t first = tim.size();
    moves.clear();
    int64_t fastest_mem = 0;
    for (int32_t q = 0; q < ns; ++q) {
      if (h->rank_of[f_of[q]] != r) continue;
      slot_pair[q] = i;
      const int32_t nc = int32_t(cand[q].size());
      fastest_mem += cand[q][0].m;
      pair_b.push_back(b_of[q]);
      pair_extra.push_back(cand[q][nc - 1].t - cand[q][0].t);
      for (int32_t j = 0; j < kMemoptMaxCands; ++j) {
        const bool in = j < nc;
        tim.push_back(in ? cand[q][j].t : 0);
        mem.push_back(in ? int32_t(cand[q][j].m) : 0);
        mkey.push_back(kMemoptNoMove);
        mdm.push_back(0);
        if (j + 1 < nc)
          moves.push_back({cand[q][j + 1].t - cand[q][j].t, cand[q][j].m - cand[q][j + 1].m,
                           i * kMemoptMaxCands + j});
      }
      ++i;
    }
    if (i >= (1 << kMemoptPairBits)) return DIP_E_UNSUPPORTED;
    if (fastest_mem > INT32_MAX) return DIP_E_RANGE;
    // exact ratio order of the rank's moves: dt_a / dm_a < dt_b / dm_b (dm > 0)
    auto less = [](const Move &x, const Move &y) {
      return __int128(x.dt) * y.dm < __int128(y.dt) * x.dm;
    };
    std::stable_sort(moves.begin(), moves.end(), less);
    uint32_t dense = 0;
    for (size_t k = 0; k < moves.size(); ++k) {
      if (k > 0 && less(moves[k - 1], moves[k])) ++dense;
      const int32_t pair = moves[k].at / kMemoptMaxCands;
      mkey[first + size_t(moves[k].at)] = (dense << kMemoptPairBits) | uint32_t(pair);
      mdm[first + size_t(moves[k].at)] = int32_t(moves[k].dm);
    }
    pair_off[r + 1] = pair_off[r] + i;
    max_pairs = std::max(max_pairs, i);
  }
  for (int32_t g = 0; g < N; ++g)
    lid_pair[g] = int32_t(uint32_t(slot_pair[h->op_slot[g]]) | (uint32_t(h->kind[g]) << 31));
  (void)hipDeviceSynchronize();
  release_memopt(h);
  auto fail = [&](hipError_t e) {
    g_last_hip = e;
    release_memopt(h);
    return int(DIP_E_HIP);
  };
  hipError_t e;
  const size_t cells = std::max<size_t>(tim.size(), 1);       // pairs x candidates
  if ((e = hipMalloc(&h->d_mo_pair_off, size_t(P + 1) * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_mo_lid_pair, size_t(std::max(N, 1)) * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_mo_time, cells * 8)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_mo_mem, cells * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_mo_key, cells * 4)) != hipSuccess) return fail(e);
  if ((e = hipMalloc(&h->d_mo_dm, cells * 4)) != hipSuccess) return fail(e);
  if ((e = hipMemcpy(h->d_mo_pair_off, pair_off.data(), size_t(P + 1) * 4, hipMemcpyHostToDevice)) ||
      (N > 0 && (e = hipMemcpy(h->d_mo_lid_pair, lid_pair.data(), size_t(N) * 4, hipMemcpyHostToDevice))) ||
      (!tim.empty() &&
       ((e = hipMemcpy(h->d_mo_time, tim.data(), tim.size() * 8, hipMemcpyHostToDevice)) ||
        (e = hipMemcpy(h->d_mo_mem, mem.data(), mem.size() * 4, hipMemcpyHostToDevice)) ||
        (e = hipMemcpy(h->d_mo_key, mkey.data(), mkey.size() * 4, hipMemcpyHostToDevice)) ||
        (e = hipMemcpy(h->d_mo_dm, mdm.data(), mdm.size() * 4, hipMemcpyHostToDevice)))))
    return fail(e);
  h->mo_max_pairs = max_pairs;
  h->mo_n_pairs = pair_off[P];
  h->mo_bb_nodes = bb_nodes > 0 ? bb_nodes : 512;
  h->mo_pair_b = pair_b;
  h->mo_pair_extra = pair_extra;
  h->mo_max_extra = 0;
  for (int64_t x : pair_extra) h->mo_max_extra = std::max(h->mo_max_extra, x);
  plan_memopt(h);
  h->mo_ok = true;
  if (h->sim_ok) alloc_selected(h);
  plan_selected(h);
  return DIP_OK;
}

int dip_sim_memopt(dip_sim *h, const int16_t *orders, int64_t n_cand, int64_t *out_time,
                   int32_t *out_peak, uint8_t *out_status, uint8_t *out_choice, void *stream) {
  if (!h || n_cand < 0) return DIP_E_INVAL;
  if (!h->mo_ok) return DIP_E_STATE;
  if (n_cand == 0) return DIP_OK;
  if (!orders || !out_time || !out_peak || !out_status) return DIP_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(out_time) & 7) || (reinterpret_cast<uintptr_t>(out_peak) & 3) ||
      (reinterpret_cast<uintptr_t>(orders) & 1))
    return DIP_E_INVAL;
  MemoptArgs a{};
  a.orders = orders;
  a.n_cand = n_cand;
  a.stride = h->stride;
  a.out_time = out_time;
  a.out_peak = out_peak;
  a.out_status = out_status;
  a.out_choice = out_choice;
  a.n_pairs = h->mo_n_pairs;
  a.bb_nodes = h->mo_bb_nodes;
  a.rank_off = h->d_rank_off;
  a.pair_off = h->d_mo_pair_off;
  a.lid_pair = h->d_mo_lid_pair;
  a.cand_time = h->d_mo_time;
  a.cand_mem = h->d_mo_mem;
  a.move_key = h->d_mo_key;
  a.move_dm = h->d_mo_dm;
  a.cap = h->d_cap;
  a.P = h->P;
  a.max_pairs = std::max(h->mo_max_pairs, 1);
  (void)hipGetLastError();
  if (a.max_pairs <= 512) {
    // Four problems a wave once the problems outnumber the resident waves of
    // one each (131,072 problems of 64 pairs: 2.98 ms against 6.30; 4,096:
    // 475 us against 363), up to 96 pairs (131,072 of 96: 4.9 ms against 7.7;
    // of 128: 10.3 against 9.0, the lanes' state having crowded out waves).
    const int g = h->mo_waves[0] && n_cand * h->P > h->mo_slots[1] ? 0 : 1;
    if (!h->mo_waves[g]) return DIP_E_UNSUPPORTED;
    if (n_cand > INT32_MAX || h->P > 65535) return DIP_E_INVAL;
    DIP_HIP(launch_memopt_group(g ? 64 : 16, h->mo_waves[g], static_cast<hipStream_t>(stream), a));
    return DIP_OK;
  }
  a.bytes_per_thread = int32_t(int64_t(a.max_pairs) * 9);
  int tpb = 64;
  while (tpb > 1 && int64_t(tpb) * a.bytes_per_thread > 65536) tpb /= 2;
  if (int64_t(tpb) * a.bytes_per_thread > 65536) return DIP_E_UNSUPPORTED;
  if (n_cand * h->P / tpb + 1 > INT32_MAX) return DIP_E_INVAL;
  DIP_HIP(launch_memopt(tpb, static_cast<hipStream_t>(stream), a));
  return DIP_OK;
}

// The re-timed evaluate through the simulation kernel: check (with each op's
// extra cost along the order), own-rank order, then the direct kernel where
// every schedule is resident with it, else 8-slot pools and the direct kernel
// for those that filled (32-slot pools and the general kernel where it does
// not fit).
static int launch_selected(dip_sim *h, const GeneralArgs &all, hipStream_t stream) {
  int32_t max_nr = 0;
  for (int32_t n : h->n_ops) max_nr = std::max(max_nr, n);
  for (int64_t c0 = 0; c0 < all.n_cand; c0 += h->sel_rows) {
    const int64_t n = std::min(h->sel_rows, all.n_cand - c0);
    const int16_t *orders = all.orders + c0 * h->stride;
    int32_t *ms = all.out_ms + c0, *bub = all.out_bub + c0 * h->P, *peak = all.out_peak + c0 * h->P;
    uint8_t *flags = all.out_flags + c0;
    const uint8_t *choice = all.choice + c0 * all.n_pairs;
    SelCheckArgs k{};
    k.orders = orders;
    k.n_cand = n;
    k.stride = h->stride;
    k.choice = choice;
    k.n_pairs = all.n_pairs;
    k.lid_pair = all.lid_pair;
    k.pair_off = all.pair_off;
    k.cand_time = all.cand_time;
    k.cand_mem = all.cand_mem;
    k.cand_key = all.cand_key;
    k.rank_off = h->d_rank_off;
    k.cap = h->d_cap;
    k.P = h->P;
    k.bm_words = (max_nr + 31) / 32;
    k.xcost = h->d_sel_x;
    k.out_ms = ms;
    k.out_bub = bub;
    k.out_peak = peak;
    k.out_flags = flags;
    k.retry_count = h->d_sel_count;
    DIP_HIP(launch_selcheck(std::min(4, h->P), stream, k));
    if (h->sim_drop_self && h->to_ok) {
      const int rc = run_order_check(h, orders, n, ms, bub, flags, stream);
      if (rc != DIP_OK) return rc;
    }
    const int64_t direct = direct_slots(h, true);
    if (n <= direct) {
      const int rc =
          run_direct(h, true, orders, n, h->d_sel_x, ms, bub, flags, nullptr, nullptr, stream);
      if (rc != DIP_OK) return rc;
      continue;
    }
    SimArgs a{};
    a.orders = orders;
    a.n_cand = n;
    a.stride = h->stride;
    a.out_ms = ms;
    a.out_bub = bub;
    a.out_flags = flags;
    a.tab = h->d_sim_tab;
    a.tab_vec = h->sim_tab_vec;
    a.off_pmap = h->sim_off_pmap;
    a.off_extra = h->sim_off_extra;
    a.lane_info = reinterpret_cast<const int32_t *>(h->d_sim_lane);
    a.state_base = uint32_t(h->sim_state_base);
    a.P = h->P;
    a.xcost = h->d_sel_x;
    a.round_limit = uint32_t(h->N) + uint32_t(h->E) + 16u;
    a.static_end = INT64_MAX;
    a.retry = h->d_sel_list;
    a.retry_count = h->d_sel_count;
    a.wpb = h->sel_wpb[0];
    const int64_t per_block = int64_t(a.wpb) * h->G;
    a.spread = n <= int64_t(h->sel_max_blocks[0]) * per_block;
    const int blocks = int(std::min<int64_t>(
        a.spread ? n : (n + per_block - 1) / per_block, h->sel_max_blocks[0]));
    DIP_HIP(launch_sim(h->pwl, 8, h->sim_paged, blocks, a.wpb, size_t(h->sel_lds[0]), stream, a, true));
    if (h->sim_max_pub <= 8) continue;
    if (direct > 0) {
      // (selections come with orders of many live items: under a binding cap
      // on 16 x 2 lanes every one of them fills 32 slots too)
      const int rc = run_direct(h, true, orders, n, h->d_sel_x, ms, bub, flags, h->d_sel_list,
                                h->d_sel_count, stream);
      if (rc != DIP_OK) return rc;
      continue;
    }
    a.list = h->d_sel_list;
    a.list_count = h->d_sel_count;
    a.retry = h->d_sel_list + h->sel_rows;
    a.retry_count = h->d_sel_count + 2;
    a.wpb = h->sel_wpb[1];
    DIP_HIP(launch_sim(h->pwl, 32, h->sim_paged, h->sel_max_blocks[1], a.wpb, size_t(h->sel_lds[1]),
                       stream, a, true));
    if (h->sim_max_pub <= 32) continue;
    GeneralArgs f = all;
    f.orders = orders;
    f.n_cand = n;
    f.out_ms = ms;
    f.out_bub = bub;
    f.out_peak = peak;
    f.out_flags = flags;
    f.choice = choice;
    f.list = a.retry;
    f.list_count = a.retry_count;
    f.tab_bytes = f.ord_bytes = 0;
    f.end_bytes = 0;
    // end times in LDS where a wave's fit; else in the general configuration's
    // scratch (which then is variant 4 too), as evaluate's own leftovers may
    // be using theirs on another stream
    const bool in_lds = h->fb_variant == 3;
    f.wpb = in_lds ? 1 : h->gen_wpb;
    DIP_HIP(launch_general(h->fb_variant, in_lds ? h->fb_blocks : h->gen_max_blocks, f.wpb,
                           size_t(in_lds ? h->fb_lds : h->gen_lds), stream, f));
  }
  return DIP_OK;
}

// The same behind the calls that used the rows before it.
static int evaluate_selected_sim(dip_sim *h, const GeneralArgs &all, hipStream_t stream) {
  std::lock_guard<std::mutex> lock(h->sel_mu);
  if (h->sel_used && stream != h->sel_stream) DIP_HIP(hipStreamWaitEvent(stream, h->sel_ev, 0));
  const int rc = launch_selected(h, all, stream);
  h->sel_used = true;
  h->sel_stream = stream;
  DIP_HIP(hipEventRecord(h->sel_ev, stream));
  return rc;
}

// whether a captured graph takes the stream's work (or that cannot be told)
static bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) == hipSuccess && st == hipStreamCaptureStatusNone)
    return false;
  (void)hipGetLastError();
  return true;
}

// Whether the general kernel is the faster one for a batch: candidates of few
// ops, where its one launch takes about 1.2 us per op and pipeline step
// (busiest rank's ops + 2 P of them), three launches 12 us and 0.4 us a step,
// and the selection check 0.45 ns per schedule and rank whatever its ops, most
// lanes of a rank's wave being idle.  Past 32 ops a rank (48 of few in all) and
// for many ranks of several ops the general kernel falls behind again once its
// lanes are full.  us, general against simulation: 4 ranks of 16 ops, 4,000
// schedules 33 and 30, 8,000 33 and 40, 100,000 64 and 290; one rank of 2 ops,
// 300,000 8 and 259; 8 ranks of 32 ops, 4,000 59 and 43, 16,000 64 and 89,
// 64,000 231 and 374; 8 of 64, 64,000 786 and 480; 64 of 4, 4,000 196 and 180,
// of 16, 4,000 329 and 293.
static bool selected_general(const dip_sim *h, int64_t n_cand) {
  const int64_t P = h->P;
  int64_t nr = 0;
  for (int32_t n : h->n_ops) nr = std::max<int64_t>(nr, n);
  return h->forced_variant == 0 && nr <= (h->N <= 336 ? 48 : 32) && h->N * P <= 16384 &&
         n_cand * P > 1400 * nr + 4000 * P - 20000;
}

int dip_sim_evaluate_selected(dip_sim *h, const int16_t *orders, const uint8_t *choice,
                              int64_t n_cand, int32_t *out_makespan, int32_t *out_bubble,
                              int32_t *out_peakmem, uint8_t *out_flags, void *stream) {
  if (!h || n_cand < 0) return DIP_E_INVAL;
  if (!h->mo_ok || !h->costs_set) return DIP_E_STATE;
  if (n_cand == 0) return DIP_OK;
  if (!orders || !choice || !out_makespan || !out_bubble || !out_peakmem || !out_flags)
    return DIP_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(orders) & 15) ||
      ((reinterpret_cast<uintptr_t>(out_makespan) | reinterpret_cast<uintptr_t>(out_bubble) |
        reinterpret_cast<uintptr_t>(out_peakmem)) & 3))
    return DIP_E_INVAL;
  // a re-timed backward stays within int32
  for (size_t p = 0; p < h->mo_pair_b.size(); ++p)
    if (int64_t(h->last_cost[size_t(h->mo_pair_b[p])]) + h->mo_pair_extra[p] > INT32_MAX)
      return DIP_E_RANGE;
  GeneralArgs a{};
  a.orders = orders;
  a.n_cand = n_cand;
  a.stride = h->stride;
  a.n_groups = (n_cand + h->G - 1) / h->G;
  a.out_ms = out_makespan;
  a.out_bub = out_bubble;
  a.out_peak = out_peakmem;
  a.out_flags = out_flags;
  a.rec = h->d_rec;
  a.edge = h->d_edge;
  a.rank_off = h->d_rank_off;
  a.busy = h->d_busy;
  a.cap = h->d_cap;
  a.gends = static_cast<int32_t *>(h->d_scratch_gen);
  a.P = h->P;
  a.pwl = h->pwl;
  a.G = h->G;
  a.N = h->N;
  a.E = h->E;
  a.wpb = h->gen_wpb;
  a.choice = choice;
  a.n_pairs = h->mo_n_pairs;
  a.lid_pair = h->d_mo_lid_pair;
  a.pair_off = h->d_mo_pair_off;
  a.cand_time = h->d_mo_time;
  a.cand_mem = h->d_mo_mem;
  a.cand_key = h->d_mo_key;
  // through the simulation kernel where it runs these costs and the times of
  // any selection fit its 32 bits (the general kernel below took 2.35 ms for
  // 32,768 schedules on 8 ranks and 3.7 ms for 1,024 on 16 x 2 lanes).  Not
  // under capture: a graph's replays come at any time beside the calls that
  // share the working rows, and the general kernel needs none.
  (void)hipGetLastError();
  if (h->sel_ok && h->variant == 9 && !selected_general(h, n_cand) &&
      !capturing(static_cast<hipStream_t>(stream)))
    return evaluate_selected_sim(h, a, static_cast<hipStream_t>(stream));
  const GenBytes b = general_bytes(h, h->gen_variant);
  a.tab_bytes = uint32_t(b.tab);
  a.ord_bytes = uint32_t(b.ord);
  a.end_bytes = uint32_t(b.end);
  const int64_t want = (a.n_groups + h->gen_wpb - 1) / h->gen_wpb;
  const int blocks = int(std::min<int64_t>(want, h->gen_max_blocks));
  (void)hipGetLastError();
  DIP_HIP(launch_general(h->gen_variant, blocks, h->gen_wpb, size_t(h->gen_lds),
                         static_cast<hipStream_t>(stream), a));
  return DIP_OK;
}

}  // extern "C"
