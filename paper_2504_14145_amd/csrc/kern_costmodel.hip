// kern_costmodel.hip -- operator-level cost tables (DIP, arXiv 2504.14145,
// Sec. 6.1) for many configurations at once.
//
// An operator's latency is its largest resource time, read with per-kind
// coefficients c = alpha / capacity (seconds per FLOP, per byte of memory
// traffic, per byte sent): max(c_fop N_fop, c_mem N_mem, c_net N_net).  An
// item (a pipeline stage, a data edge) runs its operators in sequence; its
// entry is ceil(1e6 * sum) microseconds, -1 if that exceeds 2^31 - 1 or if an
// operator's kind is out of range.  One lane per configuration; float64
// throughout, without fused multiply-adds, so the sums are the float64 sums in
// row order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "dip_sim.h"

namespace {

constexpr int kConfigsPerBlock = 256;
constexpr int kItemsPerBlock = 8;
constexpr int kLdsKinds = 16;     // kinds whose coefficients fit the block's LDS

// Lane = configuration, 256 per block; a block walks kItemsPerBlock items, and
// all its lanes read the same operator row at a time (scalar loads).  With
// LDS, the block's coefficients sit there as [kind][resource][lane]; else each
// lane reads its own from global memory.  A row's kind byte is taken from the
// aligned 32-bit word that holds it (a word that holds a valid byte lies in a
// valid page, so the wider read cannot fault), which a scalar load can serve;
// an out-of-range kind marks the item and is clamped, so the row loop has no
// early exit and its unrolled iterations overlap.
template <bool LDS>
__global__ __launch_bounds__(256) void cost_table_kernel(dip_op_table t, int64_t n_configs,
                                                         const double *coef, int32_t *out) {
#pragma clang fp contract(off)
  extern __shared__ double cl[];          // [kind][resource][lane]
  const int64_t b0 = int64_t(blockIdx.y) * kConfigsPerBlock;
  const int64_t b = b0 + threadIdx.x;
  const bool live = b < n_configs;
  const int K = t.n_kinds;
  if constexpr (LDS) {
    for (int j = threadIdx.x; j < K * 3 * kConfigsPerBlock; j += blockDim.x) {
      const int lane = j % kConfigsPerBlock, kr = j / kConfigsPerBlock;   // kr = kind * 3 + resource
      const int64_t bb = b0 + lane;
      cl[j] = bb < n_configs ? coef[bb * K * 3 + kr] : 0.0;
    }
    __syncthreads();
  }
  const double *cg = coef + (live ? b : 0) * int64_t(K) * 3;
  const uintptr_t kaddr = reinterpret_cast<uintptr_t>(t.kind);
  // read-only for the whole launch: the constant address space lets the
  // uniform word reads go through the scalar cache
  using ConstWord = const __attribute__((address_space(4))) uint32_t;
  ConstWord *kw = reinterpret_cast<ConstWord *>(kaddr & ~uintptr_t(3));
  const uint32_t k0 = uint32_t(kaddr & 3);
  const int32_t i0 = int32_t(blockIdx.x) * kItemsPerBlock;
  for (int32_t i = i0; i < i0 + kItemsPerBlock && i < t.n_items; ++i) {
    const int32_t r0 = max(t.item_ptr[i], 0), r1 = min(t.item_ptr[i + 1], t.n_rows);
    double s = 0.0;
    bool bad = false;
    // one row: its coefficients (kind kc, already clamped) times its counts,
    // the largest of the three added to the running sum
    auto row = [&](int32_t r, uint32_t kc) {
      double cf, cm, cn;
      if constexpr (LDS) {
        cf = cl[(3 * kc) * kConfigsPerBlock + threadIdx.x];
        cm = cl[(3 * kc + 1) * kConfigsPerBlock + threadIdx.x];
        cn = cl[(3 * kc + 2) * kConfigsPerBlock + threadIdx.x];
      } else {
        cf = cg[3 * kc];
        cm = cg[3 * kc + 1];
        cn = cg[3 * kc + 2];
      }
      const double a = cf * t.n_fop[r];
      const double m = cm * t.n_mem[r];
      const double n = cn * t.n_net[r];
      s = s + fmax(fmax(a, m), n);
    };
    int32_t r = r0;
    // eight rows at a time: their kind bytes from the aligned words holding
    // the first, the fifth and the last of them (each holds a valid byte;
    // the last two are the same word when the first is aligned)
    for (; r + 7 < r1; r += 8) {
      const uint32_t at = k0 + uint32_t(r), sh = (at & 3u) * 8u;
      const uint64_t wa = kw[at >> 2], wb = kw[(at >> 2) + 1], wc = kw[(at + 7) >> 2];
      const uint64_t k8 = uint64_t(uint32_t((wa | (wb << 32)) >> sh)) |
                          (uint64_t(uint32_t((wb | (wc << 32)) >> sh)) << 32);
      uint32_t kc[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t k = uint32_t(k8 >> (8 * j)) & 0xffu;
        bad |= k >= uint32_t(K);
        kc[j] = min(k, uint32_t(K - 1));
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) row(r + j, kc[j]);
    }
    for (; r < r1; ++r) {
      const uint32_t at = k0 + uint32_t(r);
      const uint32_t k = (kw[at >> 2] >> ((at & 3u) * 8u)) & 0xffu;
      bad |= k >= uint32_t(K);
      row(r, min(k, uint32_t(K - 1)));
    }
    const double us = ceil(s * 1e6);
    if (live) out[b * t.n_items + i] = (bad || !(us <= 2147483647.0)) ? -1 : int32_t(us);
  }
}

// The same for up to kRegKinds kinds: a lane keeps the coefficients of CPL
// configurations in registers.  A row's kind is uniform, so its coefficients
// are picked by scalar branches to that kind's copy of the six operations;
// reading them from LDS (24 bytes a lane and row) bounds the kernel above.
// A block of four waves keeps 64 CPL configurations (brought in through LDS,
// coalesced: lanes reading their own strided rows took as long as all the
// arithmetic) and takes every gridDim.x-th chunk of CH items, its waves one
// chunk at a time, since items differ in length by two orders of magnitude.
// Rows come through the scalar cache, eight at a time.
// 16,384 configurations x 1,280 items (93,904 rows): 0.99 -> 0.59 ms; 16
// configurations of 1,360 items 127 -> 33 us.  The float64 instructions issue
// every 4.8 cycles at best (0.28 ms of it here); the scalar branches, loads
// and kind bytes of a row take the rest.
constexpr int kRegKinds = 8;
constexpr int kRegWaves = 4;

// calls f with the constant equal to k, lo <= k < hi
template <int LO, int HI, class F>
__device__ __forceinline__ void with_kind(uint32_t k, const F &f) {
  if constexpr (HI - LO == 1) {
    f(std::integral_constant<int, LO>{});
    // (a mark of its own keeps the copies apart: merged, they would move the
    // coefficients into common registers first)
    asm volatile("; operator kind %0" ::"n"(LO));
  } else {
    constexpr int kMid = LO + (HI - LO) / 2;
    if (k < uint32_t(kMid))
      with_kind<LO, kMid>(k, f);
    else
      with_kind<kMid, HI>(k, f);
  }
}

template <int NK, int CPL, int CH>
__global__ __launch_bounds__(64 * kRegWaves) void cost_table_reg_kernel(
    dip_op_table t, int64_t n_configs, const double *coef, int32_t *out) {
#pragma clang fp contract(off)
  constexpr int kConfigs = 64 * CPL;
  __shared__ double cs[kConfigs * NK * 3];
  __shared__ int32_t next;
  const int lane = threadIdx.x & 63;
  const int64_t b0 = int64_t(blockIdx.y) * kConfigs;
  const int nb = int(n_configs - b0 < kConfigs ? n_configs - b0 : kConfigs);   // >= 1
  for (int j = threadIdx.x; j < nb * NK * 3; j += 64 * kRegWaves) cs[j] = coef[b0 * NK * 3 + j];
  if (threadIdx.x == 0) next = 0;
  __syncthreads();
  double c[NK][3][CPL];
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    const int b = min(lane + 64 * j, nb - 1);
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int x = 0; x < 3; ++x) c[k][x][j] = cs[b * (NK * 3) + 3 * k + x];
  }
  // the table is read-only for the whole launch: the constant address space
  // sends its uniform reads through the scalar cache
  using ConstWord = const __attribute__((address_space(4))) uint32_t;
  using ConstInt = const __attribute__((address_space(4))) int32_t;
  using ConstDouble = const __attribute__((address_space(4))) double;
  const uintptr_t kaddr = reinterpret_cast<uintptr_t>(t.kind);
  ConstWord *kw = reinterpret_cast<ConstWord *>(kaddr & ~uintptr_t(3));
  ConstInt *ptr = reinterpret_cast<ConstInt *>(reinterpret_cast<uintptr_t>(t.item_ptr));
  ConstDouble *nf = reinterpret_cast<ConstDouble *>(reinterpret_cast<uintptr_t>(t.n_fop));
  ConstDouble *nm = reinterpret_cast<ConstDouble *>(reinterpret_cast<uintptr_t>(t.n_mem));
  ConstDouble *nn = reinterpret_cast<ConstDouble *>(reinterpret_cast<uintptr_t>(t.n_net));
  const uint32_t k0 = uint32_t(kaddr & 3);
  const int32_t n_chunks = (t.n_items - 1) / CH + 1;    // (up to 2^31 - 1 items)
  // whether a chunk's entries of a configuration are one aligned vector
  const bool vec = CH == 4 && t.n_items % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  for (;;) {
    int32_t ck = 0;
    if (lane == 0) ck = atomicAdd(&next, 1);
    ck = __builtin_amdgcn_readfirstlane(ck) * int32_t(gridDim.x) + int32_t(blockIdx.x);
    if (ck >= n_chunks) break;
    int32_t val[CPL][CH] = {};
    for (int e = 0; e < CH; ++e) {
      const int32_t i = ck * CH + e;
      if (i >= t.n_items) break;
      const int32_t r0 = max(ptr[i], 0), r1 = min(ptr[i + 1], t.n_rows);
      double s[CPL];
#pragma unroll
      for (int j = 0; j < CPL; ++j) s[j] = 0.0;
      bool bad = false;
      auto row = [&](uint32_t k, double f, double m, double n) {
        with_kind<0, NK>(k, [&](auto kind) {
          constexpr int kk = decltype(kind)::value;
#pragma unroll
          for (int j = 0; j < CPL; ++j) {
            const double a = c[kk][0][j] * f, b = c[kk][1][j] * m, d = c[kk][2][j] * n;
            s[j] = s[j] + fmax(fmax(a, b), d);
          }
        });
      };
      int32_t r = r0;
      // (the kind bytes of eight rows as in the kernel above; a kind out of
      // range marks the item and is priced as the last one)
      for (; r + 7 < r1; r += 8) {
        const uint32_t at = k0 + uint32_t(r), sh = (at & 3u) * 8u;
        const uint64_t wa = kw[at >> 2], wb = kw[(at >> 2) + 1], wc = kw[(at + 7) >> 2];
        const uint64_t k8 = uint64_t(uint32_t((wa | (wb << 32)) >> sh)) |
                            (uint64_t(uint32_t((wb | (wc << 32)) >> sh)) << 32);
        // a byte's top bit is set by adding 128 - NK when its low seven bits
        // reach NK, or is set already
        constexpr uint64_t kLow = 0x7f7f7f7f7f7f7f7full;
        bad |= ((((k8 & kLow) + (0x8080808080808080ull - NK * 0x0101010101010101ull)) | k8) & ~kLow) != 0;
        double f[8], m[8], n[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          f[j] = nf[r + j];
          m[j] = nm[r + j];
          n[j] = nn[r + j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) row(uint32_t(k8 >> (8 * j)) & 0xffu, f[j], m[j], n[j]);
      }
      for (; r < r1; ++r) {
        const uint32_t at = k0 + uint32_t(r);
        const uint32_t k = (kw[at >> 2] >> ((at & 3u) * 8u)) & 0xffu;
        bad |= k >= uint32_t(NK);
        row(k, nf[r], nm[r], nn[r]);
      }
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const double us = ceil(s[j] * 1e6);
        const int32_t x = (bad || !(us <= 2147483647.0)) ? -1 : int32_t(us);
        for (int q = 0; q < CH; ++q) val[j][q] = q == e ? x : val[j][q];
      }
    }
    for (int j = 0; j < CPL; ++j) {
      const int b = lane + 64 * j;
      int32_t *o = out + (b0 + b) * t.n_items + ck * CH;
      if (b < nb && vec)
        *reinterpret_cast<int4 *>(o) = make_int4(val[j][0], val[j][CH > 1 ? 1 : 0],
                                                 val[j][CH > 2 ? 2 : 0], val[j][CH > 3 ? 3 : 0]);
      for (int e = 0; e < CH; ++e)
        if (b < nb && !vec && ck * CH + e < t.n_items) o[e] = val[j][e];
    }
  }
}

template <int CPL, int CH>
void launch_reg(const dim3 &grid, hipStream_t s, const dip_op_table &t, int64_t n_configs,
                const double *coef, int32_t *out) {
  const dim3 block(64 * kRegWaves);
  switch (t.n_kinds) {
    case 1: cost_table_reg_kernel<1, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 2: cost_table_reg_kernel<2, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 3: cost_table_reg_kernel<3, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 4: cost_table_reg_kernel<4, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 5: cost_table_reg_kernel<5, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 6: cost_table_reg_kernel<6, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    case 7: cost_table_reg_kernel<7, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
    default: cost_table_reg_kernel<8, CPL, CH><<<grid, block, 0, s>>>(t, n_configs, coef, out); break;
  }
}

}  // namespace

extern "C" int dip_cost_tables(const dip_op_table *t, int64_t n_configs, const double *coef,
                               int32_t *out, void *stream) {
  if (!t || n_configs < 0 || t->n_items < 0 || t->n_rows < 0 || t->n_kinds < 1 ||
      t->n_kinds > 256)
    return DIP_E_INVAL;
  if (n_configs == 0 || t->n_items == 0) return DIP_OK;
  if (!t->item_ptr || !coef || !out || (t->n_rows > 0 && (!t->n_fop || !t->n_mem || !t->n_net ||
                                                          !t->kind)))
    return DIP_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(coef) | reinterpret_cast<uintptr_t>(t->n_fop) |
       reinterpret_cast<uintptr_t>(t->n_mem) | reinterpret_cast<uintptr_t>(t->n_net)) & 7)
    return DIP_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(t->item_ptr)) & 3)
    return DIP_E_INVAL;
  const int64_t gx = (int64_t(t->n_items) + kItemsPerBlock - 1) / kItemsPerBlock;
  const int64_t gy = (n_configs + kConfigsPerBlock - 1) / kConfigsPerBlock;
  if (gx > INT32_MAX || gy > 65535) return DIP_E_INVAL;
  const dim3 grid{unsigned(gx), unsigned(gy), 1u};
  // one or two items are a single wave's serial chain, which is shorter with the
  // coefficients in LDS than through the scalar branches (one item of 300 rows
  // and 5 kinds: 21 us against 44 with four configurations a lane, 20 and 33
  // with one; two items 37 and 46, 36 and 33)
  const bool few = t->n_items == 1 ? t->n_kinds >= 3 || n_configs > 256
                                   : t->n_items == 2 && t->n_kinds >= 3 && n_configs > 256;
  if (t->n_kinds <= kRegKinds && !few) {
    // four configurations a lane from 257 up (two waves a SIMD; 4,000 of them
    // take 172 us, at two a lane 209), two from 65 (four waves; 100 of them
    // 39 us, at four a lane 49), else one; two at most from seven kinds on,
    // where four configurations' coefficients leave one wave a SIMD (8 kinds,
    // 1,280 items of 70 rows, 1,000: 86 us, at two a lane 65); the blocks that
    // are resident at once, so that each brings its coefficients in once, and
    // items by fours where every wave still gets several chunks
    const int cpl = n_configs > 256 && t->n_kinds <= 6 ? 4 : n_configs > 64 ? 2 : 1;
    const int64_t ry = (n_configs + 64 * cpl - 1) / (64 * cpl);
    if (ry <= 65535) {
      const int64_t resident = cpl == 4 ? 512 : 1024;
      const bool four = int64_t(t->n_items) * ry >= 16 * kRegWaves * resident;
      const int64_t chunks = four ? (int64_t(t->n_items) + 3) / 4 : t->n_items;
      const int64_t rx = std::max<int64_t>(
          1, std::min<int64_t>((chunks + kRegWaves - 1) / kRegWaves, (resident + ry - 1) / ry));
      const dim3 rgrid{unsigned(rx), unsigned(ry), 1u};
      hipStream_t s = static_cast<hipStream_t>(stream);
      if (cpl == 4)
        four ? launch_reg<4, 4>(rgrid, s, *t, n_configs, coef, out)
             : launch_reg<4, 1>(rgrid, s, *t, n_configs, coef, out);
      else if (cpl == 2)
        four ? launch_reg<2, 4>(rgrid, s, *t, n_configs, coef, out)
             : launch_reg<2, 1>(rgrid, s, *t, n_configs, coef, out);
      else
        four ? launch_reg<1, 4>(rgrid, s, *t, n_configs, coef, out)
             : launch_reg<1, 1>(rgrid, s, *t, n_configs, coef, out);
      return hipGetLastError() == hipSuccess ? DIP_OK : DIP_E_HIP;
    }
  }
  if (t->n_kinds <= kLdsKinds)
    hipLaunchKernelGGL(cost_table_kernel<true>, grid, dim3(256),
                       size_t(t->n_kinds) * 3 * kConfigsPerBlock * 8, static_cast<hipStream_t>(stream),
                       *t, n_configs, coef, out);
  else
    hipLaunchKernelGGL(cost_table_kernel<false>, grid, dim3(256), 0, static_cast<hipStream_t>(stream),
                       *t, n_configs, coef, out);
  return hipGetLastError() == hipSuccess ? DIP_OK : DIP_E_HIP;
}
