// Exact top-k of a small vector without sampling (plans in mode DIRECT), by
// one workgroup that holds the whole vector in registers:
//   1. every thread loads up to kSmallU 16-byte vectors and takes the maximum
//      of each of four element positions over them; the k-th largest of these
//      maxima bounds the k-th largest element from below;
//   2. the elements that reach the bound are collected in LDS (about k of
//      them while k is small against the 4096 maxima).  When ties at the
//      bound make them too many, those of smallest index are taken;
//   3. they are placed in log-scale buckets of their distance from the bound,
//      ranked within their buckets and written in order.
// A batch takes one workgroup per vector.
#include "device_common.h"
#include "filter_tile.h"
#include "launch.h"
#include "topk_block.h"

namespace profk {

constexpr int kSmallH = 8;            // 16-byte vectors per thread in each of two halves
constexpr int kSmallU = 2 * kSmallH;
constexpr uint32_t kSmallCap = 8192;  // elements collected in LDS
constexpr int kSmallDigit = 11;

struct SmallArgs {
  const void* values;
  uint64_t val_stride;  // bytes between the vectors of a batch
  uint32_t n, k;
  void* out_vals;
  int64_t* out_idx;
  profk_info_t* info;
};

struct SmallShared {
  uint32_t key[kSmallCap], idx[kSmallCap];
  alignas(16) uint32_t off[kLogBins];   // count, then first slot of each bucket
  alignas(16) uint32_t fill[kLogBins];  // entries placed in each bucket
  alignas(16) uint64_t comp[kSmallCap]; // (key, ~index) composites; before that the select's histogram and list
};

union SmallLds {
  SmallShared s;
  // the general selection over the collected elements, which the sort's
  // exchange buffers then overwrite
  struct {
    uint32_t key[kSmallCap], idx[kSmallCap];
    uint64_t sorted[kFinMaxK];            // radix histogram, then the collected top k
  } g;
  uint64_t exch[2 * kFinMaxK];
};
static_assert(2 * kFinMaxK <= kSmallCap, "exch ends before g.sorted");
static_assert(sizeof(SmallLds) + 2048 <= 160 * 1024, "LDS of a CU");

// What bounds it is one CU's load rate (a vector of 200 KB takes about 4 us)
// and the latency of the steps after it, about 2 us each.  Chunks of 8192
// elements selected by a workgroup each, with digit passes over the chunk and
// over the merged results, took 36 us (50000 fp32 values, k = 100) and a
// launch to clear their tickets before that.
template <int DT>
__global__ __launch_bounds__(kSmallBS) void k_small(SmallArgs a) {
  constexpr int ES = Elem<DT>::ES, EPV = Elem<DT>::EPV, KB = Elem<DT>::KEYBITS, H = kSmallH, U = kSmallU;
  __shared__ SmallLds sh;
  __shared__ SelectScratch scr;
  __shared__ __align__(16) uint32_t s_red[kKthRed];
  __shared__ uint32_t s_cnt, s_w[2 * (kSmallBS / kWave + 1)];
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
  const char* const values = static_cast<const char*>(a.values) + a.val_stride * blockIdx.x;
  void* const out_vals = static_cast<char*>(a.out_vals) + static_cast<size_t>(blockIdx.x) * a.k * ES;
  int64_t* const out_idx = a.out_idx + static_cast<size_t>(blockIdx.x) * a.k;
  uint32_t head = static_cast<uint32_t>(((16 - (reinterpret_cast<uintptr_t>(values) & 15)) & 15) / ES);
  if (head > a.n) head = a.n;
  const uint32_t nvec = (a.n - head) / EPV;
  const u32x4* const vec = reinterpret_cast<const u32x4*>(values + static_cast<size_t>(head) * ES);
  // past the end the last vector is read again and skipped (a vector of no
  // whole 16 bytes reads nothing)
  u32x4 v[2][H];
  if (nvec) {
#pragma unroll
    for (int u = 0; u < U; ++u) v[u / H][u % H] = vec[min(u * kSmallBS + tid, nvec - 1)];
  }
  // the elements before the first vector and after the last one, one per thread
  const uint32_t tail0 = head + nvec * EPV, ns = head + (a.n - tail0);
  const bool extra = tid < ns;
  const uint32_t xidx = tid < head ? tid : tail0 + (tid - head);
  const uint32_t xkey = extra ? key_of<DT>(load_raw<DT>(values, xidx)) : 0u;
  for (uint32_t i = tid; i < kLogBins; i += kSmallBS) {
    sh.s.off[i] = 0;
    sh.s.fill[i] = 0;
  }
  if (tid == 0) s_cnt = 0;
  // 1. the bound
  uint32_t low = 0;
  if (4 * min(nvec, static_cast<uint32_t>(kSmallBS)) >= a.k) {
    uint32_t g[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u * kSmallBS + tid < nvec) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
          const uint32_t raw = DT == 0 ? v[u / H][u % H][e & 3] : (v[u / H][u % H][e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
          g[e & 3] = max(g[e & 3], key_of<DT>(raw));
        }
      }
    }
    uint32_t* const pool = reinterpret_cast<uint32_t*>(sh.s.comp);
    low = block_kth_regs<kSmallBS, 4, kSmallDigit>(g, tid < nvec ? 0xFu : 0u, min(nvec, static_cast<uint32_t>(kSmallBS)),
                                                   a.k, pool, pool + (1 << kSmallDigit), s_red, scr)
              .x;
  } else {
    __syncthreads();
  }
  // 2. the elements that reach it
  auto slots = [&](uint32_t c) {
    const uint32_t incl = wave_incl_sum(c);
    const uint32_t tot = __builtin_amdgcn_readlane(incl, kWave - 1);
    uint32_t base = 0;
    if (lane == 0 && tot) base = atomicAdd(&s_cnt, tot);
    return __builtin_amdgcn_readlane(base, 0) + incl - c;
  };
  auto put = [&](uint32_t slot, uint32_t key, uint32_t idx) {
    if (slot < kSmallCap) {
      sh.s.key[slot] = key;
      sh.s.idx[slot] = idx;
    }
  };
  auto collect = [&](uint32_t least) {
    const Thresh<DT> th(least);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const TileSparse<DT, H, kSmallBS> ts(v[h], th, h * H * kSmallBS, nvec, tid, head);
      const bool x = h == 0 && extra && xkey >= least;
      uint32_t slot = slots(ts.count() + (x ? 1u : 0u));
      ts.emit(v[h], [&](uint32_t key, uint32_t idx) { put(slot++, key, idx); });
      if (x) put(slot, xkey, xidx);
    }
    __syncthreads();
    return s_cnt;
  };
  uint32_t n2 = collect(low);
  bool whole = false;
  if (n2 > kSmallCap) {
    // too many: if fewer than k lie above the bound it is the k-th largest
    // key, and the rest are the ties of smallest index
    const uint32_t key_max = KB == 32 ? 0xFFFFFFFFu : 0xFFFFu;
    __syncthreads();
    if (tid == 0) s_cnt = 0;
    __syncthreads();
    const uint32_t gt = low == key_max ? 0u : collect(low + 1);
    if (gt < a.k) {
      uint32_t need = a.k - gt, at = gt;  // uniform
      // c ties of this thread in index order after those of the threads below
      auto take = [&](uint32_t mask, auto index) {
        uint32_t tot;
        uint32_t r = block_excl_sum<kSmallBS>(static_cast<uint32_t>(__popc(mask)), scr.wsum, &tot);
        while (mask) {
          const uint32_t e = __builtin_ctz(mask);
          mask &= mask - 1;
          if (r < need) put(at + r, low, index(e));
          ++r;
        }
        at += min(tot, need);
        need -= min(tot, need);
      };
      take(tid < head && xkey == low ? 1u : 0u, [&](uint32_t) { return xidx; });
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (need && u * kSmallBS < nvec) {
          uint32_t mask = 0;
          if (u * kSmallBS + tid < nvec) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
              const uint32_t raw = DT == 0 ? v[u / H][u % H][e & 3] : (v[u / H][u % H][e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
              mask |= (key_of<DT>(raw) == low ? 1u : 0u) << e;
            }
          }
          take(mask, [&](uint32_t e) { return head + (u * kSmallBS + tid) * EPV + e; });
        }
      }
      if (need) take(extra && tid >= head && xkey == low ? 1u : 0u, [&](uint32_t) { return xidx; });
      n2 = a.k;
      __syncthreads();
    } else {
      whole = true;  // many distinct keys reach the bound (k is large against the maxima)
    }
  }
  bool done = false;
  if (!whole) {
    // 3. buckets of the distance from the bound
    for (uint32_t i = tid; i < n2; i += kSmallBS) atomicAdd(&sh.s.off[log_bin(sh.s.key[i] - low)], 1u);
    __syncthreads();
    // thread t owns buckets [kLogBins - 4(t+1), kLogBins - 4t)
    constexpr uint32_t kOwners = kLogBins / 4;
    const uint32_t bb = kLogBins - 4 * (min(tid, kOwners - 1) + 1);
    uint32_t h[4] = {0u, 0u, 0u, 0u};
    if (tid < kOwners) {
      const uint4 q = *reinterpret_cast<const uint4*>(&sh.s.off[bb]);
      h[0] = q.x; h[1] = q.y; h[2] = q.z; h[3] = q.w;
    }
    uint32_t run, wrun, tn, tw;
    block_excl_sum2<kSmallBS>(h[0] + h[1] + h[2] + h[3], h[0] * h[0] + h[1] * h[1] + h[2] * h[2] + h[3] * h[3], s_w, run,
                              wrun, tn, tw);
    if (tid < kOwners) {
      uint32_t o[4];
#pragma unroll
      for (int j = 3; j >= 0; --j) {
        o[j] = run;
        if (run < a.k && a.k <= run + h[j]) {
          scr.found[0] = bb + j;
          scr.found[1] = run + h[j];
          scr.found[2] = wrun + h[j] * h[j];  // (at most kSmallCap^2)
        }
        run += h[j];
        wrun += h[j] * h[j];
      }
      *reinterpret_cast<uint4*>(&sh.s.off[bb]) = uint4{o[0], o[1], o[2], o[3]};
    }
    __syncthreads();
    const uint32_t bstar = scr.found[0], n_sel = scr.found[1];
    if (scr.found[2] <= kFastCost) {
      const uint32_t thr = low + log_bin_edge(bstar);
      for (uint32_t i = tid; i < n2; i += kSmallBS) {
        const uint32_t key = sh.s.key[i];
        if (key >= thr) {
          const uint32_t bin = log_bin(key - low);
          sh.s.comp[sh.s.off[bin] + atomicAdd(&sh.s.fill[bin], 1u)] = composite(key, sh.s.idx[i]);
        }
      }
      __syncthreads();
      for (uint32_t p = tid; p < n_sel; p += kSmallBS) {
        const uint64_t c = sh.s.comp[p];
        const uint32_t bin = log_bin(comp_key(c) - low), s0 = sh.s.off[bin];
        const uint32_t dst = s0 + count_greater(sh.s.comp, s0, s0 + sh.s.fill[bin], c);
        if (dst < a.k) {
          const uint32_t bits = bits_of_key<DT>(comp_key(c));
          if (DT == 0) static_cast<uint32_t*>(out_vals)[dst] = bits;
          else static_cast<uint16_t*>(out_vals)[dst] = static_cast<uint16_t>(bits);
          out_idx[dst] = comp_idx(c);
        }
      }
      done = true;
    }
  }
  if (!done) {
    // heavy ties among the collected, or more elements than LDS holds: the
    // general selection (from memory in the latter case), then a sort
    __syncthreads();
    const TopkSmem sm{nullptr, 0, reinterpret_cast<uint32_t*>(sh.g.sorted), sh.g.sorted, &scr, &s_cnt};
    if (whole) block_topk_core<kSmallBS, kSmallDigit>(InputSrc<DT>{values, 0u}, a.n, a.k, low, KB == 32 ? 0xFFFFFFFFu : 0xFFFFu, KB, sm);
    else block_topk_core<kSmallBS, kSmallDigit>(LdsSrc<uint32_t>{sh.g.key, sh.g.idx}, n2, a.k, low, KB == 32 ? 0xFFFFFFFFu : 0xFFFFu, KB, sm);
    sort_write_any<DT, kSmallBS>(sh.g.sorted, a.k, a.k, sh.exch, out_vals, out_idx);
  }
  if (a.info && tid == 0) {
    profk_info_t* inf = a.info + blockIdx.x;
    inf->count = 0;
    inf->tau_key = 0;
    inf->status = PROFK_STATUS_DIRECT;
    inf->n_valid = a.k;
  }
}

// ------------------------------------------------------------- host -------
bool small_fits(int64_t n, int64_t k, int dtype) {
  return k <= kFinMaxK && n <= kSmallBS * kSmallU * (dtype == PROFK_F32 ? Elem<0>::EPV : Elem<1>::EPV);
}

hipError_t launch_small(const FlatCall& c) {
  (void)hipGetLastError();
  SmallArgs sa{c.values, c.stride.val, c.n, c.k, c.out_vals, c.out_idx, c.info};
  if (c.dtype == PROFK_F32) hipLaunchKernelGGL(k_small<0>, dim3(c.rows), dim3(kSmallBS), 0, c.stream, sa);
  else hipLaunchKernelGGL(k_small<1>, dim3(c.rows), dim3(kSmallBS), 0, c.stream, sa);
  return hipGetLastError();
}

}  // namespace profk
