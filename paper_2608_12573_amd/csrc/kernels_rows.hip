// Per-row Prof-K (Sec. 3: for batched inputs the procedure runs on each
// batch element).  One workgroup of 64 to 1024 threads owns one row and runs
// all four stages in LDS:
//   1. draw S indices of the row (Philox counter word 1 = row);
//   2. tau = t-th largest sampled key (from registers when they hold the
//      sample, else a radix select in LDS); lexicographic plans also find the
//      index of the threshold pair;
//   3. stream the row once with 16-byte loads, appending survivors to an
//      LDS buffer of capacity M and counting all of them; a buffer that
//      holds them all is then histogrammed by log_bin(key - tau);
//   4. k_req <= count <= M: the survivors at or above the bucket of rank k
//      are ranked within their buckets and written directly (the radix
//      refinement when those buckets are large); otherwise the exact top-k
//      of the row itself (per-row fallback, no second launch).
// The LDS layout is sized from the plan at launch (dynamic shared memory).
#include <type_traits>

#include "device_common.h"
#include "filter_tile.h"
#include "launch.h"
#include "row_common.h"
#include "topk_block.h"

namespace profk {

// The sample is held in registers (at most 8 keys per thread).
__host__ __device__ constexpr bool row_fast_tau(uint32_t S, int bs) { return S <= 8u * static_cast<uint32_t>(bs); }

// Log-scale buckets of a row workgroup: the buckets of a row key's distance,
// padded so that every thread owns the same number.
// A block of one wave takes eight log bins as one bucket: a short row's few
// hundred survivors leave them small, and clearing and scanning 3328 counters
// would cost more than the survivors do.
template <int BS> constexpr uint32_t row_bin_shift() { return BS == kRowShortBS ? 3u : 0u; }
template <int DT, int BS> constexpr uint32_t row_bins_per_thread() {
  return ((row_log_bins<DT>() >> row_bin_shift<BS>()) + BS - 1) / BS;
}
// Radix digit of the refinement and fallback in a block of one wave: eight
// bits, whose histogram fits beside its other arrays.
template <int DT, int BS> constexpr int row_block_digit() { return BS == kRowShortBS ? 8 : row_digit<DT>(); }

// Largest t whose threshold 16-bit keys take by the maxima of lane groups.
constexpr uint32_t kRowFewT = 32;

struct RowArgs {
  const void* values;
  uint32_t row;         // of the batch: the first of this launch
  uint64_t row_stride;  // elements between row starts
  uint32_t D, k, k_req, S, t, M;
  int direct;
  uint64_t seed;
  void* out_vals;
  int64_t* out_idx;
  profk_info_t* info;
  RowLayout L;
};

// PRE: the first step of the row's stream is loaded before the sample is
// drawn, so that the sample's latency and the stream's overlap; it takes
// registers that a workgroup among many on its CU has no use for.
template <int DT, bool LEX, int BS, bool PRE>
__global__ __launch_bounds__(BS, BS == kRowShortBS ? 4 : 1) void k_rows(RowArgs a) {
  constexpr int U = BS == kRowShortBS ? kRowShortU : kRowU;
  constexpr int ES = Elem<DT>::ES, EPV = Elem<DT>::EPV, KB = Elem<DT>::KEYBITS;
  constexpr int kSelDigitRow = KB == 16 ? 8 : 11;  // sample select: 2 or 3 passes
  constexpr int kDigit = row_block_digit<DT, BS>();
  constexpr int kTauDigit = BS == kRowShortBS ? kRowTauDigit : 10;  // the sample's histogram, within `hist`
  using K = RowKey<DT>;
  constexpr int NW = BS / kWave;
  constexpr uint32_t RB = row_bins_per_thread<DT, BS>();  // log bins owned per thread
  constexpr uint32_t NB = RB * BS;                        // (the bins past the last log bin stay empty)
  extern __shared__ __align__(16) uint8_t smem[];
  uint32_t* const samp = reinterpret_cast<uint32_t*>(smem + a.L.off_a);  // samples, then buffer keys
  K* const bkey = reinterpret_cast<K*>(smem + a.L.off_a);
  uint32_t* const bidx = reinterpret_cast<uint32_t*>(smem + a.L.off_b);
  uint32_t* const hist = reinterpret_cast<uint32_t*>(smem + a.L.off_hist);
  uint64_t* const collect = reinterpret_cast<uint64_t*>(smem + a.L.off_collect);
  uint64_t* const comp = reinterpret_cast<uint64_t*>(smem + a.L.off_comp);
  uint64_t* const exch = reinterpret_cast<uint64_t*>(smem + a.L.off_a);      // after the buffer is done
  __shared__ SelectScratch scr;
  __shared__ uint32_t s_cnt, s_counter, s_tie_n, s_wmax[NW];
  __shared__ __align__(16) uint32_t s_red[kKthRed];

  const uint32_t r = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  const char* row = static_cast<const char*>(a.values) + static_cast<size_t>(r) * a.row_stride * ES;
  void* out_vals = static_cast<char*>(a.out_vals) + static_cast<size_t>(r) * a.k * ES;
  int64_t* out_idx = a.out_idx + static_cast<size_t>(r) * a.k;
  const uint32_t key_max = KB == 32 ? 0xFFFFFFFFu : 0xFFFFu;
  const TopkSmem sm{nullptr, 0, hist, collect, &scr, &s_counter};

  const uintptr_t addr = reinterpret_cast<uintptr_t>(row);
  uint32_t head = static_cast<uint32_t>(((16 - (addr & 15)) & 15) / ES);
  if (head > a.D) head = a.D;
  const uint32_t nvec = (a.D - head) / EPV;
  const u32x4* vec = reinterpret_cast<const u32x4*>(row + static_cast<size_t>(head) * ES);

  uint32_t status = PROFK_STATUS_DIRECT, count = 0, tau = 0, gmax = 0;
  auto bucket = [&](uint32_t key) { return log_bin(key - tau) >> row_bin_shift<BS>(); };
  if (!a.direct) {
    u32x4 v[U];
    // one step of the stream, U vectors per thread (nvec > 0): past the
    // end the last vector is read again, and the exact test skips it.
    // (branch-free: with a branch per vector and v outside the loop the
    // compiler waits for each load before it issues the next)
    auto load_step = [&](uint32_t vb) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(vec + min(vb + u * BS + tid, nvec - 1));
    };
    if (PRE && nvec) load_step(0);
    // 1. sample: the Philox words first, then all gathers in flight at once
    const bool fast = row_fast_tau(a.S, BS);
    uint32_t keys[8], ids[8];
    uint32_t valid = 0;
    for (uint32_t blk0 = 0; 4 * blk0 < a.S; blk0 += 2 * BS) {
      U64x4 rnd[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t blk = blk0 + q * BS + tid;
        if (4 * blk < a.S) rnd[q] = philox4x64_10(blk, a.row + r, 0, 0, a.seed, 0);
      }
      uint32_t raw[8];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const uint32_t j = 4 * (blk0 + q * BS + tid) + x;
          ids[4 * q + x] = j < a.S ? index_of_word(rnd[q].w[x], a.D) : 0u;
          raw[4 * q + x] = j < a.S ? load_raw<DT>(row, ids[4 * q + x]) : 0u;
        }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const uint32_t j = 4 * (blk0 + q * BS + tid) + x;
          keys[4 * q + x] = key_of<DT>(raw[4 * q + x]);
          if (j < a.S) {
            valid |= 1u << (4 * q + x);
            if (!fast) samp[j] = keys[4 * q + x];
          }
        }
    }
    if (tid == 0) s_cnt = 0;
    // 2. threshold.  16-bit keys and t past a few: two radix passes of eight
    // bits over the registers (2432 rows of 3510, t = 129: 30.5 us with the
    // histogram of distances, 26.6; 5100 of 3734, t = 53: 43.2, 37.7; the samples
    // kept in LDS took 28.1 and 40.9).  The one-wave kernel, whose registers
    // are few and samples small, goes without the branch.
    if (KB == 16 && BS != kRowShortBS && fast && a.t > kRowFewT) {
      tau = block_select_kth<BS, kSelDigitRow>(
                [&](auto f) {
#pragma unroll
                  for (int e = 0; e < 8; ++e)
                    if ((valid >> e) & 1u) f(keys[e]);
                },
                a.t, KB, 0u, hist, scr)
                .kth;
    } else if (fast) {
      static_assert(kFastBucket * 8 >= kListWords * 4, "the list in comp");
      tau = block_kth_regs<BS, 8, kTauDigit>(keys, valid, min((a.S + 3) / 4, static_cast<uint32_t>(BS)), a.t, hist,
                                             reinterpret_cast<uint32_t*>(comp), s_red, scr)
                .x;
    } else {
      __syncthreads();
      tau = block_select_kth<BS, kSelDigitRow>(
                [&](auto f) {
                  for (uint32_t i = tid; i < a.S; i += BS) f(samp[i]);
                },
                a.t, KB, 0u, hist, scr)
                .kth;
    }
    uint32_t tie = 0xFFFFFFFFu;
    if (LEX && fast) {
      // the draws are still in registers
      auto draws = [&](auto f) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if ((valid >> e) & 1u) f(keys[e], ids[e]);
      };
      tie = tau_pair_index<BS, kDigit>(draws, tau, a.t, reinterpret_cast<uint32_t*>(smem + a.L.off_a),
                                           a.L.off_b / 4u, hist, scr, &s_tie_n);
    } else if (LEX) {
      // the draws again (Philox words and gathers), for the tied draws' indices
      auto draws = [&](auto f) {
        for (uint32_t jb = tid; 4 * jb < a.S; jb += BS) {
          const U64x4 rr = philox4x64_10(jb, a.row + r, 0, 0, a.seed, 0);
          uint32_t raw[4], ix[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bool in = 4 * jb + q < a.S;
            ix[q] = in ? index_of_word(rr.w[q], a.D) : 0u;
            raw[q] = in ? load_raw<DT>(row, ix[q]) : 0u;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (4 * jb + q < a.S) f(key_of<DT>(raw[q]), ix[q]);
        }
      };
      tie = tau_pair_index<BS, kDigit>(draws, tau, a.t, reinterpret_cast<uint32_t*>(smem + a.L.off_a),
                                           a.L.off_b / 4u, hist, scr, &s_tie_n);
    }
    for (uint32_t i = tid; i < NB; i += BS) hist[i] = 0;
    __syncthreads();

    // 3. filter the row into the LDS buffer (which reuses the sample space)
    const Thresh<DT> th(tau, tie);
    uint32_t my_max = 0;
    auto reserve = [&](uint32_t cnt) {
      const uint32_t incl = wave_incl_sum(cnt);
      const uint32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&s_cnt, total);
      return __builtin_amdgcn_readlane(base, 0) + incl - cnt;
    };
    auto store = [&](uint32_t slot, uint32_t key, uint32_t idx) {
      my_max = max(my_max, key);
      if (slot < a.M) {
        bkey[slot] = static_cast<K>(key);
        bidx[slot] = idx;
      }
    };
    for (uint32_t vb = 0; vb < nvec; vb += BS * U) {
      constexpr bool kOne = BS == kRowShortBS;  // the row is one step
      if constexpr (!kOne) {
        if (!PRE || vb) load_step(vb);
      }
      const TileSparse<DT, U, BS, LEX> tx(v, th, vb, nvec, tid, head);
      if (__ballot(tx.any()) == 0) continue;
      uint32_t slot = reserve(tx.count());
      tx.emit(v, [&](uint32_t key, uint32_t idx) { store(slot++, key, idx); });
    }
    if (tid < kWave) {
      // elements before the first aligned vector and after the last one
      const uint32_t tail0 = head + nvec * EPV;
      const uint32_t ns = head + (a.D - tail0);
      uint32_t idx = 0, key = 0;
      bool ok = false;
      if (lane < ns) {
        idx = lane < head ? lane : tail0 + (lane - head);
        key = key_of<DT>(load_raw<DT>(row, idx));
        ok = LEX ? (key > tau || (key == tau && idx <= tie)) : key >= tau;
      }
      if (__ballot(ok)) {
        const uint32_t slot = reserve(ok ? 1u : 0u);
        if (ok) store(slot, key, idx);
      }
    }
    const uint32_t wm = wave_max_u32(my_max);
    if (lane == 0) s_wmax[w] = wm;
    __syncthreads();
    count = s_cnt;
#pragma unroll
    for (int i = 0; i < NW; ++i) gmax = max(gmax, s_wmax[i]);
    status = count < a.k_req ? PROFK_STATUS_UNDERFLOW
                             : (count > a.M ? PROFK_STATUS_OVERFLOW : PROFK_STATUS_FILTERED);
    if (status == PROFK_STATUS_FILTERED) {
      // bucket histogram of the buffer (after the pass, so that the
      // streaming loop does no per-survivor histogram atomics)
      for (uint32_t i = tid; i < count; i += BS) atomicAdd(&hist[bucket(bkey[i])], 1u);
      __syncthreads();
    }
  }

  // 4. refinement, or the exact per-row fallback
  uint32_t kk = a.k;
  bool done = false;
  if (status == PROFK_STATUS_FILTERED) {
    kk = min(a.k, count);
    // Bucket offsets in descending bucket order, in place: thread t owns
    // buckets [NB - RB(t+1), NB - RB t).
    const uint32_t bb = NB - RB * (tid + 1);
    uint32_t h[RB];
    uint32_t s = 0;
#pragma unroll
    for (uint32_t j = 0; j < RB; ++j) {
      h[j] = hist[bb + j];
      s += h[j];
    }
    uint32_t run = block_excl_sum<BS>(s, scr.wsum, nullptr);
#pragma unroll
    for (int j = static_cast<int>(RB) - 1; j >= 0; --j) {
      hist[bb + j] = run;
      if (run < kk && kk <= run + h[j]) {
        scr.found[0] = bb + j;
        scr.found[1] = run;
        scr.found[2] = h[j];
      }
      run += h[j];
    }
    __syncthreads();
    const uint32_t bstar = scr.found[0], n_sel = scr.found[1] + scr.found[2];
    uint32_t big = 0;
#pragma unroll
    for (uint32_t j = 0; j < RB; ++j)
      if (bb + j >= bstar) big = max(big, h[j]);
    big = block_max<BS>(big, scr.wsum);
    if (n_sel <= a.k + kFastBucket && big <= kFastBucket) {
      // place the buckets >= b*: afterwards hist[b] is the end of bucket b
      // and hist[b + 1] its start
      for (uint32_t i = tid; i < count; i += BS) {
        const uint32_t key = bkey[i];
        const uint32_t bin = bucket(key);
        if (bin >= bstar) comp[atomicAdd(&hist[bin], 1u)] = composite(key, bidx[i]);
      }
      __syncthreads();
      for (uint32_t p = tid; p < n_sel; p += BS) {
        const uint64_t c = comp[p];
        const uint32_t bin = bucket(comp_key(c));
        const uint32_t s0 = bin + 1 < NB ? hist[bin + 1] : 0u, s1 = hist[bin];
        uint32_t rank = 0;
        for (uint32_t q = s0; q < s1; ++q) rank += comp[q] > c ? 1u : 0u;
        const uint32_t dst = s0 + rank;
        if (dst < kk) {
          const uint32_t bits = bits_of_key<DT>(comp_key(c));
          if (DT == 0) static_cast<uint32_t*>(out_vals)[dst] = bits;
          else static_cast<uint16_t*>(out_vals)[dst] = static_cast<uint16_t>(bits);
          out_idx[dst] = comp_idx(c);
        }
      }
      for (uint32_t p = kk + tid; p < a.k; p += BS) {  // relaxed recall: padding
        if (DT == 0) static_cast<uint32_t*>(out_vals)[p] = 0xFF800000u;
        else static_cast<uint16_t*>(out_vals)[p] = 0xFF80u;
        out_idx[p] = -1;
      }
      done = true;
    } else {
      block_topk<BS, kDigit>(LdsSrc<K>{bkey, bidx}, count, kk, tau, max(gmax, tau), KB, sm);
    }
  } else {
    block_topk<BS, kDigit>(InputSrc<DT>{row, 0u}, a.D, a.k, 0u, key_max, KB, sm);
  }
  if (!done) sort_write_any<DT, BS>(collect, kk, a.k, exch, out_vals, out_idx);
  if (a.info && tid == 0) {
    profk_info_t* inf = a.info + r;
    inf->count = count;
    inf->tau_key = tau;
    inf->status = static_cast<int32_t>(status);
    inf->n_valid = kk;
  }
}

// ------------------------------------------------------------- host -------
static inline uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }

RowLayout row_layout(const profk_plan_t& p, int dtype, int bs) {
  RowLayout L;
  const uint32_t S = static_cast<uint32_t>(p.S), M = static_cast<uint32_t>(p.M);
  const uint32_t k = static_cast<uint32_t>(p.k);
  const bool f32 = dtype == PROFK_F32;
  const uint32_t ubs = static_cast<uint32_t>(bs);
  uint32_t P = 1;
  while (P < (k > ubs ? k : ubs)) P <<= 1;
  const uint32_t exch = 2u * P * 8u;
  const uint32_t b_bytes = align16(M * 4u);
  const uint32_t samp_bytes = row_fast_tau(S, bs) ? 0u : S * 4u;   // samples kept in LDS
  const uint32_t key_bytes = M * (f32 ? 4u : 2u);
  uint32_t a_bytes = align16(samp_bytes > key_bytes ? samp_bytes : key_bytes);
  if (a_bytes + b_bytes < exch) a_bytes = exch - b_bytes;
  const bool wave = bs == kRowShortBS;
  const uint32_t nb = ((f32 ? row_log_bins<0>() : row_log_bins<1>()) >> (wave ? row_bin_shift<kRowShortBS>() : 0u)) + ubs - 1;
  // the radix digit's histogram; in a block of one wave the sample's is larger
  const uint32_t radix = 1u << (wave ? kRowTauDigit : f32 ? row_digit<0>() : row_digit<1>());
  uint32_t hist_words = radix;
  if (hist_words < nb / ubs * ubs) hist_words = nb / ubs * ubs;
  L.off_a = 0;
  L.off_b = a_bytes;
  L.off_hist = L.off_b + b_bytes;
  L.off_collect = L.off_hist + align16(hist_words * 4u);
  L.off_comp = L.off_collect + align16(k * 8u);
  L.bytes = L.off_comp + align16((k + kFastBucket) * 8u);
  return L;
}

// The plan's arrays in 32-bit byte sums: the buffer alone takes 4*M bytes
// (and a large sample 4*S).
static bool row_sums_fit(const profk_plan_t& p, int64_t max_k) {
  constexpr int64_t kMaxWords = kRowMaxLds / 4;
  return p.k <= max_k && p.M <= kMaxWords && p.S <= kMaxWords;
}

bool rows_fit_block(const profk_plan_t& p, int dtype) {
  return row_sums_fit(p, kRowMaxK) && row_layout(p, dtype, kRowBS).bytes <= kRowMaxLds;
}

// Threads per row.  A workgroup's rate is bound by the loads it has in flight
// (measured, fp32 rows alone on a CU: 7 GB/s with 256 threads, 37 with 1024),
// a short row's time by the latency of its stages (about 10 us, however many
// threads), so short rows want many small workgroups per CU and long or few
// rows large ones.  Measured on one MI355X (us, 256 / 512 / 1024 threads):
//   64 rows of 400 KB: 45 / 28 / 24;  256 of 128 KB: 26 / 22 / 18;
//   4096 of 256 KB (bf16): 215 / 203 / 313;  1024 of 400 KB: 90 / 83 / 105;
//   1024 of 128 KB: 36.8 / 37.0 / 62;  4096 of 64 KB: 68 / 80 / 193;
//   8192 of 16 KB: 74 / 118 / 304;  16 of 16 KB: 16 / - / 16.
// A large batch of rows that one wave holds in registers takes a wave per row:
// there a block's barriers and the passes of four waves over its counters cost
// more than the row (256 / 64 threads: 8192 rows of 16 KB 72 / 61, of 4 KB
// 70 / 34; 512 of 16 KB 17 / 19).  The lexicographic rule does not fit its
// registers.
// Under the lexicographic rule, whose blocks have more steps after the stream,
// small workgroups stay ahead for long rows too, while there are enough for
// several on each CU and four fit its LDS (256 / 512 threads, bf16: 4096 rows of
// 256 KB 231 / 281, 1214 of 162 KB 65 / 74; fp32: 1024 of 400 KB 94 / 100; but 512
// of 256 KB 55 / 49, and 1000 fp32 of 256 KB with k = 1000, 54 KB of LDS, 161 / 112).
// The vector path (sample, filter, refinement: three launches of which each
// takes R rows) shares every row out over the chip, which pays where a row is
// long and the rows are few.  Measured (us, 1024 threads / vector path, k = 32
// fp32): 4 rows of 400 KB 22 / 23, of 1 MB 37 / 23, of 4 MB 100 / 25; 64 rows
// of 400 KB 24 / 30, of 1 MB 41 / 37, of 4 MB 119 / 72; 256 rows of 1 MB 57 / 147.
// (one row after another, as before, 8 rows of 16 MB took 192 us, against 42.)
int rows_block_threads(const profk_plan_t& p, int dtype, int64_t B, int64_t R, int num_cus) {
  auto fits = [&](int bs) {
    return row_sums_fit(p, 4 * bs) && row_layout(p, dtype, bs).bytes <= kRowMaxLds;
  };
  const int64_t kb = p.N * (dtype == PROFK_F32 ? 4 : 2) / 1024;
  if (p.mode == PROFK_MODE_DIRECT && small_fits(p.N, p.k, dtype) && (kb >= kRowSmallKb || B <= num_cus)) return kRowsSmall;
  const bool small = rows_fit_block(p, dtype), wide = fits(kRowWideBS);
  if (!small && !wide) return 0;
  if (wide && R > 0) {
    const bool direct = p.mode == PROFK_MODE_DIRECT;
    const int64_t block_us = (B + num_cus - 1) / num_cus * ((direct ? 80 : 12) + kb / 37);
    const int64_t vector_us = (B + R - 1) / R * (direct ? 50 : 23) + B * kb / 5500 + B / 8;
    if (block_us > vector_us) return 0;
  }
  if (!small) return B > num_cus && fits(kRowMidBS) ? kRowMidBS : kRowWideBS;
  if (p.N * (dtype == PROFK_F32 ? 4 : 2) <= kRowShortBytes && B >= 4 * num_cus && p.mode == PROFK_MODE_FILTER &&
      !p.lexicographic && p.k <= kRowShortBS * 4 && p.S <= kRowShortBS * 8 && p.M <= kRowShortM)
    return kRowShortBS;
  if (kb >= 32 && B <= num_cus && wide) return kRowWideBS;
  const bool many = B > 2 * num_cus && row_layout(p, dtype, kRowBS).bytes <= 39 * 1024;  // (and 0.5 KB static)
  if (kb >= 128 && fits(kRowMidBS) && !(p.lexicographic && many)) return kRowMidBS;
  return kRowBS;
}

template <int DT, int BS, bool PRE>
static hipError_t launch_rows_t(const RowCall& c) {
  const profk_plan_t& p = *c.plan;
  RowArgs ra{c.values, c.row, c.row_stride, c.D, c.k, static_cast<uint32_t>(p.k_req), static_cast<uint32_t>(p.S),
             static_cast<uint32_t>(p.t), static_cast<uint32_t>(p.M), p.mode == PROFK_MODE_DIRECT ? 1 : 0,
             c.seed, c.out_vals, c.out_idx, c.info, row_layout(p, c.dtype, BS)};
  const uint32_t lds = ra.L.bytes;
  if constexpr (BS != kRowShortBS) {
    if (p.lexicographic) {
      hipLaunchKernelGGL((k_rows<DT, true, BS, PRE>), dim3(c.B), dim3(BS), lds, c.stream, ra);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_rows<DT, false, BS, PRE>), dim3(c.B), dim3(BS), lds, c.stream, ra);
  return hipGetLastError();
}

template <int DT>
static hipError_t launch_rows_dt(const RowCall& c) {
  if (c.threads == kRowShortBS) return launch_rows_t<DT, kRowShortBS, true>(c);
  if (c.threads == kRowWideBS) return launch_rows_t<DT, kRowWideBS, true>(c);
  if (c.threads == kRowMidBS) return launch_rows_t<DT, kRowMidBS, true>(c);
  return launch_rows_t<DT, kRowBS, false>(c);
}

hipError_t launch_rows(const RowCall& c) {
  (void)hipGetLastError();  // report only errors of this call's launches
  return c.dtype == PROFK_F32 ? launch_rows_dt<0>(c) : launch_rows_dt<1>(c);
}

}  // namespace profk
