// Device pieces shared by the NN-search kernels (select.hip, select_fused.hip):
// int8 code conversion, and selection over 48-bit (key, row) values.
#pragma once

#include "common.h"

namespace tav2 {

// The int8 sequence storage (codes q, Sec. 3.2.1) enters the products as bf16
// (exact: |q| <= 127); the lane also accumulates the squares of its 8 codes
// (exact in fp32: a row's sum of squares is an integer below 2^24).
__device__ __forceinline__ bf16x8 codes_to_bf16(uint2 raw, float& sq) {
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t word = j < 4 ? raw.x : raw.y;
    const float x = float(int8_t((word >> (8 * (j & 3))) & 0xFF));
    sq = fmaf(x, x, sq);
    v[j] = static_cast<__bf16>(x);
  }
  return v;
}

// Normalised score of Sec. 3.4.2's fused dequantisation: <q, c> / |q| from the
// exact dot product and the exact sum of squares ss (0 for an all-zero row).  The
// division and the square root are rounded to nearest (the build keeps them
// correctly rounded).
__device__ __forceinline__ float i8_score(float dot, float ss) {
  return ss > 0.f ? dot / sqrtf(ss) : 0.f;
}

// 48-bit selection value of a row: its 32-bit score key above 0xFFFF - row, so
// that the larger value is the row earlier in the order (score desc, row asc).
// Rows are below 65536.
__device__ __forceinline__ uint64_t sel_value(uint32_t key, int row) {
  return (uint64_t(key) << 16) | uint64_t(0xFFFFu - uint32_t(row));
}
__device__ __forceinline__ int sel_row(uint64_t v) { return int(0xFFFFu - uint32_t(v & 0xFFFFu)); }
__device__ __forceinline__ uint32_t sel_key(uint64_t v) { return uint32_t(v >> 16); }

// Orders a wave's LDS writes before its later LDS reads of words other lanes
// wrote (no workgroup barrier: the data is the wave's own).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-wide scans and reductions through DPP row shifts and row broadcasts
// (no LDS round trip): row_shr 1, 2, 4, 8 combine within rows of 16 lanes, then
// row_bcast 15 and 31 carry row totals upwards.  Lanes a shift leaves without a
// source take the identity (the `old` operand).
#define TAV2_DPP_STEPS(OP, ID)                                                          \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x111, 0xf, 0xf, false)); \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x112, 0xf, 0xf, false)); \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x114, 0xf, 0xf, false)); \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x118, 0xf, 0xf, false)); \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x142, 0xa, 0xf, false)); \
  v = v OP uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x143, 0xc, 0xf, false));
// Inclusive prefix sum over the lanes.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v) {
  TAV2_DPP_STEPS(+, 0)
  return v;
}
// OR / AND over the lanes, returned to every lane (lane 63 holds the result).
__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
  uint32_t v = uint32_t(x);
  TAV2_DPP_STEPS(|, 0)
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(v), 63));
  v = uint32_t(x >> 32);
  TAV2_DPP_STEPS(|, 0)
  return (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(v), 63))) << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_and64(uint64_t x) {
  uint32_t v = uint32_t(x);
  TAV2_DPP_STEPS(&, -1)
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(v), 63));
  v = uint32_t(x >> 32);
  TAV2_DPP_STEPS(&, -1)
  return (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(v), 63))) << 32) | lo;
}
// Smallest / largest over the lanes, returned to every lane.
#define TAV2_DPP_FN(F, ID)                                                                  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x111, 0xf, 0xf, false)));  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x112, 0xf, 0xf, false)));  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x114, 0xf, 0xf, false)));  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x118, 0xf, 0xf, false)));  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x142, 0xa, 0xf, false)));  \
  v = F(v, uint32_t(__builtin_amdgcn_update_dpp(ID, int(v), 0x143, 0xc, 0xf, false)));  \
  return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
__device__ __forceinline__ uint32_t wave_min_u(uint32_t v) { TAV2_DPP_FN(min, -1) }
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) { TAV2_DPP_FN(max, 0) }
#undef TAV2_DPP_FN
#undef TAV2_DPP_STEPS

// One digit step of a descending radix select, done by a whole wave on a
// 256-bin histogram h in LDS: the digit whose bin holds the need-th largest
// value (1 <= need <= the histogram's total) and the rank of that value among
// the bin's values (rest).  Lane l takes bins 255 - 4l .. 252 - 4l; every lane
// returns the result.
__device__ __forceinline__ void radix_digit(const uint32_t* h, uint32_t need, uint32_t& digit,
                                            uint32_t& rest) {
  const int lane = threadIdx.x % WAVE;
  const uint4 q = *reinterpret_cast<const uint4*>(h + 252 - 4 * lane);
  const uint32_t hb[4] = {q.w, q.z, q.y, q.x};   // bins 255 - 4l - i
  const uint32_t sum = hb[0] + hb[1] + hb[2] + hb[3];
  const uint32_t incl = wave_incl_sum(sum);
  const uint32_t before = incl - sum;
  uint32_t dg = 0, rs = 0, cum = before;
  bool hit = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!hit && cum + hb[i] >= need) {
      hit = true;
      dg = uint32_t(255 - 4 * lane - i);
      rs = need - cum;
    }
    cum += hb[i];
  }
  // exactly one lane holds the crossing
  const uint64_t who = __builtin_amdgcn_ballot_w64(before < need && need <= incl);
  const int src = int(__builtin_ctzll(who));
  digit = uint32_t(__builtin_amdgcn_readlane(int(dg), src));
  rest = uint32_t(__builtin_amdgcn_readlane(int(rs), src));
}

// The need-th largest (1-based) of the cnt distinct 48-bit values v[] in LDS,
// by an 8-bit radix select, most significant byte first, with NT threads.  The
// bytes above the highest bit in which the values differ are common to all of
// them and are skipped (their passes would put every value in one bin).  Every
// wave reads each histogram and finds the digit itself, and the histograms
// rotate over three buffers (a buffer is cleared in the pass after its own, two
// passes before its next use), so that a pass costs one barrier.  hist (3 x 256
// words, 16-byte aligned) and red (2 x NT / 64 values) are LDS scratch.  Starts
// and ends with a barrier; every thread returns the value.
template <int NT>
__device__ __forceinline__ uint64_t radix_select48(const uint64_t* v, int cnt, int need,
                                                   uint32_t* hist, uint64_t* red) {
  static_assert(NT >= 256, "one histogram bin per thread");
  constexpr int NW = NT / WAVE;
  const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
  __syncthreads();   // v[] is complete
  uint64_t any = 0, all = ~uint64_t(0);
  for (int i = tid; i < cnt; i += NT) {
    any |= v[i];
    all &= v[i];
  }
  any = wave_or64(any);
  all = wave_and64(all);
  if (lane == 0) {
    red[wid] = any;
    red[NW + wid] = all;
  }
  if (tid < 256) hist[tid] = hist[256 + tid] = 0u;
  __syncthreads();
  any = 0;
  all = ~uint64_t(0);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    any |= red[w];
    all &= red[NW + w];
  }
  const uint64_t diff = (any ^ all) & ((uint64_t(1) << 48) - 1);
  // first pass: the byte holding the highest differing bit (0 when cnt == 1)
  const int top = diff ? 63 - __builtin_clzll(diff) : 0;
  const int sh0 = top / 8 * 8;
  uint64_t pre = sh0 + 8 >= 48 ? 0 : all >> (sh0 + 8);
  uint32_t nd = uint32_t(need);
  int buf = 0;
  for (int sh = sh0; sh >= 0; sh -= 8) {
    uint32_t* h = hist + 256 * buf;
    for (int i = tid; i < cnt; i += NT) {
      const uint64_t x = v[i];
      if ((x >> (sh + 8)) == pre) atomicAdd(&h[(x >> sh) & 255u], 1u);
    }
    __syncthreads();
    const int clr = buf == 0 ? 2 : buf - 1;   // the previous pass's buffer: read by now
    if (tid < 256) hist[256 * clr + tid] = 0u;
    uint32_t digit, rest;
    radix_digit(h, nd, digit, rest);
    pre = (pre << 8) | uint64_t(digit);
    nd = rest;
    buf = buf == 2 ? 0 : buf + 1;
  }
  __syncthreads();
  return pre;
}

// The kk distinct selection values sel[] (LDS, any order, 16-byte aligned) to
// their ranks in the order: out_idx[rank] = row, out_score[rank] = score.  The
// rank of a value is the number of larger values (each thread reads the list
// two values per 16-byte LDS read, the same address across the wave: broadcasts).
template <int NT>
__device__ __forceinline__ void place_by_rank(const uint64_t* sel, int kk, int32_t* oi, float* os) {
  const uint4* s2 = reinterpret_cast<const uint4*>(sel);
  for (int s = threadIdx.x; s < kk; s += NT) {
    const uint64_t me = sel[s];
    int rank = 0;
    int t = 0;
    for (; t + 8 <= kk; t += 8) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 v = s2[t / 2 + u];
        rank += (uint64_t(v.y) << 32 | v.x) > me ? 1 : 0;
        rank += (uint64_t(v.w) << 32 | v.z) > me ? 1 : 0;
      }
    }
    for (; t < kk; ++t) rank += sel[t] > me ? 1 : 0;
    oi[rank] = sel_row(me);
    os[rank] = key_score(sel_key(me));
  }
}

// The kk best of a workgroup's keys to their places in the order, by bins.
//
// Keys are binned by (largest key - key) >> shift into 1024 bins of one width that
// cover the keys' range; a value's rank is then the number of values in the bins
// before its own plus its rank within the bin, so a bin of a few values takes a few
// comparisons each, whatever kk is.  Only the values of bins up to the one that holds
// the kk-th are moved.  (A radix select followed by counting, for each of the kk, how
// many are larger, costs kk^2 comparisons: a search of 4000 candidates over 16384 rows
// at kk = 512 took 234 us that way and takes 139, of 500 at kk = 1024 103 and 38, of
// 1000 at kk = 256 60 and 51.  Over short rows, against a search for the kk-th key bit
// by bit over the whole workgroup: 2800 candidates of 200 to 4000 rows at kk = 64, 62
// and 31.)
//
// Bins as wide as the whole range are too coarse where it is wide (scores of both signs:
// four bins to a factor of two), so the range is narrowed to what lies at or above the
// kk-th value's bin, and binned again, while that makes the bins finer and that bin holds
// more than a few values, and at most half of what it held (it does not shrink where it
// holds equal scores).  Scores of both signs, rows of 16: 1000 candidates of 4000 rows at
// kk = 256 and 700 at kk = 1000 take 22 and 23 us a search, and 56 and 103 with the first
// pass's bins (37 and 81 by the bitwise search and counting).
//
// Where the kk-th value's bin still holds many values (equal scores: each would be compared
// with all of them), that bin alone is binned again until the kk-th key is known, and the
// caller places the keys above it by counting and the equal ones in row order.  Half of the
// rows of one score: 8 requests of 100 to 1000 rows, 1600 candidates at kk = 100, 48 -> 20 us
// (34 by the bitwise search); 1000 of 4096 rows at kk = 512, 56 -> 48 (52).  All of one score,
// 3000 of 300 rows at kk = 8: 52 -> 15 (44).  NARROW off: one pass, for
// keys that are known to lie above a close bound (the loop costs 22 registers there).
//
// key(e), row(e): the thread's elements e = 0 .. PER - 1 (key(e) = 0: none).  kmin,
// kmax: bounds of the workgroup's keys, the same for every thread; keys below kmin are left
// out (at least kk are not).  hist (1024 words, zeroed, 16-byte aligned) and red (NT / 64
// + 3 words) are LDS scratch; sorted holds at least kk + BIN_MOST - 1 values.  The caller
// synchronises before (hist is zero).
// Returns false, with nothing written, when there is no kk-th value or its bin holds too
// many (more than BIN_MOST; with NARROW BIN_CLOSE: 64 and 256 take as long, 512 what the
// figures above say): the caller then selects another way, and knows that the kk-th key lies
// in [tlo, thi] (one key with NARROW, if there is one).
constexpr int NBINS = 1024;
constexpr int BIN_MOST = 512;
constexpr int BIN_FEW = 32;
constexpr int BIN_CLOSE = 128;
// Bins of one width over the keys kmin .. kmax, the largest keys first.
struct KeyBins {
  uint32_t kmax;
  int shift;
  __device__ __forceinline__ KeyBins(uint32_t kmin, uint32_t kmax_) : kmax(kmax_) {
    const uint32_t range = kmax_ - kmin;
    const int bits = range ? 32 - __builtin_clz(range) : 0;
    shift = bits > 10 ? bits - 10 : 0;
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t k) const { return (kmax - k) >> shift; }
  // the largest and the smallest key of bin b (the smallest: not below kmin)
  __device__ __forceinline__ uint32_t top(uint32_t b) const { return kmax - (b << shift); }
  __device__ __forceinline__ uint32_t bottom(uint32_t b, uint32_t kmin) const {
    const uint64_t past = (uint64_t(b) + 1) << shift;
    return past > uint64_t(kmax - kmin) ? kmin : kmax - uint32_t(past) + 1u;
  }
};
// One more value in bin b of hist.  The lanes that count into the first lane's bin (equal
// scores) do so at once: an LDS atomic takes its lanes' additions to one word one after the
// other.
__device__ __forceinline__ void count_in_bin(uint32_t* hist, uint32_t b) {
  const uint32_t b0 = uint32_t(__builtin_amdgcn_readfirstlane(int(b)));
  const uint64_t same = __builtin_amdgcn_ballot_w64(b == b0);
  const bool first = __builtin_amdgcn_mbcnt_hi(uint32_t(same >> 32),
                                               __builtin_amdgcn_mbcnt_lo(uint32_t(same), 0)) == 0;
  if (b != b0 || first) atomicAdd(&hist[b], b != b0 ? 1u : uint32_t(__popcll(same)));
}
// Whether many lanes of the wave hold the key of the lane before them.
__device__ __forceinline__ bool keys_repeat(uint32_t k) {
  const uint32_t prev = uint32_t(__builtin_amdgcn_update_dpp(0, int(k), 0x111, 0xf, 0xf, false));
  return __popcll(__builtin_amdgcn_ballot_w64(k == prev && k != 0u)) >= 8;
}
// hist (complete: the caller has synchronised) becomes its exclusive prefix; returns
// the bin that holds the need-th value (need >= 1) with `end` the values up to that
// bin's end and `cnt` its own, or ~0 if there are fewer.
// red: NT / 64 + 3 words.  Ends with a barrier.
template <int NT>
__device__ __forceinline__ uint32_t find_bin(uint32_t* hist, uint32_t* red, uint32_t need, int& end,
                                             int& cnt) {
  constexpr int NW = NT / WAVE, BPT = NBINS / NT;   // bins per thread
  const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
  static_assert(BPT == 4 || BPT == 2 || BPT == 1, "one vector of bins per thread");
  typedef uint32_t bins_t __attribute__((ext_vector_type(BPT)));
  const bins_t h = reinterpret_cast<const bins_t*>(hist)[tid];
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) sum += h[i];
  const uint32_t incl = wave_incl_sum(sum);
  if (lane == WAVE - 1) red[wid] = incl;
  if (tid == 0) red[NW + 1] = ~0u;
  __syncthreads();
  uint32_t at = incl - sum;
#pragma unroll
  for (int w = 0; w < NW; ++w) at += w < wid ? red[w] : 0u;
  bins_t start;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    start[i] = at;
    if (at < need && need <= at + h[i]) {
      red[NW] = at + h[i];
      red[NW + 1] = uint32_t(BPT * tid + i);
      red[NW + 2] = h[i];
    }
    at += h[i];
  }
  reinterpret_cast<bins_t*>(hist)[tid] = start;
  __syncthreads();
  end = int(red[NW]);
  cnt = int(red[NW + 2]);
  return red[NW + 1];
}
template <int NT, int PER, bool NARROW, class Key, class Row>
__device__ __forceinline__ bool place_by_bins(const Key& key, const Row& row, uint32_t kmin,
                                              uint32_t kmax, int kk, uint32_t* hist, uint32_t* red,
                                              uint64_t* sorted, int32_t* oi, float* os, uint32_t& tlo,
                                              uint32_t& thi) {
  kmin = max(kmin, 1u);
  kmax = max(kmax, kmin);
  KeyBins bin(kmin, kmax);
  // few different keys, or many equal ones (wave-uniform; looked for only where a thread has
  // many keys: with four, the look costs what the counting takes longer)
  if (bin.shift == 0 || (NARROW && PER >= 8 && keys_repeat(key(0)))) {
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (key(e) >= kmin) count_in_bin(hist, bin(key(e)));
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (key(e) >= kmin) atomicAdd(&hist[bin(key(e))], 1u);
  }
  __syncthreads();
  tlo = 0u;
  thi = ~0u;
  int total, cnt, was = 2 * NT * PER;
  uint32_t last = find_bin<NT>(hist, red, uint32_t(kk), total, cnt);
  if (last == ~0u) return false;
  tlo = bin.bottom(last, kmin);
  thi = bin.top(last);
  if constexpr (NARROW) {
    while (cnt > BIN_FEW && 2 * cnt <= was) {
      const KeyBins finer(tlo, kmax);
      if (finer.shift >= bin.shift) break;
      kmin = tlo;
      bin = finer;
      was = cnt;
      for (int b = threadIdx.x; b < NBINS; b += NT) hist[b] = 0u;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (key(e) >= kmin) count_in_bin(hist, bin(key(e)));
      __syncthreads();
      last = find_bin<NT>(hist, red, uint32_t(kk), total, cnt);
      tlo = bin.bottom(last, kmin);
      thi = bin.top(last);
    }
  }
  if constexpr (NARROW) {
    if (cnt > BIN_CLOSE) {   // the kk-th key by bins of its bin
      uint32_t need = uint32_t(kk - (total - cnt));
      while (tlo != thi) {
        const KeyBins within(tlo, thi);
        for (int b = threadIdx.x; b < NBINS; b += NT) hist[b] = 0u;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < PER; ++e)
          if (key(e) >= tlo && key(e) <= thi) count_in_bin(hist, within(key(e)));
        __syncthreads();
        int end, n;
        const uint32_t b = find_bin<NT>(hist, red, need, end, n);
        need -= uint32_t(end - n);
        tlo = within.bottom(b, tlo);
        thi = within.top(b);
      }
      return false;
    }
  } else {
    if (cnt > BIN_MOST) return false;
  }
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (key(e) >= kmin) {
      const uint32_t b = bin(key(e));
      if (b <= last) sorted[atomicAdd(&hist[b], 1u)] = sel_value(key(e), row(e));
    }
  __syncthreads();   // hist[b] is now the end of bin b <= last, and the start of the next
  for (int i = threadIdx.x; i < total; i += NT) {
    const uint64_t me = sorted[i];
    const uint32_t b = bin(sel_key(me));
    const int s0 = b ? int(hist[b - 1]) : 0, s1 = int(hist[b]);
    int rank = s0, j = s0;
    for (; j + 4 <= s1; j += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) rank += sorted[j + u] > me ? 1 : 0;
    for (; j < s1; ++j) rank += sorted[j] > me ? 1 : 0;
    if (rank < kk) {
      oi[rank] = sel_row(me);
      os[rank] = key_score(sel_key(me));
    }
  }
  return true;
}

// Workgroup-wide largest (and smallest) of a value; red: NT / 64 words each.  Ends
// with a barrier.
template <int NT>
__device__ __forceinline__ void block_min_max(uint32_t& lo, uint32_t& hi, uint32_t* red) {
  constexpr int NW = NT / WAVE;
  const int lane = threadIdx.x % WAVE, wid = threadIdx.x / WAVE;
  lo = wave_min_u(lo);
  hi = wave_max_u(hi);
  if (lane == 0) {
    red[wid] = lo;
    red[NW + wid] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    lo = min(lo, red[w]);
    hi = max(hi, red[NW + w]);
  }
}

}  // namespace tav2
