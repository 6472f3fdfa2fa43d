// NN search of Eq. 3 for narrow rows and few candidates in one kernel: a workgroup
// scores every row of the request for one candidate and keeps the products in registers,
// so there is no sample, no threshold, no survivor list in memory and no fallback launch.
//
// A thread loads whole rows (row NT j + thread).  Products: 32x32x16 MFMAs with the
// candidate in every row of the A operand; the lower lanes' rows are one tile of 32, the
// upper lanes' the other.  The operands and the k order are the other search kernels',
// and so are the scores' bits.
//
// Selection: every thread's rows fall into four groups, the groups' largest estimates
// are binned, and the bin that holds the k-th largest of them bounds the k-th key from
// below, closely (k = 256 of 16384 rows: about 300 rows reach it).  The rows that reach
// it get their exact score and are placed by bins.  Where a bin or the list overflows
// (many equal scores), the k-th key is found bit by bit below the bits that are settled
// and the equal rows go straight to their places (2000 int8 rows of d 32, a third or all of
// one score, 256 candidates: 9.9 and 8.2 us; 27 and 30 with all 32 bits searched and the
// selected rows counted; 16.5 by the launches that this kernel takes the place of).
//
// What bounds it: launch, first loads and selection are 6 to 8 us; each 1024 rows add
// about 1 us: every workgroup reads all rows from L2 and turns codes into bf16.
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "select_common.h"

namespace tav2 {
namespace sr {

struct Args {
  const void* emb;
  const int64_t* seq_off;
  const int32_t* seq_len;
  const bf16_t* cand;
  const int64_t* cand_off;
  int max_len, k, out_ld;
  int32_t* out_idx;
  float* out_score;
  int32_t* cand_req;
};
constexpr int NT = 1024;
constexpr int GROUPS = 4;    // groups of a thread's rows
constexpr int LIST = 2048;   // rows that may be among the k best, at most
static_assert(NBINS == NT && GROUPS * NT >= TAV2_K_MAX, "one bin per thread; enough groups");

// Eight codes as bf16: at most 8 significant bits, so the upper half of the float is exact.
__device__ __forceinline__ bf16x8 codes(uint32_t x, uint32_t y) {
  uint32_t p[4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const uint32_t w = j < 4 ? x : y;
    const uint32_t a = __float_as_uint(float(int8_t((w >> (8 * (j & 3))) & 0xFF)));
    const uint32_t b = __float_as_uint(float(int8_t((w >> (8 * (j & 3) + 8)) & 0xFF)));
    p[j / 2] = __builtin_amdgcn_perm(b, a, 0x07060302u);
  }
  return as_bf16x8(make_uint4(p[0], p[1], p[2], p[3]));
}

// The kk best of the workgroup's keys (key[j]: row j NT + thread, 0: none), the kk-th of
// which lies in [tlo, thi] and is found bit by bit below the bits these have in common:
// every key above it, placed by counting, then the lowest rows equal to it, in row order.
// cnt: RPT x NT / 64 words, red: 2 x NT / 64; sel: kk values.
template <int NT, int RPT>
__device__ __forceinline__ void place_by_bits(const uint32_t (&key)[RPT], int kk, uint32_t tlo,
                                              uint32_t thi, uint32_t* cnt, uint32_t* red,
                                              uint32_t* above, uint64_t* sel, int32_t* oi, float* os) {
  constexpr int NW = NT / WAVE;
  const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
  const int top = tlo == thi ? -1 : 31 - __builtin_clz(tlo ^ thi);
  uint32_t t = top < 0 ? tlo : top == 31 ? 0u : tlo & ~((2u << top) - 1u);
  __syncthreads();   // cnt, red, sel, above: nothing of them is read any more
  if (tid == 0) *above = 0u;
  for (int b = top; b >= 0; --b) {
    const uint32_t probe = t | (1u << b);
    int c = 0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) c += __popcll(__builtin_amdgcn_ballot_w64(key[j] >= probe));
    uint32_t* half = red + (b & 1) * NW;   // (the other half may still be read)
    if (lane == 0) half[wid] = uint32_t(c);
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) all += int(half[w]);
    if (all >= kk) t = probe;
  }
  // rows are ordered by (j, wave, lane): the equal keys are counted per j and wave
  uint64_t eq[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    eq[j] = __builtin_amdgcn_ballot_w64(key[j] == t);
    if (lane == 0) cnt[j * NW + wid] = uint32_t(__popcll(eq[j]));
  }
  __syncthreads();   // (*above is zero as well)
#pragma unroll
  for (int j = 0; j < RPT; ++j)
    if (key[j] > t) sel[atomicAdd(above, 1u)] = sel_value(key[j], j * NT + tid);
  uint32_t before[RPT];   // equal keys before the wave's of j: one count per lane
  {
    constexpr int N = RPT * NW, PER = (N + WAVE - 1) / WAVE;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      v[i] = PER * lane + i < N ? cnt[PER * lane + i] : 0u;
      sum += v[i];
    }
    uint32_t at = wave_incl_sum(sum) - sum;
    uint32_t ex[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      ex[i] = at;
      at += v[i];
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const int e = j * NW + wid;   // wave-uniform
      before[j] = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (e % PER == i) before[j] = uint32_t(__builtin_amdgcn_readlane(int(ex[i]), e / PER));
    }
  }
  __syncthreads();
  const int gt = int(*above);
  const float score = key_score(t);
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int pos = gt + int(before[j] + __builtin_amdgcn_mbcnt_hi(uint32_t(eq[j] >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo(uint32_t(eq[j]), 0)));
    if (key[j] == t && pos < kk) {
      oi[pos] = j * NT + tid;
      os[pos] = score;
    }
  }
  place_by_rank<NT>(sel, gt, oi, os);
}

// A row's score from its product (and, for codes, its sum of squares ss > 0): exact, and
// the estimate through the hardware reciprocal square root.  The two have the same sign and
// keys at most SLACK apart (relative error below 2^-21); a product that is not a number is
// its own score in both.  An all-zero row scores 0 whatever the candidate (its product may
// be 0 x inf): it enters as product 0 and ss 1.
constexpr uint32_t SLACK = 64;
template <bool I8>
__device__ __forceinline__ uint32_t exact_key(float dot, float ss) {
  return score_key(I8 && dot == dot ? i8_score(dot, ss) : dot);
}
template <bool I8>
__device__ __forceinline__ uint32_t estimate_key(float dot, float ss) {
  return score_key(I8 ? dot * __builtin_amdgcn_rsqf(ss) : dot);
}

// NT threads, RPT rows per thread (the rows fit NT x RPT), d = 16 KB.
template <bool I8, int KB, int RPT>
__global__ __launch_bounds__(NT) void select_resident_kernel(Args A) {
  __shared__ __attribute__((aligned(16))) uint64_t sorted[TAV2_K_MAX + BIN_MOST];
  __shared__ float list_dot[LIST], list_ss[LIST];
  __shared__ uint16_t list_row[LIST];
  __shared__ __attribute__((aligned(16))) uint32_t hist[NBINS];
  __shared__ uint32_t red[2 * NT / WAVE + 2];
  __shared__ uint32_t listed;
  const int r = blockIdx.y;
  const int64_t n = A.cand_off[r] + int64_t(blockIdx.x);
  if (n >= A.cand_off[r + 1]) return;
  const int tid = threadIdx.x, lane = tid % WAVE, hf = lane / 32;
  if (A.cand_req && tid == 0) A.cand_req[n] = r;   // the candidate's request, for the encoder
  const int L = max(0, min(A.seq_len[r], A.max_len));
  const int k = A.k, kk = k < L ? k : L;
  int32_t* oi = A.out_idx + n * A.out_ld;
  float* os = A.out_score + n * A.out_ld;
  for (int p = kk + tid; p < k; p += NT) {
    oi[p] = -1;
    os[p] = -__builtin_inff();
  }
  if (kk == 0) return;
  constexpr int d = 16 * KB;
  bf16x8 cf[KB];   // the candidate, in every row of the A operand
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
    cf[kb] = as_bf16x8(*reinterpret_cast<const uint4*>(A.cand + n * d + 16 * kb + 8 * hf));
  constexpr int ROW = I8 ? d : 2 * d;   // bytes
  constexpr int AHEAD = RPT < 16 ? 128 / ROW : 2;   // (16 rows: 128 registers)
  const uint8_t* emb = static_cast<const uint8_t*>(A.emb) + A.seq_off[r] * ROW;
  uint4 raw[AHEAD][ROW / 16];   // the lane's row NT j + tid, j modulo AHEAD
  auto load = [&](int j) {
    const uint8_t* p = emb + min(NT * j + tid, L - 1) * ROW;   // clamped; not kept
#pragma unroll
    for (int i = 0; i < ROW / 16; ++i) raw[j % AHEAD][i] = reinterpret_cast<const uint4*>(p)[i];
  };
#pragma unroll
  for (int j = 0; j < AHEAD; ++j) load(j);
  hist[tid] = 0u;
  if (tid == 0) listed = 0u;
  float dot[RPT], ss[RPT];   // of row NT j + thread
  uint32_t gm[GROUPS] = {};   // the largest estimates of rows j modulo GROUPS
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    ss[j] = 1.f;
    bool norm = true;
    f32x16 acc[2] = {f32x16{}, f32x16{}};
    uint32_t x[ROW / 4];
#pragma unroll
    for (int i = 0; i < ROW / 16; ++i) {
      const uint4 q = raw[j % AHEAD][i];
      x[4 * i] = q.x;
      x[4 * i + 1] = q.y;
      x[4 * i + 2] = q.z;
      x[4 * i + 3] = q.w;
    }
    if (j + AHEAD < RPT) load(j + AHEAD);
    if constexpr (I8) {
      int sq = 0;
#pragma unroll
      for (int i = 0; i < ROW / 4; ++i) sq = __builtin_amdgcn_sdot4(int(x[i]), int(x[i]), sq, false);
      ss[j] = float(max(sq, 1));
      norm = sq > 0;
    }
    // the lower lanes hold tile 0's rows, the upper tile 1's: words of k and k + 8
    // change places across the halves and become the two tiles' operands
    constexpr int H = I8 ? 2 : 4;   // words of 8 k
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      uint32_t t0[4], t1[4];
#pragma unroll
      for (int i = 0; i < H; ++i) {
        const auto y = __builtin_amdgcn_permlane32_swap(x[2 * H * kb + i], x[2 * H * kb + H + i], false, false);
        t0[i] = y[0];
        t1[i] = y[1];
      }
      if constexpr (I8) {
        acc[0] = mfma32(cf[kb], codes(t0[0], t0[1]), acc[0]);
        acc[1] = mfma32(cf[kb], codes(t1[0], t1[1]), acc[1]);
      } else {
        acc[0] = mfma32(cf[kb], as_bf16x8(make_uint4(t0[0], t0[1], t0[2], t0[3])), acc[0]);
        acc[1] = mfma32(cf[kb], as_bf16x8(make_uint4(t1[0], t1[1], t1[2], t1[3])), acc[1]);
      }
    }
    dot[j] = norm ? (hf ? acc[1][0] : acc[0][0]) : 0.f;
    gm[j % GROUPS] = max(gm[j % GROUPS], NT * j + tid < L ? estimate_key<I8>(dot[j], ss[j]) : 0u);
  }
  uint32_t lo = ~0u, hi = 0u;
#pragma unroll
  for (int q = 0; q < GROUPS; ++q)
    if (gm[q]) {
      lo = min(lo, gm[q]);
      hi = max(hi, gm[q]);
    }
  block_min_max<NT>(lo, hi, red);
  const KeyBins gbin(lo, hi);
#pragma unroll
  for (int q = 0; q < GROUPS; ++q)
    if (gm[q]) count_in_bin(hist, gbin(gm[q]));
  __syncthreads();
  int end, cnt;
  const uint32_t last = find_bin<NT>(hist, red, uint32_t(kk), end, cnt);
  // kk estimates reach the smallest key of that bin (min(L, GROUPS x NT) >= kk groups
  // have a row), so the kk-th exact key is at most SLACK below it, and the estimates of
  // the kk best rows 2 SLACK
  const uint64_t span = ((uint64_t(last) + 1) << gbin.shift) + 2 * SLACK;
  const uint32_t least = span >= uint64_t(hi) ? 1u : hi - uint32_t(span) + 1u;
  hist[tid] = 0u;
  // the rows whose estimate reaches it
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < RPT; ++j)
    m |= uint32_t(NT * j + tid < L && estimate_key<I8>(dot[j], ss[j]) >= least) << j;
  const uint32_t mine = uint32_t(__popc(m)), incl = wave_incl_sum(mine);
  uint32_t at = 0;
  if (lane == WAVE - 1) at = atomicAdd(&listed, incl);
  at = uint32_t(__builtin_amdgcn_readlane(int(at), WAVE - 1)) + incl - mine;
#pragma unroll
  for (int j = 0; j < RPT; ++j)
    if ((m >> j) & 1u) {
      if (at < uint32_t(LIST)) {
        list_dot[at] = dot[j];
        list_ss[at] = ss[j];
        list_row[at] = uint16_t(NT * j + tid);
      }
      ++at;
    }
  __syncthreads();
  const uint32_t total = listed;
  const uint32_t kmin = least > SLACK ? least - SLACK : 1u;   // of the kk best rows' exact keys
  const uint32_t kmax = hi < ~0u - SLACK ? hi + SLACK : ~0u;
  uint32_t tlo = kmin, thi = kmax;
  bool placed = false;
  if (total <= uint32_t(LIST)) {
    uint32_t key[LIST / NT];
    int row[LIST / NT];
#pragma unroll
    for (int e = 0; e < LIST / NT; ++e) {
      const uint32_t i = uint32_t(NT * e + tid);
      key[e] = 0u;
      row[e] = 0;
      if (i < total) {
        key[e] = exact_key<I8>(list_dot[i], list_ss[i]);
        row[e] = list_row[i];
      }
    }
    placed = place_by_bins<NT, LIST / NT, true>([&](int e) { return key[e]; }, [&](int e) { return row[e]; },
                                                kmin, kmax, kk, hist, red, sorted, oi, os, tlo, thi);
  }
  if (!placed) {
    uint32_t key[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      key[j] = NT * j + tid < L ? max(exact_key<I8>(dot[j], ss[j]), 1u) : 0u;
    place_by_bits<NT, RPT>(key, kk, tlo, thi, hist, red, &listed, sorted, oi, os);
  }
}

}  // namespace sr

// One workgroup per CU, or two where the registers of two fit (up to 64: int8 of d 32 at two
// rows a thread, bf16 at four).
// us, this kernel : the launches it takes the place of; k 128, k 1000 at 8192 rows:
//   candidates, d   rows 200     2000          4000          8192          16384
//   8,   32 int8    7.1 : 8.9    7.0 : 10.2    9.1 : 11.8    13.6 : 29.7   19.6 : 24.5
//   16,  32 int8    7.1 : 8.9    7.0 : 10.0    9.1 : 11.8    13.6 : 33.1   19.9 : 25.0
//   256, 32 int8    7.3 : 9.3    7.4 : 11.0    9.7 : 13.1    15.2 : 42.3   22.3 : 28.0
//   8,   32 bf16    6.4 : 7.6    7.1 : 8.9     9.3 : 10.3    14.2 : 33.2
//   256, 32 bf16    6.7 : 8.3    7.5 : 9.9     10.0 : 12.1   15.3 : 49.3
//   8,   64 int8    8.2 : 9.1    8.4 : 10.6    11.7 : 12.2   18.4 : 30.6
//   256, 64 int8    8.8 : 9.7    8.9 : 11.3    12.9 : 13.5   21.1 : 44.2
//   500, 32 int8                 10.7 : 12.7   (17.4 : 15.7)
//   500, 32 bf16                 (13.0 : 11.7) (14.7 : 14.8)
// Those in brackets are not taken; nor are rows above 64 bytes (256 of d 64 bf16: 21.3 us
// at 4000 rows against 17.5 then) and more than 512 KB a request (256 of d 64 int8 at 16384
// rows: 39.8 against 30.1).
bool select_resident_applies(const tav2_seq& s, const tav2_cands& c) {
  if (s.dtype != TAV2_BF16 && s.dtype != TAV2_I8) return false;
  if (s.d != 32 && s.d != 64) return false;
  const int row = s.dtype == TAV2_I8 ? s.d : 2 * s.d;   // bytes
  if (row > 64 || int64_t(s.max_len) * row > 512 * 1024) return false;
  return c.total <= 256 ||
         (c.total <= 512 && s.dtype == TAV2_I8 && s.d == 32 && s.max_len <= 2 * sr::NT);
}

hipError_t launch_select_resident(const tav2_seq& seq, const tav2_cands& c, int k, int32_t* out_idx,
                                  float* out_score, int out_ld, int32_t* cand_req, hipStream_t st) {
  if (seq.num_requests == 0 || c.total == 0) return hipSuccess;
  sr::Args A{};
  A.emb = seq.emb;
  A.seq_off = seq.offset;
  A.seq_len = seq.len;
  A.cand = static_cast<const bf16_t*>(c.emb);
  A.cand_off = c.offset;
  A.max_len = seq.max_len;
  A.k = k;
  A.out_ld = out_ld;
  A.out_idx = out_idx;
  A.out_score = out_score;
  A.cand_req = cand_req;
  const bool i8 = seq.dtype == TAV2_I8;
  const dim3 grid(unsigned(c.max_count), unsigned(seq.num_requests));
  ProfScope prof("nn_resident", st);
#define SR_LAUNCH(I8, KB)                                                                        \
  (seq.max_len <= 2 * sr::NT   ? sr::select_resident_kernel<I8, KB, 2><<<grid, sr::NT, 0, st>>>(A) \
   : seq.max_len <= 4 * sr::NT ? sr::select_resident_kernel<I8, KB, 4><<<grid, sr::NT, 0, st>>>(A) \
                               : sr::select_resident_kernel<I8, KB, 8><<<grid, sr::NT, 0, st>>>(A))
  if (!i8) SR_LAUNCH(false, 2);
  else if (seq.d == 64) SR_LAUNCH(true, 4);
  else if (seq.max_len <= 8 * sr::NT) SR_LAUNCH(true, 2);
  else sr::select_resident_kernel<true, 2, 16><<<grid, sr::NT, 0, st>>>(A);
#undef SR_LAUNCH
  return hipGetLastError();
}

}  // namespace tav2
