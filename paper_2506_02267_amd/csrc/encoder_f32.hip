// float32 encoder for small shapes (T <= 64, d_model <= 128, FFN <= 512, d <=
// 256): one workgroup per candidate runs Eq. 4's feature encoding, the causal
// post-LN layers and the linear + max-pool head (Sec. 3.2.2) on the fp32 matrix
// instructions.  Only the valid prefix of each candidate is computed: no valid
// position sees padding (under the causal mask, or in the unmasked mode, where a
// position sees the whole valid prefix).
//
// A wave owns a tile of 16 tokens from Eq. 4 to the head.  Products are taken
// transposed (weights as the A operand of 16x16x4 MFMAs): lane l then holds token
// l % 16 and features 16 f + 4 g + i (g = l / 16) in register i of accumulator f, and
// register s of accumulator f is, as it stands, the B operand of a step over the
// features 16 f + {s, 4 + s, 8 + s, 12 + s}.  The matching A operands of the four steps
// are the four floats W[row][16 f + 4 g ..], one 16-byte load per lane straight from the
// row-major matrix.  So activations stay in registers through every product, weights
// pass through neither LDS nor a barrier, and only K and V^T are shared between the
// waves (two barriers a layer).
//
// What bounds it: a candidate's chain of products on one SIMD per 16 tokens (32 cycles a
// step) and the latency of the weight stream, which is kept PF row tiles ahead, across
// the products' ends.  16 candidates of 32 positions (d_model 64, FFN 128, one layer):
// 27.5 us, where LDS-staged products on the vector units (a register tile per thread, two
// LDS reads a k step, a weight chunk's barriers) took 73; 1600 of 60 positions, two layers,
// 368 us (1545).
#include "common.h"
#include "internal.h"
#include "token_source.h"

#include <atomic>

namespace tav2 {
namespace f32e {

constexpr int MAX_LAYERS = 8;
constexpr int TT = 16;               // tokens per wave
constexpr int MAX_NW = F32_MAX_T / TT;
constexpr int LDS_MAX = 163840 - F32_MAX_T * int(sizeof(void*));   // of the accepted shapes

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mma(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct Args {
  TokenSource s;
  const float* cand;
  int d, dm, dh, H, ffn, n_layers;
  const float *W_in, *b_in, *E_act, *E_time, *E_pos, *W_pool, *b_pool;
  tav2_layer layers[MAX_LAYERS];
  float* out;
  int unmasked;   // 1: every valid position sees every valid position
  int ldv;        // row stride of V^T in LDS (floats): positions rounded up to 16, + 4
};

__host__ __device__ inline int round4(int x) { return (x + 3) / 4 * 4; }

// A matrix that a phase multiplies by: rows [0, rows) and columns [0, cols) of W (row
// stride ld), everything past them zero; cols and ld are multiples of 4, W is 16-byte
// aligned where the accepted shapes have it so (rows are whole 16-byte groups).
struct Mat {
  const float* W;
  int ld, rows, cols;
};
// Row tile r's operands over the DT k-tiles.
template <int DT>
__device__ __forceinline__ void load_rows(f32x4 (&a)[DT], const Mat& m, int r) {
  const int lane = threadIdx.x % WAVE, row = 16 * r + lane % 16, k0 = 4 * (lane / 16);
  const float* p = m.W + int64_t(row) * m.ld + k0;
#pragma unroll
  for (int f = 0; f < DT; ++f)
    a[f] = row < m.rows && 16 * f + k0 < m.cols ? *reinterpret_cast<const f32x4*>(p + 16 * f)
                                                : f32x4{0.f, 0.f, 0.f, 0.f};
}
// The weight stream: PF row tiles in flight.  A phase has DT row tiles; its last PF
// iterations load the first PF row tiles of the next phase.
template <int DT, int PF>
struct Ring {
  f32x4 a[PF][DT];
};
template <int DT, int PF>
__device__ __forceinline__ void prime(Ring<DT, PF>& q, const Mat& m) {
#pragma unroll
  for (int r = 0; r < PF; ++r) load_rows<DT>(q.a[r], m, r);
}
// acc[r] += (rows 16 r .. of cur) x; TOK: the other way round (lane holds feature 16 r +
// l % 16 of tokens 4 g + i).  The product is summed apart from acc, in two halves: added
// step by step onto the residual it would round at the residual's size every time
// (errors against 64 bits 3.3e-7 instead of 1.9e-7; the vector units' sums had 2.2e-7).
template <int DT, int PF, bool TOK = false>
__device__ __forceinline__ void phase(Ring<DT, PF>& q, f32x4 (&acc)[DT], const f32x4 (&x)[DT],
                                      const Mat& cur, const Mat& next) {
#pragma unroll
  for (int r = 0; r < DT; ++r) {
    // past the matrix a row tile is zero (skipped at widths of 100 to 124 only, 66 -> 62 us at
    // 100: elsewhere the branch costs what it saves, 26.6 -> 28.6 at 64)
    if (DT < 8 || 16 * r < cur.rows) {   // wave-uniform
      f32x4 part[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int f = 0; f < DT; ++f)
          part[f % 2] = TOK ? mma(x[f][s], q.a[r % PF][f][s], part[f % 2])
                            : mma(q.a[r % PF][f][s], x[f][s], part[f % 2]);
      acc[r] += part[0] + part[1];
    }
    load_rows<DT>(q.a[r % PF], r + PF < DT ? cur : next, r + PF < DT ? r + PF : r + PF - DT);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// v[4 f + i] of a feature vector for the lane's features (zero past dm).
template <int DT>
__device__ __forceinline__ void load_vec(f32x4 (&v)[DT], const float* p, int n) {
  const int k0 = 4 * (threadIdx.x % WAVE / 16);
#pragma unroll
  for (int f = 0; f < DT; ++f)
    v[f] = 16 * f + k0 < n ? *reinterpret_cast<const f32x4*>(p + 16 * f + k0) : f32x4{0.f, 0.f, 0.f, 0.f};
}
// The same of a side table's row: tables are float-aligned only (unlike the vectors and
// matrices); one 16-byte load all the same, which this GPU takes at any 4 bytes.
typedef float f32x4_4 __attribute__((ext_vector_type(4), aligned(4)));
template <int DT>
__device__ __forceinline__ void load_row(f32x4 (&v)[DT], const float* p, int n) {
  const int k0 = 4 * (threadIdx.x % WAVE / 16);
#pragma unroll
  for (int f = 0; f < DT; ++f) {
    v[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (16 * f + k0 < n) v[f] = *reinterpret_cast<const f32x4_4*>(p + 16 * f + k0);
  }
}
// x <- LayerNorm(x) over the dm features of the lane's token (padding features stay 0).
template <int DT>
__device__ __forceinline__ void layer_norm(f32x4 (&x)[DT], const f32x4 (&gain)[DT],
                                           const f32x4 (&off)[DT], int dm) {
  const int k0 = 4 * (threadIdx.x % WAVE / 16);
  const float inv = 1.f / float(dm);
  float s = 0.f;
#pragma unroll
  for (int f = 0; f < DT; ++f) s += (x[f][0] + x[f][1]) + (x[f][2] + x[f][3]);
  const float mu = xsum32(xsum16(s)) * inv;
  float v = 0.f;
#pragma unroll
  for (int f = 0; f < DT; ++f) {
    const bool in = 16 * f + k0 < dm;
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[f][i] = in ? x[f][i] - mu : 0.f;
      t = fmaf(x[f][i], x[f][i], t);
    }
    v += t;
  }
  const float rs = rsqrtf(xsum32(xsum16(v)) * inv + 1e-5f);
#pragma unroll
  for (int f = 0; f < DT; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[f][i] = x[f][i] * rs * gain[f][i] + off[f][i];
}

// DT: tiles of 16 features (d_model <= 16 DT); PF: row tiles of weights in flight.  Every
// product takes DT x DT tiles, so there is a kernel for each 32 features: us at one
// position and 16 candidates, with kernels for 64 and 128 only : so (one or two layers)
//   d_model 8: 32.2 : 14.0   16: 23.3 : 11.8   32: 21.7 : 11.5   68: 65.0 : 45.8   96: 78.5 : 49.6
template <int DT, int PF>
__global__ __launch_bounds__(MAX_NW* WAVE) void encode_f32_kernel(Args A) {
  constexpr int DP = 16 * DT, LDK = DP + 4;
  static_assert(DT % PF == 0, "whole rounds of the ring");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int64_t n = blockIdx.x;
  const int tid = threadIdx.x, w = tid / WAVE, lane = tid % WAVE, nw = blockDim.x / WAVE;
  const int c16 = lane % 16, g = lane / 16;
  const int dm = A.dm, d = A.d, dh = A.dh;
  const int Tv = token_valid_len(A.s, n);
  float* out = A.out + n * 2 * dm;
  if (Tv == 0) {
    for (int c = tid; c < 2 * dm; c += blockDim.x) out[c] = 0.f;
    return;
  }
  float* Ks = lds;                          // [16 nw][LDK]
  float* Vt = Ks + 16 * nw * LDK;           // [DP][ldv]
  float* pool = Vt + DP * A.ldv;            // [nw][DP]
  const int t0 = TT * w, p = t0 + c16;      // the wave's first position, the lane's
  const bool live = t0 < Tv;                // wave-uniform
  // token columns of W_in, then the candidate's, 16 DT at a time
  const int nc = (d + DP - 1) / DP;
  auto in_mat = [&](int c) {   // chunk c: of the token half, then of the candidate half
    const int k0 = (c < nc ? c : c - nc) * DP;
    return Mat{A.W_in + (c < nc ? 0 : d) + k0, 2 * d, dm, d - k0};
  };
  auto layer_mat = [&](const void* W, int row0, int rows, int cols, int ld, int k0) {
    return Mat{static_cast<const float*>(W) + int64_t(row0) * ld + k0, ld, rows, cols};
  };
  Ring<DT, PF> q;
  f32x4 x[DT];
  if (live) {
    prime(q, in_mat(0));
    TokenRef t{nullptr, 0, 0};
    if (p < Tv) t = resolve_token(A.s, n, p, d * 4);
    // ---- Eq. 4 with early fusion: [e_p ; e_c] W_in^T + b_in + side tables
    f32x4 ta[DT], tp[DT];
    load_vec<DT>(x, A.b_in, dm);
    load_row<DT>(ta, A.E_act + t.act * dm, dm);
    load_row<DT>(tp, A.E_pos + (p < Tv ? p : Tv - 1) * dm, dm);
#pragma unroll
    for (int f = 0; f < DT; ++f) x[f] += ta[f] + tp[f];
    if (A.E_time) {
      load_row<DT>(ta, A.E_time + t.time * dm, dm);
#pragma unroll
      for (int f = 0; f < DT; ++f) x[f] += ta[f];
    }
    const float* cv = A.cand + n * d;
    for (int c = 0; c < 2 * nc; ++c) {
      const int k0 = (c < nc ? c : c - nc) * DP;
      const float* src = c < nc ? reinterpret_cast<const float*>(t.emb) : cv;
      f32x4 e[DT];
#pragma unroll
      for (int f = 0; f < DT; ++f)
        e[f] = src && k0 + 16 * f + 4 * g < d
                   ? *reinterpret_cast<const f32x4*>(src + k0 + 16 * f + 4 * g)
                   : f32x4{0.f, 0.f, 0.f, 0.f};
      phase(q, x, e, in_mat(c),
            c + 1 < 2 * nc ? in_mat(c + 1) : layer_mat(A.layers[0].W_qkv, 0, dm, dm, dm, 0));
    }
  }

  const float scale = 1.f / sqrtf(float(dh));
  for (int li = 0; li < A.n_layers; ++li) {
    const tav2_layer& L = A.layers[li];
    f32x4 qv[DT];
    if (li) __syncthreads();   // every wave is past its reads of K and V^T
    if (live) {
      // ---- Q in registers, K and V^T into LDS
      load_vec<DT>(qv, L.b_qkv, dm);
      phase(q, qv, x, layer_mat(L.W_qkv, 0, dm, dm, dm, 0), layer_mat(L.W_qkv, dm, dm, dm, dm, 0));
      {
        f32x4 k[DT];
        load_vec<DT>(k, L.b_qkv + dm, dm);
        phase(q, k, x, layer_mat(L.W_qkv, dm, dm, dm, dm, 0),
              layer_mat(L.W_qkv, 2 * dm, dm, dm, dm, 0));
#pragma unroll
        for (int f = 0; f < DT; ++f)
          *reinterpret_cast<f32x4*>(Ks + p * LDK + 16 * f + 4 * g) = k[f];
      }
      {
        f32x4 v[DT];
        load_vec<DT>(v, L.b_qkv + 2 * dm, dm);
        phase(q, v, x, layer_mat(L.W_qkv, 2 * dm, dm, dm, dm, 0), layer_mat(L.W_o, 0, dm, dm, dm, 0));
#pragma unroll
        for (int f = 0; f < DT; ++f)
#pragma unroll
          for (int i = 0; i < 4; ++i) Vt[(16 * f + 4 * g + i) * A.ldv + p] = v[f][i];
      }
    }
    __syncthreads();
    if (!live) continue;
    // ---- attention, one head at a time: S^T = K Q^T (keys 16 t + 4 g + i of query c16)
    f32x4 o[DT];
#pragma unroll
    for (int f = 0; f < DT; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nt = A.unmasked ? (Tv + 15) / 16 : w + 1;   // key tiles
    const int lim = A.unmasked ? Tv : p + 1;              // keys the lane's query sees
    for (int h = 0; h < A.H; ++h) {
      const int h0 = h * dh, h1 = h0 + dh;   // heads begin and end at a multiple of 4
      f32x4 s[MAX_NW];
      float mx = -__builtin_inff();
#pragma unroll
      for (int t = 0; t < MAX_NW; ++t) {
        s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (t < nt) {   // wave-uniform
#pragma unroll
          for (int f = 0; f < DT; ++f)
            if (16 * f < h1 && 16 * f + 16 > h0) {   // uniform: the tile meets the head
              const int k0 = 16 * f + 4 * g;
              const bool in = k0 >= h0 && k0 < h1;
              // other heads' features are zero on both sides: an infinite key times a query of 0
              // would reach this head's scores.  (1600 of 60 positions at d_model 64: 364 -> 368 us
              // for the keys' part; a row of zeros to read instead 373, a branch for whole tiles 374.)
              const f32x4 a = *reinterpret_cast<const f32x4*>(Ks + (16 * t + c16) * LDK + k0);
#pragma unroll
              for (int u = 0; u < 4; ++u) s[t] = mma(in ? a[u] : 0.f, in ? qv[f][u] : 0.f, s[t]);
            }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[t][i] = 16 * t + 4 * g + i < lim ? s[t][i] * scale : -__builtin_inff();
            mx = vmax(mx, s[t][i]);
          }
        }
      }
      mx = xmax32(xmax16(mx));   // finite: key 0 is valid for every valid query
      float l = 0.f;
#pragma unroll
      for (int t = 0; t < MAX_NW; ++t)
        if (t < nt) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[t][i] = s[t][i] == -__builtin_inff() ? 0.f : expf(s[t][i] - mx);
            l += s[t][i];
          }
        }
      l = xsum32(xsum16(l));
#pragma unroll
      for (int f = 0; f < DT; ++f)
        if (16 * f < h1 && 16 * f + 16 > h0) {
          f32x4 oh = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int t = 0; t < MAX_NW; ++t)
            if (t < nt) {
              const f32x4 a = *reinterpret_cast<const f32x4*>(Vt + (16 * f + c16) * A.ldv + 16 * t + 4 * g);
#pragma unroll
              for (int u = 0; u < 4; ++u) oh = mma(a[u], s[t][u], oh);
            }
          const int k0 = 16 * f + 4 * g;
          if (k0 >= h0 && k0 < h1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[f][i] = oh[i] / l;
          }
        }
    }
    // ---- x = LayerNorm 1(x + o W_o^T + b_o)
    {
      f32x4 b[DT], gn[DT];
      load_vec<DT>(b, L.b_o, dm);
      load_vec<DT>(gn, L.ln1_g, dm);
#pragma unroll
      for (int f = 0; f < DT; ++f) x[f] += b[f];
      load_vec<DT>(b, L.ln1_b, dm);
      phase(q, x, o, layer_mat(L.W_o, 0, dm, dm, dm, 0), layer_mat(L.W_1, 0, A.ffn, dm, dm, 0));
      layer_norm<DT>(x, gn, b, dm);
    }
    // ---- x = LayerNorm 2(x + ReLU(x W_1^T + b_1) W_2^T + b_2), 16 DT hidden units at a time
    {
      f32x4 y[DT], gn[DT], b[DT];
      load_vec<DT>(y, L.b_2, dm);
      load_vec<DT>(gn, L.ln2_g, dm);
      load_vec<DT>(b, L.ln2_b, dm);
#pragma unroll
      for (int f = 0; f < DT; ++f) y[f] += x[f];
      for (int c0 = 0; c0 < A.ffn; c0 += DP) {
        const int left = A.ffn - c0;
        f32x4 hd[DT];
        load_vec<DT>(hd, L.b_1 + c0, left);
        const Mat w1 = layer_mat(L.W_1, c0, left, dm, dm, 0), w2 = layer_mat(L.W_2, 0, dm, left, A.ffn, c0);
        phase(q, hd, x, w1, w2);
#pragma unroll
        for (int f = 0; f < DT; ++f)
#pragma unroll
          for (int i = 0; i < 4; ++i) hd[f][i] = fmaxf(hd[f][i], 0.f);
        phase(q, y, hd, w2,
              left > DP ? layer_mat(L.W_1, c0 + DP, left - DP, dm, dm, 0)
                        : li + 1 < A.n_layers ? layer_mat(A.layers[li + 1].W_qkv, 0, dm, dm, dm, 0)
                                              : Mat{A.W_pool, dm, dm, dm});
      }
      layer_norm<DT>(y, gn, b, dm);
#pragma unroll
      for (int f = 0; f < DT; ++f) x[f] = y[f];
    }
  }

  // ---- head: max over valid rows of X W_pool^T + b_pool; X of the last row
  if (live) {
    const Mat wp{A.W_pool, dm, dm, dm};
    f32x4 y[DT];
#pragma unroll
    for (int f = 0; f < DT; ++f) y[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    phase<DT, PF, true>(q, y, x, wp, wp);
#pragma unroll
    for (int f = 0; f < DT; ++f) {   // lane holds feature 16 f + c16 of tokens 4 g + i
      float m = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (t0 + 4 * g + i < Tv) m = vmax(m, y[f][i]);
      m = xmax32(xmax16(m));
      if (g == 0) pool[w * DP + 16 * f + c16] = m;
    }
    if (p == Tv - 1) {
#pragma unroll
      for (int f = 0; f < DT; ++f)
        if (16 * f + 4 * g < dm) *reinterpret_cast<f32x4*>(out + dm + 16 * f + 4 * g) = x[f];
    }
  }
  __syncthreads();
  const int nl = (Tv + TT - 1) / TT;   // waves with tokens
  for (int c = tid; c < dm; c += blockDim.x) {
    float m = pool[c];
    for (int v = 1; v < nl; ++v) m = vmax(m, pool[v * DP + c]);
    out[c] = m + A.b_pool[c];
  }
}

// LDS floats of the LDS-staged form of this encoder, which sets the shapes accepted
// (the kernel needs less; what it accepts is part of the interface).
int shape_floats(int T, int d, int dm) {
  constexpr int FC = 128, WS_LD = 132, NW = 4;
  const int rows = round4(T), ldk = T % 2 ? T + 2 : T + 1;
  int region = rows * (2 * dm + 4);
  region = region > rows * (d + 4) ? region : rows * (d + 4);
  region = region > rows * (FC + 4) ? region : rows * (FC + 4);
  const int off = round4(rows * (dm + 4)) + round4(region) + round4(dm * ldk) +
                  round4(rows * (round4(T) + 4)) + round4(dm) + round4(NW * dm) + 2 * F32_MAX_T;
  return off + 16 * WS_LD;
}

}  // namespace f32e

bool encode_f32_fits(int T, const tav2_weights& w) {
  if (T < 1 || T > F32_MAX_T || w.d_model > F32_MAX_DM || w.d_ffn > F32_MAX_FFN) return false;
  if (w.n_layers > f32e::MAX_LAYERS) return false;
  // every product's k and row strides in whole 16-byte groups
  if (w.d_model % 4 || (w.d_model / w.n_heads) % 4 || w.d_ffn % 4) return false;
  return f32e::shape_floats(T, w.d_in, w.d_model) * 4 <= f32e::LDS_MAX;
}

hipError_t launch_encode_f32(const TokenSource& src, const void* cand_emb, int64_t total,
                             const tav2_weights& w, float* out, bool unmasked, hipStream_t st) {
  if (total == 0) return hipSuccess;
  f32e::Args a{};
  a.s = src;
  a.cand = static_cast<const float*>(cand_emb);
  a.d = src.d;
  a.dm = w.d_model;
  a.H = w.n_heads;
  a.dh = w.d_model / w.n_heads;
  a.ffn = w.d_ffn;
  a.n_layers = w.n_layers;
  a.W_in = static_cast<const float*>(w.W_in);
  a.b_in = w.b_in;
  a.E_act = static_cast<const float*>(w.E_act);
  a.E_time = static_cast<const float*>(w.E_time);
  a.E_pos = static_cast<const float*>(w.E_pos);
  a.W_pool = static_cast<const float*>(w.W_pool);
  a.b_pool = w.b_pool;
  for (int i = 0; i < w.n_layers; ++i) a.layers[i] = w.layers[i];
  a.out = out;
  a.unmasked = unmasked ? 1 : 0;
  const int nw = (src.T + f32e::TT - 1) / f32e::TT;
  a.ldv = 16 * nw + 4;
  const int which = (w.d_model - 1) / 32;   // 32 (which + 1) features
  const int dp = 32 * (which + 1);
  const size_t lds = size_t(16 * nw * (dp + 4) + dp * a.ldv + nw * dp) * 4;
  const size_t lds_max = size_t(64 * (128 + 4) + 128 * 68 + 4 * 128) * 4;
  void (*const kernels[4])(f32e::Args) = {f32e::encode_f32_kernel<2, 2>, f32e::encode_f32_kernel<4, 4>,
                                          f32e::encode_f32_kernel<6, 2>, f32e::encode_f32_kernel<8, 2>};
  void (*const kernel)(f32e::Args) = kernels[which];
  static std::atomic<bool> done[64][4] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !done[dev][which].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_max));
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) done[dev][which].store(true, std::memory_order_release);
  }
  ProfScope prof("encode_f32", st);
  hipLaunchKernelGGL(kernel, dim3(unsigned(total)), dim3(unsigned(nw * WAVE)), lds, st, a);
  return hipGetLastError();
}

}  // namespace tav2
