// Single-kernel encoder for the paper's production encoder shape: d_model 64,
// one or two heads, a narrow FFN, a few layers (Sec. 3.2.2 'Transformer
// Encoder'; the fused transformer of Sec. 3.4.2 keeps every transformer weight
// on chip next to the activations).  One workgroup runs Eq. 4's feature
// encoding, every causal post-LN layer and the linear + max-pool head for its
// candidates, with all layer weights resident in LDS.
//
// Layout of the work:
//  * A wave owns one tile of 16 tokens and keeps it in registers from Eq. 4 to
//    the head.  The fp32 residual stream is X^T in 16x16x32 MFMA accumulator
//    layout: lane l holds token l % 16 and 4 features per accumulator f
//    (feat4; g = l / 16).
//  * Products are taken transposed (weights as the A operand), and the rows of each
//    pair of 16-row weight tiles are dealt so (feature_row) that a lane's accumulators
//    of the pair are 8 consecutive features: rounded to bf16 they are the next
//    product's B operand as they stand, so X, Q, P, O and the FFN's hidden units never
//    pass through LDS.  The weights are held as operand fragments (16 rows x 32
//    columns = 1 KB, lane-major: conflict-free 16-byte reads, no padding).
//  * Only K and V^T are shared: each wave writes its 16 keys as fragments (4 KB),
//    32 keys (a pair of tiles) per 8 KB; two workgroup barriers a layer.
//  * A candidate of T <= 192 positions has ceil(T / 16) waves, so that all its
//    tokens run at once; one workgroup takes several short candidates when there
//    are more of them than CUs.  Longer candidates go through blocks of up to 12
//    waves (192 positions, of about one size) in turn: under the causal mask a block
//    depends on earlier ones only through their keys and values, which each block
//    leaves in a per-workgroup cache in global memory, in the same form; later blocks
//    stage them through the LDS of their own keys, half of it at a time.
//  * The workgroup is persistent: it loads the weights once and then takes
//    candidates in turn.
//
// What bounds it: one candidate is two layers of short dependent products, far below
// the matrix rate, so what counts is how many waves a SIMD can switch between, how
// few instructions a step has, and the start (arguments, lengths, token metadata and
// rows one after the other, the weights' 64 KB for the first layer next to them).
// Phase stamps at 192 positions (12 waves, 45,000 cycles in all): start 11,500; per
// layer Q / K / V 3,000, attention 1,400 (first tile) to 7,500 (last tile: seven key
// pairs), W_o + LayerNorm 1,100, FFN + LayerNorm 1,600; head 1,500.  256 candidates of 192
// positions: 21.4 us (37.8 us with 4 waves per candidate taking blocks of 64 positions
// in turn and activations passed through LDS), of 64: 12.9 us (15.2), of 256: 36.2 us
// (49.4); 200 of 300 to 1024: 175 us (318); 2000 of 192: 120 us (255); 2000 of 13 to 26:
// 23.1 us (77.9): back-to-back calls on explicit tokens, by events.  More waves (16 of at
// most 128 registers) spill: 64 us at 192 positions.  More than 128 positions a block when there are several (192 against
// 128): 173 us against 197 at 1024 positions, 565 against 665 at 2048.
#include <algorithm>
#include <atomic>

#include "common.h"
#include "internal.h"
#include "token_source.h"

namespace tav2 {
namespace sm {

constexpr int DM = 64;          // d_model
constexpr int TT = 16;          // tokens per wave
constexpr int MAX_NW = 12;      // waves per workgroup at most
constexpr int MAX_LAYERS = 4;
constexpr int MAX_DK = 8;       // token width d <= 256: at most 8 k-steps of 32 (kernels for 1, 2, 4, 8)
// From so many k-steps on, the waves share the candidates' projections (W_in's candidate
// half from memory, once a candidate) instead of each taking the product for its tile.  us,
// each product of its own : shared; one layer, FFN 32, candidates x positions:
//   d     2000 x 8     256 x 64    256 x 192   2000 x 192  300 x 1000
//   128   12.8 : 15.9              16.6 : 15.7  102 : 99    246 : 214
//   256   27.0 : 22.0  14.2 : 13.5 48.0 : 20.3  336 : 129   572 : 284  (no room for either half)
// At d 96 and 128 many short candidates would pay for the rest.
constexpr int COOP_DK = 5;
constexpr int GROUP_NW = 8;     // waves of candidates side by side at most
constexpr int FRAG = 1024;      // bytes of a 16 x 32 operand fragment
constexpr int RLD = DM + 8;           // row stride (bf16) of the packed matrices over d_model
constexpr int TABLD = DM * 2 + 16;    // bytes between the side tables' rows (their bank conflicts)
constexpr int TAB_BYTES = (72 * TABLD + FRAG - 1) / FRAG * FRAG;
constexpr int PAIR = 8 * FRAG;  // K and V^T of 32 keys: 2 x 2 K fragments, then 4 of V^T

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// The thread index through an empty asm: what is derived from it is computed where
// it is used instead of being hoisted out of the candidate, block and layer loops
// (which would keep it in registers across the whole kernel).
__device__ __forceinline__ unsigned otid() {
  unsigned t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
// Keeps the loads above it ahead of the products below it: left alone, the compiler
// saves registers by reading each LDS operand right before its product, and a wave
// then waits out the LDS latency at every one.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
// 16x16x32 operands: A[16 x 32] lane l: row l % 16, 8 k-rows 8 (l / 16) .. +7;
// B[32 x 16] lane l: column l % 16, same k-rows; D[16 x 16] lane l: column l % 16,
// rows 4 (l / 16) + i in register i.
__device__ __forceinline__ bf16x8 frag(const void* p) {
  return as_bf16x8(*reinterpret_cast<const uint4*>(p));
}
// The accumulator pair of 32 consecutive rows as the next product's operand.
__device__ __forceinline__ bf16x8 pack8(const f32x4& a, const f32x4& b) {
  return __builtin_bit_cast(bf16x8, u32x4{pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]),
                                          pack2(b[2], b[3])});
}
// Matrix row that row r of weight tile f holds: tiles 2 j and 2 j + 1 share 32 rows,
// in groups of 8 whose first four go to the first tile.  Lane group g's accumulators
// (rows 4 g + i) of the two tiles are then rows 32 j + 8 g .. + 7.
__host__ __device__ constexpr int feature_row(int f, int r) {
  return 32 * (f / 2) + 8 * (r / 4) + 4 * (f % 2) + r % 4;
}
// First of the four features that lane group g holds in accumulator f.
__device__ __forceinline__ int feat4(int f, int g) { return 32 * (f / 2) + 8 * g + 4 * (f % 2); }

struct LayerW {   // offsets (bytes) of one layer's weights
  int qkv, o, w1, w2, vec;
};
struct Args {
  TokenSource s;
  const bf16_t* cand;        // [total, d]
  const bf16_t* W_in;        // [DM, 2 d]
  const float* b_in;
  const bf16_t* E_act;       // [8, DM]
  const bf16_t* E_time;      // [64, DM] or null
  const bf16_t* E_pos;       // [max_pos, DM]
  const bf16_t* W_pool;      // [DM, DM]
  const float* b_pool;
  tav2_layer layers[MAX_LAYERS];
  const uint8_t* packed;     // the layers' weights as tav2_pack_weights wrote them, or null
  int n_layers, d, dh, ffn;
  int64_t total;
  int nwc;                   // waves (16-token tiles) per candidate
  int groups;                // candidates a workgroup takes at a time
  int npair;                 // K / V^T pairs per candidate in LDS
  int cache_pairs;           // pairs per layer in the cache of earlier blocks
  uint8_t* cache;            // [grid][layers][cache_pairs][PAIR], or null (one block)
  float* out;                // [total, 2 DM]
  LayerW pk[MAX_LAYERS];     // offsets in the packed weights
  int packed_bytes;
  // LDS layout (bytes): the side tables, b_in and the layers' vectors, the layers'
  // matrices, the candidates' projections (where shared), W_in's token half and candidate
  // half and W_pool (each < 0: no room, read from memory), K / V^T (then the pooled maxima)
  LayerW lw[MAX_LAYERS];
  int tab, bias, cvec, win_t, win_c, pool_w, kv;
  int tab16;                 // the side tables are 16-byte aligned
  int unmasked;
};

// Offsets of the layer vectors inside lw.vec (floats).
constexpr int V_BQKV = 0, V_BO = 3 * DM, V_LN1G = 4 * DM, V_LN1B = 5 * DM, V_B1 = 6 * DM;
__host__ __device__ constexpr int v_b2(int ffn) { return 6 * DM + ffn; }
__host__ __device__ constexpr int v_ln2g(int ffn) { return 7 * DM + ffn; }
__host__ __device__ constexpr int v_ln2b(int ffn) { return 8 * DM + ffn; }

// What tav2_pack_weights writes: every layer matrix as fragments in the order LDS
// holds them, its vectors, and the token half of W_in as fragments, each in a slot of
// the size of rows padded by 8 columns.
__host__ inline void plan_packed(Args& a) {
  int off = 0;
  auto take = [&](int bytes) {
    const int at = off;
    off += (bytes + 15) / 16 * 16;
    return at;
  };
  for (int l = 0; l < a.n_layers; ++l) {
    a.pk[l].qkv = take(3 * DM * RLD * 2);
    a.pk[l].o = take(DM * RLD * 2);
    a.pk[l].w1 = take(a.ffn * RLD * 2);
    a.pk[l].w2 = take(DM * (a.ffn + 8) * 2);
    a.pk[l].vec = take((9 * DM + a.ffn) * 4);
  }
  take(DM * (a.d + 8) * 2);
  a.packed_bytes = off;
}
// The LDS layout up to K / V^T; returns its size.  `room`: the bytes it may take.  W_in's
// token half, its candidate half and W_pool are held while there is room, in this order
// (every wave reads each of them once for every tile: with all three or none, 2000
// candidates of 192 positions took 171 us at two layers and d 64, and 335 at one and d
// 256; now 137 and 129).
// Matrices as fragments (row tile f, k-block kb) at (f * nkb + kb) * FRAG; W_in and
// W_2, whose k-blocks are taken one by one, at (kb * 4 + f) * FRAG.
__host__ inline int plan_lds(Args& a, int room) {
  int off = 0;
  auto take = [&](int bytes) {
    const int at = off;
    off += (bytes + 15) / 16 * 16;
    return at;
  };
  const bool coop = a.d / 32 >= COOP_DK;
  a.tab = take(TAB_BYTES);
  a.bias = off;
  off += DM * 4;
  for (int l = 0; l < a.n_layers; ++l) a.lw[l].vec = take((9 * DM + a.ffn) * 4);
  off = a.bias + (off - a.bias + FRAG - 1) / FRAG * FRAG;
  for (int l = 0; l < a.n_layers; ++l) {
    a.lw[l].qkv = take(3 * DM * DM * 2);
    a.lw[l].o = take(DM * DM * 2);
    a.lw[l].w1 = take(a.ffn * DM * 2);
    a.lw[l].w2 = take(DM * a.ffn * 2);
  }
  a.cvec = coop ? take(GROUP_NW * DM * 4) : -1;
  auto held = [&](int bytes) { return off + bytes <= room ? take(bytes) : -1; };
  a.win_t = held(a.d * DM * 2);
  a.win_c = coop ? -1 : held(a.d * DM * 2);
  a.pool_w = held(DM * DM * 2);
  a.kv = off;
  return off;
}

// The kernel's arguments through an empty asm, for the same reason (they are many
// more than the scalar registers hold; scalar loads bring them where they are used).
__device__ __forceinline__ const Args& oargs() {
  auto* p = (const __attribute__((address_space(4))) Args*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Args*)p;
}

// Waits for the wave's vector memory loads, LDS-DMA included.
__device__ __forceinline__ void wait_vm_all() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0); expcnt and lgkmcnt unconstrained
}

// One matrix's fragments into LDS by LDS-DMA, asynchronously, 1 KB per wave
// instruction: share `i` of `n` (on return: of the next matrix).  Workgroups start at
// different places of it, so that they do not all ask the same L2 channel for the
// same line at once.  The caller waits (wait_vm_all in every wave that loads, then a
// workgroup barrier) before the first LDS read.
// ld: bytes of a row, or 0 where src holds the fragments in LDS order.  Whole
// fragments come 2.5 times as fast (21 against 8 bytes per cycle and CU) as the 64-byte
// pieces of 16 rows.
__device__ __forceinline__ void dma_matrix(uint8_t* dst, const uint8_t* src, int ld, int nf, int nkb,
                                           bool kb_major, bool plain_rows, int& i, int n) {
  const int lane = threadIdx.x % WAVE, np = nf * nkb;
  int e = int((blockIdx.x / 8 * 5 + unsigned(i)) % unsigned(np));
  for (; i < np; i += n) {
    int at = e * FRAG + lane * 16;
    if (ld) {
      const int f = kb_major ? e % nf : e / nkb, kb = kb_major ? e / nf : e % nkb;
      const int row = plain_rows ? 16 * f + lane % 16 : feature_row(f, lane % 16);
      at = row * ld + kb * 64 + lane / 16 * 16;
    }
    __builtin_amdgcn_global_load_lds(src + at, dst + e * FRAG, 16, 0, 0);
    e += n;
    if (e >= np) e -= np;
  }
  i -= np;
}
// The matrices of layers [from, to), with W_in before layer 0 and W_pool after the
// last layer, where LDS holds them.
__device__ __forceinline__ void dma_layers(const Args& A, uint8_t* smem, int from, int to, int i,
                                           int n) {
  const int ffn = A.ffn;
  const bool p = A.packed != nullptr;
  if (from == 0) {
    const uint8_t* w = reinterpret_cast<const uint8_t*>(A.W_in);
    if (A.win_t >= 0)
      dma_matrix(smem + A.win_t, p ? A.packed + A.packed_bytes - DM * (A.d + 8) * 2 : w, p ? 0 : 4 * A.d,
                 4, A.d / 32, true, false, i, n);
    if (A.win_c >= 0) dma_matrix(smem + A.win_c, w + 2 * A.d, 4 * A.d, 4, A.d / 32, true, false, i, n);
  }
  for (int l = from; l < to; ++l) {
    const tav2_layer& L = A.layers[l];
    const LayerW lw = A.lw[l], pk = A.pk[l];
    auto src = [&](const void* m, int at) { return p ? A.packed + at : static_cast<const uint8_t*>(m); };
    const int ld = p ? 0 : DM * 2;
    dma_matrix(smem + lw.qkv, src(L.W_qkv, pk.qkv), ld, 12, 2, false, false, i, n);
    dma_matrix(smem + lw.o, src(L.W_o, pk.o), ld, 4, 2, false, false, i, n);
    dma_matrix(smem + lw.w1, src(L.W_1, pk.w1), ld, ffn / 16, 2, false, false, i, n);
    dma_matrix(smem + lw.w2, src(L.W_2, pk.w2), p ? 0 : ffn * 2, 4, ffn / 32, true, false, i, n);
  }
  if (to == A.n_layers && A.pool_w >= 0)
    dma_matrix(smem + A.pool_w, reinterpret_cast<const uint8_t*>(A.W_pool), DM * 2, 4, 2, false, true, i, n);
}
// 16-byte piece e of the side tables' LDS form (rows at stride TABLD; the padding
// repeats a row's last piece) and of [b_in | the layers' vectors].
__device__ __forceinline__ const uint8_t* table_piece(const Args& A, int e) {
  constexpr int PER = TABLD / 16;
  int r = e / PER, c = e - r * PER;
  c = c < DM / 8 ? c : DM / 8 - 1;
  const int last = A.E_time ? 71 : 7;
  r = r < last ? r : last;
  const bf16_t* p = r < 8 ? A.E_act + r * DM : A.E_time + (r - 8) * DM;
  return reinterpret_cast<const uint8_t*>(p + c * 8);
}
__device__ __forceinline__ int vector_pieces(const Args& A) {
  return DM / 4 + A.n_layers * (9 * DM + A.ffn) / 4;
}
__device__ __forceinline__ const uint8_t* vector_piece(const Args& A, int e) {
  const int n = vector_pieces(A);
  e = e < n ? e : n - 1;
  if (e < DM / 4) return reinterpret_cast<const uint8_t*>(A.b_in) + e * 16;
  e -= DM / 4;
  const int per = (9 * DM + A.ffn) / 4, l = e / per, r = e - l * per;
  if (A.packed) return A.packed + A.pk[l].vec + r * 16;
  const tav2_layer& L = A.layers[l];
  const int f4 = A.ffn / 4;
  const float* p;
  if (r < 48) p = L.b_qkv + 4 * r;
  else if (r < 64) p = L.b_o + 4 * (r - 48);
  else if (r < 80) p = L.ln1_g + 4 * (r - 64);
  else if (r < 96) p = L.ln1_b + 4 * (r - 80);
  else if (r < 96 + f4) p = L.b_1 + 4 * (r - 96);
  else if (r < 112 + f4) p = L.b_2 + 4 * (r - 96 - f4);
  else if (r < 128 + f4) p = L.ln2_g + 4 * (r - 112 - f4);
  else p = L.ln2_b + 4 * (r - 128 - f4);
  return reinterpret_cast<const uint8_t*>(p);
}
// Both into LDS by LDS-DMA, share i of n (their LDS regions are whole KB).
__device__ __forceinline__ void dma_vectors(const Args& A, uint8_t* smem, int& i, int n) {
  const int lane = threadIdx.x % WAVE, nt = A.tab16 ? TAB_BYTES / FRAG : 0;
  const int nv = (vector_pieces(A) + 63) / 64;
  for (; i < nt + nv; i += n) {
    if (i < nt)
      __builtin_amdgcn_global_load_lds(table_piece(A, i * 64 + lane), smem + A.tab + i * FRAG, 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(vector_piece(A, (i - nt) * 64 + lane),
                                       smem + A.bias + (i - nt) * FRAG, 16, 0, 0);
  }
  i -= nt + nv;
}
// The side tables when they are only 8-byte aligned: through registers, every thread.
__device__ __forceinline__ void copy_tables(const Args& A, uint8_t* smem) {
  for (int e = threadIdx.x; e < TAB_BYTES / 16; e += blockDim.x) {
    const uint2* p = reinterpret_cast<const uint2*>(table_piece(A, e));
    const uint2 lo = p[0], hi = p[1];
    *reinterpret_cast<uint4*>(smem + A.tab + e * 16) = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
}
// Fragment (row tile f) of k-block kb of W_in from the matrix (kb >= d / 32: its candidate
// half).
__device__ __forceinline__ bf16x8 win_frag(const Args& A, int kb, int f) {
  const int lane = otid() % WAVE;
  return frag(A.W_in + (feature_row(f, lane % 16) * 2 * A.d + 32 * kb + 8 * (lane / 16)));
}
// Four fragments (row tiles f) of k-block kb of the half of W_in that LDS holds at `at`
// (matrix k-block kb0 + kb), or of row tile pair h of W_pool (two tiles x two k-blocks): from
// LDS, or (at < 0) from the matrix.
__device__ __forceinline__ void win_frags(bf16x8 (&wf)[4], const Args& A, const uint8_t* smem, int at,
                                          int kb0, int kb) {
  const int lane = otid() % WAVE;
  if (at >= 0) {
#pragma unroll
    for (int f = 0; f < 4; ++f) wf[f] = frag(smem + at + (kb * 4 + f) * FRAG + lane * 16);
  } else {
#pragma unroll
    for (int f = 0; f < 4; ++f) wf[f] = win_frag(A, kb0 + kb, f);
  }
}
__device__ __forceinline__ void pool_frags(bf16x8 (&wf)[4], const Args& A, const uint8_t* smem, int h) {
  const int lane = otid() % WAVE;
  if (A.pool_w >= 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) wf[e] = frag(smem + A.pool_w + (4 * h + e) * FRAG + lane * 16);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      wf[e] = frag(A.W_pool + ((16 * (2 * h + e / 2) + lane % 16) * DM + 32 * (e % 2) + 8 * (lane / 16)));
  }
}

// ---------------------------------------------------------------- LayerNorm
// x[f] holds X^T of the lane's token: features feat4(f, g) + i.  Normalises over
// the 64 features (two passes: mean, then the centred squares).
__device__ __forceinline__ void layer_norm(f32x4 (&x)[4], const float* gain, const float* off) {
  const int grp = otid() % WAVE / 16;
  f32x4 gg[4], bb[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    gg[f] = *reinterpret_cast<const f32x4*>(gain + feat4(f, grp));
    bb[f] = *reinterpret_cast<const f32x4*>(off + feat4(f, grp));
  }
  fence();
  float s = 0.f;
#pragma unroll
  for (int f = 0; f < 4; ++f) s += (x[f][0] + x[f][1]) + (x[f][2] + x[f][3]);
  s = xsum32(xsum16(s));
  const float mean = s * (1.f / DM);
  float q[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[f][i] -= mean;
      q[f] = fmaf(x[f][i], x[f][i], q[f]);
    }
  const float v = xsum32(xsum16((q[0] + q[1]) + (q[2] + q[3])));
  const float rstd = rsqrtf(v * (1.f / DM) + 1e-5f);
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[f][i] = fmaf(x[f][i] * rstd, gg[f][i], bb[f][i]);
}
// The 4 bf16 of r added to v.
__device__ __forceinline__ void add4(f32x4& v, uint2 r) {
  v[0] += __uint_as_float(r.x << 16);
  v[1] += __uint_as_float(r.x & 0xFFFF0000u);
  v[2] += __uint_as_float(r.y << 16);
  v[3] += __uint_as_float(r.y & 0xFFFF0000u);
}

// ------------------------------------------------------------ token inputs
// One lane's token for Eq. 4: its embedding fragments (k-steps of 32; zeros for a
// padding position), its position's row, and its rows of the other side tables
// (which are in LDS).
template <int NK>
struct TokLoad {
  bf16x8 e[NK];
  uint2 ep[4];
  int act, time;
};
__device__ __forceinline__ TokenRef lane_token(const Args& A, int64_t n, int p, int Tv) {
  TokenRef t{nullptr, 0, 0};
  if (p < Tv) t = resolve_token(A.s, n, p, A.s.codes ? A.d : A.d * 2);
  return t;
}
// 8 int8 codes as bf16 (exact: |q| <= 127).
__device__ __forceinline__ bf16x8 codes8(uint2 raw) {
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    v[j] = static_cast<__bf16>(float(int8_t(((j < 4 ? raw.x : raw.y) >> (8 * (j & 3))) & 0xFF)));
  return v;
}
template <int NK>
__device__ __forceinline__ void load_token(TokLoad<NK>& L, int64_t n, int p, int Tv, const Args& A,
                                           int nk) {
  const int g = (otid() % WAVE) / 16;
  const int pc = p < Tv ? p : Tv - 1;   // padding: any position's row will do
#pragma unroll
  for (int f = 0; f < 4; ++f)
    L.ep[f] = *reinterpret_cast<const uint2*>(A.E_pos + (pc * DM + feat4(f, g)));
  const TokenRef t = lane_token(A, n, p, Tv);
  L.act = t.act;
  L.time = t.time;
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    L.e[k] = bf16x8{};
    if (t.emb && k < nk) {
      if (A.s.codes)   // int8 codes: dequantised after the product (Eq. 4 in the kernel)
        L.e[k] = codes8(*reinterpret_cast<const uint2*>(t.emb + 32 * k + 8 * g));
      else
        L.e[k] = frag(reinterpret_cast<const bf16_t*>(t.emb) + 32 * k + 8 * g);
    }
  }
}
// The candidate's half of Eq. 4, W_in[:, d:] c, into cv[feature]: the features of row tile
// f (every column of the product is the same).
template <int NK>
__device__ __forceinline__ void project_candidate(float* cv, const bf16_t* cand, const Args& A, int nk,
                                                  int f) {
  const int lane = otid() % WAVE, g = lane / 16;
  bf16x8 wf[NK], cf[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k)
    if (k < nk) {
      wf[k] = win_frag(A, nk + k, f);
      cf[k] = frag(cand + 32 * k + 8 * g);
    }
  f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < NK; ++k)
    if (k < nk) a = mma(wf[k], cf[k], a);
  if (lane % 16 == 0) *reinterpret_cast<f32x4*>(cv + feat4(f, g)) = a;
}
// x = X0^T of the wave's 16 tokens (Eq. 4): W_in [e ; c] + b_in + side tables.  The
// candidate (cf) enters as a product with the same column for every token (for
// int8 codes after the token product is scaled by the 0.65 / 127 of their
// quantisation, Sec. 3.2.1), or as its projection cv.
template <int NK>
__device__ __forceinline__ void encode_input(f32x4 (&x)[4], const TokLoad<NK>& tl,
                                             const bf16x8 (&cf)[NK], const float* cv,
                                             const Args& A, const uint8_t* smem, int nk) {
  const int g = otid() % WAVE / 16;
#pragma unroll
  for (int f = 0; f < 4; ++f) x[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < NK; ++k)
    if (k < nk) {
      bf16x8 wf[4];
      win_frags(wf, A, smem, A.win_t, 0, k);
      if (NK > 2) fence();
#pragma unroll
      for (int f = 0; f < 4; ++f) x[f] = mma(wf[f], tl.e[k], x[f]);
    }
  if (A.s.codes) {
#pragma unroll
    for (int f = 0; f < 4; ++f) x[f] *= 0.65f / 127.f;
  }
  if constexpr (NK >= COOP_DK) {
#pragma unroll
    for (int f = 0; f < 4; ++f) x[f] += *reinterpret_cast<const f32x4*>(cv + feat4(f, g));
  } else {
#pragma unroll
    for (int k = 0; k < NK; ++k)
      if (k < nk) {
        bf16x8 wf[4];
        win_frags(wf, A, smem, A.win_c, nk, k);
        if (NK > 2) fence();
#pragma unroll
        for (int f = 0; f < 4; ++f) x[f] = mma(wf[f], cf[k], x[f]);
      }
  }
  const float* bias = reinterpret_cast<const float*>(smem + A.bias);
  const uint8_t* ta = smem + A.tab + tl.act * TABLD;
  const uint8_t* tt = smem + A.tab + (8 + tl.time) * TABLD;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    f32x4 v = *reinterpret_cast<const f32x4*>(bias + feat4(f, g));
    add4(v, *reinterpret_cast<const uint2*>(ta + 2 * feat4(f, g)));
    add4(v, tl.ep[f]);
    if (A.E_time) add4(v, *reinterpret_cast<const uint2*>(tt + 2 * feat4(f, g)));
    x[f] += v;
  }
}

// ---------------------------------------------------------------- attention
// Online softmax state of one 16-query tile and head (queries in lane columns).
template <int DH>
struct Att {
  bf16x8 qf[DH / 32];   // Q^T fragments
  f32x4 o[DH / 16];     // O^T accumulators
  float m, l;           // reference of the exponents (log2 units), this lane's partial row sum
};
// A pair of 32 keys at kv (fragments), head h: the K operands, S^T = K Q^T (one query
// per lane column; key 16 t + 4 g + i in s[t][i]), and the V^T operands.
template <int DH>
__device__ __forceinline__ void load_k(bf16x8 (&k)[2][DH / 32], const uint8_t* kv, int h) {
  const uint8_t* p = kv + (DH == 64 ? 0 : h * FRAG) + otid() % WAVE * 16;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int kb = 0; kb < DH / 32; ++kb) k[t][kb] = frag(p + t * 2 * FRAG + kb * FRAG);
}
template <int DH>
__device__ __forceinline__ void load_v(bf16x8 (&v)[DH / 16], const uint8_t* kv, int h) {
  const uint8_t* p = kv + (4 + h * (DH / 16)) * FRAG + otid() % WAVE * 16;
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt) v[dt] = frag(p + dt * FRAG);
}
template <int DH>
__device__ __forceinline__ void scores(f32x4 (&s)[2], const bf16x8 (&k)[2][DH / 32], const Att<DH>& st) {
#pragma unroll
  for (int t = 0; t < 2; ++t) s[t] = mma(k[t][0], st.qf[0], f32x4{0.f, 0.f, 0.f, 0.f});
  if constexpr (DH == 64) {
#pragma unroll
    for (int t = 0; t < 2; ++t) s[t] = mma(k[t][DH / 32 - 1], st.qf[DH / 32 - 1], s[t]);
  }
}
// Key j of the pair is visible to the lane's query iff j < lim.
__device__ __forceinline__ void mask_scores(f32x4 (&s)[2], int lim) {
  const int g = otid() % WAVE / 16;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (16 * t + 4 * g + i >= lim) s[t][i] = -__builtin_inff();
}
// The pair's weights and its share of O and of the row sums.  The reference of the
// exponents is raised to the maximum, and the sums rescaled, only where a score has
// grown past it by more than RAISE (then P stays below 2^RAISE, and its bf16
// rounding and the 32-bit sums keep their relative precision).  It starts below every
// score and is finite: keys whose scores are -inf get weight 0 also before the first
// other one (-inf as the reference would make them not a number).  exp2 is the
// hardware instruction (results below 2^-126 flush to zero, far under the bf16
// resolution of P).
constexpr float RAISE = 6.f;
constexpr float NO_KEY = -3e38f;
template <int DH>
__device__ __forceinline__ void add_pair(Att<DH>& st, const f32x4 (&s)[2], const bf16x8 (&v)[DH / 16]) {
  constexpr float sc = (DH == 64 ? 0.125f : 0.17677669529663688f) * 1.4426950408889634f;
  const float mx = vmax(vmax(vmax(s[0][0], s[0][1]), vmax(s[0][2], s[0][3])),
                        vmax(vmax(s[1][0], s[1][1]), vmax(s[1][2], s[1][3])));
  if (__builtin_amdgcn_ballot_w64(mx * sc > st.m + RAISE)) {
    const float mnew = vmax(st.m, xmax32(xmax16(mx)) * sc);
    const float alpha = __builtin_amdgcn_exp2f(st.m - mnew);
    st.m = mnew;
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) st.o[dt] *= alpha;
  }
  f32x4 e[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) e[t][i] = __builtin_amdgcn_exp2f(fmaf(s[t][i], sc, -st.m));
  // the row sums are those of the exponentials in fp32, before P is rounded
  st.l += ((e[0][0] + e[0][1]) + (e[0][2] + e[0][3])) + ((e[1][0] + e[1][1]) + (e[1][2] + e[1][3]));
  const bf16x8 pb = pack8(e[0], e[1]);
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt) st.o[dt] = mma(v[dt], pb, st.o[dt]);
}
// Pairs `first` (if >= 0; masked by lim) and then 0 .. np - 1 (every key visible),
// each pair's scores taken while the pair before it is added.
template <int DH>
__device__ __forceinline__ void att_pairs(Att<DH>& st, const uint8_t* kv, int h, int first, int lim,
                                          int np) {
  bf16x8 k[2][DH / 32];
  f32x4 s[2];
  const uint8_t* cur = first >= 0 ? kv + first * PAIR : kv;
  const uint8_t* end = kv + np * PAIR;
  const uint8_t* nxt = first >= 0 ? kv : kv + PAIR;
  load_k<DH>(k, cur, h);
  scores<DH>(s, k, st);
  if (first >= 0) mask_scores(s, lim);
  while (true) {
    bf16x8 v[DH / 16];
    f32x4 n[2];
    const bool more = nxt < end;
    load_k<DH>(k, more ? nxt : cur, h);
    load_v<DH>(v, cur, h);
    fence();
    scores<DH>(n, k, st);
    add_pair<DH>(st, s, v);
    if (!more) break;
    s[0] = n[0];
    s[1] = n[1];
    cur = nxt;
    nxt += PAIR;
  }
}

// ---------------------------------------------------------------- the kernel
// NK: k-steps of 32 token features the kernel is built for (d / 32 <= NK).
// NW: waves per workgroup at most (what a wave's registers are set by).  MULTI: the
// candidates may have more than one block.
template <int NK, int DH, int NW, bool MULTI>
__global__ __launch_bounds__(NW* WAVE) void encoder_small_kernel(Args A) {
  constexpr int NH = DM / DH;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid % WAVE;
  const int w = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int c16 = lane % 16, g = lane / 16;
  const int ffn = A.ffn, nk = A.d / 32;
  // waves past the candidates' tiles only help to load weights (and join the barriers)
  const int ntok = A.groups * A.nwc;
  const bool loader = w >= ntok;
  const int grp = loader ? 0 : w / A.nwc;
  // this wave's tile: waves go to the SIMDs in turn, so the tiles of every second
  // four are taken in reverse, which evens out the SIMDs' causal work
  int tile = w - grp * A.nwc;
  if ((tile & 4) && (tile | 3) < A.nwc) tile ^= 3;
  const int BT = A.nwc * TT;
  uint8_t* KV = smem + A.kv + grp * A.npair * PAIR;
  float* pool = reinterpret_cast<float*>(smem + A.kv);
  uint8_t* cache = A.cache ? A.cache + int64_t(blockIdx.x) * A.n_layers * A.cache_pairs * PAIR : nullptr;
  // The weights come in two parts: up to the first layer's (every wave asks for its
  // share, awaited before the first candidate's input), and the rest, asked for after
  // the second barrier of the first layer and awaited at the next one, by the spare
  // waves, or else by the first four tiles' waves, whose attention is the shortest.
  const bool spare = ntok < int(blockDim.x) / WAVE;
  int loaded = 0;   // 1: the first part, 2: the rest is on its way, 3: all of it
  {
    int i = w;
    const int nl = int(blockDim.x) / WAVE;
    dma_vectors(oargs(), smem, i, nl);
    dma_layers(oargs(), smem, 0, 1, i, nl);
  }

  for (int64_t n0 = int64_t(blockIdx.x) * A.groups; n0 < A.total; n0 += int64_t(gridDim.x) * A.groups) {
    const int64_t n = n0 + grp;
    const int Tv = n < A.total ? token_valid_len(oargs().s, n) : 0;
    float* out = A.out + n * 2 * DM;
    if (Tv == 0 && n < A.total && !loader)
      for (int c = tile * WAVE + lane; c < 2 * DM; c += A.nwc * WAVE) out[c] = 0.f;
    // blocks of the candidate; several candidates side by side are one block each
    const int nblk = MULTI ? (Tv + BT - 1) / BT : A.groups > 1 || Tv > 0 ? 1 : 0;
    // running max of X W_pool^T over the wave's valid tokens: lane holds features 16 f + c16
    float pmax[4] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
    for (int blk = 0; blk < nblk; ++blk) {
      const int p0 = blk * BT;
      const int t0 = p0 + TT * tile;      // the wave's first position
      const bool live = !loader && t0 < Tv;   // wave-uniform
      const bool odd_end = (tile & 1) == 0 && t0 + TT >= Tv;   // no wave writes the pair's other half
      const bool keep = MULTI && blk + 1 < nblk;   // later blocks read this one's K / V^T
      const int p = t0 + c16;             // this lane's token
      f32x4 x[4];
      {
        TokLoad<NK> tl;
        bf16x8 cf[NK];
        float* cv = reinterpret_cast<float*>(smem + A.cvec);
        if (NK >= COOP_DK && blk == 0)   // every wave takes its share of the row tiles
          for (int t = w; t < 4 * A.groups && n0 + t / 4 < A.total; t += int(blockDim.x) / WAVE)
            project_candidate<NK>(cv + t / 4 * DM, A.cand + (n0 + t / 4) * A.d, oargs(), nk, t % 4);
        if (live) {
          if (NK < COOP_DK) {
            const bf16_t* cr = A.cand + n * A.d + 8 * g;
#pragma unroll
            for (int k = 0; k < NK; ++k)
              if (k < nk) cf[k] = frag(cr + 32 * k);
          }
          load_token(tl, n, p, Tv, oargs(), nk);
        }
        if (loaded == 0) {
          if (!A.tab16) copy_tables(oargs(), smem);
          wait_vm_all();
          __syncthreads();
          loaded = A.n_layers > 1 ? 1 : 3;
        } else if (NK >= COOP_DK && blk == 0) {
          __syncthreads();   // cv is complete (read last before the previous candidate's layers)
        }
        if (live) encode_input(x, tl, cf, cv + grp * DM, oargs(), smem, nk);
      }
      for (int li = 0; li < A.n_layers; ++li) {
        const int lane = otid() % WAVE, c16 = lane % 16, g = lane / 16;
        const LayerW lw = oargs().lw[li];
        const uint8_t* Wqkv = smem + lw.qkv + lane * 16;
        const uint8_t* Wo = smem + lw.o + lane * 16;
        const uint8_t* W1 = smem + lw.w1 + lane * 16;
        const uint8_t* W2 = smem + lw.w2 + lane * 16;
        const float* vec = reinterpret_cast<const float*>(smem + lw.vec);
        uint8_t* lc = cache ? cache + int64_t(li) * A.cache_pairs * PAIR : nullptr;
        if (loaded == 2) {
          wait_vm_all();
          loaded = 3;
        }
        __syncthreads();   // every wave is past its reads of the previous K / V^T
        Att<DH> st[NH];
        if (live) {
          const bf16x8 xf[2] = {pack8(x[0], x[1]), pack8(x[2], x[3])};
          uint8_t* kv = KV + (tile >> 1) * PAIR + lane * 16;
          uint8_t* ks = kv + (tile & 1) * 2 * FRAG;
          // row tiles 0..3: Q, 4..7: K (transposed), 8..11: V (untransposed: X as the
          // A operand; lane holds dim feature_row(f, c16), keys 4 g + i), two at a time, their
          // fragments read LOOK tiles ahead
          constexpr int LOOK = NW > 8 ? 2 : 4;
          bf16x8 wf[12][2];
          f32x4 acc[12];
          auto fetch = [&](int i) {
            wf[i][0] = frag(Wqkv + 2 * i * FRAG);
            wf[i][1] = frag(Wqkv + (2 * i + 1) * FRAG);
            if (i < 8) {
              acc[i] = *reinterpret_cast<const f32x4*>(vec + V_BQKV + 64 * (i / 4) + feat4(i % 4, g));
            } else {
              const float bv = vec[V_BQKV + 2 * DM + feature_row(i % 4, c16)];
              acc[i] = f32x4{bv, bv, bv, bv};
            }
          };
#pragma unroll
          for (int i = 0; i < LOOK; ++i) fetch(i);
          fence();
#pragma unroll
          for (int i = 0; i < 12; i += 2) {
            if (i + LOOK < 12) {
              fetch(i + LOOK);
              fetch(i + LOOK + 1);
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int u = i; u < i + 2; ++u)
                acc[u] = u < 8 ? mma(wf[u][kb], xf[kb], acc[u]) : mma(xf[kb], wf[u][kb], acc[u]);
            if (i < 4) {
              if constexpr (DH == 64)
                st[0].qf[i / 2] = pack8(acc[i], acc[i + 1]);
              else
                st[i / 2].qf[0] = pack8(acc[i], acc[i + 1]);
            } else if (i < 8) {
              *reinterpret_cast<uint4*>(ks + (i / 2 - 2) * FRAG) =
                  __builtin_bit_cast(uint4, pack8(acc[i], acc[i + 1]));
            } else {
#pragma unroll
              for (int u = i; u < i + 2; ++u)
                *reinterpret_cast<uint2*>(kv + (u - 4) * FRAG + 8 * (tile & 1)) =
                    make_uint2(pack2(acc[u][0], acc[u][1]), pack2(acc[u][2], acc[u][3]));
            }
            fence();
          }
          if (odd_end) {   // the missing half of the pair's V^T: finite (its P is zero)
#pragma unroll
            for (int f = 0; f < 4; ++f) *reinterpret_cast<uint2*>(kv + (4 + f) * FRAG + 8) = make_uint2(0u, 0u);
          }
        }
        __syncthreads();
        if (loaded == 1) {
          const int nl = spare ? int(blockDim.x) / WAVE - ntok : ntok < 4 ? ntok : 4;
          const int i = spare ? w - ntok : w;
          if (i >= 0 && i < nl) dma_layers(oargs(), smem, 1, A.n_layers, i, nl);
          loaded = 2;
        }
        if (keep && !loader) {   // this block's K / V^T for later blocks
          uint8_t* dst = lc + int64_t(p0 / 32) * PAIR + tid * 16;
          for (int e = tid * 16; e < A.npair * PAIR; e += A.nwc * WAVE * 16, dst += A.nwc * WAVE * 16)
            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(KV + e);
        }
        // ---- attention: the block's own keys
        if (live) {
#pragma unroll
          for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int dt = 0; dt < DH / 16; ++dt) st[h].o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            st[h].m = NO_KEY;
            st[h].l = 0.f;
            if (A.unmasked) {   // one block: every valid key
              for (int q = 0; 32 * q < Tv; ++q) {
                bf16x8 k[2][DH / 32], v[DH / 16];
                f32x4 sq[2];
                load_k<DH>(k, KV + q * PAIR, h);
                load_v<DH>(v, KV + q * PAIR, h);
                scores<DH>(sq, k, st[h]);
                mask_scores(sq, Tv - 32 * q);
                add_pair<DH>(st[h], sq, v);
              }
            } else {            // the pair of the tile's own keys, then those before it
              const int pr = tile >> 1;
              att_pairs<DH>(st[h], KV, h, pr, TT * (tile & 1) + c16 + 1, pr);
            }
          }
        }
        // ---- keys of earlier blocks, staged half of the LDS of the own keys at a
        // time (32 bytes per thread), the next half's loads in flight
        if (MULTI && blk > 0) {
          const int hp = A.npair / 2;                     // pairs per half
          const int nch = blk * 2;                        // a block is two halves
          const int64_t step = int64_t(hp) * PAIR;
          const uint8_t* src = lc + tid * 16;
          const int far = hp * PAIR / 2;                  // = 16 bytes x threads
          uint4 r0, r1;
          if (!loader) {
            r0 = *reinterpret_cast<const uint4*>(src);
            r1 = *reinterpret_cast<const uint4*>(src + far);
          }
          __syncthreads();   // every wave is past its own keys
          for (int c = 0; c < nch; ++c) {
            uint8_t* dst = KV + (c & 1) * step;
            if (!loader) {
              *reinterpret_cast<uint4*>(dst + tid * 16) = r0;
              *reinterpret_cast<uint4*>(dst + far + tid * 16) = r1;
            }
            __syncthreads();
            if (c + 1 < nch && !loader) {
              r0 = *reinterpret_cast<const uint4*>(src + (c + 1) * step);
              r1 = *reinterpret_cast<const uint4*>(src + (c + 1) * step + far);
            }
            if (live) {
#pragma unroll
              for (int h = 0; h < NH; ++h) att_pairs<DH>(st[h], dst, h, -1, 0, hp);
            }
          }
        }
        if (!live) continue;
        // ---- x += O W_o^T + b_o; LayerNorm 1
        {
          bf16x8 of[2], wf[8];
          f32x4 a[4];
#pragma unroll
          for (int f = 0; f < 4; ++f) {
            wf[2 * f] = frag(Wo + 2 * f * FRAG);
            wf[2 * f + 1] = frag(Wo + (2 * f + 1) * FRAG);
            a[f] = *reinterpret_cast<const f32x4*>(vec + V_BO + feat4(f, g));
          }
          fence();
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            const float inv = 1.f / xsum32(xsum16(st[h].l));
#pragma unroll
            for (int dt = 0; dt < DH / 16; ++dt) st[h].o[dt] *= inv;
#pragma unroll
            for (int q = 0; q < DH / 32; ++q)
              of[h * (DH / 32) + q] = pack8(st[h].o[2 * q], st[h].o[2 * q + 1]);
          }
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int f = 0; f < 4; ++f) a[f] = mma(wf[2 * f + kb], of[kb], a[f]);
#pragma unroll
          for (int f = 0; f < 4; ++f) x[f] += a[f];
          layer_norm(x, vec + V_LN1G, vec + V_LN1B);
        }
        // ---- FFN, 32 hidden units at a time: x += ReLU(x W_1^T + b_1) W_2^T + b_2; LayerNorm 2
        {
          const bf16x8 xf[2] = {pack8(x[0], x[1]), pack8(x[2], x[3])};
          f32x4 o[4];
#pragma unroll
          for (int f = 0; f < 4; ++f)
            o[f] = *reinterpret_cast<const f32x4*>(vec + v_b2(ffn) + feat4(f, g));
          for (int c = 0; c < ffn / 32; ++c) {
            f32x4 hh[2];
            bf16x8 w1f[4], w2f[4];
#pragma unroll
            for (int t = 0; t < 2; ++t)
              hh[t] = *reinterpret_cast<const f32x4*>(vec + V_B1 + feat4(2 * c + t, g));
#pragma unroll
            for (int e = 0; e < 4; ++e) w1f[e] = frag(W1 + (4 * c + e) * FRAG);
#pragma unroll
            for (int f = 0; f < 4; ++f) w2f[f] = frag(W2 + (c * 4 + f) * FRAG);
            fence();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int t = 0; t < 2; ++t) hh[t] = mma(w1f[2 * t + kb], xf[kb], hh[t]);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
              for (int i = 0; i < 4; ++i) hh[t][i] = fmaxf(hh[t][i], 0.f);
            const bf16x8 b = pack8(hh[0], hh[1]);
#pragma unroll
            for (int f = 0; f < 4; ++f) o[f] = mma(w2f[f], b, o[f]);
          }
#pragma unroll
          for (int f = 0; f < 4; ++f) x[f] += o[f];
          layer_norm(x, vec + v_ln2g(ffn), vec + v_ln2b(ffn));
        }
      }
      if (!live) continue;
      // ---- head: the last token's X; the running max of X W_pool^T over valid tokens
      if (p == Tv - 1) {
#pragma unroll
        for (int f = 0; f < 4; ++f)
          *reinterpret_cast<f32x4*>(out + DM + feat4(f, g)) = x[f];
      }
      {
        const bf16x8 xf[2] = {pack8(x[0], x[1]), pack8(x[2], x[3])};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          bf16x8 wf[4];
          pool_frags(wf, oargs(), smem, h);
#pragma unroll
          for (int f = 2 * h; f < 2 * h + 2; ++f) {
            // D[token][feature]: lane holds feature 16 f + c16 of tokens 4 g + i
            f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) y = mma(xf[kb], wf[2 * (f % 2) + kb], y);
            float m = -__builtin_inff();
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (t0 + 4 * g + i < Tv) m = vmax(m, y[i]);
            pmax[f] = vmax(pmax[f], xmax32(xmax16(m)));
          }
        }
      }
    }
    // the pooled maxima go where K / V^T were (written again only after the next
    // candidate's first barrier)
    __syncthreads();
    if (g == 0 && !loader) {
#pragma unroll
      for (int f = 0; f < 4; ++f) pool[w * DM + 16 * f + c16] = pmax[f];
    }
    __syncthreads();
    if (w == grp * A.nwc && Tv > 0 && !loader) {
      float m = pool[w * DM + lane];
      for (int q = 1; q < A.nwc; ++q) m = vmax(m, pool[(w + q) * DM + lane]);
      out[lane] = m + A.b_pool[lane];
    }
  }
  wait_vm_all();   // no LDS-DMA outlives the workgroup (every candidate empty)
}

// The packed weights: one workgroup per matrix or vector.
struct Seg {
  const uint8_t* src;
  int dst, ld;            // byte offset in the packed weights; bytes of a source row
  int nf, nkb, kb_major;  // a matrix's fragments; nf = 0: a vector of nkb 16-byte pieces
};
constexpr int MAX_SEGS = 12 * MAX_LAYERS + 1;
struct PackArgs {
  Seg seg[MAX_SEGS];
  uint8_t* blob;
};
__global__ __launch_bounds__(256) void small_pack_kernel(PackArgs P) {
  const Seg s = P.seg[blockIdx.x];
  const int n = s.nf ? s.nf * s.nkb * WAVE : s.nkb;
  for (int q = threadIdx.x; q < n; q += 256) {
    int at = q * 16;
    if (s.nf) {
      const int e = q / WAVE, lane = q % WAVE;
      const int f = s.kb_major ? e % s.nf : e / s.nkb, kb = s.kb_major ? e / s.nf : e % s.nkb;
      at = feature_row(f, lane % 16) * s.ld + kb * 64 + lane / 16 * 16;
    }
    *reinterpret_cast<uint4*>(P.blob + s.dst + q * 16) = *reinterpret_cast<const uint4*>(s.src + at);
  }
}

}  // namespace sm

// ---------------------------------------------------------------- host side
namespace {
constexpr size_t SM_CACHE_BUDGET = size_t(1) << 30;   // K/V cache bytes at most
constexpr int SM_LDS_MAX = 160 * 1024;

sm::Args small_args(const tav2_weights& w, int d) {
  sm::Args a{};
  a.n_layers = w.n_layers;
  a.d = d;
  a.ffn = w.d_ffn;
  a.dh = w.d_model / w.n_heads;
  sm::plan_packed(a);
  return a;
}

// How T positions are run: waves per candidate, and the pairs of K / V^T they
// keep in LDS next to the weights' image.  One block where ceil(T / 16) waves fit;
// else blocks of the most waves that fit (a multiple of 4: two halves of whole
// pairs).
struct SmallPlan {
  int nwc, npair, blocks;
};
int small_pairs(const sm::Args& a) {   // pairs next to what LDS has to hold
  sm::Args b = a;
  return (SM_LDS_MAX - sm::plan_lds(b, 0)) / sm::PAIR;
}
SmallPlan small_plan(int T, const sm::Args& a) {
  const int avail = small_pairs(a);
  const int tiles = (T + sm::TT - 1) / sm::TT;
  if (tiles <= sm::MAX_NW && (tiles + 1) / 2 <= avail) return SmallPlan{tiles, (tiles + 1) / 2, 1};
  const int most = std::min(sm::MAX_NW, 2 * avail) / 4 * 4;
  const int blocks = (tiles + most - 1) / most;
  const int nwc = ((tiles + blocks - 1) / blocks + 3) / 4 * 4;   // blocks of about one size
  return SmallPlan{nwc, nwc / 2, (tiles + nwc - 1) / nwc};
}
size_t small_per_wg_cache(int T, int n_layers) {
  return T <= 64 ? 0 : size_t(n_layers) * size_t((T + 63) / 64 * 2) * sm::PAIR;
}
int device_cus() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
    return v;
  return 256;
}
// Candidates side by side in a workgroup: as many as it takes to give every CU one
// workgroup, at most what the LDS and GROUP_NW waves hold.
int small_groups(int64_t total, const SmallPlan& p, const sm::Args& a, int cus) {
  if (p.blocks > 1) return 1;
  const int most = std::max(1, std::min(sm::GROUP_NW / p.nwc, small_pairs(a) / p.npair));
  const int64_t want = cdiv(total, int64_t(cus));
  return int(std::max<int64_t>(1, std::min<int64_t>(want, most)));
}
// Workgroups: one per CU at most, and no more than the cache budget allows.
int small_grid(int64_t total, int T, int n_layers, int groups, int cus) {
  int64_t g = std::min<int64_t>(cdiv(total, int64_t(groups)), cus);
  const size_t per = small_per_wg_cache(T, n_layers);
  if (per) g = std::min<int64_t>(g, std::max<int64_t>(1, int64_t(SM_CACHE_BUDGET / per)));
  return int(std::max<int64_t>(g, 1));
}
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// The pieces of the packed weights: every layer matrix and vector and the token half
// of W_in.
int small_segments(const tav2_weights& w, int d, const sm::Args& a, sm::Seg* seg) {
  int n = 0;
  constexpr int DM = sm::DM;
  const int ffn = w.d_ffn;
  auto mat = [&](const void* src, int dst, int rows, int cols, int ld, int kb_major) {
    seg[n++] = sm::Seg{static_cast<const uint8_t*>(src), dst, ld * 2, rows / 16, cols / 32, kb_major};
  };
  for (int l = 0; l < w.n_layers; ++l) {
    const tav2_layer& L = w.layers[l];
    auto vec = [&](const float* src, int at, int len) {
      seg[n++] = sm::Seg{reinterpret_cast<const uint8_t*>(src), a.pk[l].vec + at * 4, 0, 0, len / 4, 0};
    };
    mat(L.W_qkv, a.pk[l].qkv, 3 * DM, DM, DM, 0);
    mat(L.W_o, a.pk[l].o, DM, DM, DM, 0);
    mat(L.W_1, a.pk[l].w1, ffn, DM, DM, 0);
    mat(L.W_2, a.pk[l].w2, DM, ffn, ffn, 1);
    vec(L.b_qkv, sm::V_BQKV, 3 * DM);
    vec(L.b_o, sm::V_BO, DM);
    vec(L.ln1_g, sm::V_LN1G, DM);
    vec(L.ln1_b, sm::V_LN1B, DM);
    vec(L.b_1, sm::V_B1, ffn);
    vec(L.b_2, sm::v_b2(ffn), DM);
    vec(L.ln2_g, sm::v_ln2g(ffn), DM);
    vec(L.ln2_b, sm::v_ln2b(ffn), DM);
  }
  mat(w.W_in, a.packed_bytes - DM * (d + 8) * 2, DM, d, 2 * d, 1);
  return n;
}

// The shapes this encoder takes: the packed weights and 64 positions' activations in
// rows padded the same way fit the LDS, i.e. two layers of FFN 32 with d <= 64.  (The
// kernel needs less; what it accepts is part of the interface.)
int small_shape_bytes(const sm::Args& a) {
  constexpr int DM = sm::DM, RB = sm::RLD * 2;
  return a.packed_bytes + 4 * 64 * RB + 64 * (a.ffn + 8) * 2 + 32 * RB + DM * 80 + 5 * DM * 4;
}
}  // namespace

bool encode_small_supported(int d, const tav2_weights& w) {
  if (w.d_model != sm::DM || w.n_layers > sm::MAX_LAYERS) return false;
  const int dh = w.d_model / w.n_heads;
  if (dh != 32 && dh != 64) return false;
  if (w.d_ffn % 32 || w.d_ffn > 256 || d % 32 || d > 32 * sm::MAX_DK) return false;
  return small_shape_bytes(small_args(w, d)) <= SM_LDS_MAX;
}

bool encode_small_aligned(const tav2_weights& w) {
  if (!aligned16(w.W_in) || !aligned16(w.W_pool) || (reinterpret_cast<uintptr_t>(w.E_act) & 7) ||
      (reinterpret_cast<uintptr_t>(w.E_pos) & 7) || (reinterpret_cast<uintptr_t>(w.E_time) & 7))
    return false;
  for (int l = 0; l < w.n_layers; ++l) {
    const tav2_layer& L = w.layers[l];
    if (!aligned16(L.W_qkv) || !aligned16(L.W_o) || !aligned16(L.W_1) || !aligned16(L.W_2))
      return false;
  }
  return true;
}

size_t encode_small_packed_bytes(const tav2_weights& w) {
  return size_t(small_args(w, w.d_in).packed_bytes);
}

hipError_t launch_encode_small_pack(const tav2_weights& w, void* packed, hipStream_t st) {
  const sm::Args a = small_args(w, w.d_in);
  sm::PackArgs P{};
  const int n = small_segments(w, w.d_in, a, P.seg);
  P.blob = static_cast<uint8_t*>(packed);
  ProfScope prof("pack_weights", st);
  sm::small_pack_kernel<<<unsigned(n), 256, 0, st>>>(P);
  return hipGetLastError();
}

// (The size is that of a cache of every position, rounded up to 64, past the first 64;
// the blocks but the last need no more.)
size_t encode_small_workspace(int64_t total, int T, const tav2_weights& w) {
  const size_t per = small_per_wg_cache(T, w.n_layers);
  return per ? per * size_t(small_grid(total, T, w.n_layers, 1, device_cus())) : 0;
}

hipError_t launch_encode_small(const TokenSource& src, const void* cand_emb, int64_t total,
                               const tav2_weights& w, float* out, void* ws, bool unmasked,
                               hipStream_t st) {
  if (total == 0) return hipSuccess;
  sm::Args a = small_args(w, src.d);
  a.s = src;
  a.cand = static_cast<const bf16_t*>(cand_emb);
  a.W_in = static_cast<const bf16_t*>(w.W_in);
  a.b_in = w.b_in;
  a.E_act = static_cast<const bf16_t*>(w.E_act);
  a.E_time = static_cast<const bf16_t*>(w.E_time);
  a.E_pos = static_cast<const bf16_t*>(w.E_pos);
  a.W_pool = static_cast<const bf16_t*>(w.W_pool);
  a.b_pool = w.b_pool;
  for (int i = 0; i < w.n_layers; ++i) a.layers[i] = w.layers[i];
  a.packed = static_cast<const uint8_t*>(w.packed);
  a.total = total;
  a.out = out;
  a.unmasked = unmasked ? 1 : 0;
  a.tab16 = aligned16(w.E_act) && aligned16(w.E_time) ? 1 : 0;
  const int cus = device_cus();
  const SmallPlan p = small_plan(src.T, a);
  a.nwc = p.nwc;
  a.npair = p.npair;
  a.groups = small_groups(total, p, a, cus);
  a.cache_pairs = (p.blocks - 1) * p.npair;
  a.cache = p.blocks > 1 ? static_cast<uint8_t*>(ws) : nullptr;
  const int kvb = a.groups * a.npair * sm::PAIR;
  sm::plan_lds(a, SM_LDS_MAX - kvb);
  const int lds = a.kv + kvb;
  const int grid = small_grid(total, src.T, w.n_layers, a.groups, cus);
  const int nk = src.d / 32;
  // (spare waves, up to the 8 or 12 that the kernel is built for, help to load weights)
  const bool multi = p.blocks > 1;
  const int waves = !multi && a.groups * a.nwc <= 8 ? 8 : sm::MAX_NW;
  const int which = (nk <= 1 ? 0 : nk <= 2 ? 1 : nk <= 4 ? 2 : 3) + (a.dh == 64 ? 0 : 4) +
                    (multi ? 16 : waves == 8 ? 0 : 8);
#define SM_KERNELS(NW, M)                                                                  \
  sm::encoder_small_kernel<1, 64, NW, M>, sm::encoder_small_kernel<2, 64, NW, M>,          \
      sm::encoder_small_kernel<4, 64, NW, M>, sm::encoder_small_kernel<8, 64, NW, M>,      \
      sm::encoder_small_kernel<1, 32, NW, M>, sm::encoder_small_kernel<2, 32, NW, M>,      \
      sm::encoder_small_kernel<4, 32, NW, M>, sm::encoder_small_kernel<8, 32, NW, M>
  void (*const kernels[24])(sm::Args) = {SM_KERNELS(8, false), SM_KERNELS(sm::MAX_NW, false),
                                         SM_KERNELS(sm::MAX_NW, true)};
#undef SM_KERNELS
  static std::atomic<bool> done[64][24] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !done[dev][which].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernels[which]),
                            hipFuncAttributeMaxDynamicSharedMemorySize, SM_LDS_MAX);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) done[dev][which].store(true, std::memory_order_release);
  }
  ProfScope prof("encoder_small", st);
  hipLaunchKernelGGL(kernels[which], dim3(unsigned(grid)), dim3(unsigned(waves * WAVE)),
                     size_t(lds), st, a);
  return hipGetLastError();
}

}  // namespace tav2
