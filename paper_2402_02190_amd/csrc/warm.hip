// Learned warm start: per-node structural features and a small message-passing
// network (GraphSAGE form of the GNN appendix, with bias) in bfloat16 on the
// gfx950 matrix cores, with float32 accumulation, plus its backward and
// training step.  The network's output Z_w enters CPRA as fixed logits added
// to the GNN's output (cpra_model_cfg.z_offset).  The idea of a network
// trained across instances that proposes a starting point for a new instance
// is the background section's paragraph on learning generalized heuristics
// from data (meta-learned initialisation).
//
// Storage: bfloat16 activations [N, width] row-major (raw uint16 bit
// patterns, round-to-nearest-even from float32), float32 master weights and
// gradients, float32 output logits.  Kernels:
//  * k_node_features -- 16 lanes or a wavefront per node: triangle count by comparing
//    every neighbour's list with the node's own (by binary search for large degrees;
//    integer, exact), then the feature row [d/16, clustering, random channels, 0...];
//  * k_mpnn_layer -- one forward layer: each wavefront gathers the neighbour means of
//    its 32 rows (float32 sums in CSR order, one rounding) into the operands of
//    v_mfma_f32_32x32x16_bf16, next to the rows themselves, while the weights (at most
//    128 x 128) sit in LDS; bias / ReLU / bf16 or float32 store in the epilogue;
//  * k_rows_mfma, k_agg_t_bf16 -- the backward's dY [Ws | Wn] by 32-row tiles, and the
//    M^T gather of its float32 rows with an addend and a ReLU mask, bf16 result;
//  * k_wgrad_mfma -- per block of rows, the partial dY^T [X_0 | X_1] and the
//    column sums of dY (bias gradient) through LDS-staged 64-row chunks; a
//    second kernel adds the partials in block order (deterministic).
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace cpra {

cpra_status check_loss_cfg_public(const cpra_csr* g, const cpra_loss_cfg* cfg);
cpra_status check_adam_cfg(const cpra_adam_cfg* cfg);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxLayers = 8;
constexpr int kMaxWidth = 128;    // n_out and k_total limit of the row GEMM
constexpr int kMaxWgBlocks = 1024;

__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline float sigmoid_of(float z) {
  const float e = expf(-fabsf(z));
  const float r = 1.0f / (1.0f + e);
  return z >= 0.0f ? r : e * r;
}

// ------------------------------------------------------------------ features
// 2 T_i by one wavefront: lanes take neighbours, each binary-searching every entry of
// its neighbour's list in the node's own (this lane's share of the sum).
__device__ __forceinline__ long long wedges_by_search(const int32_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col_idx, int b, int e, int lane) {
  long long cnt = 0;
  for (int k = b + lane; k < e; k += 64) {
    const int j = col_idx[k];
    const int bj = row_ptr[j], ej = row_ptr[j + 1];
    for (int q = bj; q < ej; ++q) {
      const int x = col_idx[q];
      int lo = b, hi = e;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col_idx[mid] < x) lo = mid + 1; else hi = mid;
      }
      cnt += (lo < e && col_idx[lo] == x) ? 1 : 0;
    }
  }
  return cnt;
}

// 2 T_i by LPN lanes for d <= LPN H neighbours: the node's own list sits in its lanes'
// registers, lane l walks the list of neighbour l (eight entries in flight) and compares
// each entry with every own one, passed round by shuffles: three dependent loads in all,
// where the search makes log2(d) more per entry.  All 64 lanes call it; d = 0 gives 0.
template <int LPN, int H>
__device__ __forceinline__ int wedges_by_compare(const int32_t* __restrict__ row_ptr,
                                                 const int32_t* __restrict__ col_idx, int b, int d, int l) {
  int own[H], key[H], bj[H], ej[H];  // neighbours l, l + LPN, ..
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int t = LPN * h + l;
    own[h] = t < d ? col_idx[b + t] : -1;
    key[h] = t > 0 && t < d && col_idx[b + t - 1] == own[h] ? -1 : own[h];  // a repeated entry matches once
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    bj[h] = own[h] >= 0 ? row_ptr[own[h]] : 0;
    ej[h] = own[h] >= 0 ? row_ptr[own[h] + 1] : 0;
  }
  int c = 0;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    for (int q = bj[h]; __any(q < ej[h]); q += 8) {
      int x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = q + u < ej[h] ? col_idx[q + u] : -2;
#pragma unroll
      for (int p = 0; p < H; ++p)
        for (int t = 0; t < LPN && __any(LPN * p + t < d); ++t) {
          const int o = __shfl(key[p], t, LPN);
#pragma unroll
          for (int u = 0; u < 8; ++u) c += x[u] == o;
        }
    }
  }
  return c;  // this lane's share
}

// LPN lanes per node, by comparison up to 32 neighbours; the larger nodes of a wavefront
// one after the other by all its lanes, by comparison up to kWideDegree, then by search
// (comparing costs d_i d_j, searching d_j log d_i; 40-regular, N = 500: 27 us and 31,
// 64-regular 64 and 52).  With 16 lanes per node a wavefront's four nodes lie a quarter
// of the graph apart, so that a run of large ones is spread over as many wavefronts.
//
// Bound by the chain of dependent loads while the wavefronts fit the chip, then by the
// comparisons.  16 lanes per node from 8,192 nodes on up to a mean degree of 24, from
// 4,096 on up to 12, else a wavefront per node (us, 16 lanes and 64; before both, by
// search alone, in brackets; the first three rows back to back in a graph):
//   3-regular    2,000 3.7, 3.3; 5,000 3.9, 4.2; 20,000 5.2, 9.2
//   5-regular    500 3.9, 3.4; 5,000 4.2, 4.6; 12,000 4.8, 7.3; 50,000 11.5, 22
//   10-regular   2,000 6.2, 5.5; 5,000 6.6, 7.8; 20,000 10.2, 20
//   16-regular   8,000 10.6, 14.9 (19.9); 32,000 30, 42 (67)
//   20-regular   2,000 19.9, 10.8 (16.0); 8,000 22.7, 23.1 (26.4); 32,000 55, 68 (91)
//   40-regular   2,000 96, 27 (39); 32,000 232, 204 (332)
//   100-regular  2,000 657, 214 (209); 16,000 1,359, 872 (849)
//   random       9,000 of mean 28 120, 67 (80); 20,000 of mean 10 25.2, 29.0 (43.4), of
//                mean 30 178, 129 (141)
//   power law of mean 16 (largest degree 117 and 346): 2,000 147, 107 (112);
//                20,000 504, 449 (469); 4.6 of mean with 3 hubs of 2,000: 2,466, 2,456 (2,471)
constexpr int kWideDegree = 48;
template <int LPN>
__global__ __launch_bounds__(256) void k_node_features(int n, const int32_t* __restrict__ row_ptr,
                                                       const int32_t* __restrict__ col_idx,
                                                       int in_dim, int n_rand,
                                                       const float* __restrict__ rand,
                                                       int64_t ld_rand, uint16_t* __restrict__ feat,
                                                       int64_t ld_feat, int64_t* __restrict__ tri) {
  constexpr int NPW = 64 / LPN;  // nodes per wavefront
  const int lane = threadIdx.x & 63;
  const int sub = lane / LPN, l = lane % LPN;
  const int per = (n + NPW - 1) / NPW;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= per) return;  // uniform per wavefront
  const int i = w + sub * per;
  int b = 0, e = 0;
  if (i < n) {
    b = row_ptr[i];
    e = row_ptr[i + 1];
  }
  const int d = e - b;
  long long cnt = 0;  // sum over neighbours j of |N(i) n N(j)| = 2 T_i
  if constexpr (LPN == 16) {
    if (__any(d > 0 && d <= 32)) cnt = wedges_by_compare<16, 2>(row_ptr, col_idx, b, d <= 32 ? d : 0, l);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
  }
  const bool wide = LPN == 64 || __any(d > 32);
  for (int t = 0; wide && t < NPW; ++t) {
    const int dt = __shfl(d, LPN * t);  // uniform, as the branches on it
    if (LPN == 16 && dt <= 32) continue;
    const int bt = __shfl(b, LPN * t);
    long long c;
    if (dt <= kWideDegree) c = wedges_by_compare<64, 1>(row_ptr, col_idx, bt, dt, lane);
    else c = wedges_by_search(row_ptr, col_idx, bt, bt + dt, lane);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if (sub == t) cnt = c;
  }
  if (i >= n) return;
  const long long T = cnt / 2;
  if (l == 0 && tri) tri[i] = T;
  for (int c = l; c < in_dim; c += LPN) {
    float v = 0.0f;
    if (c == 0) {
      v = (float)d * 0.0625f;
    } else if (c == 1) {
      v = d >= 2 ? (float)((2.0 * (double)T) / ((double)d * (double)(d - 1))) : 0.0f;
    } else if (c - 2 < n_rand) {
      v = rand[(int64_t)i * ld_rand + (c - 2)];
    }
    feat[(int64_t)i * ld_feat + c] = f2bf(v);
  }
}

// ------------------------------------------------------------------ casts
__global__ void k_zero(int64_t n, float* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.0f;
}

__global__ void k_cast_rows_bf16(int rows, int cols, const float* __restrict__ x, int64_t ldx,
                                 uint16_t* __restrict__ y, int64_t ldy) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * cols) return;
  const int64_t r = i / cols, c = i - r * cols;
  y[r * ldy + c] = f2bf(x[r * ldx + c]);
}

__global__ void k_bce_grad(int rows, int S, const float* __restrict__ Z, int64_t ldz,
                           const uint8_t* __restrict__ target, int64_t ldt, float beta,
                           float* __restrict__ dZ, int64_t lddz) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * S) return;
  const int64_t r = i / S, s = i - r * S;
  const float p = sigmoid_of(Z[r * ldz + s]);
  dZ[r * lddz + s] += beta * (p - (float)target[r * ldt + s]);
}

// ------------------------------------------------------------------ aggregation
struct AggBfArgs {
  int n, units, lpr_log2;
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const float* inv_deg;
  const float* col_inv_deg;  // inv_deg of each entry's column, or null (gathered instead)
  const float* X;
  int64_t ldx;
  uint16_t* Y;
  int64_t ldy;
  const float* add;  // [N, width] float addend
  int64_t ld_add;
  const uint16_t* mask;  // output zeroed where mask <= 0
  int64_t ld_mask;
};

__device__ inline void load8(const uint16_t* p, float* v) {
  const u16x8 w = *reinterpret_cast<const u16x8*>(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = bf2f(w[e]);
}
__device__ inline void load8(const float* p, float* v) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// The backward's M^T dG.  Each lane owns 8 consecutive columns; the 2^lpr_log2 lanes of
// a row cover its units = width / 8 column groups.
__global__ __launch_bounds__(256) void k_agg_t_bf16(AggBfArgs a) {
  const int lane = threadIdx.x & 63;
  const int lpr = 1 << a.lpr_log2;
  const int sub = lane >> a.lpr_log2;
  const int u = lane & (lpr - 1);
  const int row = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 >> a.lpr_log2) + sub;
  if (row >= a.n || u >= a.units) return;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
  const int beg = a.row_ptr[row], end = a.row_ptr[row + 1];
  for (int k = beg; k < end; ++k) {
    const int j = a.col_idx[k];
    const float s = a.col_inv_deg ? a.col_inv_deg[k] : a.inv_deg[j];
    float v[8];
    load8(a.X + (int64_t)j * a.ldx + u * 8, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += s * v[e];
  }
  float ad[8], mk[8];
  load8(a.add + (int64_t)row * a.ld_add + u * 8, ad);
  load8(a.mask + (int64_t)row * a.ld_mask + u * 8, mk);
  u16x8 w;
#pragma unroll
  for (int e = 0; e < 8; ++e) w[e] = f2bf(mk[e] > 0.0f ? acc[e] + ad[e] : 0.0f);
  *reinterpret_cast<u16x8*>(a.Y + (int64_t)row * a.ldy + u * 8) = w;
}

// ------------------------------------------------------------------ row GEMM
// The backward's dY [Ws | Wn]: C[M, n_out] = A[M, k_total] [B0 | B1].
struct RowsArgs {
  int M, n_out, k_total;
  const uint16_t* A;
  int64_t lda;
  const uint16_t* B[2];  // [k_total, n_half] row-major, pieces along N
  int n_half;
  float* C;
  int64_t ldc;
  int tiles;  // ceil(M / 32)
};

template <int NT>  // n_out / 32 output tiles of 32 columns per wavefront
__global__ __launch_bounds__(256) void k_rows_mfma(RowsArgs a) {
  constexpr int KP = kMaxWidth + 8;  // LDS row pitch (bf16 elements) of B^T
  __shared__ __attribute__((aligned(16))) uint16_t Bt[NT * 32 * KP];
  // stage B^T [n][k] once per block
  const int kt = a.k_total;
  for (int idx = threadIdx.x; idx < NT * 32 * kt; idx += 256) {
    const int n = idx / kt, k = idx - n * kt;
    const int q = n < a.n_half ? 0 : 1;
    Bt[n * KP + k] = a.B[q][(int64_t)k * a.n_half + (q ? n - a.n_half : n)];
  }
  __syncthreads();

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int m = lane & 31;
  const int g = lane >> 5;
  for (int tile = blockIdx.x * 4 + wave; tile < a.tiles; tile += gridDim.x * 4) {
    const int row = tile * 32 + m;
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
    for (int k0 = 0; k0 < kt; k0 += 16) {
      u32x4 av = {0u, 0u, 0u, 0u};
      if (row < a.M) av = *reinterpret_cast<const u32x4*>(a.A + (int64_t)row * a.lda + k0 + 8 * g);
      const bf16x8 af = __builtin_bit_cast(bf16x8, av);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const u32x4 bv = *reinterpret_cast<const u32x4*>(&Bt[(t * 32 + m) * KP + k0 + 8 * g]);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, __builtin_bit_cast(bf16x8, bv), acc[t],
                                                         0, 0, 0);
      }
    }
    // acc[t][r] holds C[tile*32 + 8*(r/4) + 4*g + r%4][t*32 + m]
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = tile * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
        if (rr < a.M) a.C[(int64_t)rr * a.ldc + t * 32 + m] = acc[t][r];
      }
  }
}

// ------------------------------------------------------------------ forward layer
struct LayerArgs {
  int n, tiles;
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const float* inv_deg;
  const uint16_t* H;  // [n, in]
  uint16_t* A;        // [n, in]: bf16(M H), kept for the backward
  const float* Ws;    // float32 masters [n_out, in]
  const float* Wn;
  uint16_t* ws_bf;    // their bf16 shadows, written by block 0 (the backward reads them)
  uint16_t* wn_bf;
  const float* bias;
  int relu;
  uint16_t* Cb;  // bf16 output [n, n_out] or null
  float* Cf;     // float output [n, n_out] or null
};

__device__ inline u32x4 round8(const float* v) {
  u16x8 w;
#pragma unroll
  for (int e = 0; e < 8; ++e) w[e] = f2bf(v[e]);
  return __builtin_bit_cast(u32x4, w);
}

// Y = H bf16(Ws)^T + bf16(M H) bf16(Wn)^T + b in one launch.  A wavefront owns 32 rows;
// lane (row, g) gathers the neighbours' columns 16 t + 8 g .. + 7 of its row straight
// into the operand layout (FP32 sums in CSR order, four neighbours' loads in flight,
// then the one rounding), so M H is written once for the backward and never read
// here.  The weights are rounded from the float32 masters while they are staged, a
// vector of 8 per load.  Rounding points and the order of every sum are those of
// an aggregation launch followed by a product in k order, bit for bit.  Bound by the
// chain row_ptr -> col_idx -> rows at the 1,563 wavefronts that 50,000 rows give (more
// neighbours in flight or smaller blocks: no change).  64 -> 64 columns at N = 50,000,
// 5-regular: 8 + 25 us in two launches (the weights staged value by value) -> 15.7 us.
template <int NT, int KI>  // n_out / 32, in / 16
__global__ __launch_bounds__(256) void k_mpnn_layer(LayerArgs a) {
  constexpr int IN = 16 * KI, KT = 2 * IN, KP = KT + 8;  // LDS row pitch (bf16 elements)
  __shared__ __attribute__((aligned(16))) uint16_t Bt[NT * 32 * KP];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 31, g = lane >> 5;
  const int tile = blockIdx.x * 4 + wave;
  const int row = tile * 32 + m;
  const bool live = row < a.n;
  int k = 0, end = 0;
  if (live) {
    k = a.row_ptr[row];
    end = a.row_ptr[row + 1];
  }
  for (int v = threadIdx.x; v < NT * 32 * KT / 8; v += 256) {
    const int n = v / (KT / 8), c = (v % (KT / 8)) * 8;
    const bool nb = c >= IN;
    const int at = n * IN + (nb ? c - IN : c);
    const float* w = (nb ? a.Wn : a.Ws) + at;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = w[e];
    const u32x4 r = round8(x);
    *reinterpret_cast<u32x4*>(&Bt[n * KP + c]) = r;
    if (blockIdx.x == 0) *reinterpret_cast<u32x4*>((nb ? a.wn_bf : a.ws_bf) + at) = r;
  }
  u32x4 hv[KI], av[KI];
#pragma unroll
  for (int t = 0; t < KI; ++t) {
    hv[t] = u32x4{0u, 0u, 0u, 0u};
    if (live) hv[t] = *reinterpret_cast<const u32x4*>(a.H + (int64_t)row * IN + 16 * t + 8 * g);
  }
  float sum[KI][8];
#pragma unroll
  for (int t = 0; t < KI; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[t][e] = 0.0f;
  constexpr int CH = 4;
  for (; k < end; k += CH) {
    int j[CH];
    u32x4 x[CH][KI];
#pragma unroll
    for (int c = 0; c < CH; ++c) j[c] = a.col_idx[min(k + c, end - 1)];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int t = 0; t < KI; ++t) {
        x[c][t] = u32x4{0u, 0u, 0u, 0u};  // past the row's end: adds an exact zero (sums never hold -0)
        if (k + c < end) x[c][t] = *reinterpret_cast<const u32x4*>(a.H + (int64_t)j[c] * IN + 16 * t + 8 * g);
      }
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int t = 0; t < KI; ++t) {
        const u16x8 y = __builtin_bit_cast(u16x8, x[c][t]);
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[t][e] += bf2f(y[e]);
      }
  }
  const float rs = live ? a.inv_deg[row] : 0.0f;
#pragma unroll
  for (int t = 0; t < KI; ++t) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[t][e] *= rs;
    av[t] = round8(sum[t]);
    if (live) *reinterpret_cast<u32x4*>(a.A + (int64_t)row * IN + 16 * t + 8 * g) = av[t];
  }
  __syncthreads();
  if (tile >= a.tiles) return;
  // The weights are the first operand, so that a lane ends with columns of its own row:
  // acc[t][4 q + e] holds C[row][t * 32 + 8 q + 4 g + e].
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
#pragma unroll
  for (int q = 0; q < 2 * KI; ++q) {
    const bf16x8 af = __builtin_bit_cast(bf16x8, q < KI ? hv[q % KI] : av[q % KI]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const u32x4 bv = *reinterpret_cast<const u32x4*>(&Bt[(t * 32 + m) * KP + 16 * q + 8 * g]);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bv), af, acc[t], 0, 0, 0);
    }
  }
  if (!live) return;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = t * 32 + 8 * q + 4 * g;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[t][4 * q + e] + a.bias[col + e];
        if (a.relu) v[e] = fmaxf(v[e], 0.0f);
      }
      if (a.Cb) {
        uint16_t* o = a.Cb + (int64_t)row * (NT * 32) + col;
        const u16x4 y = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
        *reinterpret_cast<u16x4*>(o) = y;
      }
      if (a.Cf) __builtin_memcpy(a.Cf + (int64_t)row * (NT * 32) + col, v, sizeof v);
    }
}

// ------------------------------------------------------------------ weight gradient
struct WgArgs {
  int M, n_o, n_c, c0;
  const uint16_t* dY;  // [M, n_o] (lddy)
  int64_t lddy;
  const uint16_t* X0;  // [M, c0] (ldx0)
  int64_t ldx0;
  const uint16_t* X1;  // [M, n_c - c0] (ldx1)
  int64_t ldx1;
  int rows_per_block;
  float* partial;  // [gridDim.x][n_o][n_c + 1]
};

template <int TPW>  // output tiles (32 x 32) per wavefront
__global__ __launch_bounds__(256) void k_wgrad_mfma(WgArgs a) {
  constexpr int CH = 64;               // rows per LDS chunk
  constexpr int YP = kMaxWidth + 8;    // pitches (bf16 elements)
  constexpr int XP = 2 * 64 + 8;
  __shared__ __attribute__((aligned(16))) uint16_t Ys[CH * YP];
  __shared__ __attribute__((aligned(16))) uint16_t Xs[CH * XP];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int m = lane & 31;
  const int g = lane >> 5;
  const int tiles_c = a.n_c / 32;
  const int n_tiles = (a.n_o / 32) * tiles_c;
  f32x16 acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
  float bsum = 0.0f;  // thread o < n_o: column sum of dY (bias gradient)

  const int r_beg = blockIdx.x * a.rows_per_block;
  const int r_end = min(a.M, r_beg + a.rows_per_block);
  const int uy = a.n_o / 8, ux = a.n_c / 8;  // 16-byte units per row
  for (int c0 = r_beg; c0 < r_end; c0 += CH) {
    __syncthreads();
    for (int idx = threadIdx.x; idx < CH * uy; idx += 256) {
      const int r = idx / uy, u = idx - r * uy;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (c0 + r < r_end) v = *reinterpret_cast<const u32x4*>(a.dY + (int64_t)(c0 + r) * a.lddy + u * 8);
      *reinterpret_cast<u32x4*>(&Ys[r * YP + u * 8]) = v;
    }
    for (int idx = threadIdx.x; idx < CH * ux; idx += 256) {
      const int r = idx / ux, u = idx - r * ux;
      const int c = u * 8;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (c0 + r < r_end) {
        const uint16_t* src = c < a.c0 ? a.X0 + (int64_t)(c0 + r) * a.ldx0 + c
                                       : a.X1 + (int64_t)(c0 + r) * a.ldx1 + (c - a.c0);
        v = *reinterpret_cast<const u32x4*>(src);
      }
      *reinterpret_cast<u32x4*>(&Xs[r * XP + c]) = v;
    }
    __syncthreads();
    if (threadIdx.x < a.n_o) {
      for (int r = 0; r < CH; ++r) bsum += bf2f(Ys[r * YP + threadIdx.x]);
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int tile = wave + 4 * i;
      if (tile >= n_tiles) break;
      const int to = tile / tiles_c, tc = tile - to * tiles_c;
      const int o = to * 32 + m, c = tc * 32 + m;
#pragma unroll
      for (int ks = 0; ks < CH; ks += 16) {
        u16x8 av, bv;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int r = ks + 8 * g + e;
          av[e] = Ys[r * YP + o];
          bv[e] = Xs[r * XP + c];
        }
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                         __builtin_bit_cast(bf16x8, bv), acc[i], 0,
                                                         0, 0);
      }
    }
  }
  float* out = a.partial + (int64_t)blockIdx.x * a.n_o * (a.n_c + 1);
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int tile = wave + 4 * i;
    if (tile >= n_tiles) break;
    const int to = tile / tiles_c, tc = tile - to * tiles_c;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int o = to * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
      out[(int64_t)o * (a.n_c + 1) + tc * 32 + m] = acc[i][r];
    }
  }
  if (threadIdx.x < a.n_o) out[(int64_t)threadIdx.x * (a.n_c + 1) + a.n_c] = bsum;
}

// grads of one layer: Ws [n_o, c0], Wn [n_o, n_c - c0], b [n_o]
__global__ void k_wgrad_reduce(int blocks, int n_o, int n_c, int c0, const float* __restrict__ part,
                               float* __restrict__ dWs, float* __restrict__ dWn,
                               float* __restrict__ db) {
  const int per = n_o * (n_c + 1);
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= per) return;
  float s = 0.0f;
  for (int b = 0; b < blocks; ++b) s += part[(int64_t)b * per + idx];
  const int o = idx / (n_c + 1), c = idx - o * (n_c + 1);
  if (c < c0) dWs[o * c0 + c] = s;
  else if (c < n_c) dWn[o * (n_c - c0) + (c - c0)] = s;
  else db[o] = s;
}

// ------------------------------------------------------------------ plan
struct MLayer {
  int in, out;
  int64_t off_ws, off_wn, off_b;  // float offsets in the parameter vector
};

struct MPlan {
  int L, N;
  MLayer layer[kMaxLayers];
  int64_t n_params;
  size_t wbf_off;               // bf16 shadow of the parameters
  size_t h_off[kMaxLayers];     // bf16 input of layer k (k >= 1)
  size_t a_off[kMaxLayers];     // bf16 M H of layer k
  size_t dy_off[2];             // bf16 [N, max_out] ping-pong
  size_t g_off;                 // float [N, 2 max_in] (layers k >= 1)
  size_t part_off;              // float [kMaxWgBlocks][max_out (2 max_in + 1)]
  size_t total;
};

cpra_status check_mpnn_cfg(const cpra_mpnn_cfg* cfg) {
  if (cfg == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "mpnn: cfg is NULL");
  if (cfg->n_layers < 1 || cfg->n_layers > kMaxLayers)
    CPRA_FAIL(CPRA_ERR_PARAM, "mpnn: n_layers = %d outside 1..%d", cfg->n_layers, kMaxLayers);
  if (cfg->in_dim < 16 || cfg->in_dim > 64 || cfg->in_dim % 16 != 0)
    CPRA_FAIL(CPRA_ERR_PARAM, "mpnn: in_dim = %d must be 16, 32, 48 or 64", cfg->in_dim);
  if (cfg->n_layers > 1 && (cfg->hidden < 32 || cfg->hidden > 64 || cfg->hidden % 32 != 0))
    CPRA_FAIL(CPRA_ERR_PARAM, "mpnn: hidden = %d must be 32 or 64", cfg->hidden);
  if (cfg->S < 32 || cfg->S > kMaxWidth || cfg->S % 32 != 0)
    CPRA_FAIL(CPRA_ERR_PARAM, "mpnn: S = %d must be a multiple of 32 up to %d", cfg->S, kMaxWidth);
  return CPRA_OK;
}

void make_mplan(const cpra_mpnn_cfg* cfg, int N, MPlan* p) {
  p->L = cfg->n_layers;
  p->N = N;
  int64_t off = 0;
  int d = cfg->in_dim, max_out = 0, max_in1 = 0;
  for (int k = 0; k < p->L; ++k) {
    MLayer& l = p->layer[k];
    l.in = d;
    l.out = (k == p->L - 1) ? cfg->S : cfg->hidden;
    l.off_ws = off;
    off += (int64_t)l.out * l.in;
    l.off_wn = off;
    off += (int64_t)l.out * l.in;
    l.off_b = off;
    off += l.out;
    max_out = std::max(max_out, l.out);
    if (k >= 1) max_in1 = std::max(max_in1, l.in);
    d = l.out;
  }
  p->n_params = off;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t r = o;
    o += align_up(std::max<size_t>(bytes, 1), 256);
    return r;
  };
  p->wbf_off = take((size_t)p->n_params * 2);
  int max_in = 0;
  for (int k = 0; k < p->L; ++k) {
    const MLayer& l = p->layer[k];
    p->h_off[k] = k >= 1 ? take((size_t)N * l.in * 2) : 0;
    p->a_off[k] = take((size_t)N * l.in * 2);
    max_in = std::max(max_in, l.in);
  }
  p->dy_off[0] = take((size_t)N * max_out * 2);
  p->dy_off[1] = take((size_t)N * max_out * 2);
  p->g_off = take((size_t)N * 2 * std::max(max_in1, 1) * 4);
  p->part_off = take((size_t)kMaxWgBlocks * max_out * (2 * max_in + 1) * 4);
  p->total = o;
}

template <typename T>
inline T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

cpra_status agg_t_bf16(const cpra_csr* g, int width, const float* X, int64_t ldx, uint16_t* Y,
                       int64_t ldy, const float* add, int64_t ld_add, const uint16_t* mask,
                       int64_t ld_mask, hipStream_t st) {
  const int units = width / 8;
  int lpr_log2 = 0;
  while ((1 << lpr_log2) < units) ++lpr_log2;
  AggBfArgs a{g->n_nodes, units, lpr_log2, g->row_ptr, g->col_idx, g->inv_deg, g->col_inv_deg,
              X, ldx, Y, ldy, add, ld_add, mask, ld_mask};
  const int rows_per_block = 4 * (64 >> lpr_log2);
  const int blocks = (int)ceil_div(g->n_nodes, rows_per_block);
  const double bytes = (double)g->n_nodes * width * 12.0 + 4.0 * (double)g->nnz + 8.0 * g->n_nodes;
  ProfScope ps("mpnn_aggregate_transposed", st, 0.0, bytes);
  hipLaunchKernelGGL(k_agg_t_bf16, dim3(blocks), dim3(256), 0, st, a);
  CPRA_CHECK_LAUNCH("mpnn aggregate");
  return CPRA_OK;
}

cpra_status rows_gemm(const RowsArgs& a0, hipStream_t st) {
  RowsArgs a = a0;
  a.tiles = (int)ceil_div(a.M, 32);
  if (a.M == 0) return CPRA_OK;
  const int blocks = (int)std::min<int64_t>(ceil_div(a.tiles, 4), 2048);
  const double flops = 2.0 * a.M * (double)a.n_out * a.k_total;
  const double bytes = (double)a.M * (2.0 * a.k_total + 4.0 * a.n_out);
  ProfScope ps("mpnn_gemm_bf16", st, flops, bytes);
  switch (a.n_out / 32) {
    case 1: hipLaunchKernelGGL((k_rows_mfma<1>), dim3(blocks), dim3(256), 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_rows_mfma<2>), dim3(blocks), dim3(256), 0, st, a); break;
    case 3: hipLaunchKernelGGL((k_rows_mfma<3>), dim3(blocks), dim3(256), 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_rows_mfma<4>), dim3(blocks), dim3(256), 0, st, a); break;
    default: CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn gemm: n_out %d", a.n_out);
  }
  CPRA_CHECK_LAUNCH("mpnn gemm");
  return CPRA_OK;
}

cpra_status wgrad(const MPlan& p, int k, const uint16_t* dY, const uint16_t* H, float* grads,
                  void* ws, hipStream_t st) {
  const MLayer& l = p.layer[k];
  WgArgs a{};
  a.M = p.N;
  a.n_o = l.out;
  a.n_c = 2 * l.in;
  a.c0 = l.in;
  a.dY = dY;
  a.lddy = l.out;
  a.X0 = H;
  a.ldx0 = l.in;
  a.X1 = at<uint16_t>(ws, p.a_off[k]);
  a.ldx1 = l.in;
  a.rows_per_block = (int)std::max<int64_t>(64, ceil_div(ceil_div(p.N, kMaxWgBlocks), 64) * 64);
  a.partial = at<float>(ws, p.part_off);
  const int blocks = std::max(1, (int)ceil_div(p.N, a.rows_per_block));
  const int n_tiles = (a.n_o / 32) * (a.n_c / 32);
  const int tpw = (n_tiles + 3) / 4;
  {
    const double flops = 2.0 * p.N * (double)a.n_o * a.n_c;
    const double bytes = (double)p.N * 2.0 * (a.n_o + a.n_c) + 4.0 * blocks * a.n_o * (a.n_c + 1);
    ProfScope ps("mpnn_wgrad_bf16", st, flops, bytes);
    switch (tpw) {
      case 1: hipLaunchKernelGGL((k_wgrad_mfma<1>), dim3(blocks), dim3(256), 0, st, a); break;
      case 2: hipLaunchKernelGGL((k_wgrad_mfma<2>), dim3(blocks), dim3(256), 0, st, a); break;
      case 3: hipLaunchKernelGGL((k_wgrad_mfma<3>), dim3(blocks), dim3(256), 0, st, a); break;
      case 4: hipLaunchKernelGGL((k_wgrad_mfma<4>), dim3(blocks), dim3(256), 0, st, a); break;
      default: CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn wgrad: %d tiles", n_tiles);
    }
    CPRA_CHECK_LAUNCH("mpnn wgrad");
  }
  const int per = a.n_o * (a.n_c + 1);
  ProfScope ps("mpnn_wgrad_reduce", st, 0.0, 4.0 * (double)blocks * per + 4.0 * per);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)ceil_div(per, 256)), dim3(256), 0, st, blocks,
                     a.n_o, a.n_c, a.c0, a.partial, grads + l.off_ws, grads + l.off_wn,
                     grads + l.off_b);
  CPRA_CHECK_LAUNCH("mpnn wgrad reduce");
  return CPRA_OK;
}

template <int NT>
cpra_status launch_layer(int ki, const LayerArgs& a, dim3 grid, hipStream_t st) {
  switch (ki) {
    case 1: hipLaunchKernelGGL((k_mpnn_layer<NT, 1>), grid, dim3(256), 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_mpnn_layer<NT, 2>), grid, dim3(256), 0, st, a); break;
    case 3: hipLaunchKernelGGL((k_mpnn_layer<NT, 3>), grid, dim3(256), 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_mpnn_layer<NT, 4>), grid, dim3(256), 0, st, a); break;
    default: CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn layer: in %d", 16 * ki);
  }
  CPRA_CHECK_LAUNCH("mpnn layer");
  return CPRA_OK;
}

cpra_status mpnn_forward_impl(const cpra_csr* g, const MPlan& p, const float* params,
                              const uint16_t* feat, float* Zw, void* ws, hipStream_t st) {
  uint16_t* wbf = at<uint16_t>(ws, p.wbf_off);
  const uint16_t* H = feat;
  for (int k = 0; k < p.L; ++k) {
    const MLayer& l = p.layer[k];
    const bool last = k == p.L - 1;
    LayerArgs a{};
    a.n = p.N;
    a.tiles = (int)ceil_div(p.N, 32);
    a.row_ptr = g->row_ptr;
    a.col_idx = g->col_idx;
    a.inv_deg = g->inv_deg;
    a.H = H;
    a.A = at<uint16_t>(ws, p.a_off[k]);
    a.Ws = params + l.off_ws;
    a.Wn = params + l.off_wn;
    a.ws_bf = wbf + l.off_ws;
    a.wn_bf = wbf + l.off_wn;
    a.bias = params + l.off_b;
    a.relu = last ? 0 : 1;
    if (last) a.Cf = Zw; else a.Cb = at<uint16_t>(ws, p.h_off[k + 1]);
    const double n = p.N;
    ProfScope ps("mpnn_layer_bf16", st, 4.0 * n * l.out * l.in,
                 n * (4.0 * l.in + (last ? 4.0 : 2.0) * l.out) + 4.0 * (double)g->nnz + 8.0 * n,
                 2.0 * (double)g->nnz * l.in);
    const dim3 grid((unsigned)ceil_div(a.tiles, 4));
    switch (l.out / 32) {
      case 1: CPRA_CHECK(launch_layer<1>(l.in / 16, a, grid, st)); break;
      case 2: CPRA_CHECK(launch_layer<2>(l.in / 16, a, grid, st)); break;
      case 3: CPRA_CHECK(launch_layer<3>(l.in / 16, a, grid, st)); break;
      case 4: CPRA_CHECK(launch_layer<4>(l.in / 16, a, grid, st)); break;
      default: CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn layer: n_out %d", l.out);
    }
    if (!last) H = at<uint16_t>(ws, p.h_off[k + 1]);
  }
  return CPRA_OK;
}

cpra_status mpnn_backward_impl(const cpra_csr* g, const MPlan& p, const uint16_t* feat,
                               const float* dZw, float* grads, void* ws, hipStream_t st) {
  const uint16_t* wbf = at<uint16_t>(ws, p.wbf_off);
  const MLayer& lo = p.layer[p.L - 1];
  uint16_t* dY = at<uint16_t>(ws, p.dy_off[0]);
  {
    const int64_t total = (int64_t)p.N * lo.out;
    ProfScope ps("mpnn_cast", st, 0.0, 6.0 * (double)total);
    hipLaunchKernelGGL(k_cast_rows_bf16, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, st,
                       p.N, lo.out, dZw, (int64_t)lo.out, dY, (int64_t)lo.out);
    CPRA_CHECK_LAUNCH("mpnn cast");
  }
  int cur = 0;
  for (int k = p.L - 1; k >= 0; --k) {
    const MLayer& l = p.layer[k];
    const uint16_t* H = k == 0 ? feat : at<uint16_t>(ws, p.h_off[k]);
    CPRA_CHECK(wgrad(p, k, dY, H, grads, ws, st));
    if (k == 0) break;
    float* G = at<float>(ws, p.g_off);
    RowsArgs r{};
    r.M = p.N;
    r.n_out = 2 * l.in;
    r.k_total = l.out;
    r.A = dY;
    r.lda = l.out;
    r.B[0] = wbf + l.off_ws;
    r.B[1] = wbf + l.off_wn;
    r.n_half = l.in;
    r.C = G;
    r.ldc = 2 * l.in;
    CPRA_CHECK(rows_gemm(r, st));
    uint16_t* dYn = at<uint16_t>(ws, p.dy_off[cur ^ 1]);
    CPRA_CHECK(agg_t_bf16(g, l.in, G + l.in, 2 * l.in, dYn, l.in, G, 2 * l.in, H, l.in, st));
    dY = dYn;
    cur ^= 1;
  }
  return CPRA_OK;
}

cpra_status check_graph_mpnn(const cpra_csr* g, const cpra_mpnn_cfg* cfg, const char* who) {
  CPRA_CHECK(check_csr(g, who, true, false));
  CPRA_CHECK(check_mpnn_cfg(cfg));
  return CPRA_OK;
}

}  // namespace
}  // namespace cpra

extern "C" {

cpra_status cpra_node_features(const cpra_csr* g, int32_t in_dim, int32_t n_rand,
                               const float* rand, int64_t ld_rand, uint16_t* feat, int64_t ld_feat,
                               int64_t* triangles, cpra_stream_t stream) {
  using namespace cpra;
  CPRA_CHECK(check_csr(g, "node_features", false, false));
  if (n_rand < 0 || in_dim < 2 + n_rand)
    CPRA_FAIL(CPRA_ERR_SHAPE, "node_features: in_dim %d < 2 + n_rand %d", in_dim, n_rand);
  if (ld_feat < in_dim || (n_rand > 0 && ld_rand < n_rand))
    CPRA_FAIL(CPRA_ERR_SHAPE, "node_features: leading dimension smaller than the row");
  if (g->n_nodes == 0) return CPRA_OK;
  if (feat == nullptr || (n_rand > 0 && rand == nullptr))
    CPRA_FAIL(CPRA_ERR_NULL, "node_features: feat or rand is NULL");
  hipStream_t st = as_stream(stream);
  const double bytes = 2.0 * g->n_nodes * (double)in_dim + 4.0 * g->n_nodes * (double)n_rand +
                       (triangles ? 8.0 : 0.0) * g->n_nodes + 4.0 * (double)g->nnz +
                       4.0 * (g->n_nodes + 1.0);
  ProfScope ps("node_features", st, 0.0, bytes);
  const int64_t n = g->n_nodes;
  const bool four = (n >= 8192 && g->nnz <= 24 * n) || (n >= 4096 && g->nnz <= 12 * n);
  auto* const kernel = four ? k_node_features<16> : k_node_features<64>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(g->n_nodes, four ? 16 : 4)), dim3(256), 0, st,
                     g->n_nodes, g->row_ptr, g->col_idx, in_dim, n_rand, rand, ld_rand, feat,
                     ld_feat, triangles);
  CPRA_CHECK_LAUNCH("node_features");
  return CPRA_OK;
}

int64_t cpra_mpnn_param_count(const cpra_mpnn_cfg* cfg) {
  if (cpra::check_mpnn_cfg(cfg) != CPRA_OK) return -1;
  cpra::MPlan p{};
  cpra::make_mplan(cfg, 0, &p);
  return p.n_params;
}

cpra_status cpra_mpnn_param_offsets(const cpra_mpnn_cfg* cfg, int64_t* offsets) {
  using namespace cpra;
  CPRA_CHECK(check_mpnn_cfg(cfg));
  if (offsets == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "mpnn_param_offsets: offsets is NULL");
  MPlan p{};
  make_mplan(cfg, 0, &p);
  for (int k = 0; k < p.L; ++k) {
    offsets[3 * k] = p.layer[k].off_ws;
    offsets[3 * k + 1] = p.layer[k].off_wn;
    offsets[3 * k + 2] = p.layer[k].off_b;
  }
  return CPRA_OK;
}

size_t cpra_mpnn_workspace_bytes(const cpra_csr* g, const cpra_mpnn_cfg* cfg) {
  if (g == nullptr || cpra::check_mpnn_cfg(cfg) != CPRA_OK) return 0;
  cpra::MPlan p{};
  cpra::make_mplan(cfg, g->n_nodes, &p);
  return p.total;
}

cpra_status cpra_mpnn_forward(const cpra_csr* g, const cpra_mpnn_cfg* cfg, const float* params,
                              const uint16_t* feat, float* Zw, void* ws, size_t ws_bytes,
                              cpra_stream_t stream) {
  using namespace cpra;
  CPRA_CHECK(check_graph_mpnn(g, cfg, "mpnn_forward"));
  MPlan p{};
  make_mplan(cfg, g->n_nodes, &p);
  if (ws == nullptr || ws_bytes < p.total)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "mpnn_forward: workspace %zu < %zu bytes", ws_bytes, p.total);
  if (!params || !feat || (g->n_nodes > 0 && !Zw)) CPRA_FAIL(CPRA_ERR_NULL, "mpnn_forward: NULL buffer");
  if (reinterpret_cast<uintptr_t>(feat) % 16 != 0)
    CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn_forward: feat must be 16-byte aligned");
  if (g->n_nodes == 0) return CPRA_OK;
  return mpnn_forward_impl(g, p, params, feat, Zw, ws, as_stream(stream));
}

cpra_status cpra_mpnn_backward(const cpra_csr* g, const cpra_mpnn_cfg* cfg, const uint16_t* feat,
                               const float* dZw, float* grads, void* ws, size_t ws_bytes,
                               cpra_stream_t stream) {
  using namespace cpra;
  CPRA_CHECK(check_graph_mpnn(g, cfg, "mpnn_backward"));
  MPlan p{};
  make_mplan(cfg, g->n_nodes, &p);
  if (ws == nullptr || ws_bytes < p.total)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "mpnn_backward: workspace %zu < %zu bytes", ws_bytes, p.total);
  if (!feat || !grads || (g->n_nodes > 0 && !dZw)) CPRA_FAIL(CPRA_ERR_NULL, "mpnn_backward: NULL buffer");
  if (reinterpret_cast<uintptr_t>(feat) % 16 != 0)
    CPRA_FAIL(CPRA_ERR_SHAPE, "mpnn_backward: feat must be 16-byte aligned");
  if (g->n_nodes == 0) {  // no rows: every gradient is an empty sum
    hipLaunchKernelGGL(k_zero, dim3((unsigned)ceil_div(p.n_params, 256)), dim3(256), 0,
                       as_stream(stream), p.n_params, grads);
    CPRA_CHECK_LAUNCH("mpnn_backward");
    return CPRA_OK;
  }
  return mpnn_backward_impl(g, p, feat, dZw, grads, ws, as_stream(stream));
}

cpra_status cpra_mpnn_saved(const cpra_csr* g, const cpra_mpnn_cfg* cfg, void* ws, size_t ws_bytes,
                            int32_t layer, int32_t which, const uint16_t** out, int64_t* ld) {
  using namespace cpra;
  CPRA_CHECK(check_graph_mpnn(g, cfg, "mpnn_saved"));
  if (out == nullptr || ld == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "mpnn_saved: NULL output");
  MPlan p{};
  make_mplan(cfg, g->n_nodes, &p);
  if (ws == nullptr || ws_bytes < p.total)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "mpnn_saved: workspace %zu < %zu bytes", ws_bytes, p.total);
  if (layer < 0 || layer >= p.L || which < 0 || which > 1 || (which == 0 && layer == 0))
    CPRA_FAIL(CPRA_ERR_PARAM, "mpnn_saved: no saved tensor (%d, %d)", layer, which);
  *out = at<uint16_t>(ws, which == 0 ? p.h_off[layer] : p.a_off[layer]);
  *ld = p.layer[layer].in;
  return CPRA_OK;
}

cpra_status cpra_bce_grad(int32_t n_rows, int32_t S, const float* Z, int64_t ldz,
                          const uint8_t* target, int64_t ldt, float beta, float* dZ, int64_t lddz,
                          cpra_stream_t stream) {
  using namespace cpra;
  if (n_rows < 0 || S < 0 || ldz < S || ldt < S || lddz < S)
    CPRA_FAIL(CPRA_ERR_SHAPE, "bce_grad: bad sizes");
  if (!std::isfinite(beta)) CPRA_FAIL(CPRA_ERR_NONFINITE, "bce_grad: beta is not finite");
  const int64_t total = (int64_t)n_rows * S;
  if (total == 0) return CPRA_OK;
  if (!Z || !target || !dZ) CPRA_FAIL(CPRA_ERR_NULL, "bce_grad: NULL buffer");
  hipStream_t st = as_stream(stream);
  ProfScope ps("bce_grad", st, 0.0, 13.0 * (double)total);
  hipLaunchKernelGGL(k_bce_grad, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, st, n_rows, S,
                     Z, ldz, target, ldt, beta, dZ, lddz);
  CPRA_CHECK_LAUNCH("bce_grad");
  return CPRA_OK;
}

size_t cpra_mpnn_train_step_workspace_bytes(const cpra_csr* g, const cpra_mpnn_step_cfg* cfg) {
  if (g == nullptr || cfg == nullptr || cpra::check_mpnn_cfg(&cfg->net) != CPRA_OK) return 0;
  cpra::MPlan p{};
  cpra::make_mplan(&cfg->net, g->n_nodes, &p);
  return cpra::align_up(p.total, 256) + cpra::loss_workspace_bytes(g, cfg->net.S, true);
}

cpra_status cpra_mpnn_train_step(const cpra_csr* g, const cpra_mpnn_step_cfg* cfg, float* params,
                                 float* grads, float* m, float* v, const uint16_t* feat,
                                 const uint8_t* target, float* Zw, float* dZw, double* terms,
                                 int32_t t, int32_t* step_counter, void* ws, size_t ws_bytes,
                                 cpra_stream_t stream) {
  using namespace cpra;
  if (cfg == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "mpnn_train_step: cfg is NULL");
  CPRA_CHECK(check_graph_mpnn(g, &cfg->net, "mpnn_train_step"));
  cpra_loss_cfg lc = cfg->loss;
  lc.step_counter = step_counter;
  if (lc.S != cfg->net.S) CPRA_FAIL(CPRA_ERR_PARAM, "mpnn_train_step: loss.S != net.S");
  CPRA_CHECK(check_loss_cfg_public(g, &lc));
  CPRA_CHECK(check_adam_cfg(&cfg->adam));
  if (!std::isfinite(cfg->beta)) CPRA_FAIL(CPRA_ERR_NONFINITE, "mpnn_train_step: beta is not finite");
  if (step_counter == nullptr && t < 1) CPRA_FAIL(CPRA_ERR_PARAM, "mpnn_train_step: t must be >= 1");
  if (g->n_nodes == 0) return CPRA_OK;
  if (!params || !grads || !m || !v || !feat || !Zw || !dZw)
    CPRA_FAIL(CPRA_ERR_NULL, "mpnn_train_step: NULL buffer");
  MPlan p{};
  make_mplan(&cfg->net, g->n_nodes, &p);
  const size_t net_bytes = align_up(p.total, 256);
  const size_t need = net_bytes + loss_workspace_bytes(g, cfg->net.S, true);
  if (ws == nullptr || ws_bytes < need)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "mpnn_train_step: workspace %zu < %zu bytes", ws_bytes, need);
  hipStream_t st = as_stream(stream);
  const int S = cfg->net.S;
  void* loss_ws = static_cast<char*>(ws) + net_bytes;
  CPRA_CHECK(mpnn_forward_impl(g, p, params, feat, Zw, ws, st));
  CPRA_CHECK(loss_fwd_bwd(g, &lc, Zw, S, nullptr, 0, dZw, S, nullptr, loss_ws, ws_bytes - net_bytes,
                          st, terms != nullptr));
  if (terms) {
    CPRA_CHECK(loss_terms_reduce(g, &lc, terms, loss_ws, st, step_counter));
  } else if (step_counter) {
    CPRA_CHECK(increment_counter(step_counter, st));
  }
  if (target && cfg->beta != 0.0f) {
    const int64_t total = (int64_t)g->n_nodes * S;
    ProfScope ps("bce_grad", st, 0.0, 13.0 * (double)total);
    hipLaunchKernelGGL(k_bce_grad, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, st,
                       g->n_nodes, S, Zw, (int64_t)S, target, (int64_t)S, cfg->beta, dZw, (int64_t)S);
    CPRA_CHECK_LAUNCH("bce_grad");
  }
  CPRA_CHECK(mpnn_backward_impl(g, p, feat, dZw, grads, ws, st));
  CPRA_CHECK(adam_step(p.n_params, params, grads, m, v, &cfg->adam, t, step_counter, st,
                       /*t_offset=*/0));
  return CPRA_OK;
}

}  // extern "C"
