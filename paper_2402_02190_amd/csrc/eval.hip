// Threshold rounding and exact integer evaluation of the S solutions
// (training-setting appendix: P <= 0.5 -> 0, P > 0.5 -> 1, i.e. x = [Z > 0];
// objective table; Sec. 4.1 Evaluation Metrics; Proposition 3.2).
//
// Same lane layout as the loss kernel: 64/LPR nodes per wavefront, the LPR
// lanes of a node cover its heads.  Each edge {i, j} is visited from its
// smaller endpoint only.  Integer counts are summed per block and added with
// 64-bit integer atomics (exact, so order does not matter); weighted values
// (the cut weight of MaxCut, the set weight of weighted MIS) go through
// per-item FP64 partials and the fixed-order segmented reduction.  With
// per-head edge weights head s is evaluated on its own instance: only edges
// with a nonzero weight in head s count, with that weight.
#include <algorithm>

#include "common.hpp"

namespace cpra {

namespace {

// x = [Z > 0] decided on the bit pattern: +0 and negatives (sign bit set) give
// 0, every positive value from the smallest subnormal to +inf gives 1, NaN 0.
// The result does not depend on the wavefront's denormal mode.
__device__ inline bool rounds_to_one(float z) {
  const int32_t b = __float_as_int(z);
  return b > 0 && b <= 0x7f800000;
}

struct EvalArgs {
  int n, S, problem, lpr_log2;
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const float* weight;
  const float* Z;
  int64_t ldz;
  uint8_t* X;
  int64_t ldx;
  int64_t* value;
  int64_t* viol;
  int64_t* pairham;
  double* wpart;
  int64_t items_cap;
  int n_graphs;
  const int32_t* graph_ptr;
  const int32_t* item_ptr;
  int R;
  const float* node_w;  // MIS node weights or null (weight 1)
  int64_t ld_nw;        // 0: one weight per node
  const float* edge_w;  // per-head edge weights [nnz, ld_ew] or null
  int64_t ld_ew;
};

template <typename T>
__device__ inline T xor_sum(T v, int from_mask, int to_mask) {
  for (int m = from_mask; m < to_mask; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

template <int NC>
__global__ __launch_bounds__(256) void k_round_eval(EvalArgs a) {
  int g, r0, r1;
  if (!item_rows(blockIdx.x, a.n_graphs, a.n, a.graph_ptr, a.item_ptr, a.R, &g, &r0, &r1)) return;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int lpr = 1 << a.lpr_log2;
  const int rpw = 64 >> a.lpr_log2;
  const int sub = lane >> a.lpr_log2;
  const int cl = lane & (lpr - 1);
  const int S = a.S;
  const bool mis = a.problem == CPRA_MIS;

  int c_val[NC], c_vio[NC];
  double c_w[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    c_val[c] = 0;
    c_vio[c] = 0;
    c_w[c] = 0.0;
  }
  long long pair = 0;

  for (int base = r0; base < r1; base += 4 * rpw) {
    const int row = base + wave * rpw + sub;
    const bool active = row < r1;
    int x[NC];
    int k_row = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int s = c * lpr + cl;
      x[c] = (active && s < S && rounds_to_one(a.Z[(int64_t)row * a.ldz + s])) ? 1 : 0;
      k_row += x[c];
      if (active && s < S && a.X) a.X[(int64_t)row * a.ldx + s] = (uint8_t)x[c];
    }
    if (active) {
      if (mis) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int s = c * lpr + cl;
          c_val[c] += x[c];
          if (x[c] && s < S)
            c_w[c] += a.node_w ? (double)a.node_w[a.ld_nw ? (int64_t)row * a.ld_nw + s
                                                            : (int64_t)row]
                               : 1.0;
        }
      }
      const int beg = a.row_ptr[row], end = a.row_ptr[row + 1];
      for (int k = beg; k < end; ++k) {
        const int j = a.col_idx[k];
        if (j <= row) continue;
        const float w0 = a.weight ? a.weight[k] : 1.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int s = c * lpr + cl;
          if (s >= S) continue;
          const float w = a.edge_w ? a.edge_w[(int64_t)k * a.ld_ew + s] : w0;
          if (a.edge_w && w == 0.0f) continue;  // not an edge of head s's instance
          const int xj = rounds_to_one(a.Z[(int64_t)j * a.ldz + s]) ? 1 : 0;
          if (mis) {
            c_vio[c] += x[c] & xj;
          } else if (x[c] != xj) {
            c_val[c] += 1;
            c_w[c] += (double)w;
          }
        }
      }
    }
    k_row = xor_sum<int>(k_row, 1, lpr);
    if (active && cl == 0) pair += (long long)k_row * (long long)(S - k_row);
  }

  __shared__ int sh_val[4][NC * 64];
  __shared__ int sh_vio[4][NC * 64];
  __shared__ double sh_w[4][NC * 64];
  __shared__ long long sh_pair[4];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int v1 = xor_sum<int>(c_val[c], lpr, 64);
    const int v2 = xor_sum<int>(c_vio[c], lpr, 64);
    const double v3 = xor_sum<double>(c_w[c], lpr, 64);
    if (sub == 0) {
      sh_val[wave][c * lpr + cl] = v1;
      sh_vio[wave][c * lpr + cl] = v2;
      sh_w[wave][c * lpr + cl] = v3;
    }
  }
  const long long pr = xor_sum<long long>(pair, 1, 64);
  if (lane == 0) sh_pair[wave] = pr;
  __syncthreads();
  for (int s = threadIdx.x; s < NC * lpr; s += 256) {
    if (s >= S) continue;
    const long long v1 = (long long)sh_val[0][s] + sh_val[1][s] + sh_val[2][s] + sh_val[3][s];
    const long long v2 = (long long)sh_vio[0][s] + sh_vio[1][s] + sh_vio[2][s] + sh_vio[3][s];
    if (a.value && v1) atomicAdd(reinterpret_cast<unsigned long long*>(a.value + (int64_t)g * S + s),
                                 (unsigned long long)v1);
    if (a.viol && v2) atomicAdd(reinterpret_cast<unsigned long long*>(a.viol + (int64_t)g * S + s),
                                (unsigned long long)v2);
    if (a.wpart)
      a.wpart[(int64_t)s * a.items_cap + blockIdx.x] =
          ((sh_w[0][s] + sh_w[1][s]) + sh_w[2][s]) + sh_w[3][s];
  }
  if (threadIdx.x == 0 && a.pairham) {
    const long long t = sh_pair[0] + sh_pair[1] + sh_pair[2] + sh_pair[3];
    if (t) atomicAdd(reinterpret_cast<unsigned long long*>(a.pairham + g), (unsigned long long)t);
  }
}

// ---- unweighted scoring on bit-packed solutions ------------------------------
// Two passes: k_round_pack rounds Z once, writes X and one 64-bit word per row and
// 64 heads (ballots), and counts set sizes and pair products; k_edge_counts gathers
// 8 bytes per neighbour instead of a row of Z and counts x_i & x_j (MIS violations)
// or x_i ^ x_j (cut edges) for 64 heads at a time in bit-sliced counters.  What bounds
// it: the one read of Z (25.6 MB at N = 100,000, S = 64) and, in the second pass, the
// latency of two dependent loads per neighbour chunk.  N = 100,000, 20-regular,
// S = 64: 298 us for the row-gathering kernel above, 34 for the whole call here
// (47 with one head per lane in the first pass, 14 of it the second pass).
constexpr int kPackRows = 256;  // rows per item

struct PackArgs {
  int n, S, words, lpr_log2;
  const float* Z;
  int64_t ldz;
  uint8_t* X;
  int64_t ldx;
  int64_t* value;  // set sizes (MIS), or null
  int64_t* pairham;
  uint64_t* bits;  // [words][n]
  int n_graphs;
  const int32_t* graph_ptr;
  const int32_t* item_ptr;
};

// The bit of a word's head h: h itself, or with float4 rows (V4, 16 lanes of 4 heads)
// bit 16 e + c for head 4 c + e, as the four ballots of a row give them.
template <bool V4>
__global__ __launch_bounds__(256) void k_round_pack(PackArgs a) {
  int g, r0, r1;
  if (!item_rows(blockIdx.x, a.n_graphs, a.n, a.graph_ptr, a.item_ptr, kPackRows, &g, &r0, &r1)) return;
  constexpr int E = V4 ? 4 : 1;  // heads per lane
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lpr_log2 = V4 ? 4 : a.lpr_log2;
  const int lpr = 1 << lpr_log2, rpw = 64 >> lpr_log2;
  const int sub = lane >> lpr_log2, cl = lane & (lpr - 1);
  const int S = a.S;
  __shared__ int ones[kPackRows];       // ones of each row over the heads
  __shared__ int sh_val[4][64];
  __shared__ long long sh_pair[4];
  ones[threadIdx.x] = 0;
  __syncthreads();
  constexpr int U = 8;  // rows in flight per lane
  for (int w = 0; w < a.words; ++w) {
    const int s = w * 64 + E * cl;
    int cnt[E] = {};
    for (int base = r0 + wave * rpw; base < r1; base += 4 * rpw * U) {
      float z[U][E];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int row = base + u * 4 * rpw + sub;
        const bool in = row < r1 && s < S;
        const float* p = a.Z + (int64_t)row * a.ldz + s;
        if constexpr (V4) {
          const float4 x = in ? *reinterpret_cast<const float4*>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
          z[u][0] = x.x;
          z[u][1] = x.y;
          z[u][2] = x.z;
          z[u][3] = x.w;
        } else {
          z[u][0] = in ? *p : 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int row = base + u * 4 * rpw + sub;
        uint64_t word = 0;
        uint32_t bytes = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const bool one = rounds_to_one(z[u][e]);
          const uint64_t row_bits = (__ballot(one) >> (sub << lpr_log2)) & (~0ull >> (64 - lpr));
          word |= row_bits << (16 * e);
          bytes |= (uint32_t)one << (8 * e);
          cnt[e] += one;
        }
        if (row >= r1) continue;
        if (a.X && s < S) {
          uint8_t* x = a.X + (int64_t)row * a.ldx + s;
          if constexpr (V4) *reinterpret_cast<uint32_t*>(x) = bytes;
          else *x = (uint8_t)bytes;
        }
        if (cl == 0) {
          a.bits[(int64_t)w * a.n + row] = word;
          ones[row - r0] += __popcll(word);  // this lane's row only
        }
      }
    }
    if (a.value) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        for (int m = lpr; m < 64; m <<= 1) cnt[e] += __shfl_xor(cnt[e], m, 64);
        if (sub == 0) sh_val[wave][E * cl + e] = cnt[e];
      }
      __syncthreads();
      if (threadIdx.x < E * lpr && w * 64 + (int)threadIdx.x < S) {
        const int t = threadIdx.x;
        const long long v = (long long)sh_val[0][t] + sh_val[1][t] + sh_val[2][t] + sh_val[3][t];
        if (v) atomicAdd(reinterpret_cast<unsigned long long*>(a.value + (int64_t)g * S + w * 64 + t),
                         (unsigned long long)v);
      }
      __syncthreads();
    }
  }
  if (!a.pairham) return;
  __syncthreads();
  const long long k = ones[threadIdx.x];  // 0 past the item's rows
  const long long p = xor_sum<long long>(k * (S - k), 1, 64);
  if (lane == 0) sh_pair[wave] = p;
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long t = sh_pair[0] + sh_pair[1] + sh_pair[2] + sh_pair[3];
    if (t) atomicAdd(reinterpret_cast<unsigned long long*>(a.pairham + g), (unsigned long long)t);
  }
}

struct EdgeArgs {
  int n, S, cut;  // cut: count x_i ^ x_j, else x_i & x_j
  int v4;         // head order of the words (k_round_pack)
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const uint64_t* bits;
  int64_t* out;  // [n_graphs, S]
  int n_graphs;
  const int32_t* graph_ptr;
  const int32_t* item_ptr;
};

// Bit-sliced counters: plane p holds bit p of 64 counts.  Adds one word.
template <int NP>
__device__ __forceinline__ void bit_add(uint64_t (&c)[NP], uint64_t v) {
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const uint64_t t = c[p] & v;
    c[p] ^= v;
    v = t;
  }
}
// c += the counters of lane ^ mask (one plane more).
template <int NP>
__device__ __forceinline__ void bit_merge(const uint64_t (&c)[NP], uint64_t (&r)[NP + 1], int mask) {
  uint64_t carry = 0;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const uint64_t o = __shfl_xor((unsigned long long)c[p], mask, 64);
    const uint64_t x = c[p] ^ o;
    r[p] = x ^ carry;
    carry = (c[p] & o) | (carry & x);
  }
  r[NP] = carry;
}

// One thread per row, one 64-head word per blockIdx.y; each edge from its smaller
// endpoint.  A thread's counts stay below 64 between flushes; a flush sums the
// wavefront's counters (six butterfly stages) and lane s takes head s.
__global__ __launch_bounds__(256) void k_edge_counts(EdgeArgs a) {
  int g, r0, r1;
  if (!item_rows(blockIdx.x, a.n_graphs, a.n, a.graph_ptr, a.item_ptr, kPackRows, &g, &r0, &r1)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t* bits = a.bits + (int64_t)blockIdx.y * a.n;
  const int row = r0 + threadIdx.x;
  int k = 0, end = 0;
  uint64_t xi = 0;
  if (row < r1) {
    k = a.row_ptr[row];
    end = a.row_ptr[row + 1];
    xi = bits[row];
  }
  int total = 0;
  uint64_t c[6] = {0, 0, 0, 0, 0, 0};
  constexpr int CH = 8;  // neighbours per chunk; 7 chunks stay below 64
  int chunks = 0;
  auto flush = [&]() {
    uint64_t c1[7], c2[8], c3[9], c4[10], c5[11], c6[12];
    bit_merge(c, c1, 1);
    bit_merge(c1, c2, 2);
    bit_merge(c2, c3, 4);
    bit_merge(c3, c4, 8);
    bit_merge(c4, c5, 16);
    bit_merge(c5, c6, 32);
#pragma unroll
    for (int p = 0; p < 12; ++p) total += (int)((c6[p] >> lane) & 1) << p;
#pragma unroll
    for (int p = 0; p < 6; ++p) c[p] = 0;
    chunks = 0;
  };
  while (__any(k < end)) {
    int j[CH];
    uint64_t x[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) j[i] = k + i < end ? a.col_idx[k + i] : -1;
#pragma unroll
    for (int i = 0; i < CH; ++i) x[i] = j[i] > row ? bits[j[i]] : (a.cut ? xi : 0ull);
#pragma unroll
    for (int i = 0; i < CH; ++i) bit_add(c, a.cut ? xi ^ x[i] : xi & x[i]);
    k = min(k + CH, end);
    if (++chunks == 7) flush();  // uniform
  }
  if (chunks) flush();
  __shared__ int sh[4][64];
  sh[wave][lane] = total;
  __syncthreads();
  const int s = blockIdx.y * 64 + (a.v4 ? 4 * (lane & 15) + (lane >> 4) : lane);
  if (threadIdx.x < 64 && s < a.S) {
    const long long v = (long long)sh[0][lane] + sh[1][lane] + sh[2][lane] + sh[3][lane];
    if (v) atomicAdd(reinterpret_cast<unsigned long long*>(a.out + (int64_t)g * a.S + s), (unsigned long long)v);
  }
}

// p[0 .. n) = 0 for up to three arrays.
__global__ void k_clear3(int64_t* p0, int64_t n0, int64_t* p1, int64_t n1, int64_t* p2, int64_t n2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p0 && i < n0) p0[i] = 0;
  if (p1 && i < n1) p1[i] = 0;
  if (p2 && i < n2) p2[i] = 0;
}

struct EvalGeom {
  int lpr, lpr_log2, nc, R;
  int64_t items_cap;
};

EvalGeom eval_geom(const cpra_csr* g, int S) {
  EvalGeom G{};
  G.lpr = 1;
  while (G.lpr < S && G.lpr < 64) G.lpr <<= 1;
  while ((1 << G.lpr_log2) < G.lpr) ++G.lpr_log2;
  int need = (int)ceil_div(S, G.lpr);
  G.nc = 1;
  while (G.nc < need) G.nc <<= 1;
  G.R = 4 * (64 / G.lpr) * 2;
  G.items_cap = max_items(g, G.R);
  return G;
}

size_t eval_ws(const cpra_csr* g, int S, size_t* item_off, size_t* part_off) {
  EvalGeom G = eval_geom(g, S);
  size_t off = 0;
  *item_off = off;
  off += align_up((size_t)(g->n_graphs + 1) * sizeof(int32_t), 256);
  *part_off = off;
  off += align_up((size_t)S * G.items_cap * sizeof(double), 256);
  return off;
}

// The bit-packed path keeps its words in the place of the FP64 partials, which it has
// no use for.  Up to 16 heads they need more than those; a workspace without that
// room runs the row-gathering kernel.
inline size_t bits_bytes(const cpra_csr* g, int S) {
  return (size_t)g->n_nodes * ceil_div(S, 64) * sizeof(uint64_t);
}

}  // namespace

}  // namespace cpra

extern "C" {

size_t cpra_round_eval_workspace_bytes(const cpra_csr* g, int32_t S) {
  if (g == nullptr || S < 1) return 0;
  size_t item_off, part_off;
  const size_t need = cpra::eval_ws(g, S, &item_off, &part_off);
  return std::max(need, cpra::align_up(part_off + cpra::bits_bytes(g, S), 256));
}

cpra_status cpra_round_eval(const cpra_csr* g, int32_t problem, int32_t S, const float* Z,
                            int64_t ldz, uint8_t* X, int64_t ldx, int64_t* value,
                            int64_t* violations, double* wvalue, int64_t* pair_hamming,
                            const float* node_weight, int64_t ld_node_weight,
                            const float* edge_weight, int64_t ld_edge_weight, void* ws,
                            size_t ws_bytes, cpra_stream_t stream) {
  using namespace cpra;
  CPRA_CHECK(check_csr(g, "round_eval", false, false));
  if (problem != CPRA_MIS && problem != CPRA_MAXCUT)
    CPRA_FAIL(CPRA_ERR_PARAM, "round_eval: unknown problem %d", problem);
  if (S < 1 || S > 1024) CPRA_FAIL(CPRA_ERR_PARAM, "round_eval: S = %d outside 1..1024", S);
  if (g->n_nodes > 0 && Z == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "round_eval: Z is NULL");
  if (ldz < S || (X && ldx < S)) CPRA_FAIL(CPRA_ERR_SHAPE, "round_eval: leading dimension < S");
  if (node_weight && problem != CPRA_MIS)
    CPRA_FAIL(CPRA_ERR_PARAM, "round_eval: node weights are defined for MIS only");
  if (node_weight && ld_node_weight != 0 && ld_node_weight < S)
    CPRA_FAIL(CPRA_ERR_SHAPE, "round_eval: ld_node_weight must be 0 or >= S");
  if (edge_weight && ld_edge_weight < S)
    CPRA_FAIL(CPRA_ERR_SHAPE, "round_eval: ld_edge_weight must be >= S");
  size_t item_off, part_off;
  size_t need = eval_ws(g, S, &item_off, &part_off);
  if (ws == nullptr || ws_bytes < need)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "round_eval: workspace %zu < %zu bytes", ws_bytes, need);
  hipStream_t st = as_stream(stream);
  EvalGeom G = eval_geom(g, S);
  char* base = static_cast<char*>(ws);
  int32_t* item_ptr = reinterpret_cast<int32_t*>(base + item_off);
  double* wpart = wvalue ? reinterpret_cast<double*>(base + part_off) : nullptr;
  const bool packed = wvalue == nullptr && edge_weight == nullptr && g->n_nodes > 0 &&
                      bits_bytes(g, S) <= ws_bytes - part_off;
  CPRA_CHECK(launch_item_ptr(g, packed ? kPackRows : G.R, item_ptr, st));
  const int64_t n_gs = (int64_t)g->n_graphs * S;
  if (value || violations || pair_hamming) {
    hipLaunchKernelGGL(k_clear3, dim3((unsigned)ceil_div(n_gs, 256)), dim3(256), 0, st, value, n_gs, violations,
                       n_gs, pair_hamming, (int64_t)g->n_graphs);
    CPRA_CHECK_LAUNCH("round_eval clear");
  }
  const double work = 4.0 * (double)g->n_nodes * S + (X ? (double)g->n_nodes * S : 0.0) +
                      4.0 * (double)g->nnz * (edge_weight ? 1.0 + S : 1.0) + 4.0 * g->n_nodes;
  if (packed) {
    const int items = (int)max_items(g, kPackRows);
    const int32_t* gp = g->n_graphs > 1 ? g->graph_ptr : nullptr;
    uint64_t* bits = reinterpret_cast<uint64_t*>(base + part_off);
    const bool mis = problem == CPRA_MIS;
    int64_t* edges = mis ? violations : value;
    ProfScope ps("round_eval", st, 0.0, work);
    const PackArgs pa{g->n_nodes, S, (int)ceil_div(S, 64), G.lpr_log2, Z, ldz, X, ldx, mis ? value : nullptr,
                      pair_hamming, bits, g->n_graphs, gp, item_ptr};
    // float4 rows of Z and 4-byte stores of X where alignment allows
    const bool v4 = S % 4 == 0 && ldz % 4 == 0 && reinterpret_cast<uintptr_t>(Z) % 16 == 0 &&
                    (X == nullptr || (ldx % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 4 == 0));
    if (v4) hipLaunchKernelGGL(k_round_pack<true>, dim3(items), dim3(256), 0, st, pa);
    else hipLaunchKernelGGL(k_round_pack<false>, dim3(items), dim3(256), 0, st, pa);
    CPRA_CHECK_LAUNCH("round_pack");
    if (edges) {
      const EdgeArgs ea{g->n_nodes, S, mis ? 0 : 1, v4 ? 1 : 0, g->row_ptr, g->col_idx, bits, edges, g->n_graphs, gp, item_ptr};
      hipLaunchKernelGGL(k_edge_counts, dim3(items, (unsigned)ceil_div(S, 64)), dim3(256), 0, st, ea);
      CPRA_CHECK_LAUNCH("edge_counts");
    }
    return CPRA_OK;
  }
  EvalArgs a{};
  a.n = g->n_nodes;
  a.S = S;
  a.problem = problem;
  a.lpr_log2 = G.lpr_log2;
  a.row_ptr = g->row_ptr;
  a.col_idx = g->col_idx;
  a.weight = g->weight;
  a.Z = Z;
  a.ldz = ldz;
  a.X = X;
  a.ldx = ldx;
  a.value = value;
  a.viol = violations;
  a.pairham = pair_hamming;
  a.wpart = wpart;
  a.items_cap = G.items_cap;
  a.n_graphs = g->n_graphs;
  a.graph_ptr = g->n_graphs > 1 ? g->graph_ptr : nullptr;
  a.item_ptr = item_ptr;
  a.R = G.R;
  a.node_w = node_weight;
  a.ld_nw = ld_node_weight;
  a.edge_w = edge_weight;
  a.ld_ew = ld_edge_weight;
  const int blocks = (int)G.items_cap;
  ProfScope ps("round_eval", st, 0.0, work);
  switch (G.nc) {
#define CPRA_EVAL_CASE(NCV)                                                          \
  case NCV:                                                                          \
    hipLaunchKernelGGL(k_round_eval<NCV>, dim3(blocks), dim3(256), 0, st, a);        \
    break;
    CPRA_EVAL_CASE(1)
    CPRA_EVAL_CASE(2)
    CPRA_EVAL_CASE(4)
    CPRA_EVAL_CASE(8)
    CPRA_EVAL_CASE(16)
#undef CPRA_EVAL_CASE
    default:
      CPRA_FAIL(CPRA_ERR_PARAM, "round_eval: S too large");
  }
  CPRA_CHECK_LAUNCH("round_eval");
  if (wvalue)
    CPRA_CHECK(launch_segment_reduce(g, G.R, item_ptr, nullptr, wpart, G.items_cap, S, wvalue, st));
  return CPRA_OK;
}

}  // extern "C"
