// Mean aggregation M X and its transpose M^T X over a CSR graph (GNN appendix:
// Aggregate step with the 1/|N(v)| normalisation).
//
// Layout: a 64-lane wavefront holds 64/LPR rows; the LPR lanes of one row
// cover its columns in VEC-float vectors, NC vectors per lane.  A row's
// neighbour list is walked in chunks, a chunk's row gathers issued together;
// every gathered row segment is read as contiguous, coalesced vectors.  Sums
// run in CSR order, so results are deterministic.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace cpra {

namespace {

template <int VEC>
struct Vec;
template <>
struct Vec<1> {
  using T = float;
  __device__ static T zero() { return 0.0f; }
  __device__ static void axpy(T& acc, float s, const T& x) { acc += s * x; }
  __device__ static void add(T& acc, const T& x) { acc += x; }
};
template <>
struct Vec<2> {
  using T = float2;
  __device__ static T zero() { return make_float2(0.f, 0.f); }
  __device__ static void axpy(T& acc, float s, const T& x) { acc.x += s * x.x; acc.y += s * x.y; }
  __device__ static void add(T& acc, const T& x) { acc.x += x.x; acc.y += x.y; }
};
template <>
struct Vec<4> {
  using T = float4;
  __device__ static T zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ static void axpy(T& acc, float s, const T& x) {
    acc.x += s * x.x; acc.y += s * x.y; acc.z += s * x.z; acc.w += s * x.w;
  }
  __device__ static void add(T& acc, const T& x) {
    acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
  }
};

template <int VEC>
__device__ inline float comp(const typename Vec<VEC>::T& v, int e) {
  if constexpr (VEC == 1) return v;
  else if constexpr (VEC == 2) return e == 0 ? v.x : v.y;
  else return e == 0 ? v.x : (e == 1 ? v.y : (e == 2 ? v.z : v.w));
}
template <int VEC>
__device__ inline void set_comp(typename Vec<VEC>::T& v, int e, float x) {
  if constexpr (VEC == 1) v = x;
  else if constexpr (VEC == 2) { if (e == 0) v.x = x; else v.y = x; }
  else { if (e == 0) v.x = x; else if (e == 1) v.y = x; else if (e == 2) v.z = x; else v.w = x; }
}

// The mean's factor, rounded by itself (never fused with the addend that follows).
template <int VEC>
__device__ inline void scale(typename Vec<VEC>::T& v, float s) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < VEC; ++e) set_comp<VEC>(v, e, comp<VEC>(v, e) * s);
}

constexpr double kStreamOutBytes = 32.0 * 1024 * 1024;

constexpr int kSlice = 32;  // columns of a slice: one 128-byte line of a row

struct AggArgs {
  int n;
  int width;
  int lpr_log2;
  int slices_log2;  // column slices dealt to the XCDs (0: whole rows)
  int relu;
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const float* inv_deg;
  const float* col_inv_deg;  // inv_deg of each entry's column, or null (gathered instead)
  const float* X;
  int64_t ldx;
  float* Y;
  int64_t ldy;
  const float* add;
  int64_t ld_add;
  const float* bias;
  const float* mask;
  int64_t ld_mask;
  float* sig_out;  // optional sigmoid(Y) [N, width] (ld_sig)
  int64_t ld_sig;
  const float* add2;  // optional second addend [N, width] (ld_add2)
  int64_t ld_add2;
  unsigned nnz_bytes;  // of col_idx, where that fits
  int32_t* queue;  // persistent launches: the work queue (kQueueInts counters)
  int units;       // persistent launches: row blocks of 4 wavefronts
  int chunk;       // persistent launches: row blocks per dequeue
  int stream_out;  // streaming output stores (tables larger than L2)
};

// A streaming (nontemporal) store of one VEC-float vector.  Above kStreamOutBytes of
// output (more than the 8 XCDs' L2 together) the output rows, which this launch does
// not read again, are stored this way so that they take no L2 lines from the gathered
// table: C3 (a 182 MB table) 1.775 -> 1.751 ms per step, C4 (51 MB) and C3s (22 MB)
// unchanged; on C2 (10 MB) it cost 0.8%.  The index stream goes the same way with 64-bit
// addresses only: by buffer loads (NARROW) it is kept, as the slices of a row read it
// again (100,000 x 128, 20-regular: 145 us nontemporal, 103 kept).
template <int VEC>
__device__ inline void store_nt(const typename Vec<VEC>::T& v, float* p) {
  if constexpr (VEC == 1) {
    __builtin_nontemporal_store(v, p);
  } else {
    typedef float nv __attribute__((ext_vector_type(VEC)));
    nv x;
#pragma unroll
    for (int e = 0; e < VEC; ++e) x[e] = comp<VEC>(v, e);
    __builtin_nontemporal_store(x, reinterpret_cast<nv*>(p));
  }
}

__device__ inline float sigmoid_of(float z) {
  const float e = expf(-fabsf(z));
  const float r = recip_1_2(1.0f + e);
  return z >= 0.0f ? r : e * r;
}

// Row block `unit` (4 wavefronts of 64/LPR rows each).
//
// A row's entries go in chunks of CH, all gathers of a chunk in flight; the adds run in
// CSR order.  With one vector per lane each lane loads one of the chunk's entries and
// the row's others receive it by a permute.  Entries past the row's end are not gathered
// and add an exact zero (the sums never hold -0, so x + 0 = x).
//
// On sparse graphs the instructions bound it as much as memory does: with 64-bit
// addresses a gather spent about 60 cycles on multiplies for 16 of loading, every lane
// loaded every entry, and a chunk of the transposed gather waited for its entries before
// it asked for their factors.  NARROW (every operand below 4 GiB, n and the row strides
// in bytes below 2^24): one 24-bit multiply-add per gather, entries and factors loaded
// together.  252 graphs of 2,750 nodes, mean degree 7, 32 columns: 129 -> 113 us, and
// transposed 79 -> 73 us.  On one large 20-regular graph the L2 misses bound it
// (100,000 x 128: 137 us, 7.5 TB/s of rows; in column slices 103).
template <int VEC, int NC, bool TRANS, bool NARROW, int CH>
__device__ __forceinline__ void agg_unit(const AggArgs& a, int unit) {
  using V = typename Vec<VEC>::T;
  using O = Vec<VEC>;
  constexpr bool kEarly = !TRANS && NC <= 2;  // addends and mask in flight along with the gathers
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int lpr = 1 << a.lpr_log2;
  const int sub = lane >> a.lpr_log2;
  const int cl = lane & (lpr - 1);
  const int rpw = 64 >> a.lpr_log2;
  const int row = (unit * 4 + wave) * rpw + sub;
  const int units = a.width / VEC;
  const bool spread = NC == 1 && lpr >= CH;  // uniform
  const int first = (lane & ~(lpr - 1)) << 2;

  int k = 0, end = 0;
  if (row < a.n) {
    k = a.row_ptr[row];
    end = a.row_ptr[row + 1];
  }
  // Entry `at` of the CSR arrays and its factor (0 past the row's end).
  const unsigned nnz_b = NARROW ? a.nnz_bytes : 0;
  const __amdgpu_buffer_rsrc_t J = __builtin_amdgcn_make_buffer_rsrc((void*)a.col_idx, (short)0, nnz_b, 0x00020000);
  const __amdgpu_buffer_rsrc_t W = __builtin_amdgcn_make_buffer_rsrc((void*)a.col_inv_deg, (short)0, nnz_b, 0x00020000);
  auto entry = [&](int at, int* j, float* s) {
    const bool in = at < end;
    if constexpr (NARROW) {
      const unsigned off = in ? (unsigned)at * 4u : ~0u;  // past the buffer: reads as 0
      *j = (int)__builtin_amdgcn_raw_buffer_load_b32(J, off, 0, 0);
      if (TRANS) {
        if (a.col_inv_deg) *s = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(W, off, 0, 0));
        else *s = in ? a.inv_deg[*j] : 0.f;
      }
    } else {
      *j = 0;
      *s = 0.f;
      if (!in) return;
      *j = a.stream_out ? __builtin_nontemporal_load(a.col_idx + at) : a.col_idx[at];
      if (TRANS) *s = a.col_inv_deg ? a.col_inv_deg[at] : a.inv_deg[*j];
    }
  };

  // element u of row `row` of an operand of leading dimension ld
  auto at = [&](auto* p, int64_t ld, int u) {
    using P = decltype(p);
    using C = typename std::conditional<std::is_const<std::remove_pointer_t<P>>::value, const char, char>::type;
    if constexpr (NARROW)
      return reinterpret_cast<P>(reinterpret_cast<C*>(p) +
                                 (__umul24((unsigned)row, (unsigned)ld * 4u) + (unsigned)u * (VEC * 4u)));
    else
      return p + (int64_t)row * ld + u * VEC;
  };
  V acc[NC], ad[NC], ad2[NC], mk[NC];
  auto extras = [&](int c, int u) {
    if (a.add) ad[c] = *reinterpret_cast<const V*>(at(a.add, a.ld_add, u));
    if (a.add2) ad2[c] = *reinterpret_cast<const V*>(at(a.add2, a.ld_add2, u));
    if (a.mask) mk[c] = *reinterpret_cast<const V*>(at(a.mask, a.ld_mask, u));
  };
  unsigned col[NC];  // byte offset of the lane's vectors in a row (past the width: the last one again)
  float rs = 1.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    acc[c] = ad[c] = ad2[c] = mk[c] = O::zero();
    const int u = c * lpr + cl;
    col[c] = (unsigned)min(u, units - 1) * (VEC * 4u);
    if (kEarly && row < a.n && u < units) extras(c, u);
  }
  if (!TRANS && row < a.n) rs = a.inv_deg[row];

  const unsigned ldb = (unsigned)a.ldx * 4u;
  for (; k < end; k += CH) {
    int j[CH];
    float s[CH];
    if (spread) {
      int jl;
      float sl;
      entry(k + (cl & (CH - 1)), &jl, &sl);
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        j[i] = __builtin_amdgcn_ds_bpermute(first + 4 * i, jl);
        if (TRANS) s[i] = __int_as_float(__builtin_amdgcn_ds_bpermute(first + 4 * i, __float_as_int(sl)));
      }
    } else {
#pragma unroll
      for (int i = 0; i < CH; ++i) entry(k + i, &j[i], &s[i]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      V x[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        x[i] = O::zero();
        if (k + i < end) {
          const char* r = NARROW ? reinterpret_cast<const char*>(a.X) + (__umul24((unsigned)j[i], ldb) + col[c])
                                 : reinterpret_cast<const char*>(a.X + (int64_t)j[i] * a.ldx) + col[c];
          x[i] = *reinterpret_cast<const V*>(r);
        }
      }
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        if constexpr (TRANS) O::axpy(acc[c], s[i], x[i]); else O::add(acc[c], x[i]);
      }
    }
  }
  if (row >= a.n) return;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int u = c * lpr + cl;
    if (u >= units) continue;
    if (!kEarly) extras(c, u);
    V r = acc[c];
    if constexpr (!TRANS) scale<VEC>(r, rs);
    if (a.add) O::add(r, ad[c]);
    if (a.add2) O::add(r, ad2[c]);
    if (a.bias) O::add(r, *reinterpret_cast<const V*>(a.bias + u * VEC));
    if (a.relu || a.mask) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        float x = comp<VEC>(r, e);
        if (a.relu) x = fmaxf(x, 0.0f);
        if (a.mask && !(comp<VEC>(mk[c], e) > 0.0f)) x = 0.0f;
        set_comp<VEC>(r, e, x);
      }
    }
    if (a.stream_out) store_nt<VEC>(r, at(a.Y, a.ldy, u));
    else *reinterpret_cast<V*>(at(a.Y, a.ldy, u)) = r;
    if (a.sig_out) {
      V sg;
#pragma unroll
      for (int e = 0; e < VEC; ++e) set_comp<VEC>(sg, e, sigmoid_of(comp<VEC>(r, e)));
      *reinterpret_cast<V*>(at(a.sig_out, a.ld_sig, u)) = sg;
    }
  }
}

// One block per row block, in XCD order; with column slices, XCD x takes slice
// x % slices of its share of the rows, so that the table it gathers from is that much
// smaller against its L2.
template <int VEC, int NC, bool TRANS, bool NARROW, int CH>
__global__ __launch_bounds__(256) void k_aggregate(AggArgs a) {
  int unit = xcd_unit(blockIdx.x, gridDim.x);
  if (a.slices_log2) {
    const int xcd = blockIdx.x & 7;
    const int c0 = (xcd & ((1 << a.slices_log2) - 1)) * kSlice;
    unit = (xcd >> a.slices_log2) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    a.X += c0;
    a.Y += c0;
    if (a.add) a.add += c0;
    if (a.add2) a.add2 += c0;
    if (a.bias) a.bias += c0;
    if (a.mask) a.mask += c0;
    if (a.sig_out) a.sig_out += c0;
    a.width = kSlice;
  }
  agg_unit<VEC, NC, TRANS, NARROW, CH>(a, unit);
}

// Persistent: at most the resident blocks, each taking row blocks from the queue.
template <int VEC, int NC, bool TRANS, bool NARROW, int CH>
__global__ __launch_bounds__(256) void k_aggregate_persistent(AggArgs a) {
  __shared__ int s_chunk;
  const int chunks = (a.units + a.chunk - 1) / a.chunk;
  for (bool first = true;; first = false) {
    if (threadIdx.x == 0) s_chunk = queue_next(a.queue, chunks, first);
    __syncthreads();
    const int c = s_chunk;
    if (c < 0) break;  // uniform across the block
    const int u1 = min(a.units, (c + 1) * a.chunk);
    for (int u = c * a.chunk; u < u1; ++u) agg_unit<VEC, NC, TRANS, NARROW, CH>(a, u);
    __syncthreads();  // s_chunk is rewritten by the next dequeue
  }
}

inline bool aligned(const void* p, int bytes) {
  return p == nullptr || (reinterpret_cast<uintptr_t>(p) % bytes) == 0;
}

template <int VEC, bool TRANS, bool NARROW>
cpra_status launch_nc(const AggArgs& a, int nc, int blocks, hipStream_t stream, int64_t nnz) {
  // compulsory bytes: X once, Y written, add/mask read, CSR, inv_deg
  const double nw = (double)a.n * a.width * 4.0;
  const double bytes = nw * (2.0 + (a.add ? 1.0 : 0.0) + (a.add2 ? 1.0 : 0.0) +
                             (a.mask ? 1.0 : 0.0) + (a.sig_out ? 1.0 : 0.0)) +
                       4.0 * (double)nnz * (TRANS && a.col_inv_deg ? 2.0 : 1.0) +
                       8.0 * (double)a.n + 4.0;
  ProfScope ps(TRANS ? "aggregate_transposed" : "aggregate", stream, 0.0, bytes,
               4.0 * (double)nnz * a.width);
  if (a.queue) CPRA_CHECK(zero_queue(a.queue, stream));
  auto launch = [&](auto nc_, auto ch_) {
    constexpr int NCV = decltype(nc_)::value, CHV = decltype(ch_)::value;
    if (a.queue) {
      const int cap = resident_blocks(
          reinterpret_cast<const void*>(&k_aggregate_persistent<VEC, NCV, TRANS, NARROW, CHV>), 256);
      AggArgs ap = a;
      const int grid = std::min(a.units, cap);
      ap.chunk = queue_chunk(a.units, grid);
      hipLaunchKernelGGL((k_aggregate_persistent<VEC, NCV, TRANS, NARROW, CHV>), dim3(grid), dim3(256), 0, stream,
                         ap);
    } else {
      hipLaunchKernelGGL((k_aggregate<VEC, NCV, TRANS, NARROW, CHV>), dim3(blocks), dim3(256), 0, stream, a);
    }
  };
  // Chunks of 8 entries (of 4 for four vectors and more per lane, for the registers).
  // Column slices take chunks of 2 (100,000 x 128: 103 us, with 4 111, with 8 121, with
  // 1 112).  With two vectors per lane and a table of twice an XCD's L2 and more, 8
  // gathers per lane in flight only push each other's lines out: 20-regular, 100,000 x 32: 44 us
  // with chunks of 8 and 33 with chunks of 2 (transposed 45 and 42), 10,000 x 256: 20.6
  // and 17.4.  Below, the latency counts: 10,000 x 128: 10.2 and 11.7, 2,000 x 64: 4.9
  // and 5.6.
  const bool misses = (double)a.n * a.width * 4.0 > 8.0 * 1024 * 1024;
  switch (nc) {
    case 1:
      if (a.slices_log2) launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
      else launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
      break;
    case 2:
      if (misses) launch(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
      else launch(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
      break;
    case 4: launch(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{}); break;
    case 16: launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 4>{}); break;
    default:
      CPRA_FAIL(CPRA_ERR_SHAPE, "aggregate: width too large");
  }
  CPRA_CHECK_LAUNCH("aggregate");
  return CPRA_OK;
}

// Slices of 32 columns, one 128-byte line of a row, dealt to the XCDs: the XCDs of a
// slice share the rows, and each gathers from n lines instead of n rows, of which its
// 4 MB L2 holds that much more; a row's entries are read once per slice.  (One graph:
// the rows of a batch's graphs are dealt to the XCDs, and their tables are small.)
// Measured whole rows against slices, us, transposed gather in brackets:
//   256 columns from 8 MB on:  10,000 nodes, 5-regular 9.1, 6.7 (9.2, 6.8);
//                              50,000, 20-regular 130, 93 (135, 105)
//   128 columns from 12 MB on: 30,000, 5-regular 13.4, 11.1 (13.8, 11.5); 100,000,
//                              20-regular 133, 102 (141, 116); at 10 MB 16.7, 18.6
//   64 columns from 16 MB on and mean degree 12: 100,000, 20-regular 59, 52 (69, 57);
//                              50,000, 20-regular 22.0, 24.0; 100,000, 5-regular 22.0, 22.9
// Sparse graphs past 131,072 nodes keep whole rows (200,000, 5-regular, 128 columns: 83,
// 84 (85, 87)).
int slices_log2_of(const cpra_csr* g, int width, const float* X, int64_t ldx) {
  const bool dense = g->nnz >= 12 * (int64_t)g->n_nodes;
  const double mb = (double)g->n_nodes * width * 4.0 / (1024 * 1024);
  if (g->n_graphs != 1 || ldx % kSlice != 0 || !aligned(X, 4 * kSlice)) return 0;
  if (!dense && g->n_nodes > 131072) return 0;
  if (width == 8 * kSlice) return mb >= 8 ? 3 : 0;
  if (width == 4 * kSlice) return mb >= 12 ? 2 : 0;
  if (width == 2 * kSlice) return dense && mb >= 16 ? 1 : 0;
  return 0;
}

template <bool NARROW>
cpra_status launch_vec(const AggArgs& a, bool transpose, int vec, int nc, int blocks, hipStream_t stream,
                       int64_t nnz) {
  if (transpose) {
    if (vec == 4) return launch_nc<4, true, NARROW>(a, nc, blocks, stream, nnz);
    if (vec == 2) return launch_nc<2, true, NARROW>(a, nc, blocks, stream, nnz);
    return launch_nc<1, true, NARROW>(a, nc, blocks, stream, nnz);
  }
  if (vec == 4) return launch_nc<4, false, NARROW>(a, nc, blocks, stream, nnz);
  if (vec == 2) return launch_nc<2, false, NARROW>(a, nc, blocks, stream, nnz);
  return launch_nc<1, false, NARROW>(a, nc, blocks, stream, nnz);
}

}  // namespace

cpra_status aggregate(const cpra_csr* g, bool transpose, int width, const float* X, int64_t ldx,
                      float* Y, int64_t ldy, const float* add, int64_t ld_add, const float* bias,
                      bool relu, const float* mask, int64_t ld_mask, hipStream_t stream,
                      float* sig_out, int64_t ld_sig, const float* add2, int64_t ld_add2,
                      int32_t* queue) {
  if (g->n_nodes == 0 || width == 0) return CPRA_OK;
  int vec = 1;
  for (int v : {4, 2}) {
    int vb = v * 4;
    if (width % v == 0 && ldx % v == 0 && ldy % v == 0 && (add == nullptr || ld_add % v == 0) &&
        (mask == nullptr || ld_mask % v == 0) && (sig_out == nullptr || ld_sig % v == 0) &&
        (add2 == nullptr || ld_add2 % v == 0) && aligned(X, vb) && aligned(Y, vb) &&
        aligned(add, vb) && aligned(bias, vb) && aligned(mask, vb) && aligned(sig_out, vb) &&
        aligned(add2, vb)) {
      vec = v;
      break;
    }
  }
  int units = width / vec;
  // On graphs of mean degree >= 12, two vectors per lane (twice the rows, and
  // their independent gathers, in flight per wavefront) measured faster: the
  // 20-regular 100,000-node aggregation 167 -> 151 us.  On sparser graphs
  // (mean degree ~7) the one-vector layout was faster (150 vs 178 us).
  const int per_lane = g->nnz >= 12 * (int64_t)g->n_nodes ? 2 : 1;
  const bool queued = queue && persistent_enabled();
  const int slices_log2 = vec == 4 && !queued ? slices_log2_of(g, width, X, ldx) : 0;
  if (slices_log2) units = kSlice / vec;
  int lpr = 1;
  while ((slices_log2 ? 1 : per_lane) * lpr < units && lpr < 64) lpr <<= 1;
  int lpr_log2 = 0;
  while ((1 << lpr_log2) < lpr) ++lpr_log2;
  int need = (int)ceil_div(units, lpr);
  int nc = 1;
  while (nc < need) nc <<= 1;
  if (nc > 16) CPRA_FAIL(CPRA_ERR_SHAPE, "aggregate: width %d exceeds 4096", width);
  int rows_per_block = 4 * (64 / lpr);
  const int units_rb = (int)ceil_div(g->n_nodes, rows_per_block);
  const int blocks =
      slices_log2 ? 8 * (int)ceil_div(units_rb, 8 >> slices_log2) : (int)xcd_grid(units_rb);
  AggArgs a{g->n_nodes, width, lpr_log2, slices_log2, relu ? 1 : 0, g->row_ptr, g->col_idx, g->inv_deg,
            g->col_inv_deg, X, ldx, Y, ldy, add, ld_add, bias, mask, ld_mask, sig_out, ld_sig, add2, ld_add2,
            (unsigned)(g->nnz * 4), queued ? queue : nullptr, units_rb, 1,
            (double)g->n_nodes * width * 4.0 > kStreamOutBytes ? 1 : 0};
  // 32-bit byte offsets where every one fits, from 24-bit factors.
  bool narrow = g->n_nodes < (1 << 24) && (int64_t)g->nnz * 4 < (int64_t)1 << 32;
  for (int64_t ld : {ldx, ldy, add ? ld_add : 0, mask ? ld_mask : 0, sig_out ? ld_sig : 0, add2 ? ld_add2 : 0})
    narrow = narrow && ld * 4 < (1 << 24) && (int64_t)g->n_nodes * ld * 4 < (int64_t)1 << 32;
  if (narrow) return launch_vec<true>(a, transpose, vec, nc, blocks, stream, g->nnz);
  return launch_vec<false>(a, transpose, vec, nc, blocks, stream, g->nnz);
}

}  // namespace cpra

extern "C" cpra_status cpra_aggregate_mean(const cpra_csr* g, int32_t transpose, int32_t width,
                                           const float* X, int64_t ldx, float* Y, int64_t ldy,
                                           const float* add, int64_t ld_add, const float* bias,
                                           int32_t relu, const float* mask, int64_t ld_mask,
                                           cpra_stream_t stream) {
  CPRA_CHECK(cpra::check_csr(g, "aggregate_mean", true, false));
  if (width < 0) CPRA_FAIL(CPRA_ERR_SHAPE, "aggregate_mean: width < 0");
  if (g->n_nodes > 0 && width > 0) {
    if (X == nullptr || Y == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "aggregate_mean: X or Y is NULL");
    if (ldx < width || ldy < width || (add && ld_add < width) || (mask && ld_mask < width))
      CPRA_FAIL(CPRA_ERR_SHAPE, "aggregate_mean: leading dimension smaller than width");
    if (X == Y) CPRA_FAIL(CPRA_ERR_PARAM, "aggregate_mean: X must not alias Y");
  }
  return cpra::aggregate(g, transpose != 0, width, X, ldx, Y, ldy, add, ld_add, bias, relu != 0,
                         mask, ld_mask, cpra::as_stream(stream));
}
