// FP32 GEMM on the bfloat16 matrix cores by exact three-way splitting, and on the FP32
// ones in the same structure.  Shared by
// the translation units of the plain and the grouped launches; not part of the ABI.
//
// Every FP32 operand value, times 2^16, is written as x = hi + mid + lo, three bfloat16
// values rounded to nearest: hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid.  Both
// differences are exact in FP32 and the last remainder has at most 8 significant
// bits, so hi + mid + lo = x: the scaling puts the last bit of every FP32 number, 2^-149
// and up, at or above bfloat16's smallest subnormal, 2^-133 (without it an operand of
// 1e-35 kept 18 bits and one of 1e-37 11; it costs a product 1 to 3%: 100,000x128,
// K = 256: 51.5 -> 52.4 us).
// A product a b is then hi hi + (hi mid + mid hi + hi lo + lo hi + mid mid) plus
// mid lo + lo mid, at most 2^-25 |a b| each and as often positive as negative, and
// lo lo, which are left out: six v_mfma_f32_32x32x16_bf16 for
// 16 k, 192 matrix-pipe cycles where v_mfma_f32_32x32x2f32 needs 512 (with the two
// of them taken in, that product takes 61 us).  The products
// of bfloat16 values are exact in FP32; the hi hi sums and the corrections have an
// FP32 accumulator each, added once at the end, so the small terms are not rounded
// at the size of the large sum.  Measured against FP64 on 32x32 tiles of normal
// data (relative 2-norm; FP32 MFMA -> this): K = 32 1.1e-7 -> 3.9e-8, K = 256
// 2.9e-7 -> 8.3e-8, K = 4,096 1.2e-6 -> 4.0e-7, K = 131,072 6.2e-6 -> 2.4e-6; with
// all six products in one accumulator the errors are those of the FP32 MFMA.  The
// largest error of a sum of K products, in 2^-24 of their magnitudes: K = 1 1.0 -> 1.8,
// K = 2 1.9 -> 2.4, K = 3 2.6 -> 2.3, K = 8 4.0 -> 2.1, K = 32 5.0 -> 2.2; so a block
// with one or two k takes FP32 MFMAs (tile_fp32).
//
// So does a 32x32 tile for its results that are not finite (an infinity meets a zero
// mid part, operands from 2^112 on round to an infinite hi, and scaled sums from 2^96
// on overflow): large results, infinities and NaNs come out as an FP32 sum gives them.
//
// Structure (k_gemm_oct): a block computes BM x BN with WM x WN wavefronts; K advances
// in BK-deep steps.  Global values are loaded two steps ahead into registers with
// buffer loads (rows, columns and, where K is not the contiguous axis, k past the
// edge are past the buffer's range and read as 0), split once per block when they
// are written to LDS (double-buffered, one barrier per step), and read back as MFMA
// operands.  The unit of all three is an octet: 8 consecutive k of one row or column,
// a lane's operand of one MFMA and 16 bytes of each of the three planes.  A plane is
// [k octet][row][8], each octet's rows followed by 128 / OCT bytes, so that the operand
// reads (32 consecutive rows of one octet) and the stores (consecutive rows of one
// octet, or 8 / OCT rows of all octets) meet every bank once.  The splitting of the
// next tile (6.5 VALU instructions per value) is placed between the MFMAs of the
// current one.  What bounds it is a wavefront's instruction issue (one VALU
// instruction per 5-8 cycles, so the loop is kept lean: cursors in scalar registers,
// no selects at the edges) and, at K <= 64, memory.  100,000x128, K = 256, NT: 58 us
// with 64x64 tiles, 50 (131 TFLOP/s) with A in registers (k_gemm_rows) against 78-97
// for the FP32 loops of gemm_kernel.hpp; matrix pipes busy 22 to 32% of the time in the
// products of a step over 100,000 nodes.  (Remainders by v_dot2_f32_bf16 take 4.5
// instructions per value, but 1 to 10% more time.)
//
// The same structure without splitting (SP = false) feeds v_mfma_f32_32x32x2f32 with k
// in order, which gives the bits of the one- and two-deep loops of gemm_kernel.hpp for
// every tile shape: 63 us at that shape (104 TFLOP/s, two thirds of the FP32 MFMA
// peak), 5.4 us against 8.2 for a 100x32 product (K = 64), whose time is the
// instructions of one short loop.
#pragma once

#include "gemm_kernel.hpp"

namespace cpra {
namespace gemmk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// hi, mid and lo of two values, packed.  The low halves are widened by a byte
// permute: given a shift, the compiler converts that value a second time instead.
__device__ inline unsigned pack_bf16(float a, float b) {
  bf16x2 r;
  r[0] = (__bf16)a;
  r[1] = (__bf16)b;
  return __builtin_bit_cast(unsigned, r);
}
__device__ inline float low_bf16(unsigned p) {
  return __uint_as_float(__builtin_amdgcn_perm(0u, p, 0x01000c0cu));
}
__device__ inline float high_bf16(unsigned p) { return __uint_as_float(p & 0xffff0000u); }
// hi hi | hi mid | mid hi | mid mid | hi lo | lo hi
constexpr int kTerms = 6, kPlaneA[kTerms] = {0, 0, 1, 1, 0, 2}, kPlaneB[kTerms] = {0, 1, 0, 1, 2, 0};
constexpr float kScale = 0x1p16f, kUnscale = 0x1p-32f;  // of an operand, and back from a product of two
constexpr int kBrief = 2;  // up to so many products in a sum, FP32's error is the smaller
__device__ inline void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  a *= kScale;
  b *= kScale;
  h = pack_bf16(a, b);
  const float ra = a - low_bf16(h), rb = b - high_bf16(h);
  m = pack_bf16(ra, rb);
  l = pack_bf16(ra - low_bf16(m), rb - high_bf16(m));
}

__device__ inline int clamp_bytes(int64_t b) {
  return b < 0 ? 0 : b > 0x7fffffff ? 0x7fffffff : (int)b;
}

#if defined(__HIP_DEVICE_COMPILE__)
// base + voff + soff bytes; voff past the buffer's end: 0
__device__ inline float buf1(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff = 0) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
}
__device__ inline u32x4 buf4(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff = 0) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
}
#endif

// Position of an operand's loads: k of its piece, [k, kn) remaining for this block.
// K contiguous: p is the tile's first row at k = 0, else its first column at k.
struct Cursor {
  const float* p;
  int k, kn, kt;
  unsigned ld4;  // leading dimension in bytes
};

// One operand tile: R rows or columns by BK steps of K, staged by NT threads.
// KC: K is the contiguous axis.  VEC: its octets are read as two float4s (16-byte
// aligned, K a multiple of 4), else value by value.
// SP: staged as the three bfloat16 planes; else as FP32 in two planes, the even k of
// each octet and the odd k, so that half-wavefront h reads the operands of four
// v_mfma_f32_32x32x2f32 (k = 2 e + h of the octet) as one 16-byte chunk.
template <int R, int BK, int NT, bool KC, bool VEC, bool SP>
struct OctTile {
  static constexpr int NP = SP ? 3 : 2;        // planes
  static constexpr int OCT = BK / 8;
  static constexpr int UNITS = R * OCT;
  static constexpr int NU = UNITS >= NT ? UNITS / NT : 1;  // octets per thread
  static_assert(UNITS >= NT ? UNITS % NT == 0 : NT % UNITS == 0, "octets and threads");
  static constexpr int ROWP = R + 8 / OCT;     // 16-byte slots per octet row of a plane
  static constexpr int PLANE = OCT * ROWP;     // slots per plane
  static constexpr int SLOTS = NP * PLANE;     // slots per stage

  // With fewer octets than threads several threads stage the same octet (the same
  // values to the same place).
  __device__ static inline int unit(int tid, int u) { return (tid + u * NT) % UNITS; }
  __device__ static inline int row_of(int i) { return KC ? i / OCT : i % R; }
  __device__ static inline int oct_of(int i) { return KC ? i % OCT : i / R; }

  // Byte offset of each octet from the step's first value; bit 31 (past the buffer's
  // range) for a row or column past the edge.
  unsigned voff[NU];
  __device__ inline void setup(unsigned ld4, int mn0, int mn_lim, int tid) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = unit(tid, u);
      const int r = row_of(i), o = oct_of(i);
      voff[u] = (KC ? (unsigned)r * ld4 + 32u * o : (unsigned)(8 * o) * ld4 + 4u * r) |
                (mn0 + r < mn_lim ? 0u : 0x80000000u);
    }
  }

  // Loads of the next step's octets.
  __device__ inline void load_all(float (&raw)[NU][8], const Cursor& c, int tid) const {
#if defined(__HIP_DEVICE_COMPILE__)
    const int left = c.kn - c.k;
    // K not contiguous: rows of K from `left` on are past the buffer's end
    const int bytes = KC ? 0x7fffffff : (left > 0 ? (left < BK ? left : BK) : 0) * (int)c.ld4;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)c.p, (short)0,
                                                                        __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
    const unsigned so = KC ? 4u * c.k : 0u;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if constexpr (KC) {
        // k past the end: bit 31 puts the offset past the buffer's range
        const int l = left - 8 * oct_of(unit(tid, u));
        if constexpr (VEC) {
          const u32x4 a = buf4(rs, voff[u] | ((unsigned)(l - 1) & 0x80000000u), so);
          const u32x4 b = buf4(rs, (voff[u] + 16u) | ((unsigned)(l - 5) & 0x80000000u), so);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            raw[u][j] = __uint_as_float(a[j]);
            raw[u][4 + j] = __uint_as_float(b[j]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            raw[u][j] = buf1(rs, (voff[u] + 4u * j) | ((unsigned)(l - 1 - j) & 0x80000000u), so);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) raw[u][j] = buf1(rs, voff[u] + j * c.ld4);
      }
    }
#endif
  }

  struct Planes {
    u32x4 p[NP];
  };
  // Half an octet: two pairs, whose dependent chains interleave.
  template <int u, int hf>
  __device__ static inline void split(const float (&raw)[NU][8], Planes (&pl)[NU]) {
#pragma unroll
    for (int pr = 2 * hf; pr < 2 * hf + 2; ++pr) {
      if constexpr (SP) {
        unsigned h, m, l;
        split_pair(raw[u][2 * pr], raw[u][2 * pr + 1], h, m, l);
        pl[u].p[0][pr] = h;
        pl[u].p[1][pr] = m;
        pl[u].p[2][pr] = l;
      } else {
        pl[u].p[0][pr] = __float_as_uint(raw[u][2 * pr]);
        pl[u].p[1][pr] = __float_as_uint(raw[u][2 * pr + 1]);
      }
    }
  }
  template <int u>
  __device__ static inline void store(const Planes (&pl)[NU], u32x4* st, int tid) {
    const int i = unit(tid, u);
    u32x4* p = st + oct_of(i) * ROWP + row_of(i);
#pragma unroll
    for (int q = 0; q < NP; ++q) p[q * PLANE] = pl[u].p[q];
  }
  __device__ static inline void stage_all(const float (&raw)[NU][8], u32x4* st, int tid) {
    Planes pl[NU];
    static_for<NU>([&](auto u) {
      static_for<2>([&](auto hf) { split<decltype(u)::value, decltype(hf)::value>(raw, pl); });
      store<decltype(u)::value>(pl, st, tid);
    });
  }
  // Chunk f of the operands of half-wavefront h for row or column mn and 16 k: plane f
  // of the octet k = 16 ks + 8 h .. (SP), or the half's k of octet 2 ks + f.
  __device__ static inline u32x4 read(const u32x4* st, int f, int ks, int h, int mn) {
    return SP ? st[f * PLANE + (2 * ks + h) * ROWP + mn] : st[h * PLANE + (2 * ks + f) * ROWP + mn];
  }
};

// Where step kt of a block lies: its piece, its first k and the end of the piece's K
// for this block (no k at or past kt_end).
struct StepAt {
  bool p1;
  int kt, k, kn;
};
__device__ inline StepAt step_at(int kt, int nt0, int kn0, int kn1, int kt_end, int bk) {
  StepAt s;
  s.kt = kt;
  s.p1 = kt >= nt0;
  const int first = s.p1 ? nt0 : 0;
  s.k = (kt - first) * bk;
  s.kn = min(s.p1 ? kn1 : kn0, (kt_end - first) * bk);
  return s;
}
template <bool KC>
__device__ inline Cursor cursor_at(const StepAt& s, const float* X, int64_t ld, int mn0) {
  return Cursor{X + (KC ? mn0 * ld : s.k * ld + mn0), s.k, s.kn, s.kt, 4u * (unsigned)ld};
}
template <bool KC>
__device__ inline void advance(Cursor& c, int bk) {
  c.k += bk;
  ++c.kt;
  if constexpr (!KC) c.p = reinterpret_cast<const float*>(reinterpret_cast<const char*>(c.p) + (size_t)bk * c.ld4);
}

// 32x32 results by FP32 MFMAs in k order straight from memory, over [b0, e0) of the
// first piece and [b1, e1) of the second: rows `row` .. (m_left of them inside), columns
// `col` .. (n_left), in the accumulator layout of the 32x32 MFMA.
template <bool A_T, bool B_T>
__device__ __attribute__((noinline)) floatx16 tile_fp32(const float* A0, const float* A1, const float* B0,
                                                        const float* B1, int64_t lda0, int64_t lda1,
                                                        int64_t ldb0, int64_t ldb1, int64_t row, int64_t col,
                                                        int m_left, int n_left, int b0, int e0, int b1, int e1) {
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#if defined(__HIP_DEVICE_COMPILE__)
  const int l32 = threadIdx.x & 31, half = (threadIdx.x >> 5) & 1;
  const bool m_in = l32 < m_left, n_in = l32 < n_left;
  auto piece = [&](const float* A, const float* B, int64_t lda, int64_t ldb, int b, int e) {
    constexpr int U = 4;  // MFMAs of two k each per trip
    for (int k0 = b; k0 < e; k0 += 2 * U) {
      float x[U], y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = k0 + 2 * u + half;
        x[u] = m_in && k < e ? A[A_T ? k * lda + row + l32 : (row + l32) * lda + k] : 0.f;
        y[u] = n_in && k < e ? B[B_T ? (col + l32) * ldb + k : k * ldb + col + l32] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u], y[u], acc, 0, 0, 0);
    }
  };
  piece(A0, B0, lda0, ldb0, b0, e0);
  piece(A1, B1, lda1, ldb1, b1, e1);
#endif
  return acc;
}

// This block's work: problem, tile and K range.
struct Work {
  bool live;
  int prob, grp, split, tm, tn;
  int m0, n0, m_lim;       // first row and column, end of the rows
  int kn0, kn1;            // K of the two pieces
  const float *A0, *A1, *B0, *B1;  // their operands, at this block's graph
  float* C;
  const float* bias;
  float* bias_grad;
};

// Work units in XCD order (each XCD takes one contiguous eighth of them).  Without
// split-K: row tile, problem, column tile -- the column tiles and the problems of a
// row tile, which read the same rows of A, run together on one XCD.  Else: split,
// graph, problem, tile -- the tiles and problems of one K range run together.
template <int BM, int BN, bool A_T, bool B_T, int GM>
__device__ __forceinline__ Work find_work(const LaunchArgs& args) {
  Work w{};
  const int inner = args.grid_x;
  int q = xcd_unit(blockIdx.x, gridDim.x);
  int in = q % inner;
  q /= inner;
  w.prob = q % args.n_prob;
  q /= args.n_prob;
  if (GM != 2 && args.splits == 1) {
    w.tm = q;
    w.tn = in;
  } else {
    if constexpr (GM == 2) {
      w.grp = q % args.G;
      q /= args.G;
    }
    w.split = q;
    const int tn_of = max(1, args.p[w.prob].tiles_n);
    w.tm = in / tn_of;
    w.tn = in - w.tm * tn_of;
  }
  // uniform across the block; said so, as the divisions above run in vector registers
  w.prob = __builtin_amdgcn_readfirstlane(w.prob);
  w.grp = __builtin_amdgcn_readfirstlane(w.grp);
  w.split = __builtin_amdgcn_readfirstlane(w.split);
  w.tm = __builtin_amdgcn_readfirstlane(w.tm);
  w.tn = __builtin_amdgcn_readfirstlane(w.tn);
  if (w.split >= args.splits) return w;
  const ProbDev& P = args.p[w.prob];
  if (w.tm >= P.tiles_m || w.tn >= P.tiles_n) return w;
  w.m0 = w.tm * BM;
  w.n0 = w.tn * BN;
  w.m_lim = P.M;
  w.kn0 = P.K[0];
  w.kn1 = P.n_pieces > 1 ? P.K[1] : 0;
  w.C = P.C;
  w.bias = P.bias;
  w.bias_grad = P.bias_grad;
  int kb = 0;
  int64_t b_off = 0;
  if constexpr (GM == 1) {
    const int4 e = args.row_map[w.tm];
    if (e.x < 0) return w;  // past the last row tile of the batch
    w.m0 = e.y;
    w.m_lim = e.z;
    b_off = (int64_t)e.x * P.b_stride;
    if (w.bias) w.bias += (int64_t)e.x * P.bias_stride;
  } else if constexpr (GM == 2) {
    kb = args.gptr[w.grp];
    const int kn = args.gptr[w.grp + 1] - kb;
    w.kn0 = kn;
    w.kn1 = P.n_pieces > 1 ? kn : 0;
    w.C += (int64_t)w.grp * P.c_stride;
    if (w.bias_grad) w.bias_grad += (int64_t)w.grp * P.bg_stride;
  }
  w.A0 = P.A[0] + (A_T ? (int64_t)kb * P.lda[0] : kb);
  w.A1 = P.A[1] + (A_T ? (int64_t)kb * P.lda[1] : kb);
  w.B0 = P.B[0] + b_off + (B_T ? kb : (int64_t)kb * P.ldb[0]);
  w.B1 = P.B[1] + b_off + (B_T ? kb : (int64_t)kb * P.ldb[1]);
  w.live = true;
  return w;
}

// This block's split-K partial tile (args.splits > 1).
template <int GM>
__device__ inline float* partial_of(const LaunchArgs& args, const Work& w) {
  const ProbDev& P = args.p[w.prob];
  return args.partial + P.part_off + ((int64_t)w.split * (GM == 2 ? args.G : 1) + w.grp) * P.M * P.n_eff;
}

// Epilogue of one 32x32 tile at row0, col0 of the block's tile: acc + cor (or FP32 sums
// over the block's steps [kt_begin, kt_end) of bk, see above), then the
// partial tile or bias, addend, beta C, ReLU, mask, result and sigmoid.
// Accumulator layout of the 32x32 MFMA: register r of lane l holds
// D[8*(r/4) + 4*(l/32) + r%4][l%32].  Rows past the edge lie past the range of the
// tile's buffers, columns past it get bit 31 in their offset: stores there are
// dropped and loads give 0, with no branch per value, and the loads of an epilogue
// operand are all in flight together.
template <bool A_T, bool B_T, bool SP, int GM>
__device__ __forceinline__ void oct_epilogue(const LaunchArgs& args, const Work& w, const floatx16& acc,
                                             const floatx16& cor, int row0, int col0, int bk, int nt0,
                                               int kt_begin, int kt_end) {
#if defined(__HIP_DEVICE_COMPILE__)
  const ProbDev& P = args.p[w.prob];
  const int lane = threadIdx.x & 63;
  const int m_valid = w.m_lim - w.m0;
  const int col = w.n0 + col0 + (lane & 31);
  const unsigned edge = col < P.N ? 0u : 0x80000000u;
  const int r0 = row0 + 4 * (lane >> 5);
  struct Buf {
    __amdgpu_buffer_rsrc_t rs;
    unsigned base, ld4;
    // row (r >> 2) * 8 + (r & 3) below the lane's first
    __device__ inline unsigned at(int r) const { return base + ((r >> 2) * 8 + (r & 3)) * ld4; }
  };
  auto buf = [&](const float* X, int64_t ld) {
    const unsigned ld4 = 4u * (unsigned)ld;
    return Buf{__builtin_amdgcn_make_buffer_rsrc((void*)(X + (int64_t)w.m0 * ld), (short)0,
                                                 clamp_bytes(4 * ((int64_t)(m_valid - 1) * ld + P.N)), 0x00020000),
               ((unsigned)r0 * ld4 + 4u * col) | edge, ld4};
  };
  auto read = [&](const Buf& b, float (&x)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = buf1(b.rs, b.at(r));
  };
  float v[16];
  if constexpr (SP) {
    const int b0 = min(w.kn0, kt_begin * bk), e0 = min(w.kn0, kt_end * bk);
    const int b1 = max(0, min(w.kn1, (kt_begin - nt0) * bk)), e1 = max(0, min(w.kn1, (kt_end - nt0) * bk));
    const bool brief = e0 - b0 + e1 - b1 <= kBrief;
    float nf = 0.f;  // NaN if one of them is not finite
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      v[r] = (acc[r] + cor[r]) * kUnscale;
      nf = fmaf(v[r], 0.f, nf);
    }
    if (brief || __any(nf != nf)) {  // uniform
      const floatx16 f = tile_fp32<A_T, B_T>(w.A0, w.A1, w.B0, w.B1, P.lda[0], P.lda[1], P.ldb[0], P.ldb[1],
                                             w.m0 + row0, w.n0 + col0, m_valid - row0, P.N - w.n0 - col0, b0, e0, b1,
                                             e1);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = !brief && fabsf(v[r]) <= 3.402823466e38f ? v[r] : f[r];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = acc[r];
  }
  if (args.splits > 1) {
    const Buf b = buf(partial_of<GM>(args, w), P.n_eff);
#pragma unroll
    for (int r = 0; r < 16; ++r) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r]), b.rs, b.at(r), 0, 0);
    return;
  }
  if (w.bias) {
    const float bv = col < P.N ? w.bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] += bv;
  }
  float x[16];
  if (P.add) {
    read(buf(P.add, P.ld_add), x);
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] += x[r];
  }
  const Buf c = buf(w.C, P.ldc);
  if (P.beta != 0.f) {
    read(c, x);
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] += P.beta * x[r];
  }
  if (P.relu) {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = fmaxf(v[r], 0.f);
  }
  if (P.mask) {
    read(buf(P.mask, P.ld_mask), x);
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = x[r] > 0.f ? v[r] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r]), c.rs, c.at(r), 0, 0);
  if (P.sig_out) {
    const Buf b = buf(P.sig_out, P.ld_sig);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e = expf(-fabsf(v[r]));
      const float s = 1.0f / (1.0f + e);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r] >= 0.0f ? s : e * s), b.rs, b.at(r), 0, 0);
    }
  }
#endif
}

// A_T, B_T, GM as for k_gemm.  VEC: float4 loads of the K-contiguous operands.
// SP: split operands; else plain FP32 MFMAs, whose sums run over k in order (the bits
// of the k_gemm loops 1 and 2).
template <int BM, int BN, int BK, int WM, int WN, bool A_T, bool B_T, bool VEC, bool SP, int GM>
__global__ __launch_bounds__(64 * WM * WN) void k_gemm_oct(LaunchArgs args) {
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / (32 * WM), TN = BN / (32 * WN);
  static_assert(TM >= 1 && TN >= 1 && TM * 32 * WM == BM && TN * 32 * WN == BN, "bad tiling");
  using TA = OctTile<BM, BK, NT, !A_T, VEC, SP>;
  using TB = OctTile<BN, BK, NT, B_T, VEC, SP>;
  __shared__ u32x4 As[2][TA::SLOTS];
  __shared__ u32x4 Bs[2][TB::SLOTS];

  const Work w = find_work<BM, BN, A_T, B_T, GM>(args);
  if (!w.live) return;
  const ProbDev& P = args.p[w.prob];
  const int m0 = w.m0, n0 = w.n0, m_lim = w.m_lim, kn0 = w.kn0, kn1 = w.kn1;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int half = lane >> 5, l32 = lane & 31;

  const int nt0 = (kn0 + BK - 1) / BK;
  const int nt1 = (kn1 + BK - 1) / BK;
  const int KT = nt0 + nt1;
  // uniform, although the division runs in vector registers; steps run in pairs (an
  // odd count's last one multiplies zeros), so split ranges are even, except where the
  // order of the sums is to stay that of the other FP32 loops
  const int ceil_split = (KT + args.splits - 1) / args.splits;
  const int per_split = __builtin_amdgcn_readfirstlane(SP ? (ceil_split + 1) & ~1 : ceil_split);
  const int kt_begin = min(KT, w.split * per_split);
  const int kt_end = min(KT, kt_begin + per_split);

  floatx16 acc[TM][TN], cor[SP ? TM : 1][SP ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] = 0.f;
        if constexpr (SP) cor[i][j][r] = 0.f;
      }

  const int64_t lda0 = P.lda[0], lda1 = P.lda[1], ldb0 = P.ldb[0], ldb1 = P.ldb[1];
  const int n_lim = P.N;

  using RawA = float[TA::NU][8];
  using RawB = float[TB::NU][8];
  TA ta;
  TB tb;
  Cursor ca, cb;
  auto seek = [&](int kt) {
    const StepAt at = step_at(kt, nt0, w.kn0, w.kn1, kt_end, BK);
    ca = cursor_at<!A_T>(at, at.p1 ? w.A1 : w.A0, at.p1 ? lda1 : lda0, m0);
    cb = cursor_at<B_T>(at, at.p1 ? w.B1 : w.B0, at.p1 ? ldb1 : ldb0, n0);
    ta.setup(ca.ld4, m0, m_lim, tid);
    tb.setup(cb.ld4, n0, n_lim, tid);
  };
  auto load_next = [&](RawA& ra, RawB& rb) {
    ta.load_all(ra, ca, tid);
    tb.load_all(rb, cb, tid);
    advance<!A_T>(ca, BK);
    advance<B_T>(cb, BK);
    if (ca.kt == nt0 && nt1 > 0) seek(nt0);  // uniform
  };

  // Bias gradient (row sums of op(A) over this block's K range, A stored [K, M]):
  // thread t of a first-column block adds the octets it stages, all of row t % BM.
  constexpr int BG = NT / BM > 0 ? NT / BM : 1;
  const bool do_bias = A_T && w.bias_grad != nullptr && w.tn == 0;
  float bsum = 0.f;
  auto add_bias = [&](const RawA& ra) {
    if constexpr (A_T) {
      static_assert(!A_T || (NT % BM == 0 && TA::UNITS % NT == 0), "bias slices");
#pragma unroll
      for (int u = 0; u < TA::NU; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) bsum += ra[u][j];
    }
  };

  // One step: operands of the first 16 k read, the loads of step kt + 2 issued into
  // the free set while they arrive, then the MFMAs; after each of them a share of the
  // step's other work: the operand reads of the next 16 k, the splitting of step
  // kt + 1 and its stores to the other LDS stage.
  constexpr int KS = BK / 16;
  constexpr int NF = TA::NP;
  constexpr int PER = (SP ? kTerms : 8) * TM * TN;                 // MFMAs per 16 k
  constexpr int NCONV = 2 * (TA::NU + TB::NU);       // half octets to split per thread and step
  constexpr int NREAD = NF * (TM + TN);
  constexpr int NSLOT = PER * KS;
  struct Frags {
    u32x4 a[TM][NF], b[TN][NF];
  };
  auto read_frag = [&](auto rc, Frags& f, const u32x4* as, const u32x4* bs, int ks) {
    constexpr int r = decltype(rc)::value;  // chunk 0 of every operand first
    constexpr int p = r / (TM + TN), q = r % (TM + TN);
    if constexpr (q < TM) f.a[q][p] = TA::read(as, p, ks, half, (wm * TM + q) * 32 + l32);
    else f.b[q - TM][p] = TB::read(bs, p, ks, half, (wn * TN + q - TM) * 32 + l32);
  };
  auto step = [&](int cur, RawA& fra, RawB& frb, const RawA& nxa, const RawB& nxb) {
    const u32x4* as = As[cur];
    const u32x4* bs = Bs[cur];
    u32x4* const as_st = As[cur ^ 1];
    u32x4* const bs_st = Bs[cur ^ 1];
    typename TA::Planes pa[TA::NU];
    typename TB::Planes pb[TB::NU];
    Frags f[2];
    static_for<NREAD>([&](auto rc) { read_frag(rc, f[0], as, bs, 0); });
    __builtin_amdgcn_sched_barrier(0);
    load_next(fra, frb);
    __builtin_amdgcn_sched_barrier(0);
    static_for<NSLOT>([&](auto sc) {
      constexpr int slot = decltype(sc)::value;
      constexpr int ks = slot / PER, sl = slot % PER;
      constexpr int term = sl / (TM * TN), i = (sl / TN) % TM, j = sl % TN;
      if constexpr (SP) {
        floatx16& c = term == 0 ? acc[i][j] : cor[i][j];
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[ks % 2].a[i][kPlaneA[term]]),
                                                    __builtin_bit_cast(bf16x8, f[ks % 2].b[j][kPlaneB[term]]), c, 0, 0, 0);
      } else {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f[ks % 2].a[i][term / 4][term % 4]),
                                                         __uint_as_float(f[ks % 2].b[j][term / 4][term % 4]),
                                                         acc[i][j], 0, 0, 0);
      }
      if constexpr (ks + 1 < KS) {
        static_for<NREAD>([&](auto rc) {
          if constexpr (decltype(rc)::value * PER / NREAD == sl) read_frag(rc, f[(ks + 1) % 2], as, bs, ks + 1);
        });
      }
      static_for<NCONV>([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if constexpr (o * NSLOT / NCONV == slot) {
          if constexpr (o < 2 * TA::NU) {
            TA::template split<o / 2, o % 2>(nxa, pa);
            if constexpr (o % 2 == 1) TA::template store<o / 2>(pa, as_st, tid);
          } else {
            constexpr int q = o - 2 * TA::NU;
            TB::template split<q / 2, q % 2>(nxb, pb);
            if constexpr (q % 2 == 1) TB::template store<q / 2>(pb, bs_st, tid);
          }
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    if (do_bias) add_bias(nxa);  // zeros past the last step
    __syncthreads();
  };
  // Steps run in pairs, so that every register set is named statically; with an odd
  // count the last one multiplies zeros (peeling it made the compiler copy the
  // accumulators at the join).
  RawA ra0, ra1;
  RawB rb0, rb1;
  seek(kt_begin);
  load_next(ra0, rb0);
  load_next(ra1, rb1);
  TA::stage_all(ra0, As[0], tid);
  TB::stage_all(rb0, Bs[0], tid);
  if (do_bias) add_bias(ra0);
  __syncthreads();
  int kt = kt_begin;
  do {
    step(0, ra0, rb0, ra1, rb1);
    step(1, ra1, rb1, ra0, rb0);
    kt += 2;
  } while (kt < kt_end);
  static_for<TM>([&](auto ic) {
    static_for<TN>([&](auto jc) {
      constexpr int i = decltype(ic)::value, j = decltype(jc)::value;
      oct_epilogue<A_T, B_T, SP, GM>(args, w, acc[i][j], cor[SP ? i : 0][SP ? j : 0], (wm * TM + i) * 32, (wn * TN + j) * 32, BK, nt0,
                                   kt_begin, kt_end);
    });
  });
  if (do_bias) {  // fixed-order sum of the BG slices of each row
    __syncthreads();
    float* red = reinterpret_cast<float*>(&As[0][0]);
    red[(tid / BM) * BM + tid % BM] = bsum;
    __syncthreads();
    if (tid < BM && m0 + tid < m_lim) {
      float v = 0.f;
      for (int g2 = 0; g2 < BG; ++g2) v += red[g2 * BM + tid];
      if (args.splits > 1) partial_of<GM>(args, w)[(int64_t)(m0 + tid) * P.n_eff + P.N] = v;
      else w.bias_grad[m0 + tid] = v;
    }
  }
}

// Tall products with a K-contiguous A (the node products: X W^T, dY W).  Each of the
// WM wavefronts owns 32 rows and all BN columns of the block's tile and loads its A
// values straight into the MFMA layout, so that A passes through no LDS and is split
// once; only B's octets are staged (as in k_gemm_oct, one step ahead).  Lane
// (row, h) takes the 16 values at k = 16 h .. 16 h + 15 of a 32-deep step, 64
// consecutive bytes; its first octet is the operand of the step's first MFMAs, its
// second of the others, and B's octets are read in the same order (any order of k
// works when both operands use it).  While one octet is multiplied the next one is
// split, so two octets of planes and two steps of raw values are held.
template <int BN, int WM, bool B_T, bool VEC, int GM>
__global__ __launch_bounds__(64 * WM, BN >= 64 ? 2 : 4) void k_gemm_rows(LaunchArgs args) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BK = 32, NT = 64 * WM, BM = 32 * WM, TN = BN / 32;
  using TB = OctTile<BN, BK, NT, B_T, VEC, true>;
  __shared__ u32x4 Bs[2][TB::SLOTS];
  const Work w = find_work<BM, BN, false, B_T, GM>(args);
  if (!w.live) return;
  const ProbDev& P = args.p[w.prob];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int nt0 = (w.kn0 + BK - 1) / BK, nt1 = (w.kn1 + BK - 1) / BK;
  const int KT = nt0 + nt1;
  // steps run in pairs; uniform, although the division runs in vector registers
  const int per_split = __builtin_amdgcn_readfirstlane(((KT + args.splits - 1) / args.splits + 1) & ~1);
  const int kt_begin = min(KT, w.split * per_split);
  const int kt_end = min(KT, kt_begin + per_split);

  floatx16 acc[TN], cor[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[j][r] = 0.f;
      cor[j][r] = 0.f;
    }

  const int64_t lda0 = P.lda[0], lda1 = P.lda[1], ldb0 = P.ldb[0], ldb1 = P.ldb[1];
  Cursor ca, cb;
  unsigned va = 0;
  TB tb;
  const int arow = wave * 32 + l32;
  auto seek_a = [&](int kt) {
    const StepAt at = step_at(kt, nt0, w.kn0, w.kn1, kt_end, BK);
    ca = cursor_at<true>(at, at.p1 ? w.A1 : w.A0, at.p1 ? lda1 : lda0, w.m0);
    va = ((unsigned)arow * ca.ld4 + 64u * half) | (w.m0 + arow < w.m_lim ? 0u : 0x80000000u);
  };
  auto seek_b = [&](int kt) {
    const StepAt at = step_at(kt, nt0, w.kn0, w.kn1, kt_end, BK);
    cb = cursor_at<B_T>(at, at.p1 ? w.B1 : w.B0, at.p1 ? ldb1 : ldb0, w.n0);
    tb.setup(cb.ld4, w.n0, P.N, tid);
  };
  auto load_a = [&](float (&x)[16]) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)ca.p, (short)0, 0x7fffffff, 0x00020000);
    const int l = ca.kn - ca.k - 16 * half;
    const unsigned so = 4u * ca.k;
    if constexpr (VEC) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x4 y = buf4(rs, (va + 16u * q) | ((unsigned)(l - 1 - 4 * q) & 0x80000000u), so);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[4 * q + j] = __uint_as_float(y[j]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = buf1(rs, (va + 4u * j) | ((unsigned)(l - 1 - j) & 0x80000000u), so);
    }
    advance<true>(ca, BK);
    if (ca.kt == nt0 && nt1 > 0) seek_a(nt0);  // uniform
  };
  auto load_b = [&](float (&x)[TB::NU][8]) {
    tb.load_all(x, cb, tid);
    advance<B_T>(cb, BK);
    if (cb.kt == nt0 && nt1 > 0) seek_b(nt0);
  };

  struct Planes {
    u32x4 p[3];
  };
  auto split_a = [&](auto hfc, const float* x, Planes& a) {  // half hf of the octet at x
    constexpr int hf = decltype(hfc)::value;
#pragma unroll
    for (int pr = 2 * hf; pr < 2 * hf + 2; ++pr) {
      unsigned h, m, l;
      split_pair(x[2 * pr], x[2 * pr + 1], h, m, l);
      a.p[0][pr] = h;
      a.p[1][pr] = m;
      a.p[2][pr] = l;
    }
  };
  // Step kt (LDS stage cur): a0 holds its first octet split, `now` its raw values,
  // `nxt` those of step kt + 1; `now` then receives step kt + 2.
  constexpr int PER = kTerms * TN;
  constexpr int NSLOT = 2 * PER;
  constexpr int NB = 2 * TB::NU;
  Planes a0, a1;
  float rb[TB::NU][8];
  auto step = [&](int cur, float (&now)[16], const float (&nxt)[16]) {
    const u32x4* bs = Bs[cur];
    u32x4* const st = Bs[cur ^ 1];
    typename TB::Planes pb[TB::NU];
    u32x4 f[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) f[0][p] = bs[p * TB::PLANE + (2 * half) * TB::ROWP + l32];
    load_b(rb);
    __builtin_amdgcn_sched_barrier(0);
    static_for<NSLOT>([&](auto sc) {
      constexpr int slot = decltype(sc)::value;
      constexpr int ks = slot / PER, j = slot % PER / kTerms, term = slot % kTerms, g = slot / kTerms;
      const Planes& a = ks == 0 ? a0 : a1;
      floatx16& c = term == 0 ? acc[j] : cor[j];
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.p[kPlaneA[term]]),
                                                  __builtin_bit_cast(bf16x8, f[g % 2][kPlaneB[term]]), c, 0, 0, 0);
      if constexpr (term % 2 == 0 && g + 1 < 2 * TN) {  // next column tile's operands
        constexpr int p = term / 2, g1 = g + 1;
        f[g1 % 2][p] = bs[p * TB::PLANE + (2 * half + g1 / TN) * TB::ROWP + 32 * (g1 % TN) + l32];
      }
      // A: the second octet of this step, then the first of the next one
      static_for<4>([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if constexpr (o * NSLOT / 4 == slot) {
          if constexpr (o < 2) split_a(std::integral_constant<int, o % 2>{}, now + 8, a1);
          else split_a(std::integral_constant<int, o % 2>{}, nxt, a0);
        }
      });
      if constexpr (slot == PER - 1) load_a(now);
      // B: staged in the second half (its loads were issued at the step's start)
      static_for<NB>([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if constexpr (PER + o * PER / NB == slot) {
          TB::template split<o / 2, o % 2>(rb, pb);
          if constexpr (o % 2 == 1) TB::template store<o / 2>(pb, st, tid);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
  };
  float r0[16], r1[16];
  seek_a(kt_begin);
  seek_b(kt_begin);
  load_b(rb);
  load_a(r0);
  load_a(r1);
  TB::stage_all(rb, Bs[0], tid);
  static_for<2>([&](auto hf) { split_a(hf, r0, a0); });
  __syncthreads();
  int kt = kt_begin;
  do {  // in pairs, as in k_gemm_oct
    step(0, r0, r1);
    step(1, r1, r0);
    kt += 2;
  } while (kt < kt_end);
  static_for<TN>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    oct_epilogue<false, B_T, true, GM>(args, w, acc[j], cor[j], wave * 32, 32 * j, BK, nt0, kt_begin, kt_end);
  });
#endif
}

// 16 k of one operand of k_gemm_direct: x[s] of lane l is the value of row (column)
// l % 16 at k = g + 4 s + l / 16; k from `left` on and rows with `edge` read as 0.
// K-contiguous operands are read as one float4 per lane, k = g + 4 (l / 16) .., whose 4x4
// blocks over the quarters of the wavefront are then transposed.
template <bool KC, bool VEC>
__device__ __forceinline__ void direct_operand(__amdgpu_buffer_rsrc_t rs, unsigned edge, unsigned ld4, int l16,
                                               int quad, int g, int left, float* x) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (KC && VEC) {
    const int k = g + 4 * quad;
    const u32x4 v = buf4(rs, (l16 * ld4 + 4u * k) | edge | (k < left ? 0u : 0x80000000u));
    const auto p02 = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const auto p13 = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const auto p01 = __builtin_amdgcn_permlane16_swap(p02[0], p13[0], false, false);
    const auto p23 = __builtin_amdgcn_permlane16_swap(p02[1], p13[1], false, false);
    x[0] = __uint_as_float(p01[0]);
    x[1] = __uint_as_float(p01[1]);
    x[2] = __uint_as_float(p23[0]);
    x[3] = __uint_as_float(p23[1]);
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = g + 4 * s + quad;
      x[s] = buf1(rs, (KC ? l16 * ld4 + 4u * k : k * ld4 + 4u * l16) | edge | (k < left ? 0u : 0x80000000u));
    }
  }
#endif
}

// Small products: a wavefront computes one 16x16 tile straight from global memory, every
// operand of 64 k in flight at once, with the 16x16x4 FP32 MFMA (whose sums run over k in
// order, like those of the 32x32x2: the bits are the same).  A launch of a few dozen
// 32x32 tiles lasts as long as one wavefront takes to find its work and to issue a tile's
// loads, LDS traffic and MFMAs; here that is a quarter, with no barrier, on four times
// as many CUs.  Back to back in a graph: C = A^T B, 32x64 over K = 100: 5.6 -> 4.6 us;
// A B^T, 100x64, K = 64: 4.5 -> 4.4 (2.7 of them are an empty kernel's).
template <bool A_T, bool B_T, bool VEC>
__global__ __launch_bounds__(64) void k_gemm_direct(LaunchArgs args) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BK = 32, CHUNK = 64, GROUP = 16;  // K step of the split ranges, k in flight, k per branch
  // Blocks: column tile within problem, row tile, split (no divisions, which cost as much
  // as the tile's loads).
  Work w{};
  int tn = blockIdx.x;
  while (tn >= args.grid_x) {
    tn -= args.grid_x;
    ++w.prob;
  }
  w.split = blockIdx.z;
  const ProbDev& P = args.p[w.prob];
  if ((int)blockIdx.y >= P.tiles_m || tn >= P.tiles_n) return;
  w.m0 = blockIdx.y * 16;
  w.n0 = tn * 16;
  w.m_lim = P.M;
  w.kn0 = P.K[0];
  w.kn1 = P.n_pieces > 1 ? P.K[1] : 0;
  w.C = P.C;
  w.bias = P.bias;
  const int lane = threadIdx.x;
  const int l16 = lane & 15, quad = lane >> 4;
  const int m_valid = min(16, w.m_lim - w.m0), n_valid = min(16, P.N - w.n0);

  const int nt0 = (w.kn0 + BK - 1) / BK;
  const int KT = nt0 + (w.kn1 + BK - 1) / BK;
  const int per_split = args.splits == 1 ? KT : __builtin_amdgcn_readfirstlane((KT + args.splits - 1) / args.splits);
  const int kt_begin = min(KT, w.split * per_split);
  const int kt_end = min(KT, kt_begin + per_split);

  // The lane's results are rows 4 quad .. + 3 of column l16; their addends are loaded first.
  const int row = w.m0 + 4 * quad, col = w.n0 + l16;
  const bool final_ = args.splits == 1;
  bool ok[4];
  float add[4], old[4], msk[4], bias = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ok[i] = l16 < n_valid && 4 * quad + i < m_valid;
    add[i] = old[i] = msk[i] = 0.f;
    if (!final_ || !ok[i]) continue;
    if (P.add) add[i] = P.add[(int64_t)(row + i) * P.ld_add + col];
    if (P.beta != 0.f) old[i] = w.C[(int64_t)(row + i) * P.ldc + col];
    if (P.mask) msk[i] = P.mask[(int64_t)(row + i) * P.ld_mask + col];
  }
  if (final_ && w.bias && l16 < n_valid) bias = w.bias[col];

  typedef float floatx4 __attribute__((ext_vector_type(4)));
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  // k in [b, e) of one piece.  Rows and columns past the edge, and k past the end, are
  // past the buffers' ranges (bit 31) and read as 0.
  auto piece = [&](const float* A, const float* B, int64_t lda, int64_t ldb, int b, int e) {
    const unsigned la = 4u * (unsigned)lda, lb = 4u * (unsigned)ldb;
    const unsigned a0 = l16 < m_valid ? 0u : 0x80000000u, b0 = l16 < n_valid ? 0u : 0x80000000u;
    auto load = [&](int k0, float (&x)[CHUNK / 4], float (&y)[CHUNK / 4]) {
      const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(A + (A_T ? (int64_t)k0 * lda + w.m0 : (int64_t)w.m0 * lda + k0)), (short)0, 0x7fffffff, 0x00020000);
      const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(B + (B_T ? (int64_t)w.n0 * ldb + k0 : (int64_t)k0 * ldb + w.n0)), (short)0, 0x7fffffff, 0x00020000);
#pragma unroll
      for (int g = 0; g < CHUNK; g += GROUP) {
        if (k0 + g >= e) break;
        direct_operand<!A_T, VEC>(ra, a0, la, l16, quad, g, e - k0, x + g / 4);
        direct_operand<B_T, VEC>(rb, b0, lb, l16, quad, g, e - k0, y + g / 4);
      }
    };
    auto multiply = [&](int k0, const float (&x)[CHUNK / 4], const float (&y)[CHUNK / 4]) {
#pragma unroll
      for (int g = 0; g < CHUNK; g += GROUP) {
        if (k0 + g >= e) break;
#pragma unroll
        for (int s = g / 4; s < (g + GROUP) / 4; ++s)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s], y[s], acc, 0, 0, 0);
      }
    };
    float x[2][CHUNK / 4] = {}, y[2][CHUNK / 4] = {};
    if (b < e) load(b, x[0], y[0]);
    for (int k0 = b; k0 < e; k0 += 2 * CHUNK) {
      if (k0 + CHUNK < e) load(k0 + CHUNK, x[1], y[1]);
      multiply(k0, x[0], y[0]);
      if (k0 + CHUNK >= e) break;
      if (k0 + 2 * CHUNK < e) load(k0 + 2 * CHUNK, x[0], y[0]);
      multiply(k0 + CHUNK, x[1], y[1]);
    }
  };
  piece(P.A[0], P.B[0], P.lda[0], P.ldb[0], min(w.kn0, kt_begin * BK), min(w.kn0, kt_end * BK));
  if (P.n_pieces > 1)
    piece(P.A[1], P.B[1], P.lda[1], P.ldb[1], max(0, min(w.kn1, (kt_begin - nt0) * BK)),
          max(0, min(w.kn1, (kt_end - nt0) * BK)));

#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!ok[i]) continue;
    float v = acc[i];
    if (!final_) {
      partial_of<0>(args, w)[(int64_t)(row + i) * P.n_eff + col] = v;
      continue;
    }
    if (w.bias) v += bias;
    if (P.add) v += add[i];
    if (P.beta != 0.f) v += P.beta * old[i];
    if (P.relu) v = fmaxf(v, 0.f);
    if (P.mask) v = msk[i] > 0.f ? v : 0.f;
    w.C[(int64_t)(row + i) * P.ldc + col] = v;
    if (P.sig_out) {
      const float z = expf(-fabsf(v));
      const float s = recip_1_2(1.0f + z);
      P.sig_out[(int64_t)(row + i) * P.ld_sig + col] = v >= 0.0f ? s : z * s;
    }
  }
#endif
}

// Whether every K-contiguous operand may be read as float4s.
inline bool split_vec(const LaunchArgs& args, bool a_t, bool b_t) {
  for (int i = 0; i < args.n_prob; ++i) {
    const ProbDev& d = args.p[i];
    for (int pc = 0; pc < d.n_pieces; ++pc) {
      if (!a_t && (!d.vecA[pc] || d.K[pc] % 4 != 0)) return false;
      if (b_t && (!d.vecB[pc] || d.K[pc] % 4 != 0)) return false;
    }
  }
  return true;
}

// The grid of a BM x BN tiling (in find_work's order).
template <int BM, int BN, int GM>
dim3 split_grid(LaunchArgs& args) {
  int tm = 0, tn = 0, tiles = 0;
  for (int i = 0; i < args.n_prob; ++i) {
    ProbDev& d = args.p[i];
    d.tiles_m = GM == 1 ? args.row_counts[bm_index(BM)] : (int)ceil_div(d.M, BM);
    d.tiles_n = (int)ceil_div(d.N, BN);
    tm = max(tm, d.tiles_m);
    tn = max(tn, d.tiles_n);
    tiles = max(tiles, d.tiles_m * d.tiles_n);
  }
  if (GM == 1) args.row_map = args.row_maps[bm_index(BM)];
  const bool plain = GM != 2 && args.splits == 1;
  args.grid_x = plain ? tn : tiles;
  return dim3((unsigned)xcd_grid((int64_t)args.n_prob * args.grid_x * (plain ? tm : (int64_t)args.splits * args.G)));
}

template <int BM, int BN, int BK, int WM, int WN, bool SP, bool A_T, bool B_T, int GM>
void launch_oct(LaunchArgs& args, hipStream_t stream) {
  const dim3 grid = split_grid<BM, BN, GM>(args), block(64 * WM * WN);
  if constexpr (!A_T || B_T) {
    if (!split_vec(args, A_T, B_T)) {
      hipLaunchKernelGGL((k_gemm_oct<BM, BN, BK, WM, WN, A_T, B_T, false, SP, GM>), grid, block, 0, stream, args);
      return;
    }
  }
  hipLaunchKernelGGL((k_gemm_oct<BM, BN, BK, WM, WN, A_T, B_T, true, SP, GM>), grid, block, 0, stream, args);
}

template <int BN, int WM, bool B_T, int GM>
void launch_rows(LaunchArgs& args, hipStream_t stream) {
  const dim3 grid = split_grid<32 * WM, BN, GM>(args), block(64 * WM);
  if (split_vec(args, false, B_T))
    hipLaunchKernelGGL((k_gemm_rows<BN, WM, B_T, true, GM>), grid, block, 0, stream, args);
  else
    hipLaunchKernelGGL((k_gemm_rows<BN, WM, B_T, false, GM>), grid, block, 0, stream, args);
}

template <bool A_T, bool B_T>
void launch_direct(LaunchArgs& args, hipStream_t stream) {
  int tm = 0, tn = 0;
  for (int i = 0; i < args.n_prob; ++i) {
    ProbDev& d = args.p[i];
    d.tiles_m = (int)ceil_div(d.M, 16);
    d.tiles_n = (int)ceil_div(d.N, 16);
    tm = max(tm, d.tiles_m);
    tn = max(tn, d.tiles_n);
  }
  args.grid_x = tn;
  const dim3 grid((unsigned)(tn * args.n_prob), (unsigned)tm, (unsigned)args.splits);
  if (split_vec(args, A_T, B_T))
    hipLaunchKernelGGL((k_gemm_direct<A_T, B_T, true>), grid, dim3(64), 0, stream, args);
  else
    hipLaunchKernelGGL((k_gemm_direct<A_T, B_T, false>), grid, dim3(64), 0, stream, args);
}

// cfg as resolve_cfg gives it.
template <bool A_T, bool B_T, int GM>
void launch_split_any(int cfg, LaunchArgs& args, hipStream_t stream) {
  switch (cfg) {
#define CPRA_SPLIT_CFG(I, BM, BN, BK, WM, WN, SP) \
  case I: launch_oct<BM, BN, BK, WM, WN, SP, A_T, B_T, GM>(args, stream); break;
    CPRA_SPLIT_CFG(32, 64, 64, 32, 2, 2, true)
    CPRA_SPLIT_CFG(33, 128, 64, 32, 2, 2, true)
    CPRA_SPLIT_CFG(34, 64, 128, 32, 2, 2, true)
    CPRA_SPLIT_CFG(35, 128, 128, 32, 2, 4, true)
    CPRA_SPLIT_CFG(36, 128, 32, 32, 4, 1, true)
    CPRA_SPLIT_CFG(37, 32, 64, 32, 1, 2, true)
    CPRA_SPLIT_CFG(38, 32, 32, 32, 1, 1, true)
    CPRA_SPLIT_CFG(39, 64, 64, 16, 2, 1, true)
    CPRA_SPLIT_CFG(45, 64, 64, 32, 2, 2, false)
    CPRA_SPLIT_CFG(46, 128, 64, 32, 2, 2, false)
    CPRA_SPLIT_CFG(47, 32, 64, 32, 1, 2, false)
    CPRA_SPLIT_CFG(48, 32, 32, 32, 1, 1, false)
    CPRA_SPLIT_CFG(49, 128, 128, 32, 2, 4, false)
    CPRA_SPLIT_CFG(50, 128, 32, 32, 4, 1, false)
#undef CPRA_SPLIT_CFG
    default:
      if constexpr (!A_T) {
        if (cfg == 40) launch_rows<128, 4, B_T, GM>(args, stream);
        if (cfg == 41) launch_rows<64, 4, B_T, GM>(args, stream);
        if (cfg == 42) launch_rows<32, 4, B_T, GM>(args, stream);
        if (cfg == 43) launch_rows<64, 2, B_T, GM>(args, stream);
        if (cfg == 44) launch_rows<32, 1, B_T, GM>(args, stream);
      }
      if constexpr (GM == 0) {
        if (cfg == kDirect) launch_direct<A_T, B_T>(args, stream);
      }
  }
}

}  // namespace gemmk
}  // namespace cpra
