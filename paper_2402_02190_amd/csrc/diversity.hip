// Solution-diversity analytics over the S rounded solutions: pairwise Hamming
// distances, their histogram over the S(S-1)/2 pairs and the number of distinct
// solutions (Sec. 4.1 Evaluation Metrics; the Hamming-distance and unique-
// solution analyses of the diversity appendix).  The pairwise distances are
// the O(N S^2) quantity that Proposition 3.2 lets the loss avoid; here they
// are computed once per evaluation, on bit-packed columns: each solution is
// packed into ceil(N/64) 64-bit words and d(s, l) is a sum of popcounts of
// XORed words.  Everything is integer and exact.
#include "common.hpp"

namespace cpra {

namespace {

// B[s * W + w] = bits of rows 64 w .. 64 w + 63 of column s (row r -> bit r % 64).
// One block per word row: 4 groups of 64 threads take 16 rows each (16 loads in
// flight per thread) for 64 heads at a time.  The same launch clears the histogram.
__global__ __launch_bounds__(256) void k_pack_columns(int N, int S, int W, const uint8_t* __restrict__ X,
                                                      int64_t ldx, uint64_t* __restrict__ B,
                                                      int64_t* __restrict__ hist) {
  const int w = blockIdx.x;
  if (hist && blockIdx.y == 0 && threadIdx.x < 64) {
    const int64_t i = (int64_t)w * 64 + threadIdx.x;
    if (i <= N) hist[i] = 0;
    if (w == W - 1 && threadIdx.x == 0) hist[N] = 0;  // a 65th bin when N is a multiple of 64
  }
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int s = blockIdx.y * 64 + lane;
  const int r0 = w * 64 + part * 16;
  uint8_t x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = s < S && r0 + r < N ? X[(int64_t)(r0 + r) * ldx + s] : 0;
  unsigned bits = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) bits |= (x[r] ? 1u : 0u) << r;
  __shared__ unsigned sh[4][64];
  sh[part][lane] = bits;
  __syncthreads();
  if (part == 0 && s < S)
    B[(int64_t)s * W + w] = (uint64_t)(sh[0][lane] | (sh[1][lane] << 16)) |
                            ((uint64_t)(sh[2][lane] | (sh[3][lane] << 16)) << 32);
}

// One block per 16 x 16 tile of pairs on or above the diagonal, 4 groups of 256
// threads (one pair each) sharing the words: chunks of 64 words of the 32 columns are
// staged in LDS with coalesced loads, group q sums words q, q + 4, .. of a chunk, and
// the four sums are added at the end.  At S = 100 there are 28 tiles, so the time is
// the chain of one tile's chunks: 3 for N = 10,000 (40 -> 7 us; a thread per ordered
// pair walked all 157 words of two columns from memory).
__global__ __launch_bounds__(1024) void k_pair_distances(int S, int W, int tiles, const uint64_t* __restrict__ B,
                                                         int32_t* __restrict__ D, int64_t ldd,
                                                         int64_t* __restrict__ hist) {
  constexpr int CW = 64;
  __shared__ uint64_t xs[16][CW + 1], xl[16][CW + 1];
  __shared__ int part[4][256];
  int ti = 0, rest = blockIdx.x;  // tile (ti, tj), ti <= tj, row by row
  while (rest >= tiles - ti) {
    rest -= tiles - ti;
    ++ti;
  }
  const int tj = ti + rest;
  const int pair = threadIdx.x & 255, q = threadIdx.x >> 8;
  const int ps = pair >> 4, pl = pair & 15;
  int d = 0;
  for (int w0 = 0; w0 < W; w0 += CW) {
    {
      const int c = threadIdx.x >> 6, w = threadIdx.x & 63;  // column and word of the chunk
      const int s = ti * 16 + c, l = tj * 16 + c;
      xs[c][w] = s < S && w0 + w < W ? B[(int64_t)s * W + w0 + w] : 0;
      xl[c][w] = l < S && w0 + w < W ? B[(int64_t)l * W + w0 + w] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CW / 4; ++i) d += __popcll(xs[ps][4 * i + q] ^ xl[pl][4 * i + q]);
    __syncthreads();
  }
  part[q][pair] = d;
  __syncthreads();
  if (q != 0) return;
  d = part[0][pair] + part[1][pair] + part[2][pair] + part[3][pair];
  const int s = ti * 16 + ps, l = tj * 16 + pl;
  if (s >= S || l >= S) return;
  D[(int64_t)s * ldd + l] = d;
  if (ti != tj) D[(int64_t)l * ldd + s] = d;
  if (hist && s < l) atomicAdd(reinterpret_cast<unsigned long long*>(hist + d), 1ull);
}

// n_unique = number of heads s with no earlier head l < s at distance 0: a wavefront
// per head reads its row of the (symmetric) matrix up to the diagonal.
__global__ __launch_bounds__(1024) void k_count_unique(int S, const int32_t* __restrict__ D, int64_t ldd,
                                                       int32_t* __restrict__ n_unique) {
  __shared__ int cnt[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int first = 0;
  for (int s = wave; s < S; s += 16) {
    bool dup = false;
    for (int l = lane; l < s; l += 64) dup |= D[(int64_t)s * ldd + l] == 0;
    first += !__any(dup);
  }
  if (lane == 0) cnt[wave] = first;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < 16; ++w) t += cnt[w];
    *n_unique = t;
  }
}

size_t div_ws(int N, int S, bool need_d, size_t* d_off) {
  const int W = (int)ceil_div(N, 64);
  size_t off = align_up((size_t)S * W * sizeof(uint64_t), 256);
  *d_off = off;
  if (need_d) off += align_up((size_t)S * S * sizeof(int32_t), 256);
  return std::max<size_t>(off, 256);
}

}  // namespace

}  // namespace cpra

extern "C" {

size_t cpra_pairwise_hamming_workspace_bytes(int32_t N, int32_t S) {
  if (N < 0 || S < 1 || S > 1024) return 0;
  size_t d;
  return cpra::div_ws(N, S, true, &d);
}

cpra_status cpra_pairwise_hamming(int32_t N, int32_t S, const uint8_t* X, int64_t ldx, int32_t* D,
                                  int64_t ldd, int64_t* hist, int32_t* n_unique, void* ws,
                                  size_t ws_bytes, cpra_stream_t stream) {
  using namespace cpra;
  if (N < 0) CPRA_FAIL(CPRA_ERR_SHAPE, "pairwise_hamming: N < 0");
  if (S < 1 || S > 1024) CPRA_FAIL(CPRA_ERR_PARAM, "pairwise_hamming: S = %d outside 1..1024", S);
  if (ldx < S || (D && ldd < S)) CPRA_FAIL(CPRA_ERR_SHAPE, "pairwise_hamming: leading dimension < S");
  if (N > 0 && X == nullptr) CPRA_FAIL(CPRA_ERR_NULL, "pairwise_hamming: X is NULL");
  const bool need_d = D == nullptr && (hist || n_unique);
  size_t d_off;
  const size_t need = div_ws(N, S, need_d, &d_off);
  if (ws == nullptr || ws_bytes < need)
    CPRA_FAIL(CPRA_ERR_WORKSPACE, "pairwise_hamming: workspace %zu < %zu bytes", ws_bytes, need);
  if (!D && !hist && !n_unique) return CPRA_OK;
  hipStream_t st = as_stream(stream);
  const int W = (int)ceil_div(N, 64);
  uint64_t* B = reinterpret_cast<uint64_t*>(ws);
  int32_t* Dm = D ? D : reinterpret_cast<int32_t*>(static_cast<char*>(ws) + d_off);
  const int64_t ld = D ? ldd : S;
  if (hist && W == 0) CPRA_CHECK(fill_i64(hist, 1, 0, st));  // else the packing clears it
  {
    ProfScope ps("pack_columns", st, 0.0, (double)N * S + 8.0 * S * W);
    if (W > 0)
      hipLaunchKernelGGL(k_pack_columns, dim3(W, (unsigned)ceil_div(S, 64)), dim3(256), 0, st, N, S,
                         W, X, ldx, B, hist);
    CPRA_CHECK_LAUNCH("pack_columns");
  }
  {
    ProfScope ps("pair_distances", st, 0.0, 4.0 * S * S + 8.0 * S * W);
    const int t = (int)ceil_div(S, 16);
    hipLaunchKernelGGL(k_pair_distances, dim3((unsigned)(t * (t + 1) / 2)), dim3(1024), 0, st, S, W, t, B, Dm, ld,
                       hist);
    CPRA_CHECK_LAUNCH("pair_distances");
  }
  if (n_unique) {
    hipLaunchKernelGGL(k_count_unique, dim3(1), dim3(1024), 0, st, S, Dm, ld, n_unique);
    CPRA_CHECK_LAUNCH("count_unique");
  }
  return CPRA_OK;
}

}  // extern "C"
