// Grouped expert GEMMs on few rows (token generation) for bf16 and fp16:
//
//   C[r, n] = act( sum_k A[r, k] * B[i][n, k] ),  offsets[i] <= r < offsets[i+1]
//
// With a handful of rows per expert the work is one pass over the weights: it is bound by the HBM stream and by
// the latencies in front of it.  The kernel of the large tiles spends some 50 us per launch on those (one
// block per CU: row list, first k-tile, hand-over, output transpose one after another).  Here a block owns 32
// columns of one expert: no staging, no barrier in the loop; its eight wavefronts split the contraction, fetch both
// MFMA operands straight from memory (a lane's operand is 16 bytes of a row, 256 bytes of each of 32 rows at a
// time) and meet once, to add their partial sums in wavefront order (fixed float32 summation order).  Two blocks on
// a CU have 128 KiB of loads in flight.  Measured (layer, 8 experts, d = 2048, F = 8192, bf16, 537 MB of weights):
// 16 tokens top-1 194 -> 127 us, 128 tokens 197 -> 137 us.  Tried and slower: the next span prefetched into a second
// register set (157 us), a block per 32 rows instead of passes (128 tokens: 372 us), non-temporal loads of the weights
// (131 us), 16 wavefronts a block (142 us).
// An expert with many rows is bound by the fetches instead: every block of 32 columns reads all its rows.  A pass takes
// up to 64 rows, half the contraction at a time, so that a fetched weight feeds four products (128 rows on one expert of
// 2048 x 8192: layer 161 us with 32 rows a pass, 128 us now; wavefronts side by side on groups of 32 rows: 157 us).

#include <type_traits>

#include "common.h"

namespace ppmoe {

namespace few {

constexpr int BN = 32;           // columns of a block: two 16-row weight fragments per wavefront
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kTok = 32;         // rows whose partial sums are in LDS at a time
constexpr int kLd = BN + 4;      // floats per row of partial sums in LDS

// FUSE: as in the kernel of the large tiles.  0: packed tensors.  1: packed row r of A is row
// aux_rows[r] / aux_div of the matrix given as A.  2: packed row r belongs to assignment a = aux_rows[r] of
// token a / aux_div; if it is that token's only kept pick here it is stored, times aux_w[a], as row `token`
// of C, else unweighted as packed row r of C2.
template <bool GELU, int FUSE, int DT>
__global__ __launch_bounds__(kThreads, 4) void grouped_gemm_few_rows_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
    const int32_t* __restrict__ offsets, int n_exp, int Nout, int K, int most, const int32_t* __restrict__ aux_rows,
    const float* __restrict__ aux_w, int aux_div, const int32_t* __restrict__ aux_inv, bf16_t* __restrict__ C2,
    unsigned long long* __restrict__ clock_words) {
  typedef typename Elem16<DT>::vec8 vec8;
  __shared__ __attribute__((aligned(16))) float part[kWaves][kTok][kLd];
  if (most > 0 && !no_expert_above(offsets, n_exp, most)) return;
  const int n_tiles = (Nout + BN - 1) / BN;
  const int expert = blockIdx.x / n_tiles, col0 = (blockIdx.x - expert * n_tiles) * BN;
  const int lo = offsets[expert], cnt = offsets[expert + 1] - lo;
  // (read back by moe_ffn_clock: the first block of the first expert with rows)
  const bool clocked = threadIdx.x == 0 && col0 == 0 && lo == offsets[0] && (cnt > 0 || expert == n_exp - 1);
  if (clocked) {
    clock_words[0] = clock64();
    clock_words[1] = wall_clock64();
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;   // operand layout of the 16x16x32 MFMA: row r, k-values 8 g .. 8 g + 7
  const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
  const bf16_t* wrow[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
    wrow[nt] = B + (static_cast<size_t>(expert) * Nout + min(col0 + nt * 16 + r, Nout - 1)) * K + g * 8;

  // Finishes four columns of packed row `row`.
  auto store = [&](int row, int n, f32x4 v) __attribute__((always_inline)) {
    if (GELU) v = gelu_tanh4(v);
    bf16_t* base = C;
    if (FUSE == 2) {
      const int a = aux_rows[row], t = a / aux_div;
      int kept = 1;
      if (aux_div > 1) {
        kept = 0;
        for (int j = 0; j < aux_div; ++j) kept += aux_inv[t * aux_div + j] >= 0;
      }
      if (kept == 1) {
        v *= aux_w[a];
        row = t;
      } else {
        base = C2;
      }
    }
    uint2 o;
    o.x = Elem16<DT>::pack2(v[0], v[1]);
    o.y = Elem16<DT>::pack2(v[2], v[3]);
    *reinterpret_cast<uint2*>(base + static_cast<size_t>(row) * Nout + col0 + n) = o;
  };
  // One pass over the block's weights: MT groups of 16 of the expert's rows, J k-steps of 32 fetched at a time.
  auto pass = [&](int t0, int rows, auto mt_c, auto j_c) __attribute__((always_inline)) {
    constexpr int MT = decltype(mt_c)::value, J = decltype(j_c)::value;
    constexpr int kStep = 32 * J;
    const bf16_t* trow[MT];
    f32x4 acc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int p = lo + t0 + min(mt * 16 + r, rows - 1);   // (rows past the end re-read the last one)
      trow[mt] = A + static_cast<size_t>(FUSE == 1 ? aux_rows[p] / aux_div : p) * K + g * 8;
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // WHOLE: the span ends inside the row.
    auto span = [&](int k0, auto whole_c) __attribute__((always_inline)) {
      constexpr bool WHOLE = decltype(whole_c)::value;
      u32x4 w[J][2], x[J][MT];
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = k0 + 32 * j;
        const bool ok = WHOLE || k + g * 8 < K;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          w[j][nt] = ok ? *reinterpret_cast<const u32x4*>(wrow[nt] + k) : zero;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) x[j][mt] = ok ? *reinterpret_cast<const u32x4*>(trow[mt] + k) : zero;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt)
            acc[mt][nt] = Elem16<DT>::mfma16(__builtin_bit_cast(vec8, w[j][nt]), __builtin_bit_cast(vec8, x[j][mt]),
                                             acc[mt][nt]);
    };
    int k0 = wave * kStep;
    for (; k0 + kStep <= K; k0 += kWaves * kStep) span(k0, std::true_type{});
    if (k0 < K) span(k0, std::false_type{});
    // The wavefronts' partial sums meet in LDS, 32 rows at a time.
#pragma unroll
    for (int half = 0; half < (MT + 1) / 2; ++half) {
      if (t0 > 0 || half > 0) __syncthreads();   // the partial sums before these have been read
      // D = W_frag (16 n) x Tok_frag^T (16 m): lane holds token m = lane % 16, columns 4 (lane / 16) + i
#pragma unroll
      for (int mt = 2 * half; mt < min(MT, 2 * half + 2); ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          *reinterpret_cast<f32x4*>(&part[wave][(mt & 1) * 16 + r][nt * 16 + g * 4]) = acc[mt][nt];
      __syncthreads();
      const int m = threadIdx.x >> 3, n = (threadIdx.x & 7) * 4;   // four columns of one row per thread
      if (m < min(kTok, rows - half * kTok) && col0 + n < Nout) {   // (Nout is a multiple of 8: four are all in or all out)
        f32x4 v = *reinterpret_cast<const f32x4*>(&part[0][m][n]);
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += *reinterpret_cast<const f32x4*>(&part[w][m][n]);
        store(lo + t0 + half * kTok + m, n, v);
      }
    }
  };
  for (int t0 = 0; t0 < cnt; t0 += 2 * kTok) {
    const int rows = min(2 * kTok, cnt - t0);
    if (rows > kTok) pass(t0, rows, std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    else if (rows > 16) pass(t0, rows, std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    else pass(t0, rows, std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
  }
  if (clocked) {
    clock_words[2] = clock64();
    clock_words[3] = wall_clock64();
  }
}

}  // namespace few

hipError_t launch_grouped_gemm_few_rows(int in_dtype, bool gelu, const bf16_t* A, const bf16_t* B, bf16_t* C,
                                        const int32_t* offsets, int n_exp, int Nout, int K, int most,
                                        void* workspace, hipStream_t s, int fuse,
                                        const int32_t* aux_rows, const float* aux_w, int aux_div,
                                        const int32_t* aux_inv, bf16_t* C2) {
  using namespace few;
  if ((fuse == 1 && !gelu) || (fuse == 2 && gelu) || fuse < 0 || fuse > 2 || (fuse != 0 && aux_rows == nullptr) ||
      (fuse == 2 && aux_w == nullptr) || aux_div < 1 ||
      (fuse == 2 && aux_div != 1 && (aux_inv == nullptr || C2 == nullptr)))
    return hipErrorInvalidValue;
  const hipError_t e = grouped_gemm_set_up(s);
  if (e != hipSuccess) return e;
  unsigned long long* clock_words = gemm_clock_words(workspace);
  const unsigned grid = static_cast<unsigned>(n_exp) * static_cast<unsigned>((Nout + BN - 1) / BN);
#define PPMOE_LAUNCH(G, F)                                                                                 \
  do {                                                                                                     \
    if (in_dtype == MOE_F16)                                                                               \
      grouped_gemm_few_rows_kernel<G, F, MOE_F16><<<grid, kThreads, 0, s>>>(                               \
          A, B, C, offsets, n_exp, Nout, K, most, aux_rows, aux_w, aux_div, aux_inv, C2, clock_words);                  \
    else                                                                                                   \
      grouped_gemm_few_rows_kernel<G, F, MOE_BF16><<<grid, kThreads, 0, s>>>(                              \
          A, B, C, offsets, n_exp, Nout, K, most, aux_rows, aux_w, aux_div, aux_inv, C2, clock_words);                  \
  } while (0)
  if (fuse == 1) PPMOE_LAUNCH(true, 1);
  else if (fuse == 2) PPMOE_LAUNCH(false, 2);
  else if (gelu) PPMOE_LAUNCH(true, 0);
  else PPMOE_LAUNCH(false, 0);
#undef PPMOE_LAUNCH
  return hipGetLastError();
}

}  // namespace ppmoe
