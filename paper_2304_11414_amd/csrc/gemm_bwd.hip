// Backward of the local experts' FFN (Section 3.2, footnote to Eq. 1: the backward pass costs about
// twice the forward; the paper trains through automatic differentiation and prints no algorithm, so
// this is the chain rule of  U = X A,  H = GeLU(U),  Y = H B  per expert):
//
//   dH = dY B^T,   dU = dH * GeLU'(U),   dX = dU A^T,   dA = X^T dU,   dB = H^T dY.
//
// With the library's [out, in] weight layout (W1[i] = A_i^T: [F, d]; W2[i] = B_i^T: [d, F]) the two
// data gradients are products with a weight matrix whose CONTRACTION index is its row index
//   dH[r, f] = sum_c dY[r, c] W2[i][c, f],        dX[r, c] = sum_f dU[r, f] W1[i][f, c],
// and the two weight gradients contract over the packed rows of the expert
//   dW2[i][c, f] = sum_r dY[r, c] H[r, f],        dW1[i][f, c] = sum_r dU[r, f] X[r, c],
// so in both an operand reaches the matrix cores across its rows.  Both run on the K loop of gemm_core.h, which reads
// such an operand from LDS with the transposing read: the data gradients as the forward's persistent kernel with
// weights by rows (gemm_fast.hip), the weight gradients as weight_gradient_kernel below.  What those do not take
// (contractions of the data gradient that are no multiple of 64; too few tiles) goes to a plain kernel
// with 128 x 128 x 64 tiles (two blocks per CU, scheduled by the compiler; MODE 0: data gradient, MODE 1: weight
// gradient): four wavefronts (2 x 2), each a quarter of the tile as MFMA 32x32x16 blocks; operand
// tiles go through LDS as [row][k] with k contiguous (rows 144 bytes apart, 16-byte chunks
// XOR-swizzled: fragment reads and staging writes are free of bank conflicts); an operand whose k
// runs along memory rows is transposed in registers on its way into LDS (a thread loads an 8 x 8
// block as eight 16-byte pieces, one per memory row, and writes eight 16-byte chunks, one per tile
// row).  Weight gradients are float32 (the precision gradients are accumulated in); data gradients
// have the layer's 16-bit type.  Sums have a fixed order: bitwise reproducible.

#include <type_traits>

#include "gemm_core.h"

namespace ppmoe {

namespace bwd {

constexpr int BK = 64;
constexpr int kThreads = 256;
constexpr int kRowBytes = 144;                // one tile row in LDS: 64 k-values (128 bytes) + 16 bytes of skew
constexpr int kStages = 2;
constexpr int kTile = 128;                    // rows and columns of a block's tile
constexpr int kTileBytes = kTile * kRowBytes;
constexpr int kStageBytes = 2 * kTileBytes;
constexpr int kPlainLdsBytes = kStages * kStageBytes;   // 72 KiB: two blocks per CU

// Byte offset of 16-byte chunk `ch` (8 k-values) of tile row `row`: chunks are XOR-swizzled with the
// row's group of 16, so that the eight rows a thread writes after its in-register transpose, 16 rows
// apart from the next lane's, and the 16 consecutive rows a fragment read serves per cycle both
// spread over all banks.
__device__ __forceinline__ int lds_chunk(int row, int ch) {
  return row * kRowBytes + ((ch ^ ((row >> 4) & 7)) << 4);
}

// What one operand tile looks like in memory.  `base` points at element (tile row 0, k = 0).
// K-contiguous: element (row, k) at base + row * ld + k; else the tile row index is contiguous:
// element (row, k) at base + k * ld + row.  rows / ks: how many tile rows / k values are valid from
// base on (the rest reads as zero).
struct Operand {
  const bf16_t* base;
  int64_t ld;
  int rows, ks;
};

// One operand tile is 128 rows x 64 k = 1024 chunks of 16 bytes, staged by two wavefronts
// (half: which of the two), eight chunks per thread.
//  * k contiguous in memory: lane = (row % 8) * 8 + chunk; eight lanes read one whole 128-byte line.
//  * rows contiguous in memory: a thread reads an 8 (k) x 8 (rows) block, one 16-byte piece from each of
//    eight consecutive memory rows (16 lanes read 256 contiguous bytes of
//    each), transposes it in registers (v_perm_b32) and writes eight 16-byte chunks, one per tile row.
template <bool K_CONTIGUOUS>
__device__ __forceinline__ void load_tile(const Operand& op, int k0, int half, int lane, u32x4* v) {
  const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
  if (K_CONTIGUOUS) {
    const int ch = lane & 7;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = (lane >> 3) + 8 * half + 16 * i;
      const bool ok = row < op.rows && k0 + ch * 8 < op.ks;
      v[i] = ok ? *reinterpret_cast<const u32x4*>(op.base + static_cast<int64_t>(row) * op.ld + k0 + ch * 8) : zero;
    }
  } else {
    const int rg = lane & 15, kg = half * 4 + (lane >> 4);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int k = k0 + kg * 8 + kk;
      const bool ok = k < op.ks && rg * 8 < op.rows;
      v[kk] = ok ? *reinterpret_cast<const u32x4*>(op.base + static_cast<int64_t>(k) * op.ld + rg * 8) : zero;
    }
  }
}

template <bool K_CONTIGUOUS>
__device__ __forceinline__ void store_tile(unsigned char* lds_tile, int half, int lane, const u32x4* v) {
  if (K_CONTIGUOUS) {
    const int ch = lane & 7;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = (lane >> 3) + 8 * half + 16 * i;
      *reinterpret_cast<u32x4*>(lds_tile + lds_chunk(row, ch)) = v[i];
    }
  } else {
    const int rg = lane & 15, kg = half * 4 + (lane >> 4);
    // v[kk] dword q holds tile rows 2q (low half) and 2q + 1 (high half) at k = kk; the chunk
    // of tile row r wants, in dword q, k = 2q (low) and 2q + 1 (high).
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      u32x4 o;
      const uint32_t sel = (r & 1) ? 0x07060302u : 0x05040100u;
      o.x = __builtin_amdgcn_perm(v[1][r >> 1], v[0][r >> 1], sel);
      o.y = __builtin_amdgcn_perm(v[3][r >> 1], v[2][r >> 1], sel);
      o.z = __builtin_amdgcn_perm(v[5][r >> 1], v[4][r >> 1], sel);
      o.w = __builtin_amdgcn_perm(v[7][r >> 1], v[6][r >> 1], sel);
      *reinterpret_cast<u32x4*>(lds_tile + lds_chunk(rg * 8 + r, kg)) = o;
    }
  }
}

// Which output tile a block computes, and where its operand tiles start.
struct TileInfo {
  int expert, row0, rows, col0, m0, kt_count;
  Operand opA, opB;   // opA: the operand whose tile rows are the output rows; opB: the output columns
};

template <int MODE>
__device__ __forceinline__ bool locate_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                            const int32_t* __restrict__ offsets, int n_exp, int M, int N,
                                            int K, TileInfo& ti) {
  const int n_tiles = (N + kTile - 1) / kTile;
  ti.expert = ti.row0 = ti.rows = ti.col0 = ti.m0 = ti.kt_count = 0;
  // Consecutive block ids land on different XCDs (round robin over 8): remap so that each XCD works on
  // a contiguous run of the tile list and its L2 sees the same panels from many CUs.
  auto xcd_tile = [](int bid, int total) {
    const int per = (total + 7) >> 3;
    const int t = (bid & 7) * per + (bid >> 3);
    return ((bid >> 3) < per && t < total) ? t : -1;
  };
  if (MODE == 0) {
    // tiles ordered expert-major, then n-tile, then m-tile; blocks past the last tile leave
    int total = 0;
    for (int i = 0; i < n_exp; ++i) total += (offsets[i + 1] - offsets[i] + kTile - 1) / kTile * n_tiles;
    int tile = xcd_tile(blockIdx.x, total);
    if (tile < 0) return false;
    bool found = false;
    int lo = offsets[0];
    for (int i = 0; i < n_exp && !found; ++i) {
      const int hi = offsets[i + 1];
      const int m_tiles = (hi - lo + kTile - 1) / kTile;
      const int here = m_tiles * n_tiles;
      if (tile < here) {
        const int nt = tile / m_tiles, mt = tile - nt * m_tiles;
        ti.expert = i;
        ti.row0 = lo + mt * kTile;
        ti.rows = min(kTile, hi - ti.row0);
        ti.col0 = nt * kTile;
        found = true;
      } else {
        tile -= here;
        lo = hi;
      }
    }
    if (!found) return false;
    ti.opA = Operand{A + static_cast<int64_t>(ti.row0) * K, K, ti.rows, K};
    ti.opB = Operand{B + static_cast<int64_t>(ti.expert) * K * N + ti.col0, N, min(kTile, N - ti.col0), K};
    ti.kt_count = (K + BK - 1) / BK;
  } else {
    const int m_tiles = (M + kTile - 1) / kTile;
    int tile = xcd_tile(blockIdx.x, n_exp * m_tiles * n_tiles);
    if (tile < 0) return false;
    // Tiles ordered in blocks of up to 32 (ba row tiles x bb column tiles of one expert: what the 32
    // CUs of an XCD hold at a time, sharing ba + bb operand panels), the blocks of a position going
    // through all the experts before the next position: each XCD's run of the list visits every
    // expert, so an expert with many rows (a long contraction) is not one XCD's alone.
    int bb = n_tiles % 8 == 0 ? 8 : n_tiles % 4 == 0 ? 4 : n_tiles % 2 == 0 ? 2 : 1;
    int ba = 32 / bb;
    while (ba > 1 && m_tiles % ba != 0) ba >>= 1;
    const int per_block = ba * bb, blocks_n = n_tiles / bb;
    const int blk = tile / (n_exp * per_block);
    tile -= blk * n_exp * per_block;
    ti.expert = tile / per_block;
    const int w = tile - ti.expert * per_block;
    const int mt = (blk / blocks_n) * ba + w / bb, nt = (blk % blocks_n) * bb + w % bb;
    ti.m0 = mt * kTile;
    ti.col0 = nt * kTile;
    const int lo = offsets[ti.expert], hi = offsets[ti.expert + 1];
    ti.rows = min(kTile, M - ti.m0);
    // the contraction runs over the expert's packed rows: k = r - lo
    ti.opA = Operand{A + static_cast<int64_t>(lo) * M + ti.m0, M, ti.rows, hi - lo};
    ti.opB = Operand{B + static_cast<int64_t>(lo) * N + ti.col0, N, min(kTile, N - ti.col0), hi - lo};
    ti.kt_count = (hi - lo + BK - 1) / BK;
  }
  return true;
}

// Stores a block's accumulators.  A lane holds output row m = lane & 31 of each 32-row block and, in
// register v, column n = (v / 4) * 8 + (lane >> 5) * 4 + v % 4: four consecutive columns per group.
template <int MODE, int DT>
__device__ __forceinline__ void store_tile_output(const f32x16 (&acc)[2][2], void* __restrict__ C,
                                                  const TileInfo& ti, int N, int M, int wm, int wn, int frow,
                                                  int half) {
  const int cols = min(kTile, N - ti.col0);
#pragma unroll
  for (int mi = 0; mi < 2; ++mi) {
    const int m = wm * 64 + mi * 32 + frow;
    if (m >= ti.rows) continue;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = wn * 64 + ni * 32 + q * 8 + half * 4;
        if (n >= cols) continue;   // (N is a multiple of 8: a group of 4 columns is all in or all out)
        const float v0 = acc[mi][ni][q * 4 + 0], v1 = acc[mi][ni][q * 4 + 1];
        const float v2 = acc[mi][ni][q * 4 + 2], v3 = acc[mi][ni][q * 4 + 3];
        if (MODE == 0) {
          bf16_t* c = static_cast<bf16_t*>(C) + static_cast<int64_t>(ti.row0 + m) * N + ti.col0 + n;
          uint2 p;
          p.x = Elem16<DT>::pack2(v0, v1);
          p.y = Elem16<DT>::pack2(v2, v3);
          *reinterpret_cast<uint2*>(c) = p;
        } else {
          float* c = static_cast<float*>(C) + (static_cast<int64_t>(ti.expert) * M + ti.m0 + m) * N + ti.col0 + n;
          *reinterpret_cast<float4*>(c) = make_float4(v0, v1, v2, v3);
        }
      }
    }
  }
}

// One output tile's products into `acc` (2 x 2 blocks of 32 x 32 per wavefront): two LDS stages, the next
// k-tile's loads in flight while the current one is multiplied.
template <int MODE, int DT>
__device__ __forceinline__ void accumulate_tile(const TileInfo& ti, f32x16 (&acc)[2][2], unsigned char* lds) {
  typedef typename Elem16<DT>::vec8 vec8;
  const Operand opA = ti.opA, opB = ti.opB;
  constexpr bool kAContig = MODE == 0;   // A[r, k]: k contiguous only for the data gradient

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int frow = lane & 31, half = lane >> 5;
  // staging: wavefronts 0, 1 bring in the A tile, 2, 3 the B tile
  const bool stage_b = wave >= 2;
  const int stage_half = wave & 1;

#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

  u32x4 g[8];
  auto load = [&](int kt) {
    if (stage_b) load_tile<false>(opB, kt * BK, stage_half, lane, g);
    else load_tile<kAContig>(opA, kt * BK, stage_half, lane, g);
  };
  auto store = [&](unsigned char* buf) {
    if (stage_b) store_tile<false>(buf + kTileBytes, stage_half, lane, g);
    else store_tile<kAContig>(buf, stage_half, lane, g);
  };
  if (ti.kt_count > 0) {
    load(0);
    store(lds);
  }
  __syncthreads();
  for (int kt = 0; kt < ti.kt_count; ++kt) {
    unsigned char* cur = lds + (kt & 1) * kStageBytes;
    unsigned char* nxt = lds + ((kt + 1) & 1) * kStageBytes;
    if (kt + 1 < ti.kt_count) load(kt + 1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      vec8 fa[2], fb[2];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
        fa[mi] = *reinterpret_cast<const vec8*>(cur + lds_chunk(wm * 64 + mi * 32 + frow, ks * 2 + half));
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        fb[ni] = *reinterpret_cast<const vec8*>(cur + kTileBytes + lds_chunk(wn * 64 + ni * 32 + frow, ks * 2 + half));
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = Elem16<DT>::mfma32(fb[ni], fa[mi], acc[mi][ni]);   // D[n][m]: lane = row m, registers = columns n
      }
    }
    if (kt + 1 < ti.kt_count) store(nxt);
    __syncthreads();
  }
}

// MODE 0 (data gradient):   C[r, n]    = sum_k A[r, k] * B[i][k, n]   for the rows r of expert i
//                           A [rows, K] 16-bit, B [n_exp, K, N] 16-bit, C [rows, N] 16-bit
// MODE 1 (weight gradient): C[i][m, n] = sum_{r in expert i} A[r, m] * B[r, n]
//                           A [rows, M] 16-bit, B [rows, N] 16-bit, C [n_exp, M, N] float32
template <int MODE, int DT>
__global__ __launch_bounds__(kThreads) void grouped_gemm_bwd_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, void* __restrict__ C,
    const int32_t* __restrict__ offsets, int n_exp, int M, int N, int K, int pick_cus) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  TileInfo ti;
  if (MODE == 0 && pick_cus > 0 && !few_big_tiles(offsets, n_exp, N, K, pick_cus)) return;
  if (!locate_tile<MODE>(A, B, offsets, n_exp, M, N, K, ti)) return;
  f32x16 acc[2][2];
  accumulate_tile<MODE, DT>(ti, acc, lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  store_tile_output<MODE, DT>(acc, C, ti, N, M, wave >> 1, wave & 1, lane & 31, lane >> 5);
}

// The weight gradients C[i][m, n] = sum_{r in expert i} A[r, m] * B[r, n] on 256 x 256 tiles: persistent, one block per CU,
// the K loop of gemm_core.h with both operands by rows; a tile's first two k-tiles are requested before the previous
// tile's epilogue.  k-rows past the expert's last one read zeros (the descriptors end there).
//
// What bounds it: the K loop at the clock the power limit leaves, and the float32 result (256 KiB per tile, drained at the
// HBM's rate: 537 MB per launch at 8 experts of 2048 x 8192).
//
// Tiles are ordered in blocks of up to 32 (ba row tiles x bb column tiles of one expert: what the 32 CUs of an XCD hold at
// a time, sharing ba + bb operand panels), the blocks of a position going through all the experts before the next
// position: an XCD's eighth of the list visits every expert, so an expert with many rows (a long contraction) is not
// one XCD's alone, and the CUs of an XCD take their tiles in turn.
constexpr int kWgradOutBytes = 4096;   // per wavefront: 16 rows of 64 float32 columns
constexpr int kWgradLdsBytes = core::kRing + 4 * kWgradOutBytes;

template <int DT>
__global__ __launch_bounds__(kThreads) void weight_gradient_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                                   float* __restrict__ C,
                                                                   const int32_t* __restrict__ offsets, int n_exp, int M,
                                                                   int N) {
  using core::IC;
  constexpr int BM = core::BM, BN = core::BN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t lds0 = core::lds_address(lds);

  const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
  const int total = n_exp * m_tiles * n_tiles, per_xcd = (total + 7) >> 3;
  const int bb = n_tiles % 8 == 0 ? 8 : n_tiles % 4 == 0 ? 4 : n_tiles % 2 == 0 ? 2 : 1;
  int ba = 32 / bb;
  while (ba > 1 && m_tiles % ba != 0) ba >>= 1;
  const int per_block = ba * bb, blocks_n = n_tiles / bb;
  const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
  const int end = min(total, (xcd + 1) * per_xcd);

  struct Tile {
    int expert, m0, col0, lo, rows;
  };
  auto locate = [&](int tile) -> Tile {
    Tile t;
    const int blk = tile / (n_exp * per_block);
    tile -= blk * n_exp * per_block;
    t.expert = tile / per_block;
    const int w = tile - t.expert * per_block;
    t.m0 = ((blk / blocks_n) * ba + w / bb) * BM;
    t.col0 = ((blk % blocks_n) * bb + w % bb) * BN;
    t.lo = offsets[t.expert];
    t.rows = offsets[t.expert + 1] - t.lo;
    return t;
  };

  const unsigned char *ga = nullptr, *gb = nullptr;
  int64_t bytes_a = 0, bytes_b = 0;   // from the tile's first column at the expert's first row to the end of its last row
  const int64_t step_a = static_cast<int64_t>(BK) * M * 2, step_b = static_cast<int64_t>(BK) * N * 2;
  uint32_t off_a[8], off_b[8];        // by half * 4 + chunk
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    off_a[n] = core::staged_by_rows(wave, lane, n >> 2, n & 3, M * 2u);
    off_b[n] = core::staged_by_rows(wave, lane, n >> 2, n & 3, N * 2u);
  }
  auto load = [&](auto j_c, auto n_c, int i) __attribute__((always_inline)) {
    constexpr int j = decltype(j_c)::value, n = decltype(n_c)::value;
    constexpr bool is_a = j == 0 || j == 3;
    const int64_t at = i * (is_a ? step_a : step_b), left = (is_a ? bytes_a : bytes_b) - at;
    const int records = static_cast<int>(left < 0 ? 0 : left < 0x7fffffff ? left : 0x7fffffff);
    core::load_to_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>((is_a ? ga : gb) + at), 0, records, 0x00020000),
                      lds + (i & 1) * core::kKTile + j * core::kHalfTile + (wave * 4 + n) * 1024,
                      is_a ? off_a[(j == 3) * 4 + n] : off_b[(j == 2) * 4 + n], 0);
  };
  auto begin = [&](const Tile& t) __attribute__((always_inline)) {
    ga = reinterpret_cast<const unsigned char*>(A + static_cast<int64_t>(t.lo) * M + t.m0);
    gb = reinterpret_cast<const unsigned char*>(B + static_cast<int64_t>(t.lo) * N + t.col0);
    bytes_a = (static_cast<int64_t>(t.rows) * M - t.m0) * 2;
    bytes_b = (static_cast<int64_t>(t.rows) * N - t.col0) * 2;
    core::each<16>([&](auto i) __attribute__((always_inline)) { load(IC<i.value / 4>{}, IC<i.value % 4>{}, 0); });
    core::each<16>([&](auto i) __attribute__((always_inline)) { load(IC<i.value / 4>{}, IC<i.value % 4>{}, 1); });
  };

  uint32_t a_base[4], b_base[4];
  core::fragment_base(lds0, lane, wm, a_base);
  core::fragment_base(lds0, lane, wn, b_base);
  int tile = xcd * per_xcd + static_cast<int>(blockIdx.x >> 3);
  if (tile >= end) return;
  Tile nxt = locate(tile);
  bool stores_behind = false;
  bool begun = false;
  while (tile < end) {
    const Tile cur = nxt;
    if (!begun) begin(cur);
    tile += step;
    if (tile < end) nxt = locate(tile);
    f32x4 acc[8][8];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
      for (int ni = 0; ni < 8; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (an expert without rows: one k-tile of zeros)
    core::k_loop<DT, true, true, 64>(acc, a_base, b_base, max(1, (cur.rows + BK - 1) / BK), stores_behind, load);
    __builtin_amdgcn_s_barrier();   // every wavefront is done with the ring
    begun = tile < end;
    if (begun) begin(nxt);

    // ---- epilogue: 16 rows x 64 columns at a time through 4 KiB of LDS of the wavefront's own (rows of 256 bytes, 16-byte
    // chunk c of row r at chunk c ^ r), so that a store instruction covers 4 rows x 256 contiguous bytes.  LDS operations
    // of a wavefront complete in order: the next piece is written without waiting for the reads of this one.
    int lane_l = lane;
    asm volatile("" : "+v"(lane_l));
    const int fr = lane_l & 15, fq = lane_l >> 4;
    const uint32_t epi = lds0 + core::kRing + wave * kWgradOutBytes;
    const int nrow = M - cur.m0 - wm * 128, ncol = N - cur.col0 - wn * 128;   // valid rows and columns (may be <= 0)
    const bool full = M - cur.m0 >= BM && N - cur.col0 >= BN;
    float* out = C + (static_cast<int64_t>(cur.expert) * M + cur.m0 + wm * 128 + fq) * N + cur.col0 + wn * 128 + fr * 4;
    u32x4 back[2][4];
    auto write_read = [&](auto s_c) __attribute__((always_inline)) {
      constexpr int s = decltype(s_c)::value, mi = s >> 1, n0 = (s & 1) * 4;
      core::each<4>([&](auto b_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value;
        f32x4 v;
        v[0] = core::read_acc(acc[mi][n0 + b][0]);
        v[1] = core::read_acc(acc[mi][n0 + b][1]);
        v[2] = core::read_acc(acc[mi][n0 + b][2]);
        v[3] = core::read_acc(acc[mi][n0 + b][3]);
        core::lds_write16(epi + fr * 256 + (((b * 4 + fq) ^ fr) << 4), v);
      });
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = i * 4 + fq;
        core::lds_read16<0>(back[s & 1][i], epi + r * 256 + ((fr ^ r) << 4));
      }
    };
    auto store = [&](auto s_c, auto full_c) __attribute__((always_inline)) {
      constexpr int s = decltype(s_c)::value, mi = s >> 1, n0 = (s & 1) * 64;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = mi * 16 + i * 4;   // (+ fq)
        if (decltype(full_c)::value || (r + fq < nrow && n0 + fr * 4 < ncol))
          *reinterpret_cast<u32x4*>(out + static_cast<int64_t>(r) * N + n0) = back[s & 1][i];
      }
    };
    auto drain = [&](auto full_c) __attribute__((always_inline)) {
      write_read(IC<0>{});
      core::each<16>([&](auto s_c) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
        if constexpr (s < 15) {
          write_read(IC<(s < 15 ? s + 1 : 0)>{});
          asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");
        } else {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        core::tie(back[s & 1]);
        store(s_c, full_c);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    if (full) drain(std::true_type{});
    else drain(std::false_type{});
    stores_behind = full;
  }
}

// H = GeLU(U) (not stored when H is NULL: the caller has it) and dU = dH * GeLU'(U) over the packed
// rows [0, offsets[n_exp]) x F, one row per block
// iteration; dH and dU may be the same buffer.  tanh form:  s = 1 / (1 + exp(-2 z)),
// z = sqrt(2/pi) (u + 0.044715 u^3):   GeLU = u s,   GeLU' = s + 2 u s (1 - s) sqrt(2/pi) (1 + 3 * 0.044715 u^2).
// row_dot (may be NULL): row_dot[r] = sum_f dH[r, f] * H[r, f], the derivative with respect to a
// scale factor of the row's expert output (what the gate weight's gradient is made of), added up in a
// fixed order (butterfly inside a wavefront, wavefronts in order).
template <int DT>
__global__ __launch_bounds__(256) void act_backward_kernel(const bf16_t* __restrict__ U, const bf16_t* dH,
                                                           bf16_t* __restrict__ H, bf16_t* dU,
                                                           float* __restrict__ row_dot,
                                                           const int32_t* __restrict__ offsets, int n_exp,
                                                           int F) {
  __shared__ float part[4];
  const int rows = offsets[n_exp];
  const int pieces = F / 8;   // 16-byte pieces per row
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    float dot = 0.f;
    for (int i = threadIdx.x; i < pieces; i += 256) {
      const int64_t at = static_cast<int64_t>(r) * pieces + i;
      const u32x4 u4 = reinterpret_cast<const u32x4*>(U)[at];
      const u32x4 g4 = reinterpret_cast<const u32x4*>(dH)[at];
      const uint32_t uw[4] = {u4.x, u4.y, u4.z, u4.w}, gw[4] = {g4.x, g4.y, g4.z, g4.w};
      uint32_t hw[4], dw[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float u[2], g[2], h[2], du[2];
        Elem16<DT>::widen2(uw[j], u[0], u[1]);
        Elem16<DT>::widen2(gw[j], g[0], g[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float sg = gelu_sigmoid(u[e]);
          h[e] = u[e] * sg;
          const float dz2 = 1.5957691216057308f * fmaf(3.0f * 0.044715f * u[e], u[e], 1.0f);  // d(2 z)/du
          du[e] = g[e] * (sg + h[e] * (1.0f - sg) * dz2);
          dot = fmaf(g[e], h[e], dot);
        }
        hw[j] = Elem16<DT>::pack2(h[0], h[1]);
        dw[j] = Elem16<DT>::pack2(du[0], du[1]);
      }
      if (H != nullptr) reinterpret_cast<u32x4*>(H)[at] = u32x4{hw[0], hw[1], hw[2], hw[3]};   // (uniform)
      reinterpret_cast<u32x4*>(dU)[at] = u32x4{dw[0], dw[1], dw[2], dw[3]};
    }
    if (row_dot != nullptr) {   // (uniform)
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) dot += __shfl_xor(dot, off, 64);
      if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = dot;
      __syncthreads();
      if (threadIdx.x == 0) row_dot[r] = ((part[0] + part[1]) + part[2]) + part[3];
      __syncthreads();
    }
  }
}

// H = GeLU(U) alone, the same arithmetic.
template <int DT>
__global__ __launch_bounds__(256) void gelu_rows_kernel(const bf16_t* __restrict__ U, bf16_t* __restrict__ H,
                                                        const int32_t* __restrict__ offsets, int n_exp, int F) {
  const int64_t pieces = static_cast<int64_t>(offsets[n_exp]) * (F / 8);   // 16-byte pieces
  for (int64_t at = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; at < pieces;
       at += static_cast<int64_t>(gridDim.x) * 256) {
    const u32x4 u4 = reinterpret_cast<const u32x4*>(U)[at];
    const uint32_t uw[4] = {u4.x, u4.y, u4.z, u4.w};
    uint32_t hw[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float u[2], h[2];
      Elem16<DT>::widen2(uw[j], u[0], u[1]);
#pragma unroll
      for (int e = 0; e < 2; ++e) h[e] = u[e] * gelu_sigmoid(u[e]);
      hw[j] = Elem16<DT>::pack2(h[0], h[1]);
    }
    reinterpret_cast<u32x4*>(H)[at] = u32x4{hw[0], hw[1], hw[2], hw[3]};
  }
}

}  // namespace bwd

hipError_t launch_gelu_rows(const moe_config& c, const void* U, void* H, const int32_t* offsets, int64_t rows,
                            hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int64_t pieces = rows * (c.F / 8);
  const int blocks = static_cast<int>(pieces / 256 < 256 * 16 ? (pieces + 255) / 256 : 256 * 16);
  if (c.in_dtype == MOE_F16)
    bwd::gelu_rows_kernel<MOE_F16><<<blocks, 256, 0, s>>>(static_cast<const bf16_t*>(U), static_cast<bf16_t*>(H),
                                                          offsets, c.local_count, c.F);
  else
    bwd::gelu_rows_kernel<MOE_BF16><<<blocks, 256, 0, s>>>(static_cast<const bf16_t*>(U), static_cast<bf16_t*>(H),
                                                           offsets, c.local_count, c.F);
  return hipGetLastError();
}

// Compute units of the current device (asked once per device: the launcher may run under stream capture).
static int cus_of_current_device() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int cus = cached[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    cached[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

size_t expert_ffn_backward_gemm_offset(const moe_config& c, int64_t rows) {
  // U, H, dU: three [rows, F] 16-bit buffers (256-byte aligned), then the persistent GEMM's scratch
  return 3 * ((static_cast<size_t>(rows) * c.F * 2 + 255) & ~size_t(255));
}

size_t expert_ffn_backward_scratch_bytes(const moe_config& c, int64_t rows) {
  return expert_ffn_backward_gemm_offset(c, rows) + ((grouped_gemm_workspace_bytes() + 255) & ~size_t(255));
}

hipError_t launch_expert_ffn_backward(const moe_config& c, int64_t rows, const void* x_sliced,
                                      const int32_t* offsets, const void* W1, const void* W2,
                                      const void* dY, void* dX, float* dW1, float* dW2, void* scratch,
                                      hipStream_t s, float* row_dot, const void* U_saved, const void* H_saved) {
  using namespace bwd;
  // (rows == 0: no packed row can exist; every launch below is then empty except the two weight
  // gradients, whose tiles store zeros)
  const size_t one = (static_cast<size_t>(rows) * c.F * 2 + 255) & ~size_t(255);
  unsigned char* ws = static_cast<unsigned char*>(scratch);
  const bool saved = U_saved != nullptr && H_saved != nullptr;
  const bf16_t* U = saved ? static_cast<const bf16_t*>(U_saved) : reinterpret_cast<const bf16_t*>(ws);
  const bf16_t* H = saved ? static_cast<const bf16_t*>(H_saved) : reinterpret_cast<const bf16_t*>(ws + one);
  bf16_t* H_out = saved ? nullptr : reinterpret_cast<bf16_t*>(ws + one);
  bf16_t* dU = reinterpret_cast<bf16_t*>(ws + 2 * one);
  void* gemm_ws = ws + expert_ffn_backward_gemm_offset(c, rows);
  const int N = c.local_count;
  const bf16_t* xs = static_cast<const bf16_t*>(x_sliced);
  const bf16_t* w1 = static_cast<const bf16_t*>(W1);
  const bf16_t* w2 = static_cast<const bf16_t*>(W2);
  const bf16_t* dy = static_cast<const bf16_t*>(dY);

  // U = X A (the forward's first GEMM without its activation), unless the forward kept it
  if (!saved) {
    hipError_t e = launch_grouped_gemm(c.in_dtype, false, x_sliced, W1, ws, offsets, N, rows, c.F, c.d, gemm_ws, s);
    if (e != hipSuccess) return e;
  }

  const int n_cus = cus_of_current_device() & ~7;
  static std::atomic<uint64_t> attrs_done{0};
  const hipError_t attrs = once_per_device(attrs_done, [] {
    const void* small[] = {reinterpret_cast<const void*>(grouped_gemm_bwd_kernel<0, MOE_BF16>),
                           reinterpret_cast<const void*>(grouped_gemm_bwd_kernel<1, MOE_BF16>),
                           reinterpret_cast<const void*>(grouped_gemm_bwd_kernel<0, MOE_F16>),
                           reinterpret_cast<const void*>(grouped_gemm_bwd_kernel<1, MOE_F16>)};
    const void* big[] = {reinterpret_cast<const void*>(weight_gradient_kernel<MOE_BF16>),
                         reinterpret_cast<const void*>(weight_gradient_kernel<MOE_F16>)};
    for (const void* k : small) {
      hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kPlainLdsBytes);
      if (err != hipSuccess) return err;
    }
    for (const void* k : big) {
      hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kWgradLdsBytes);
      if (err != hipSuccess) return err;
    }
    return hipSuccess;
  });
  if (attrs != hipSuccess) return attrs;
  // An operand by rows on the persistent kernels: 32-bit offsets up to 63 rows past a k-tile's first (63 * 2^25 + 512 < 2^31,
  // where the descriptors end); beyond that the 128 x 128 tiles, whose offsets have 64 bits.
  constexpr int kColumnsByRows = 1 << 24;
  // cc[rows, n] = a[rows, k] b[i][k, n].  The persistent kernel takes contractions of whole k-tiles, unless that
  // would leave more than half of the CUs without a tile; then 128 x 128 tiles, two blocks per CU.  The host knows the row
  // count only as a bound (the counts live on the device).  Where the rank holds some of the experts that is every
  // assignment there is: if an even share of them would be too few tiles, both shapes are launched and the row counts decide
  // (few_big_tiles; the launch that leaves costs about 5 us).
  auto data_gradient = [&](const bf16_t* a, const bf16_t* b, bf16_t* cc, int n, int k) -> hipError_t {
    if (rows == 0) return hipSuccess;
    auto few = [&](int64_t r) { return 2 * ((r + 255) / 256 + N) * ((n + 255) / 256) < n_cus; };
    const bool big = k % BK == 0 && k < (1 << 22) && n < kColumnsByRows && !few(rows);
    const int pick_cus = big && N < c.E && few(rows * N / c.E) ? n_cus : 0;
    if (big) {
      const hipError_t e = launch_grouped_gemm_fast(c.in_dtype, false, a, b, cc, offsets, N, 0, n, k, gemm_ws, s, 0, nullptr,
                                                    nullptr, 1, nullptr, nullptr, true, pick_cus);
      if (e != hipSuccess || pick_cus == 0) return e;
    }
    // (as a second shape it has fewer than n_cus / 2 tiles of 256 x 256 to do, each four of its own)
    const int64_t tiles = big ? 2 * n_cus : ((rows + 127) / 128 + N) * ((n + 127) / 128);
    const unsigned grid = static_cast<unsigned>((tiles + 7) / 8 * 8);
    if (c.in_dtype == MOE_F16)
      grouped_gemm_bwd_kernel<0, MOE_F16><<<grid, kThreads, kPlainLdsBytes, s>>>(a, b, cc, offsets, N, 0, n, k, pick_cus);
    else
      grouped_gemm_bwd_kernel<0, MOE_BF16><<<grid, kThreads, kPlainLdsBytes, s>>>(a, b, cc, offsets, N, 0, n, k, pick_cus);
    return hipGetLastError();
  };
  // cc[i][m, n] = sum over the rows of expert i of a[r, m] b[r, n].  The persistent kernel (one block per CU) unless
  // that would leave more than half of the CUs without a tile; then 128 x 128 tiles, two blocks per CU.
  auto weight_gradient = [&](const bf16_t* a, const bf16_t* b, float* cc, int m, int n) -> hipError_t {
    const int64_t tiles = static_cast<int64_t>(N) * ((m + 255) / 256) * ((n + 255) / 256);
    if (2 * tiles >= n_cus && m < kColumnsByRows && n < kColumnsByRows) {
      const unsigned grid = static_cast<unsigned>(tiles < n_cus ? (tiles + 7) / 8 * 8 : n_cus);
      if (c.in_dtype == MOE_F16) weight_gradient_kernel<MOE_F16><<<grid, kThreads, kWgradLdsBytes, s>>>(a, b, cc, offsets, N, m, n);
      else weight_gradient_kernel<MOE_BF16><<<grid, kThreads, kWgradLdsBytes, s>>>(a, b, cc, offsets, N, m, n);
      return hipGetLastError();
    }
    const int64_t small_tiles = static_cast<int64_t>(N) * ((m + 127) / 128) * ((n + 127) / 128);
    const unsigned grid = static_cast<unsigned>((small_tiles + 7) / 8 * 8);
    if (c.in_dtype == MOE_F16)
      grouped_gemm_bwd_kernel<1, MOE_F16><<<grid, kThreads, kPlainLdsBytes, s>>>(a, b, cc, offsets, N, m, n, 0, 0);
    else
      grouped_gemm_bwd_kernel<1, MOE_BF16><<<grid, kThreads, kPlainLdsBytes, s>>>(a, b, cc, offsets, N, m, n, 0, 0);
    return hipGetLastError();
  };

  // dH = dY B^T  (into the dU buffer), then H = GeLU(U), dU = dH * GeLU'(U) in place
  hipError_t e = data_gradient(dy, w2, dU, c.F, c.d);
  if (e != hipSuccess) return e;
  {
    const int blocks = static_cast<int>(rows < 256 * 16 ? (rows > 0 ? rows : 1) : 256 * 16);
    if (c.in_dtype == MOE_F16)
      act_backward_kernel<MOE_F16><<<blocks, 256, 0, s>>>(U, dU, H_out, dU, row_dot, offsets, N, c.F);
    else
      act_backward_kernel<MOE_BF16><<<blocks, 256, 0, s>>>(U, dU, H_out, dU, row_dot, offsets, N, c.F);
  }
  e = data_gradient(dU, w1, static_cast<bf16_t*>(dX), c.d, c.F);   // dX = dU A^T
  if (e != hipSuccess) return e;
  // dB^T[i] = dY_i^T H_i  ([d, F]);  dA^T[i] = dU_i^T X_i  ([F, d])
  e = weight_gradient(dy, H, dW2, c.d, c.F);
  if (e != hipSuccess) return e;
  return weight_gradient(dU, xs, dW1, c.F, c.d);
}

}  // namespace ppmoe
