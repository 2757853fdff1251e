// Fast path of the grouped expert GEMMs (Section 3.3.2; FFN = GeLU(X A) B, Section 3.1.3) for bf16
// and fp16:
//
//   C[r, n] = act( sum_k A[r, k] * B[i][n, k] ),  offsets[i] <= r < offsets[i+1]
//
// Block tile 256 x 256 x 64 with the K loop of gemm_core.h, which says what bounds it.
//
// Scheduling: the kernel is persistent (one block per CU; consecutive block ids go round-robin over
// the 8 XCDs, checked once per process with the XCC_ID register).  Row tiles are "big" (up to 256
// rows) or, for the last at most 128 rows of an expert, "small" (computed as 32/64/128 rows x 256
// columns with the four wavefronts side by side: a tail of a few rows costs a few MFMAs, not a tile).
// Big tiles are taken whole, in rounds of the whole chip; the tile list is ordered in blocks of a
// few row tiles x a few column tiles and an XCD runs one block per round, so the CUs sharing an L2
// work on the same panels and neighbouring XCDs on neighbouring blocks.  What is left (big tiles
// when there are fewer than CUs, and the small tiles) is one stream of k-tiles per XCD cut into
// shares (stream-K); an XCD runs its stream between two of its rounds, each XCD at another point of
// the launch, so that this HBM-bound work runs beside the other XCDs' MFMA-bound rounds instead of as
// a phase of the whole chip.  A tile cut between CUs is finished by the CU that holds its first k-tile; the
// others store their partial accumulators to a scratch slot and raise a flag.  Writer and reader of
// a slot sit on the same XCD, so the hand-over goes through their shared L2 without device-scope
// cache maintenance (the device-scope fences are kept as a fallback for any other placement).
//
// A hand-over that does not arrive within the spin limit (the persistent blocks were not all resident:
// another kernel held compute units), or that would come from another XCD's L2, is not waited for:
// the reading CU computes the missing shares itself, each as its owner would have and added in the same order, so
// the output tile is always complete, has the same bits, and the error word only reports lost time.
//
// A CU goes from one tile to the next without draining: the next tile is looked up while the current one
// starts, its first two k-tiles are requested (the ring of the K loop is free by then) before the current tile's
// epilogue, which has LDS of its own, and the epilogue's stores drain under the next tile's first k-tiles.  (Not so with
// FUSE 2: place_rows waits for loads of its own behind them, and loads return in order.)

#include <atomic>
#include <mutex>

#include "gemm_core.h"

namespace ppmoe {


namespace fast {

using namespace core;

// LDS: the K loop's ring, then 4 KiB per wavefront for the output transpose.
constexpr int kOutBytes = 4096;                              // 16 rows of 128 columns
constexpr int kLdsBytes = kRing + 4 * kOutBytes;             // 144 KiB
// A small tile's k-tiles in the ring: three stages of weight rows (32 KiB), two of token rows (up to 16 KiB).
constexpr int kSmallWeights = 256 * BK * 2, kSmallTokens = 128 * BK * 2;
static_assert(3 * kSmallWeights + 2 * kSmallTokens <= kRing, "a small tile's stages fit in the ring");

// How a tile is computed.  0: "big", the wavefronts form a 2 x 2 grid of 128 x 128 sub-tiles.
// 1, 2, 4: "small", at most 32, 64, 128 rows: the wavefronts stand side by side, each owning all
// the rows and 64 of the 256 columns (2 KIND x 4 accumulator blocks instead of 8 x 8), so a tail of a
// few rows costs its share of MFMAs and the fetch of its weight panel, not a whole tile.
__device__ __forceinline__ int tile_kind(int rows) { return rows <= 32 ? 1 : rows <= 64 ? 2 : 4; }

// An expert's rows are cut into m-tiles of BM; its last m-tile is "small" when it has at most
// kSmallRows rows.  The tile list has two parts: all the other ("big") tiles, ordered expert-major,
// in blocks of row tiles x column tiles; then the small tiles, ordered
// expert-major, then n-tile.
constexpr int kSmallRows = 128;
constexpr int kMinShare = 16;   // k-tiles: the smallest share of a cut stream a CU is given (8, 12, 24 and 32 measured slower)

__device__ __forceinline__ void expert_tiles(int cnt, int small_rows, int& big_m, int& small) {
  const int m_tiles = (cnt + BM - 1) / BM;
  small = (m_tiles > 0 && cnt - (m_tiles - 1) * BM <= small_rows) ? 1 : 0;
  big_m = m_tiles - small;
}

// A segment: k-tiles [kb, ke) of one output tile.  stream: index of the tile in the XCD's stream (cut tiles).
struct Segment {
  int expert, row0, rows, col0, kind;
  int kb, ke, stream;
  int list;        // which of the two row lists in LDS is its
  bool resumed;    // another CU's share of a tile whose hand-over did not arrive
  bool valid;
};

// Inclusive prefix sum over the wavefront.
__device__ __forceinline__ int sum_over_lanes_up_to(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Scratch for tiles cut between CUs: per block one slot of 256 x 256 float accumulators for the
// partial sums it hands over and one flag, plus a second slot where it parks its own partial sums
// when a hand-over it waited for did not arrive (the first slot may still be unread by its reader).
constexpr int kSlotFloats = BM * BN;
constexpr int kSlotsPerBlock = 2;
// Behind the flags and the error word: four 64-bit words in which block 0 leaves the shader-clock
// and wall-clock counters at its start and at its end (what clock the launch ran at).
constexpr int kClockWord = 2 * kMaxPersistentBlocks + 2;   // (32-bit word index in `flags`, 8-byte aligned)
constexpr int kDefaultSpinLimit = 1 << 17;   // polls of a flag (a few tenths of a second) before giving up

// The XCD (accelerator complex die) this wavefront runs on.
__device__ __forceinline__ uint32_t xcc_id() {
  uint32_t v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(v));
  return v;
}

// Set-up check of the placement rule the hand-over of partial sums relies on (block b runs on XCD
// b mod 8, so blocks b and b' with b = b' mod 8 share an L2): every block reports where it ran.
__device__ uint32_t g_xcc_of_block[kMaxPersistentBlocks];   // (each device holds its own copy)
__global__ __launch_bounds__(kThreads) void xcc_probe_kernel() {
  if (threadIdx.x == 0) g_xcc_of_block[blockIdx.x] = xcc_id();
}

// FUSE: 0: A and C are the packed tensors.  1: the rows of A are read through a list (packed row r is
// row aux_rows[r] / aux_div of the matrix given as A): the index selection of Algorithm 1 done by
// the loads of the first GEMM.  2: the placement of the expert outputs into the layer output done by
// the stores of the second GEMM: packed row r belongs to assignment a = aux_rows[r] of token
// a / aux_div; if it is that token's only kept pick on this device (aux_inv[token, :] has no other
// entry >= 0; always so with aux_div == 1) it is multiplied by aux_w[a] and stored as row `token` of
// C, which nobody else writes; otherwise it is stored unweighted as packed row r of C2 and left to
// the combine kernel, which has to add it to the token's other picks.
// RAGGED: K is not a multiple of 64 (it is one of 8).  The pieces of the last k-tile that lie past the
// end of a row belong to the next row: their loads get an offset no descriptor covers and read zeros,
// which costs one vector OR per load (a variant of its own, so that the other one does not pay it).
// B_BY_ROWS: B is [n_exp, K, Nout] (its contraction index is its row): the data gradients of the backward pass.
// ACT: 0: no activation; 1: GeLU; 2: the pre-activations are stored as C2, and GeLU of them as stored (see gelu_sigmoid) as C
// (no FUSE): a training step keeps both.
template <int ACT, int FUSE, int DT, bool RAGGED, bool B_BY_ROWS>
__global__ __launch_bounds__(kThreads) void grouped_gemm_fast_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
    const int32_t* __restrict__ offsets, int n_exp, int few_most, int Nout, int K, float* __restrict__ slots,
    uint32_t* __restrict__ flags, uint32_t epoch, int same_l2, int spin_limit,
    const int32_t* __restrict__ aux_rows, const float* __restrict__ aux_w, int aux_div,
    const int32_t* __restrict__ aux_inv, bf16_t* __restrict__ C2, int pick_cus) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  __shared__ int contrib[kMaxPersistentBlocks / 8 + 1];   // [0] = how many, then the block ids whose slots to add
  __shared__ int contrib_failed;
  // Per expert: its first packed row, the next expert's, big row tiles and small row tiles before it.
  __shared__ u32x4 table[kMaxExperts];
  __shared__ int wave_sums[2][4];
  // Per tile row (of this tile and the next): FUSE 1: aux_rows; FUSE 2: where it goes (>= 0: row of C; else ~packed row
  // of C2) and its weight.
  __shared__ uint32_t row_list[FUSE == 0 ? 1 : 2 * BM], row_weight[FUSE == 2 ? 2 * BM : 1];
  if (few_most > 0 && no_expert_above(offsets, n_exp, few_most)) return;   // (the kernel for few rows has done it)
  if (B_BY_ROWS && few_big_tiles(offsets, n_exp, Nout, K, pick_cus)) return;   // (the 128 x 128 tiles do it)
  const uint32_t my_xcc = xcc_id();
  // A block's flag is down before it can be looked at: whatever the caller's workspace held, a stale
  // word cannot pass for this launch's epoch (the readers poll tens of microseconds from now).
  if (threadIdx.x == 0)
    __hip_atomic_store(flags + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    unsigned long long* cw = reinterpret_cast<unsigned long long*>(flags + kClockWord);
    cw[0] = clock64();
    cw[1] = wall_clock64();
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 15, fq = lane >> 4;
  const uint32_t lds0 = lds_address(lds);

  constexpr int kStores = ACT == 2 ? 64 : 32;   // of a wavefront, for a whole tile

  // ---- the tile list ---------------------------------------------------------------------------
  const int n_tiles = (Nout + BN - 1) / BN;
  const int KT = (K + BK - 1) / BK;
  int total_big, total_small;
  {
    int big_m = 0, small = 0, lo = 0, hi = 0;
    if (tid < n_exp) {
      lo = offsets[tid];
      hi = offsets[tid + 1];
      expert_tiles(hi - lo, kSmallRows, big_m, small);
    }
    int big_sum = sum_over_lanes_up_to(big_m), small_sum = sum_over_lanes_up_to(small);
    if (lane == 63) {
      wave_sums[0][wave] = big_sum;
      wave_sums[1][wave] = small_sum;
    }
    __syncthreads();
    total_big = total_small = 0;
    for (int w = 0; w < 4; ++w) {
      if (w == wave) {
        big_sum += total_big;
        small_sum += total_small;
      }
      total_big += wave_sums[0][w];
      total_small += wave_sums[1][w];
    }
    if (tid < n_exp)
      table[tid] = u32x4{static_cast<uint32_t>(lo), static_cast<uint32_t>(hi), static_cast<uint32_t>(big_sum - big_m),
                         static_cast<uint32_t>(small_sum - small)};
    __syncthreads();
    total_big = __builtin_amdgcn_readfirstlane(total_big) * n_tiles;
    total_small = __builtin_amdgcn_readfirstlane(total_small) * n_tiles;
  }
  // The expert that holds the nth big (COL 2) or small (COL 3) row tile: the last one whose entry is at most nth.
  struct Expert {
    int index, lo, hi, before;
  };
  auto find_expert = [&](auto col_c, int nth) -> Expert {
    constexpr int COL = decltype(col_c)::value;
    Expert e = {0, 0, 0, 0};
    for (int i0 = 0; i0 < n_exp; i0 += 64) {
      const u32x4 v = lds_read_quad(lds_address(table) + 16 * min(i0 + lane, n_exp - 1));
      const int n = __popcll(__ballot(i0 + lane < n_exp && static_cast<int>(v[COL]) <= nth));
      if (n == 0) break;
      e.index = i0 + n - 1;
      e.lo = __builtin_amdgcn_readlane(v[0], n - 1);
      e.hi = __builtin_amdgcn_readlane(v[1], n - 1);
      e.before = __builtin_amdgcn_readlane(v[COL], n - 1);
    }
    return e;
  };

  // ---- this block's work -----------------------------------------------------------------------
  // Consecutive block ids go round-robin over the 8 XCDs, so `cus` = gridDim/8 blocks share an L2.
  //  * Big tiles are taken whole, in rounds of the whole chip: in round j, XCD x runs the cus tiles
  //    starting at (8 j + x) cus of the tile list, one per CU.  The list is ordered so that those
  //    cus tiles are a block of a few row tiles x a few column tiles (see big_tile): they run at
  //    the same time and in step along K, which is what lets the L2 serve a panel once for several
  //    CUs.  What is left after the whole rounds (fewer than 8 cus tiles) is split evenly over the
  //    XCDs: one more, partial round per XCD -- unless an XCD's part is at most a quarter of its
  //    CUs, see below.
  //  * The small tiles (an eighth per XCD), and before them those few left-over big tiles, form one
  //    stream of k-tiles that is cut into shares, so that a 3-row tail of an expert, or one tile more
  //    than the chip has CUs, does not cost a whole tile slot and every CU has work.  A tile cut
  //    this way is finished by the CU that holds its first k-tile.
  const int xcd = blockIdx.x & 7, cu = blockIdx.x >> 3, cus = gridDim.x >> 3;
  // Big tiles: whole rounds of the chip first -- in round j XCD x takes the cus tiles starting at
  // (8 j + x) cus of the list, so at any time the eight XCDs work on neighbouring blocks -- then the
  // remainder (fewer than 8 cus tiles), an eighth to each XCD.
  const int chip = 8 * cus;
  const int full_rounds = total_big / chip, rem = total_big - full_rounds * chip;
  const int lx0 = full_rounds * chip + ((rem * xcd) >> 3);
  const int lx1 = full_rounds * chip + ((rem * (xcd + 1)) >> 3);
  const int sx0 = ((total_small * xcd) >> 3);
  const int sx1 = ((total_small * (xcd + 1)) >> 3);
  // The XCD's part of the remainder (r tiles) either runs as one more, partial round, in which
  // cus - r CUs idle for a tile's KT k-tiles, or joins the stream and is cut among all CUs, which
  // costs the hand-over of the big tiles' partial sums (256 KiB each, and an epilogue that waits for
  // them: about 25 k-tiles' time) and, where tiles share panels, the L2's help: the CUs of a stream
  // are not in step along K.  It is cut when it is small (up to a quarter of the CUs: one tile more
  // than the chip has CUs must not cost a round); and, when there is no whole round at all (few tiles
  // per expert: the tiles share little), when the idle time of the partial round would be larger
  // than that price (long contractions).  Measured: with whole rounds before it, cutting 12 tiles of
  // 320 k-tiles per XCD costs 6 % of the launch, running them as a round 3 %.
  const int rem_x = lx1 - lx0;
  const bool cut_big = rem_x > 0 && (rem_x * 4 <= cus ||
                                     (full_rounds == 0 && KT * (cus - rem_x) >= 25 * cus));
  const int rounds = full_rounds + (!cut_big && lx1 > lx0 ? 1 : 0);
  const int stream_big = cut_big ? lx1 - lx0 : 0;                  // big tiles at the head of the stream
  const int stream_tiles = stream_big + sx1 - sx0;
  // (32 bits: KT <= 2^16, up to cus big tiles, and an eighth of the n_exp * n_tiles panels of weights; these fit the card's
  // 288 GB, so units * cus stays below 2^31 also with 8 columns.  64-bit divisions are 100 instructions each, before the first load.)
  const int units = stream_tiles * KT;
  // With a short contraction a hand-over costs more than the rest of the tile, and a share of kMinShare k-tiles is
  // several tiles one after another while other CUs idle: the stream is then dealt out in whole tiles.  Up to 20 k-tiles
  // always; up to 32 where a partial round keeps the other CUs from their shares; up to 40 where big tiles are in it.  Whole
  // k-tiles, whole against cut: 61 layers of 40 to 900 rows on one expert 0.89 of the time in the mean, 60 of 40 to 6000 tokens over 1 to
  // 12 experts 0.73, 120 FFN backwards of up to 6000 rows 0.81 (8 experts of about 256 rows of 512 x 2048: first product 42 us
  // cut, 20 whole); slower in 5 of the 241, by up to 3 % (1300 tokens of 768 x 2112, top-2 over 6 experts: 103 cut, 106 whole).
  // The lines themselves lie where rows of no whole k-tiles turn: 3000 rows of 520 x 1000 over 4 experts 83 cut, 26 whole, 700 of 1304 x
  // 4000 67 and 38, 3000 of 1992 x 4000 over 12 93 and 63; beyond them 136 of 1992 x 1000 over 12 33 and 46, 12000
  // of 1800 x 4000 over 12 241 and 255, 1500 of 3528 x 1000 over 2 68 and 80.
  // (A spin limit of 0 is the diagnostic setting in which nobody waits for a hand-over: it cuts all the same.)
  const bool whole = spin_limit > 0 && KT <= (stream_big > 0 ? 40 : full_rounds == 0 && rounds > 0 ? 32 : 20);
  // Shares shorter than kMinShare k-tiles are not worth their hand-over: fewer CUs then take part.
  const int takers = max(1, min(cus, whole ? stream_tiles : units / kMinShare));
  const int deal = whole ? KT : 1;   // k-tiles dealt out together
  const int deals = whole ? stream_tiles : units;
  auto share_begin = [&](int c) -> int {
    return static_cast<int>(static_cast<uint32_t>(deals * min(c, takers)) / static_cast<uint32_t>(takers)) * deal;
  };
  // When an XCD runs its share of the stream: before big round `stream_slot` (= rounds: after the
  // last one), the XCDs spread over the launch.  The stream's small tiles are bound by the HBM stream
  // of their weight panels and leave CUs without a share idle; the big tiles are bound by the matrix
  // cores: spread over the XCDs in time, one kind of work runs beside the other instead of as a
  // phase of the whole chip at the end (measured on four workloads: up to 9 % of a launch).
  const int stream_slot = ((7 - xcd) * (rounds + 1)) >> 3;
  int round = 0;
  // The partial round's tiles go to the first CUs of an XCD, so the shares are dealt out from the last one:
  // where there are fewer shares than CUs, a CU with a tile of that round is the last to get one as well.
  const int share = cus - 1 - cu;
  int u = share_begin(share);
  const int u_end = share_begin(share + 1);

  // Big tiles of one expert are listed in blocks of hm row tiles x hn column tiles (hm = up to 8,
  // hm * hn = the CUs of an XCD), row tile fastest inside a block, blocks along the columns first:
  // `cus` consecutive tiles -- what an XCD runs at the same time -- share hm token panels and hn
  // weight panels, and the blocks the eight XCDs run at the same time share their token panels.
  // (Listing an expert column by column instead gives every CU of an XCD its own token panel: with
  // 100 row tiles per expert each token panel was fetched again for every column tile.)
  auto big_tile = [&](int tile, Segment& s) {
    const Expert e = find_expert(IC<2>{}, tile / n_tiles);
    const int lo = e.lo, hi = e.hi;
    s.expert = e.index;
    tile -= e.before * n_tiles;
    int big_m, small;
    expert_tiles(hi - lo, kSmallRows, big_m, small);
    const int hm = min(big_m, 8), hn = max(1, cus / hm);
    const int mb = tile / (hm * n_tiles);              // block row
    const int t2 = tile - mb * hm * n_tiles;
    const int hmb = min(hm, big_m - mb * hm);          // its height (the last one may be lower)
    const int nb = t2 / (hmb * hn);                    // block inside the block row
    const int t3 = t2 - nb * hmb * hn;
    const int n_in = t3 / hmb, m_in = t3 - n_in * hmb;
    s.row0 = lo + (mb * hm + m_in) * BM;
    s.rows = min(BM, hi - s.row0);
    s.col0 = (nb * hn + n_in) * BN;
    s.kind = 0;
  };
  // The small tiles: expert-major, then column tile.
  auto small_tile = [&](int tile, Segment& s) {
    const int nth = tile / n_tiles;
    const Expert e = find_expert(IC<3>{}, nth);
    int big_m, small;
    expert_tiles(e.hi - e.lo, kSmallRows, big_m, small);
    s.expert = e.index;
    s.row0 = e.lo + big_m * BM;
    s.rows = e.hi - s.row0;
    s.col0 = (tile - nth * n_tiles) * BN;
    s.kind = tile_kind(s.rows);
  };
  auto next_segment = [&]() -> Segment {
    Segment s = {};
    while (round < rounds || u < u_end) {
      if (round < rounds && !(u < u_end && round >= stream_slot)) {
        const int b = round < full_rounds ? (round * 8 + xcd) * cus + cu : lx0 + cu;
        const bool none = round >= full_rounds && b >= lx1;   // the last round may be partial
        ++round;
        if (none) continue;   // (the stream, if any, still follows)
        big_tile(b, s);
        s.kb = 0;
        s.ke = KT;
      } else {
        s.stream = static_cast<int>(static_cast<uint32_t>(u) / static_cast<uint32_t>(KT));
        s.kb = u - s.stream * KT;
        s.ke = min(KT, s.kb + (u_end - u));
        u += s.ke - s.kb;
        if (s.stream < stream_big) big_tile(lx0 + s.stream, s);
        else small_tile(sx0 + s.stream - stream_big, s);
      }
      s.valid = true;
      break;
    }
    return s;
  };

  // ---- loads -----------------------------------------------------------------------------------
  // Buffer loads: a scalar descriptor of the tile's panel (base = its first row), this lane's
  // 32-bit byte offset in a register and the k-tile offset as a scalar -- one address register
  // per lane and no 64-bit vector add per load.  (Offsets are 32-bit: a panel of 256 rows must
  // stay below 2 GiB, i.e. K < 4M.)  The descriptor ends with the last valid row of the panel: an offset beyond it
  // (there is none, rows are clamped) would read zeros instead of touching memory.  k-tiles past the end of the
  // segment are loaded through an empty descriptor: every lane is out of range and gets zeros.
  // (a gathered panel is the whole matrix: the rows the list names are rows of A, nothing to clamp)
  const unsigned char *ga = nullptr, *gb = nullptr;
  int rec_a = 0, rec_b = 0, load_kb = 0, load_ke = 0;
  int64_t bytes_b = 0;
  uint32_t off_a[8], off_b[8];       // by chunk (big tile: half * 4 + n)
  uint32_t past_a[2], past_b[2];     // RAGGED, by parity of the chunk: this lane's piece of the last k-tile is past the row's end
  auto load_a = [&](int n, int kt, unsigned char* dst) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(ga), 0, kt < load_ke ? rec_a : 0, 0x00020000);
    load_to_lds(rsrc, dst, RAGGED ? off_a[n] | (kt == KT - 1 ? past_a[n & 1] : 0u) : off_a[n], kt * (BK * 2));
  };
  auto load_b = [&](int n, int kt, unsigned char* dst) __attribute__((always_inline)) {
    if (B_BY_ROWS) {   // (the descriptor starts at the k-tile and ends with the expert's last k-row)
      const int64_t step = static_cast<int64_t>(BK) * Nout * 2, left = bytes_b - kt * step;
      const int rec = kt < load_ke ? static_cast<int>(left < 0x7fffffff ? left : 0x7fffffff) : 0;
      load_to_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(gb + kt * step), 0, rec, 0x00020000), dst,
                  off_b[n], 0);
      return;
    }
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(gb), 0, kt < load_ke ? rec_b : 0, 0x00020000);
    load_to_lds(rsrc, dst, RAGGED ? off_b[n] | (kt == KT - 1 ? past_b[n & 1] : 0u) : off_b[n], kt * (BK * 2));
  };
  auto load_big = [&](auto j_c, auto n_c, int i) __attribute__((always_inline)) {
    constexpr int j = decltype(j_c)::value, n = decltype(n_c)::value;
    unsigned char* dst = lds + (i & 1) * kKTile + j * kHalfTile + (wave * 4 + n) * 1024;
    if constexpr (j == 0 || j == 3) load_a((j == 3) * 4 + n, load_kb + i, dst);
    else load_b((j == 2) * 4 + n, load_kb + i, dst);
  };
  // Small tile: a wavefront fetches the 64 weight rows it multiplies, and a quarter of the token rows.
  auto load_small_weights = [&](int i, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < 8; ++n) load_b(n, load_kb + i, lds + stage * kSmallWeights + (wave * 8 + n) * 1024);
  };
  auto load_small_tokens = [&](auto kind_c, int i) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_c)::value;
#pragma unroll
    for (int n = 0; n < KIND; ++n)
      load_a(n, load_kb + i, lds + 3 * kSmallWeights + (i & 1) * kSmallTokens + (wave * KIND + n) * 1024);
  };

  // A small tile's weights by rows: a wavefront's 64 columns are 64 k-rows of 128 bytes, 32-byte block b of k-row k at block
  // b ^ (((k >> 1) & 1) + 2 ((k >> 3) & 1)): the eight k-rows that 32 lanes of a transposing read touch fall on different banks.
  auto small_by_rows = [](int wave, int lane, int n, uint32_t row_bytes) -> uint32_t {
    const int k = n * 8 + (lane >> 3);
    const int piece = (lane & 7) ^ ((((k >> 1) & 1) + 2 * ((k >> 3) & 1)) << 1);
    return k * row_bytes + (wave * 64 + piece * 8) * 2;
  };
  // Addresses of a segment, and the loads of its first two k-tiles.
  auto begin = [&](const Segment& s) __attribute__((always_inline)) {
    const int cols = min(BN, Nout - s.col0);
    ga = reinterpret_cast<const unsigned char*>(FUSE == 1 ? A : A + static_cast<size_t>(s.row0) * K);
    gb = reinterpret_cast<const unsigned char*>(
        B + (B_BY_ROWS ? static_cast<size_t>(s.expert) * Nout * K + s.col0 : (static_cast<size_t>(s.expert) * Nout + s.col0) * K));
    const int64_t bytes_a = FUSE == 1 ? 0x7fffffff : static_cast<int64_t>(s.rows) * K * 2;
    bytes_b = B_BY_ROWS ? (static_cast<int64_t>(K) * Nout - s.col0) * 2 : static_cast<int64_t>(cols) * K * 2;
    rec_a = static_cast<int>(bytes_a < 0x7fffffff ? bytes_a : 0x7fffffff);
    rec_b = static_cast<int>(bytes_b < 0x7fffffff ? bytes_b : 0x7fffffff);
    load_kb = s.kb;
    load_ke = s.ke;
    int lane_s = lane;   // (opaque: what is derived from the lane alone would otherwise stay live across the K loop)
    asm volatile("" : "+v"(lane_s));
    const int lrow = lane_s >> 3, slot = lane_s & 7;
    uint32_t row_a[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int big_row = (wave >> 1) * 128 + (wave & 1) * 32 + (n >> 2) * 64 + (n & 3) * 8;
      const int ra = (s.kind == 0 ? big_row : (wave * s.kind + (n & (s.kind - 1))) * 8) + lrow;
      const int rb = (s.kind == 0 ? big_row : (wave * 8 + n) * 8) + lrow;
      const int piece_a = slot ^ ((ra >> 1) & 7), piece_b = slot ^ ((rb >> 1) & 7);
      row_a[n] = min(ra, s.rows - 1);
      off_a[n] = piece_a * 16;
      if (!B_BY_ROWS) off_b[n] = static_cast<uint32_t>(min(rb, cols - 1)) * K * 2 + piece_b * 16;
      else if (s.kind == 0) off_b[n] = staged_by_rows(wave, lane_s, n >> 2, n & 3, Nout * 2u);
      else off_b[n] = small_by_rows(wave, lane_s, n, Nout * 2u);
      if (RAGGED && n < 2) {
        past_a[n] = (KT - 1) * BK + piece_a * 8 >= K ? 0x80000000u : 0u;
        past_b[n] = (KT - 1) * BK + piece_b * 8 >= K ? 0x80000000u : 0u;
      }
    }
    if (FUSE == 1) {
      const uint32_t list = lds_address(row_list) + s.list * (BM * 4);
      lds_read_words(row_a, list);
#pragma unroll
      for (int n = 0; n < 8; ++n) row_a[n] = aux_div == 1 ? row_a[n] : row_a[n] / static_cast<uint32_t>(aux_div);
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) off_a[n] += row_a[n] * K * 2;
    if (s.kind == 0) {
      each<16>([&](auto i) __attribute__((always_inline)) { load_big(IC<i.value / 4>{}, IC<i.value % 4>{}, 0); });
      each<16>([&](auto i) __attribute__((always_inline)) { load_big(IC<i.value / 4>{}, IC<i.value % 4>{}, 1); });
    } else {
      load_small_weights(0, 0);
      if (s.kind == 1) load_small_tokens(IC<1>{}, 0);
      else if (s.kind == 2) load_small_tokens(IC<2>{}, 0);
      else load_small_tokens(IC<4>{}, 0);
      load_small_weights(1, 1);
    }
  };
  // FUSE 1: the list of a segment's rows goes to LDS while the segment before it runs.
  auto fetch_list = [&](const Segment& s) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(aux_rows + s.row0), 0, s.rows * 4, 0x00020000);
    unsigned char* dst = reinterpret_cast<unsigned char*>(row_list) + s.list * (BM * 4) + wave * 256;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 4,
                                             min(tid, s.rows - 1) * 4, 0, 0, 0);
  };
  // FUSE 2: where the rows of a segment go, and their weights.
  auto place_rows = [&](const Segment& s) __attribute__((always_inline)) {
    const int r = s.row0 + min(tid, s.rows - 1);
    const int a = aux_rows[r];
    int dst = a;
    float w = aux_w[a];
    if (aux_div != 1) {
      const int t = a / aux_div;
      int kept = 0;
      for (int j = 0; j < aux_div; ++j) kept += aux_inv[t * aux_div + j] >= 0;
      dst = kept == 1 ? t : ~r;
      if (kept != 1) w = 1.f;
    }
    lds_write_word(lds_address(row_list) + (s.list * BM + tid) * 4, static_cast<uint32_t>(dst));
    lds_write_word(lds_address(row_weight) + (s.list * BM + tid) * 4, __float_as_uint(w));
  };

  uint32_t a_base[2], b_base[Fragments<B_BY_ROWS>::kBases];
  fragment_base(lds0, lane, wm, a_base);
  fragment_base(lds0, lane, wn, b_base);

  // The K loop of a small tile: a wavefront multiplies all the token rows (KIND x 2 blocks of 16) by its own 64
  // weight rows.  It is bound by the HBM stream of the weights, so two k-tiles of them are in flight and the rest is
  // left simple: the fragments of a k-tile are read and multiplied after one barrier (for the token rows; the weight
  // rows are the wavefront's own).
  auto small_loop = [&](auto kind_c, f32x4 (&acc)[8][4], int tiles, bool stores_behind) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_c)::value;
    typedef typename Elem16<DT>::vec8 vec8;
    u32x4 ft[2][2 * KIND], fw[2][4];
    u32x2 fwt[2][8];                      // (B_BY_ROWS: a fragment in two halves)
    uint32_t wb[B_BY_ROWS ? 4 : 2], tb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const uint32_t at = lds0 + fr * 128 + (((4 * ks + fq) ^ ((fr >> 1) & 7)) << 4);
      if (!B_BY_ROWS) wb[ks] = at + wave * 64 * 128;
      tb[ks] = at + 3 * kSmallWeights;
    }
    if (B_BY_ROWS) {
      const int j = (lane >> 2) & 3;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        wb[B_BY_ROWS ? b : 0] = lds0 + wave * 8192 + (fq * 8 + j) * 128 + ((b ^ ((j >> 1) + 2 * (fq & 1))) << 5) + (lane & 3) * 8;
    }
    const int behind = in_scalar(stores_behind ? 1 : 0);
    int stage = 0;
#pragma clang loop unroll(disable)
    for (int t = 0; t < tiles; ++t) {
      // the weights and tokens of k-tile t have landed (younger: the 8 weight loads of the next one)
      wait_loads<8, (8 + kStores < 63 ? 8 + kStores : 63)>(t, behind);
      __builtin_amdgcn_s_barrier();
      const uint32_t ws = stage * kSmallWeights, ts = (t & 1) * kSmallTokens;
      const uint32_t t0 = tb[0] + ts, t1 = tb[1] + ts;
      auto read_weights = [&](auto ks_c) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value;
        if constexpr (B_BY_ROWS)
          each<8>([&](auto i) __attribute__((always_inline)) {
            lds_read_transposed<KS * 4096 + (i.value & 1) * 512>(fwt[KS][i.value], wb[(i.value >> 1) & 3] + ws);
          });
        else
          each<4>([&](auto i) __attribute__((always_inline)) { lds_read16<i.value * 2048>(fw[KS][i.value], wb[KS] + ws); });
      };
      read_weights(IC<0>{});
      each<2 * KIND>([&](auto i) __attribute__((always_inline)) { lds_read16<i.value * 2048>(ft[0][i.value], t0); });
      read_weights(IC<1>{});
      each<2 * KIND>([&](auto i) __attribute__((always_inline)) { lds_read16<i.value * 2048>(ft[1][i.value], t1); });
      load_small_tokens(kind_c, t + 1);
      load_small_weights(t + 2, stage == 0 ? 2 : stage - 1);
      stage = stage == 2 ? 0 : stage + 1;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        // (the reads of the second k-step may still be under way: lgkmcnt counts to 15)
        constexpr int kYounger = (B_BY_ROWS ? 8 : 4) + 2 * KIND;
        if (ks == 0) asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(kYounger < 15 ? kYounger : 15) : "memory");
        else asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        if (B_BY_ROWS) {
          asm volatile("" : PPMOE_TIE8(fwt[ks]) : : "memory");
#pragma unroll
          for (int i = 0; i < 4; ++i) fw[ks][i] = __builtin_shufflevector(fwt[ks][2 * i], fwt[ks][2 * i + 1], 0, 1, 2, 3);
        } else {
          asm volatile("" : PPMOE_TIE4(fw[ks]) : : "memory");
        }
#pragma unroll
        for (int i = 0; i < 2 * KIND; ++i) asm volatile("" : "+v"(ft[ks][i]) : : "memory");
        each<8 * KIND>([&](auto x) __attribute__((always_inline)) {
          constexpr int mi = x.value / 4, ni = (mi & 1) ? 3 - x.value % 4 : x.value % 4;
          acc[mi][ni] = Elem16<DT>::mfma16(__builtin_bit_cast(vec8, fw[ks][ni]), __builtin_bit_cast(vec8, ft[ks][mi]), acc[mi][ni]);
        });
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  };

  Segment nxt = next_segment(), pending = {};
  if (FUSE == 1 && nxt.valid) {
    fetch_list(nxt);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
  }
  // A segment that does not hold the first k-tile of its output tile hands its partial sums to the
  // CU that does (through this block's scratch slot) and raises its flag: mode 1.  The one that
  // holds it writes the output tile (mode 0), after adding the partial sums of the CUs after it, if
  // the rest of the k range went there (their first segment, which they finished long ago).  If
  // those do not arrive it takes nobody's: it parks its own partial sums in its own slot (mode 2,
  // no flag) and runs the other CUs' shares of the tile as segments of its own, one after another, each of
  // which ends by adding the parked sums: the same sums in the same order, so the result has the same bits.
  bool stores_behind = false;   // exactly kStores stores per wavefront were issued after the loads of a segment's first two k-tiles
  bool begun = false;           // the loads of the next segment's first two k-tiles are under way
  while (nxt.valid) {
    // ---- a segment's products --------------------------------------------------------------------
    const Segment cur = nxt;
    if (!begun) begin(cur);
    if (pending.valid) {
      nxt = pending;
      pending.valid = false;
    } else {
      nxt = next_segment();
      nxt.list = cur.list ^ 1;
      if (FUSE == 1 && nxt.valid) fetch_list(nxt);
    }
    if (FUSE == 2) place_rows(cur);
    const int tiles = cur.ke - cur.kb;
    // What follows a segment's K loop: who writes the tile, the next segment's loads, the epilogue.  (One copy for big
    // tiles and one for small ones: accumulators that both kinds of K loop feed cost the compiler copies inside the loops.)
    auto finish_segment = [&](auto& acc, auto ni_c) __attribute__((always_inline)) {
    constexpr int NI = decltype(ni_c)::value;   // 16-column blocks of a wavefront
    __builtin_amdgcn_s_barrier();   // every wavefront is done with the ring

    int mode = (cur.kb > 0 && !cur.resumed) ? 1 : 0;
    int n_contrib = 0;
    // The next CU's share of the tile is computed here as well: its k range follows cur's.
    auto resume = [&]() {
      mode = 2;
      pending = nxt;
      nxt = cur;
      nxt.kb = cur.ke;
      const int first = cur.stream * KT;   // of the tile in the stream
      int c2 = share + 1;
      while (share_begin(c2) <= first + cur.ke) ++c2;   // (the shares end with the stream, behind the tile)
      nxt.ke = min(KT, share_begin(c2) - first);
      nxt.resumed = true;
    };
    if (cur.resumed) {
      if (tid == 0) {
        contrib[0] = 1;
        contrib[1] = kMaxPersistentBlocks + blockIdx.x;   // its parking slot
      }
      __syncthreads();
      n_contrib = 1;   // (this CU's own stores, complete since the barrier that followed them)
      if (cur.ke < KT) resume();
    } else if (mode == 0 && cur.ke < KT) {
      if (tid == 0) {
        // One thread lists the CUs of the shares after this one that begin inside this tile (skipping empty
        // shares) and polls their flags (relaxed loads that go to L2, no cache maintenance in the loop).
        int n = 0, failed = 0;
        for (int c2 = share + 1; c2 < cus && share_begin(c2) < (cur.stream + 1) * KT; ++c2) {
          if (share_begin(c2 + 1) == share_begin(c2)) continue;
          const int b2 = ((cus - 1 - c2) << 3) | xcd;
          contrib[++n] = b2;
          int spins = 0;
          uint32_t f = 0;
          bool up = false;
          while (spins < spin_limit) {
            f = __hip_atomic_load(flags + b2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((f >> 4) == epoch) {
              up = true;
              break;
            }
            ++spins;
            __builtin_amdgcn_s_sleep(16);
          }
          if (!up) {   // not delivered in time (the writer's block may not even be resident yet)
            failed = 1;
            flags[kMaxPersistentBlocks] = kGemmErrorMagic | 1u;
            break;
          }
          if (same_l2 && (f & 15u) != my_xcc) {
            // The partial sums sit in another XCD's L2 and their writer released them at workgroup
            // scope only (the set-up check of the placement was wrong): they cannot be read safely.
            failed = 1;
            flags[kMaxPersistentBlocks] = kGemmErrorMagic | 2u;
            break;
          }
        }
        contrib[0] = n;
        contrib_failed = failed;
      }
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(contrib_failed)) {
        resume();
      } else {
        // Once per thread, after the flags are up.  Within an XCD the partial sums are in the shared L2
        // (stores write through the L1, and this CU has never read these lines since its L1 was
        // invalidated at the start of the kernel), so ordering against the barrier is all it takes;
        // the device-scope acquire invalidates the L2, which then misses on every panel being streamed.
        if (same_l2)
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        else
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        n_contrib = __builtin_amdgcn_readfirstlane(contrib[0]);
      }
    }

    // The ring is free: the next segment's first two k-tiles are under way during the epilogue -- unless somebody waits
    // for its stores, or it starts with loads of its own (partial sums).
    begun = nxt.valid && mode == 0 && n_contrib == 0;
    if (begun) begin(nxt);

    // ---- epilogue of the current segment ---------------------------------------------------------
    stores_behind = false;
    {
      // Per-segment opaque copies: they stop the compiler from hoisting the address arithmetic of the
      // code below out of the segment loop, where it would cost live registers.
      int tid_l = tid;
      asm volatile("" : "+v"(tid_l));
      const int lane_l = tid_l & 63, fr_l = tid_l & 15, fq_l = lane_l >> 4;
      // Where this wavefront's accumulator blocks sit in the tile (see tile_kind).
      const int row_base = NI == 8 ? wm * 128 : 0, col_base = NI == 8 ? wn * 128 : wave * 64;
      const int cols = min(BN, Nout - cur.col0);
      const int ncol = min(cols - col_base, NI * 16);   // valid columns of this wavefront's part (may be <= 0)
      const int nrow = cur.rows - row_base;               // valid rows of it (may be <= 0)
      const bool full = NI == 8 && cur.rows == BM && cols == BN;
      const int my_slot_id = __builtin_amdgcn_readfirstlane((mode == 2 ? kMaxPersistentBlocks : 0) + static_cast<int>(blockIdx.x));
      f32x4* my_slot = reinterpret_cast<f32x4*>(slots + static_cast<size_t>(my_slot_id) * kSlotFloats) + tid_l;
      // The accumulators leave 16 rows at a time (all 128, or 64, columns of the wavefront) through 4 KiB of LDS of
      // the wavefront's own: rows of 256 bytes, 16-byte chunk c of row r at chunk c ^ r, written 8 bytes per lane,
      // read back 16 (a store instruction covers 4 rows x 256 contiguous bytes).  LDS operations of a wavefront complete in
      // order: nothing is waited for between the writes and the reads; the stores of a block go out after the arithmetic
      // of the next one.
      const uint32_t epi = lds0 + kRing + wave * kOutBytes;
      const uint32_t wr = epi + fr_l * 256 + (fq_l & 1) * 8;
      const int ec = lane_l & 15, er = fq_l;              // (read back: row i * 4 + er, chunk ec)
      const uint32_t list = lds_address(row_list) + cur.list * (BM * 4), weight = lds_address(row_weight) + cur.list * (BM * 4);
      u32x4 back[4];
      // stores block mi (rows mi * 16 ..) of this wavefront's part from `back`, as rows of C or (pre) of the pre-activations
      auto store_rows = [&](int mi, auto full_c, bool pre) __attribute__((always_inline)) {
        int dst[4];
        if (FUSE == 2) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            asm volatile("ds_read_b32 %0, %1" : "=v"(dst[i]) : "v"(list + (row_base + mi * 16 + i * 4 + er) * 4) : "memory");
          asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(dst[0]), "+v"(dst[1]), "+v"(dst[2]), "+v"(dst[3]) : : "memory");
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : PPMOE_TIE4(back) : : "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = mi * 16 + i * 4 + er;
          bf16_t* base = (FUSE == 2 && dst[i] < 0) || (ACT == 2 && pre) ? C2 : C;
          const int row = FUSE == 2 ? (dst[i] >= 0 ? dst[i] : ~dst[i]) : cur.row0 + row_base + r;
          bf16_t* at = base + static_cast<size_t>(row) * Nout + cur.col0 + col_base + ec * 8;
          if (decltype(full_c)::value || (r < nrow && ec * 8 < ncol)) *reinterpret_cast<u32x4*>(at) = back[i];
        }
      };
      auto as_is = [&](f32x4 y) __attribute__((always_inline)) -> uint64_t {
        return static_cast<uint64_t>(Elem16<DT>::pack2(y[0], y[1])) |
               (static_cast<uint64_t>(Elem16<DT>::pack2(y[2], y[3])) << 32);
      };
      // GeLU of pre-activations as they are stored (ACT 2)
      auto gelu_of_stored = [&](uint64_t pre) __attribute__((always_inline)) -> uint64_t {
        float a[4];
        Elem16<DT>::widen2(static_cast<uint32_t>(pre), a[0], a[1]);
        Elem16<DT>::widen2(static_cast<uint32_t>(pre >> 32), a[2], a[3]);
        f32x4 y;
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = a[i] * gelu_sigmoid(a[i]);
        return as_is(y);
      };
      // the final values of 16 x 16 block (mi, ni) as 16-bit elements
      auto finish = [&](f32x4 y, float w) __attribute__((always_inline)) -> uint64_t {
        if (ACT == 1) y = gelu_tanh4(y);
        if (FUSE == 2) y *= w;
        return as_is(y);
      };
      auto weight_of = [&](int mi) __attribute__((always_inline)) -> float {
        return FUSE == 2 ? __int_as_float(lds_read_word(weight + (row_base + mi * 16 + fr_l) * 4)) : 1.f;
      };
      auto write_block = [&](int ni, uint64_t v) __attribute__((always_inline)) {
        const uint32_t a = wr + (((ni * 2 + (fq_l >> 1)) ^ fr_l) << 4);
        asm volatile("ds_write_b64 %0, %1" : : "v"(a), "v"(v) : "memory");
      };
      auto read_back = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = i * 4 + er;
          asm volatile("ds_read_b128 %0, %1" : "=v"(back[i]) : "v"(epi + r * 256 + ((ec ^ r) << 4)) : "memory");
        }
      };
      // v[ni] += the partial sums of block row mi, CN contributors at a time
      auto add_partials = [&](int mi, f32x4 (&v)[NI]) __attribute__((always_inline)) {
        constexpr int CN = NI == 8 ? 3 : 7;
        for (int c0 = 0; c0 < n_contrib; c0 += CN) {
          f32x4 p[CN][NI];
#pragma unroll
          for (int j = 0; j < CN; ++j) {
            const int b2 = __builtin_amdgcn_readfirstlane(contrib[1 + min(c0 + j, n_contrib - 1)]);
            const f32x4* slot = reinterpret_cast<const f32x4*>(slots + static_cast<size_t>(b2) * kSlotFloats) + tid_l;
            if (c0 + j < n_contrib) {
#pragma unroll
              for (int ni = 0; ni < NI; ++ni) p[j][ni] = slot[(mi * 8 + ni) * kThreads];
            } else {
#pragma unroll
              for (int ni = 0; ni < NI; ++ni) p[j][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
          }
#pragma unroll
          for (int j = 0; j < CN; ++j)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) v[ni] += p[j][ni];
        }
      };
      const bool plain = full && mode == 0 && n_contrib == 0;
      if (plain) {
        if constexpr (NI == 8) {
        // (no branches: they cost a wavefront that is alone on its SIMD more than the work they would skip)
        each<8>([&](auto mi_c) __attribute__((always_inline)) {
          constexpr int mi = decltype(mi_c)::value;
          uint64_t packed[8], before[8];   // (before: ACT 2)
          const float w = weight_of(mi);
          each<8>([&](auto ni_c) __attribute__((always_inline)) {
            constexpr int ni = decltype(ni_c)::value;
            f32x4 v;
            v[0] = read_acc(acc[mi][ni][0]);
            v[1] = read_acc(acc[mi][ni][1]);
            v[2] = read_acc(acc[mi][ni][2]);
            v[3] = read_acc(acc[mi][ni][3]);
            if (ACT == 2) {
              before[ni] = as_is(v);
              packed[ni] = gelu_of_stored(before[ni]);
            } else {
              packed[ni] = finish(v, w);
            }
          });
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (mi > 0) store_rows(mi - 1, std::true_type{}, false);
          if constexpr (ACT == 2) {
            each<8>([&](auto ni_c) __attribute__((always_inline)) { write_block(ni_c.value, before[ni_c.value]); });
            read_back();
            store_rows(mi, std::true_type{}, true);
          }
          each<8>([&](auto ni_c) __attribute__((always_inline)) { write_block(ni_c.value, packed[ni_c.value]); });
          read_back();
          __builtin_amdgcn_sched_barrier(0);
        });
        store_rows(7, std::true_type{}, false);
        }
      } else {
        // A loop, the accumulators of a block picked by a switch.  Unrolled, this path and its copy for small tiles are 45 KB of 124 that a
        // short launch runs through once, as fast as instructions come from the L2: layer on one expert, 136 tokens of 1024 x 512
        // 69.6 -> 67.7 us, 189 of 256 x 128 50.5 -> 48.4, 700 and more unchanged or up to 4 % faster.
        // (Blocks of 16 rows with no valid row are neither sent nor fetched.)
        const int blocks = in_scalar(nrow <= 0 ? 0 : min(8, (nrow + 15) >> 4));
#pragma clang loop unroll(disable)
        for (int mi = 0; mi < blocks; ++mi) {
          f32x4 v[NI];
          auto fetch = [&](auto mi_c) __attribute__((always_inline)) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
              for (int e = 0; e < 4; ++e) v[ni][e] = read_acc(acc[decltype(mi_c)::value][ni][e]);
          };
          switch (mi) {
            case 0: fetch(IC<0>{}); break;
            case 1: fetch(IC<1>{}); break;
            case 2: fetch(IC<2>{}); break;
            case 3: fetch(IC<3>{}); break;
            case 4: fetch(IC<4>{}); break;
            case 5: fetch(IC<5>{}); break;
            case 6: fetch(IC<6>{}); break;
            default: fetch(IC<7>{}); break;
          }
          // Partial sums are added in CU order (fixed summation order); the loads of several CUs' slots go out
          // together, so that the wait is one memory latency for them all.
          if (n_contrib > 0) add_partials(mi, v);
          if (mode == 0) {
            uint64_t packed[NI], before[NI];
            const float w = weight_of(mi);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
              if (ACT == 2) {
                before[ni] = as_is(v[ni]);
                packed[ni] = gelu_of_stored(before[ni]);
              } else {
                packed[ni] = finish(v[ni], w);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (mi > 0) store_rows(mi - 1, std::false_type{}, false);
            if (ACT == 2) {
#pragma unroll
              for (int ni = 0; ni < NI; ++ni) write_block(ni, before[ni]);
              read_back();
              store_rows(mi, std::false_type{}, true);
            }
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) write_block(ni, packed[ni]);
            read_back();
          } else {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) my_slot[(mi * 8 + ni) * kThreads] = v[ni];
          }
          __builtin_amdgcn_sched_barrier(0);   // one block at a time keeps the register footprint small
        }
        if (mode == 0 && blocks > 0) store_rows(blocks - 1, std::false_type{}, false);
      }
      if (mode == 0) {
        stores_behind = plain;
        if (n_contrib > 0 && !cur.resumed) {
          // every thread has read the partial sums: lower the flags (the scratch may be reused by a
          // replay of the same launch, whose flags carry the same value)
          __syncthreads();
          if (tid == 0)
            for (int i = 1; i <= n_contrib; ++i)
              __hip_atomic_store(flags + contrib[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else if (mode == 2) {
        // Parked: a thread reads back what it stored itself, once vmcnt is 0; the block meets, then goes on with
        // the same tile.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      } else {
        // Release: every thread makes its own stores visible device-wide, then the block meets, then
        // one thread raises the flag (a relaxed store is enough after the fences).
        // (Within an XCD: the stores have reached the shared L2 once vmcnt is 0.  The device-scope
        // release would write back every dirty line of the L2 -- the output tiles -- once per hand-over.)
        if (same_l2) {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        } else {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        }
        __syncthreads();
        if (tid == 0) {
          uint32_t up = (epoch << 4) | my_xcc;
          asm volatile("" : "+s"(up));   // (formed here: hoisted out of the segment loop it would cost a vector register)
          __hip_atomic_store(flags + blockIdx.x, up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    };
    if (cur.kind == 0) {
      f32x4 acc[8][8];
#pragma unroll
      for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int ni = 0; ni < 8; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
      k_loop<DT, false, B_BY_ROWS, kStores>(acc, a_base, b_base, tiles, stores_behind, load_big);
      finish_segment(acc, IC<8>{});
    } else {
      f32x4 acc[8][4];
#pragma unroll
      for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (cur.kind == 1) small_loop(IC<1>{}, acc, tiles, stores_behind);
      else if (cur.kind == 2) small_loop(IC<2>{}, acc, tiles, stores_behind);
      else small_loop(IC<4>{}, acc, tiles, stores_behind);
      finish_segment(acc, IC<4>{});
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    unsigned long long* cw = reinterpret_cast<unsigned long long*>(flags + kClockWord);
    cw[2] = clock64();
    cw[3] = wall_clock64();
  }
}

}  // namespace fast

hipError_t read_gemm_error_word(const void* workspace, uint32_t* word, hipStream_t s) {
  const float* slots = static_cast<const float*>(workspace);
  const uint32_t* flags = reinterpret_cast<const uint32_t*>(
      slots + static_cast<size_t>(fast::kSlotsPerBlock) * kMaxPersistentBlocks * fast::kSlotFloats);
  hipError_t e = hipMemcpyAsync(word, flags + kMaxPersistentBlocks, sizeof(uint32_t),
                                hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  if ((*word & 0xffffff00u) == kGemmErrorMagic) {   // reported once: lower it again
    static const uint32_t zero = 0;
    e = hipMemcpyAsync(const_cast<uint32_t*>(flags) + kMaxPersistentBlocks, &zero, sizeof(uint32_t),
                       hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
  }
  return e;
}

unsigned long long* gemm_clock_words(void* workspace) {
  uint32_t* flags = reinterpret_cast<uint32_t*>(
      static_cast<float*>(workspace) +
      static_cast<size_t>(fast::kSlotsPerBlock) * kMaxPersistentBlocks * fast::kSlotFloats);
  return reinterpret_cast<unsigned long long*>(flags + fast::kClockWord);
}

// Shader-clock and wall-clock ticks a block of the last fast-path launch on this workspace counted
// between its start and its end.  Synchronises the stream.
hipError_t read_gemm_clock_words(const void* workspace, uint64_t* shader_ticks, uint64_t* wall_ticks,
                                 hipStream_t s) {
  const float* slots = static_cast<const float*>(workspace);
  const uint32_t* flags = reinterpret_cast<const uint32_t*>(
      slots + static_cast<size_t>(fast::kSlotsPerBlock) * kMaxPersistentBlocks * fast::kSlotFloats);
  uint64_t w[4] = {0, 0, 0, 0};
  hipError_t e = hipMemcpyAsync(w, flags + fast::kClockWord, sizeof(w), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  *shader_ticks = w[2] - w[0];
  *wall_ticks = w[3] - w[1];
  return hipSuccess;
}

size_t grouped_gemm_fast_workspace_bytes() {
  // slots, flags (+1 word: the error word), and inside the padding the four clock words
  return static_cast<size_t>(fast::kSlotsPerBlock) * kMaxPersistentBlocks * fast::kSlotFloats * sizeof(float) +
         (2 * kMaxPersistentBlocks + 1) * sizeof(uint32_t) + 256;
}

// ---- per-device set-up --------------------------------------------------------------------------
// Once per device: the dynamic-LDS attribute of the kernels, the number of persistent blocks, and the
// placement check (do blocks b and b + 8 share an XCD, as the workgroup-scope hand-over assumes?).
// The check launches a probe and waits for it, so it is the one thing here that synchronises; it
// runs from moe_init, or from the first launch on a device that finds it not done -- unless that
// launch is being captured into a graph, in which case the launch uses device-scope fences and
// leaves the check for later.
namespace {

constexpr int kMaxDevices = 64;
struct FastSetup {
  bool attrs = false;   // kernel attributes set, `blocks` valid
  bool probed = false;  // same_l2 valid
  int blocks = 0;
  int same_l2 = 0;
};
FastSetup g_setup[kMaxDevices];
std::mutex g_setup_mutex;
std::atomic<int> g_force_device_scope{0};
std::atomic<int> g_spin_limit{fast::kDefaultSpinLimit};

hipError_t setup_attrs(FastSetup& st, int dev) {
  using namespace fast;
  if (st.attrs) return hipSuccess;
#define PPMOE_KERNELS(DT, R)                                                               \
  reinterpret_cast<const void*>(grouped_gemm_fast_kernel<1, 0, DT, R, false>),          \
      reinterpret_cast<const void*>(grouped_gemm_fast_kernel<0, 0, DT, R, false>),     \
      reinterpret_cast<const void*>(grouped_gemm_fast_kernel<1, 1, DT, R, false>),      \
      reinterpret_cast<const void*>(grouped_gemm_fast_kernel<0, 2, DT, R, false>)
  const void* kernels[] = {PPMOE_KERNELS(MOE_BF16, false), PPMOE_KERNELS(MOE_BF16, true),
                           PPMOE_KERNELS(MOE_F16, false), PPMOE_KERNELS(MOE_F16, true),
                           reinterpret_cast<const void*>(grouped_gemm_fast_kernel<2, 0, MOE_BF16, false, false>),
                           reinterpret_cast<const void*>(grouped_gemm_fast_kernel<2, 0, MOE_F16, false, false>),
                           reinterpret_cast<const void*>(grouped_gemm_fast_kernel<0, 0, MOE_BF16, false, true>),
                           reinterpret_cast<const void*>(grouped_gemm_fast_kernel<0, 0, MOE_F16, false, true>)};
#undef PPMOE_KERNELS
  for (const void* k : kernels) {
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
  }
  int cus = 0;
  hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (cus > kMaxPersistentBlocks) cus = kMaxPersistentBlocks;
  st.blocks = cus & ~7;   // one block per CU, the same number on each of the 8 XCDs
  if (st.blocks < 8) return hipErrorInvalidConfiguration;
  st.attrs = true;
  return hipSuccess;
}

// Launches the placement probe on `s` and waits for it.  Must not be called while `s` is capturing.
hipError_t setup_probe(FastSetup& st, hipStream_t s) {
  if (st.probed) return hipSuccess;
  uint32_t host[kMaxPersistentBlocks];
  fast::xcc_probe_kernel<<<st.blocks, fast::kThreads, 0, s>>>();
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipMemcpyFromSymbolAsync(host, HIP_SYMBOL(fast::g_xcc_of_block), st.blocks * sizeof(uint32_t), 0,
                               hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  st.same_l2 = 1;
  for (int b = 8; b < st.blocks; ++b)
    if (host[b] != host[b & 7]) st.same_l2 = 0;
  st.probed = true;
  return hipSuccess;
}

}  // namespace

// The set-up as a launch on `s` finds it or, outside a capture, makes it.
static hipError_t set_up_for_launch(hipStream_t s, int* blocks, int* same_l2) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_setup_mutex);
  FastSetup& st = g_setup[dev];
  e = setup_attrs(st, dev);
  if (e != hipSuccess) return e;
  if (!st.probed) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(s, &cap);
    if (e != hipSuccess) return e;
    if (cap == hipStreamCaptureStatusNone) {
      e = setup_probe(st, s);
      if (e != hipSuccess) return e;
    }
  }
  *blocks = st.blocks;
  *same_l2 = st.probed ? st.same_l2 : 0;   // unknown placement: device-scope fences are always right
  return hipSuccess;
}

hipError_t grouped_gemm_set_up(hipStream_t s) {
  int blocks = 0, same_l2 = 0;
  return set_up_for_launch(s, &blocks, &same_l2);
}

hipError_t grouped_gemm_fast_init(hipStream_t s) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_setup_mutex);
  e = setup_attrs(g_setup[dev], dev);
  if (e != hipSuccess) return e;
  return setup_probe(g_setup[dev], s);
}

void grouped_gemm_fast_set_handover(int force_device_scope, int spin_limit) {
  if (force_device_scope >= 0) g_force_device_scope = force_device_scope ? 1 : 0;
  if (spin_limit >= 0) g_spin_limit = spin_limit;
}

hipError_t launch_grouped_gemm_fast(int in_dtype, bool gelu, const bf16_t* A, const bf16_t* B, bf16_t* C,
                                    const int32_t* offsets, int n_exp, int few_most, int Nout,
                                    int K, void* workspace, hipStream_t s, int fuse,
                                    const int32_t* aux_rows, const float* aux_w, int aux_div,
                                    const int32_t* aux_inv, bf16_t* C2, bool b_by_rows, int pick_cus) {
  using namespace fast;
  int blocks = 0, same_l2 = 0;
  hipError_t e = set_up_for_launch(s, &blocks, &same_l2);
  if (e != hipSuccess) return e;
  if (g_force_device_scope.load()) same_l2 = 0;
  const int spin_limit = g_spin_limit.load();
  static std::atomic<uint32_t> launches{0};
  // 28 bits (the flag word also carries the XCD id), spread over the word so that small integers
  // left in a recycled workspace do not look like an epoch; 0 means "flag down".
  uint32_t epoch = (++launches * 0x9E3779B1u) >> 4;
  if (epoch == 0) epoch = (++launches * 0x9E3779B1u) >> 4;
  float* slots = static_cast<float*>(workspace);
  uint32_t* flags = reinterpret_cast<uint32_t*>(
      slots + static_cast<size_t>(kSlotsPerBlock) * kMaxPersistentBlocks * kSlotFloats);
  const bool ragged = K % BK != 0;
  // fuse: 0 none; 1 rows of A through aux_rows (first GEMM only); 2 rows of the result placed through
  // aux_rows (second GEMM only; with aux_div > 1 it needs the inverse permutation and a place for
  // the rows it cannot place)
  if ((fuse == 1 && !gelu) || (fuse == 2 && gelu) || fuse < 0 || fuse > 2 ||
      (fuse != 0 && aux_rows == nullptr) || (fuse == 2 && aux_w == nullptr) || aux_div < 1 ||
      (fuse == 2 && aux_div != 1 && (aux_inv == nullptr || C2 == nullptr)))
    return hipErrorInvalidValue;
#define PPMOE_LAUNCH_KERNEL(...)                                                      \
  __VA_ARGS__<<<blocks, kThreads, kLdsBytes, s>>>(     \
      A, B, C, offsets, n_exp, few_most, Nout, K, slots, flags, epoch, same_l2, spin_limit, aux_rows, aux_w, aux_div, \
      aux_inv, C2, pick_cus)
#define PPMOE_LAUNCH_DT(G, F, DT, R) PPMOE_LAUNCH_KERNEL(grouped_gemm_fast_kernel<G, F, DT, R, false>)
#define PPMOE_LAUNCH(G, F)                            \
  do {                                                \
    if (in_dtype == MOE_F16 && ragged) PPMOE_LAUNCH_DT(G, F, MOE_F16, true); \
    else if (in_dtype == MOE_F16) PPMOE_LAUNCH_DT(G, F, MOE_F16, false);     \
    else if (ragged) PPMOE_LAUNCH_DT(G, F, MOE_BF16, true);                  \
    else PPMOE_LAUNCH_DT(G, F, MOE_BF16, false);                             \
  } while (0)
  if (b_by_rows) {
    if (gelu || fuse != 0 || ragged) return hipErrorInvalidValue;
    if (in_dtype == MOE_F16) PPMOE_LAUNCH_KERNEL(grouped_gemm_fast_kernel<0, 0, MOE_F16, false, true>);
    else PPMOE_LAUNCH_KERNEL(grouped_gemm_fast_kernel<0, 0, MOE_BF16, false, true>);
  } else if (fuse == 1) PPMOE_LAUNCH(1, 1);
  else if (fuse == 2) PPMOE_LAUNCH(0, 2);
  else if (gelu && C2 != nullptr) {   // (the pre-activations as well)
    if (ragged) return hipErrorInvalidValue;
    if (in_dtype == MOE_F16) PPMOE_LAUNCH_KERNEL(grouped_gemm_fast_kernel<2, 0, MOE_F16, false, false>);
    else PPMOE_LAUNCH_KERNEL(grouped_gemm_fast_kernel<2, 0, MOE_BF16, false, false>);
  } else if (gelu) PPMOE_LAUNCH(1, 0);
  else PPMOE_LAUNCH(0, 0);
#undef PPMOE_LAUNCH_DT
#undef PPMOE_LAUNCH_KERNEL
#undef PPMOE_LAUNCH
  return hipGetLastError();
}

}  // namespace ppmoe
