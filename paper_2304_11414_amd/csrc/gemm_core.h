// The K loop of the large-tile GEMMs (16-bit operands, float32 accumulators): block tile 256 x 256 x 64, four
// wavefronts (one per SIMD), each owning a 128 x 128 sub-tile as 8 x 8 MFMA 16x16x32 accumulators (256 accumulator
// registers).
//
// What bounds it is power: with random operands the chip lowers its clock to 1.6 to 2.1 GHz, so what counts is the
// energy per k-tile as much as its cycles.  Hence
//   * the 16x16x32 instruction, not 32x32x16: half the accumulator traffic per flop.  Register-resident loops with
//     random operands: 2.11 PFLOP/s at 2.07 GHz against 1.84 at 1.77 GHz (both 2.45 with constant operands);
//   * the operand that changes from one MFMA to the next is the first one: with the second changing the instruction
//     takes 22 cycles instead of 16 (2862 cycles per k-tile instead of 2096, no memory traffic);
//   * operand tiles go from memory to LDS without passing through registers (buffer loads with an LDS
//     destination): no staging registers, no LDS write instructions.
// 8192 x 8192 x 8192: 1.37 PFLOP/s with 32x32x16 and register staging, 1.41 with LDS loads, 1.47 to 1.55 with both (by card);
// 2340 cycles per k-tile (2048 are MFMAs, 107 go to the 32 fragment reads of a wavefront, 139 to its 16 loads) at 1.8 GHz.
//
// A k-tile of the block is four half-tiles of 16 KiB: A0, B0, B1, A1 (j = 0..3), half h of an operand holding the
// tile rows w * 128 + h * 64 + (0..63), w = 0, 1: the 64 rows that each of the two wavefronts along that operand
// multiplies in one phase.  Four phases per k-tile, 32 MFMAs each: (A0, B0), (A0, B1), (A1, B1), (A1, B0); phase p
// reads the fragments phase p + 1 needs from LDS (a register set holds one half-tile's share of a wavefront for the
// whole k-tile; B0's is overwritten in the last phase, k-step by k-step as it is used up).  LDS holds two k-tiles;
// a half-tile's slot is refilled with the k-tile after the next one as soon as its fragments are read: loads are
// in flight for one and a half k-tiles (3500 cycles), up to 96 KiB per CU.  Two barriers per k-tile.
//
// LDS: rows of 128 bytes (64 k-values), 16-byte piece p of row r at slot p ^ ((r >> 1) & 7): the 16 lanes that a
// ds_read_b128 serves per cycle (16 consecutive rows, one piece) touch 16 different slots.  A load instruction fills
// 1 KiB of LDS in lane order (8 rows), so the swizzle is in the lanes' memory offsets: still whole 128-byte lines.
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"

namespace ppmoe {
namespace core {

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int kThreads = 256;
constexpr int kHalfTile = 128 * BK * 2;          // 16 KiB
constexpr int kKTile = 4 * kHalfTile;            // 64 KiB
constexpr int kRing = 2 * kKTile;                // 128 KiB

template <int N>
using IC = std::integral_constant<int, N>;
template <typename F, int... I>
__device__ __forceinline__ void each_of(F f, std::integer_sequence<int, I...>) {
  (f(IC<I>{}), ...);
}
// f(IC<0>{}), f(IC<1>{}), ..., f(IC<N - 1>{})
template <int N, typename F>
__device__ __forceinline__ void each(F f) {
  each_of(f, std::make_integer_sequence<int, N>{});
}

// Reads one accumulator element where it lives (an accumulator register), at this point of the
// program: without it the compiler copies all 256 accumulators to vector registers right after the
// K loop and spills half of them.
__device__ __forceinline__ float read_acc(float a) {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

template <int OFF, typename V>
__device__ __forceinline__ void lds_read16(V& dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
__device__ __forceinline__ void lds_write16(uint32_t addr, const f32x4& v) {
  asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
// One 32-bit word, waited for (inline assembly: the compiler would first wait for every load into LDS that is in flight).
__device__ __forceinline__ int lds_read_word(uint32_t addr) {
  int v;
  asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
__device__ __forceinline__ u32x4 lds_read_quad(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
  return v;
}
__device__ __forceinline__ void lds_write_word(uint32_t addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) unsigned char*)p));
}

// v[n] = the word at base + 4 * v[n], n = 0..7, waited for.
__device__ __forceinline__ void lds_read_words(uint32_t (&v)[8], uint32_t base) {
#pragma unroll
  for (int n = 0; n < 8; ++n) v[n] = base + 4 * v[n];
  asm volatile(
      "ds_read_b32 %0, %0\n\tds_read_b32 %1, %1\n\tds_read_b32 %2, %2\n\tds_read_b32 %3, %3\n\t"
      "ds_read_b32 %4, %4\n\tds_read_b32 %5, %5\n\tds_read_b32 %6, %6\n\tds_read_b32 %7, %7\n\ts_waitcnt lgkmcnt(0)"
      : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])
      :
      : "memory");
}

#define PPMOE_TIE4(f) "+v"((f)[0]), "+v"((f)[1]), "+v"((f)[2]), "+v"((f)[3])
#define PPMOE_TIE8(f) \
  "+v"((f)[0]), "+v"((f)[1]), "+v"((f)[2]), "+v"((f)[3]), "+v"((f)[4]), "+v"((f)[5]), "+v"((f)[6]), "+v"((f)[7])

__device__ __forceinline__ void tie(u32x4 (&v)[4]) { asm volatile("" : PPMOE_TIE4(v) : : "memory"); }

// 16 bytes per lane from memory (descriptor, byte offset of the lane, scalar offset) to LDS at `dst` + 16 * lane.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t rsrc, unsigned char* dst, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, soff, 0, 0);
}

// An operand whose contraction index is its column (k contiguous in memory): the row of the 256-row tile that this
// lane fetches for chunk n (0..3) of half h, and its 16-byte piece in that row's 128 bytes (the swizzle's inverse).
__device__ __forceinline__ int staged_row(int wave, int lane, int h, int n) {
  return (wave >> 1) * 128 + h * 64 + (wave & 1) * 32 + n * 8 + (lane >> 3);
}
__device__ __forceinline__ int staged_piece(int lane, int n) { return (lane & 7) ^ (((n & 1) * 4 + (lane >> 4)) & 7); }

// An operand whose contraction index is its row: a half-tile is 64 k-rows of 256 bytes, the 128 columns
// w * 128 + h * 64 + (0..63), w = 0, 1, side by side.  Its fragments are read with the transposing LDS read: of a group
// of 16 lanes, lanes 4 j .. 4 j + 3 name the 32 bytes (16 columns) of k-row j, and lane i receives column i at the four k's.
// 32-byte block b of k-row k sits at block b ^ ((k & 3) + 4 ((k >> 3) & 1)): the eight k-rows that 32 lanes
// read at a time then touch all banks once.  This lane's byte offset from the tile's first column at the k-tile's first row.
__device__ __forceinline__ uint32_t staged_by_rows(int wave, int lane, int h, int n, uint32_t row_bytes) {
  const int k = wave * 16 + n * 4 + (lane >> 4);
  const int piece = (lane & 15) ^ (((k & 3) + 4 * ((k >> 3) & 1)) << 1);
  return k * row_bytes + ((piece >> 3) * 128 + h * 64 + (piece & 7) * 8) * 2;
}

template <int OFF>
__device__ __forceinline__ void lds_read_transposed(u32x2& dst, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}

// A wavefront's fragments of one half-tile: eight (k-step * 4 + 16-row block) of 8 k-values per lane, read with kReads
// LDS instructions.  BY_ROWS: the operand's contraction index is its row.
template <bool BY_ROWS>
struct Fragments;
template <>
struct Fragments<false> {
  static constexpr int kReads = 8, kBases = 2;
  u32x4 v[8];
  template <int SLOT, int I>
  __device__ __forceinline__ void read(const uint32_t (&base)[2]) {
    lds_read16<SLOT * kHalfTile + (I & 3) * 2048>(v[I], base[I >> 2]);
  }
  __device__ __forceinline__ u32x4 get(int r) const { return v[r]; }
  template <int H>   // the fragments of k-step H
  __device__ __forceinline__ void tie_half() { asm volatile("" : PPMOE_TIE4(v + 4 * H) : : "memory"); }
  __device__ __forceinline__ void tie() {
    tie_half<0>();
    tie_half<1>();
  }
};
template <>
struct Fragments<true> {
  static constexpr int kReads = 16, kBases = 4;
  u32x2 v[16];
  template <int SLOT, int I>
  __device__ __forceinline__ void read(const uint32_t (&base)[4]) {
    lds_read_transposed<SLOT * kHalfTile + (I >> 3) * 8192 + (I & 1) * 1024>(v[I], base[(I >> 1) & 3]);
  }
  __device__ __forceinline__ u32x4 get(int r) const { return __builtin_shufflevector(v[2 * r], v[2 * r + 1], 0, 1, 2, 3); }
  template <int H>
  __device__ __forceinline__ void tie_half() { asm volatile("" : PPMOE_TIE8(v + 8 * H) : : "memory"); }
  __device__ __forceinline__ void tie() {
    tie_half<0>();
    tie_half<1>();
  }
};

// This lane's fragment addresses in half-tile 0 of the ring's first k-tile.  w: the wavefront's half of the tile.
// By columns: k-steps 0 and 1 (32 k-values each): row (lane & 15) of a 16-row block, the 8 k-values of piece 4 ks + (lane >> 4).
__device__ __forceinline__ void fragment_base(uint32_t lds0, int lane, int w, uint32_t (&base)[2]) {
  const int fr = lane & 15, fq = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    base[ks] = lds0 + (w * 64 + fr) * 128 + (((4 * ks + fq) ^ ((fr >> 1) & 7)) << 4);
}
// By rows: the four 16-column blocks; k-row 8 (lane >> 4) + (0..3) of a k-step, 8 of the block's 32 bytes.
__device__ __forceinline__ void fragment_base(uint32_t lds0, int lane, int w, uint32_t (&base)[4]) {
  const int fq = lane >> 4, j = (lane >> 2) & 3, sub = lane & 3;
#pragma unroll
  for (int b = 0; b < 4; ++b) base[b] = lds0 + (fq * 8 + j) * 256 + (((w * 4 + b) ^ (j + 4 * (fq & 1))) << 5) + sub * 8;
}

// A value that is the same in all lanes, in a scalar register.  (The builtin is dropped where the compiler sees that its
// operand is uniform, and the value may then reach a scalar operand of inline assembly in a vector register.  The wait
// states that the instruction needs after a write of its operand, and its result before a read, are written out: the compiler
// does not look into inline assembly for them.)
__device__ __forceinline__ int in_scalar(int v) {
  int s;
  asm volatile("s_nop 4\n\tv_readfirstlane_b32 %0, %1\n\ts_nop 4" : "=s"(s) : "v"(v));
  return s;
}

// At most N vector memory operations outstanding; only M while t < behind.  (One branch, not taken in the steady state:
// a taken one costs some 40 cycles of a wavefront that has nobody to hide them behind.)
template <int N, int M>
__device__ __forceinline__ void wait_loads(int t, int behind) {
  asm volatile(
      "s_cmp_lt_i32 %0, %1\n\ts_cbranch_scc1 .Lbehind%=\n\ts_waitcnt vmcnt(%2)\n.Lbehind%=:\n\ts_waitcnt vmcnt(%3)"
      :
      : "s"(t), "s"(behind), "n"(N), "n"(M)
      : "memory", "scc");
}

// acc[mi][ni] += the products of `tiles` k-tiles.  The loads of k-tiles 0 and 1 are under way (in the order j, n);
// load(j, n, i) issues those of half-tile j, chunk n, of k-tile i into ring slot (i & 1, j); past the last k-tile it
// fetches zeros.  stores_behind: exactly STORES stores of every wavefront were issued after the loads of k-tiles 0 and 1
// (vmcnt counts in order: they need not have drained for those loads to have landed; it counts to 63).
// A_BY_ROWS, B_BY_ROWS: the operand's contraction index is its row.
// D = B_frag (16 columns) x A_frag^T (16 rows): lane: row mi * 16 + (lane & 15), in register v of acc[mi][ni] column
// ni * 16 + (lane >> 4) * 4 + v.
template <int DT, bool A_BY_ROWS, bool B_BY_ROWS, int STORES, typename LOAD>
__device__ __forceinline__ void k_loop(f32x4 (&acc)[8][8], const uint32_t (&a_base)[Fragments<A_BY_ROWS>::kBases],
                                       const uint32_t (&b_base)[Fragments<B_BY_ROWS>::kBases], int tiles,
                                       bool stores_behind, LOAD load) {
  typedef typename Elem16<DT>::vec8 vec8;
  constexpr int NA = Fragments<A_BY_ROWS>::kBases, NB = Fragments<B_BY_ROWS>::kBases;
  constexpr int RA = Fragments<A_BY_ROWS>::kReads, RB = Fragments<B_BY_ROWS>::kReads;
  constexpr int SA = 16 / RA, SB = 16 / RB;            // MFMAs per fragment read
  constexpr auto up_to_63 = [](int n) { return n < 63 ? n : 63; };
  Fragments<A_BY_ROWS> fa[2];   // by half
  Fragments<B_BY_ROWS> fb[2];
  uint32_t par = 0;
  const int behind = in_scalar(stores_behind ? 2 : 0);
  wait_loads<24, up_to_63(24 + STORES)>(0, behind);
  __builtin_amdgcn_s_barrier();
  each<RA>([&](auto i) __attribute__((always_inline)) { fa[0].template read<0, i.value>(a_base); });
  each<RB / 2>([&](auto i) __attribute__((always_inline)) { fb[0].template read<1, i.value>(b_base); });
  // MFMA x (0..31) of the phase that multiplies halves ha and hb, pinned where it is written (without the
  // sched_barriers the compiler sinks the fragment reads below the MFMAs).  B fragments in a snake, A's held for four.
  auto mfma = [&](auto ha_c, auto hb_c, auto x_c) __attribute__((always_inline)) {
    constexpr int ha = decltype(ha_c)::value, hb = decltype(hb_c)::value, x = decltype(x_c)::value;
    constexpr int ks = x >> 4, i = (x >> 2) & 3, k = (i & 1) ? 3 - (x & 3) : (x & 3);
    constexpr int mi = ha * 4 + i, ni = hb * 4 + k;
    __builtin_amdgcn_sched_barrier(0);
    acc[mi][ni] = Elem16<DT>::mfma16(__builtin_bit_cast(vec8, fb[hb].get(ks * 4 + k)),
                                     __builtin_bit_cast(vec8, fa[ha].get(ks * 4 + i)), acc[mi][ni]);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma clang loop unroll(disable)
  for (int t = 0; t < tiles; ++t) {
    const uint32_t nx = kKTile - par;
    uint32_t at[NA], an[NA], bt[NB], bn[NB];   // fragment addresses of this k-tile and the next
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      at[i] = a_base[i] + par;
      an[i] = a_base[i] + nx;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      bt[i] = b_base[i] + par;
      bn[i] = b_base[i] + nx;
    }
    // B1 and A1 of this k-tile have landed (younger: the 16 loads of the next one), and every wavefront has read
    // A0 of this one and (but for k-step 1) B0.
    wait_loads<16, up_to_63(16 + STORES)>(t, behind);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fa[0].tie();   // (the ties keep the MFMAs that use these fragments behind the wait)
    fb[0].template tie_half<0>();
    __builtin_amdgcn_s_barrier();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<0>{}, IC<0>{}, x);
      if constexpr (X < RB / 2) fb[0].template read<1, RB / 2 + (X < RB / 2 ? X : 0)>(bt);
      constexpr int Y = X - RB / 2;
      if constexpr (Y >= 0 && Y < 16 && Y % SB == 0) fb[1].template read<2, (Y >= 0 && Y < 16 ? Y / SB : 0)>(bt);
      // (the reads of B0's k-step 1 are followed by 6 or 8 others when the MFMAs that need them come up)
      if constexpr (X == 15) {
        if constexpr (B_BY_ROWS) asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt lgkmcnt(6)" ::: "memory");
        fb[0].template tie_half<1>();
      }
      if constexpr (X % 8 == 3) load(IC<0>{}, IC<X / 8>{}, t + 2);
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fb[1].tie();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<0>{}, IC<1>{}, x);
      if constexpr (X < 16 && X % SA == 0) fa[1].template read<3, (X < 16 ? X / SA : 0)>(at);
    });
    // A0 and B0 of the next k-tile have landed (younger: its B1 and A1 and A0 of the one after), and every
    // wavefront has read all of this one.
    wait_loads<12, up_to_63(12 + STORES)>(t + 1, behind);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fa[1].tie();
    __builtin_amdgcn_s_barrier();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<1>{}, IC<1>{}, x);
      if constexpr (X < 16 && X % SA == 0) fa[0].template read<0, (X < 16 ? X / SA : 0)>(an);
      if constexpr (X < 24 && X % 4 == 3) load(IC<1 + X / 16>{}, IC<(X / 4) & 3>{}, t + 2);
    });
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<1>{}, IC<0>{}, x);
      constexpr int Y = X - 16;
      if constexpr (Y >= 0 && Y < 8 && Y % SB == 0) fb[0].template read<1, (Y >= 0 && Y < 8 ? Y / SB : 0)>(bn);
      if constexpr (X < 24 && X % 4 == 3) load(IC<(X < 8 ? 2 : 3)>{}, IC<(X < 8 ? 2 + X / 4 : X / 4 - 2)>{}, t + 2);
    });
    par = nx;
  }
  // (the fragments read last are not used; they land before the registers die, and the phantom loads before their slots are
  // reused.  The accumulators are named as such: left to itself the register allocator keeps some of them elsewhere.)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  fa[0].tie();
  fb[0].template tie_half<0>();
#pragma unroll
  for (int mi = 0; mi < 8; ++mi)
    asm volatile("" : "+a"(acc[mi][0]), "+a"(acc[mi][1]), "+a"(acc[mi][2]), "+a"(acc[mi][3]), "+a"(acc[mi][4]),
                 "+a"(acc[mi][5]), "+a"(acc[mi][6]), "+a"(acc[mi][7]));
}

}  // namespace core
}  // namespace ppmoe
