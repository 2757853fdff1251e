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
// 8192 x 8192 x 8192: 1.37 PFLOP/s with 32x32x16 and register staging, 1.41 with LDS loads, 1.55 with both;
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

// 16 bytes per lane from memory (descriptor, byte offset of the lane, scalar offset) to LDS at `dst` + 16 * lane.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t rsrc, unsigned char* dst, uint32_t off, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, soff, 0, 0);
}

// The row of a 256-row tile that this lane fetches for chunk n (0..3) of half h, and the byte offset in that row.
__device__ __forceinline__ int staged_row(int wave, int lane, int h, int n) {
  return (wave >> 1) * 128 + h * 64 + (wave & 1) * 32 + n * 8 + (lane >> 3);
}
__device__ __forceinline__ int staged_piece(int lane, int n) {   // 16-byte piece: the swizzle's inverse
  return (lane & 7) ^ (((n & 1) * 4 + (lane >> 4)) & 7);
}

// This lane's fragment addresses in half-tile 0 of the ring's first k-tile, k-steps 0 and 1 (32 k-values each):
// row (lane & 15) of a 16-row block, the 8 k-values of piece 4 ks + (lane >> 4).  w: the wavefront's half of the tile.
__device__ __forceinline__ void fragment_base(uint32_t lds0, int lane, int w, uint32_t (&base)[2]) {
  const int fr = lane & 15, fq = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    base[ks] = lds0 + (w * 64 + fr) * 128 + (((4 * ks + fq) ^ ((fr >> 1) & 7)) << 4);
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
// fetches zeros.  stores_behind: exactly 32 stores of every wavefront were issued after the loads of k-tiles 0 and 1
// (vmcnt counts in order: they need not have drained for those loads to have landed).
// D = B_frag (16 columns) x A_frag^T (16 rows): lane: row mi * 16 + (lane & 15), in register v of acc[mi][ni] column
// ni * 16 + (lane >> 4) * 4 + v.
template <int DT, typename LOAD>
__device__ __forceinline__ void k_loop(f32x4 (&acc)[8][8], const uint32_t (&a_base)[2], const uint32_t (&b_base)[2],
                                       int tiles, bool stores_behind, LOAD load) {
  typename Elem16<DT>::vec8 f[4][8];   // [half-tile j][k-step * 4 + 16-row block]
  uint32_t par = 0;
  const int behind = stores_behind ? 2 : 0;
  if (stores_behind) asm volatile("s_waitcnt vmcnt(56)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  // fragment r (k-step * 4 + block) of half-tile j
#define PPMOE_RD(j, r, ad) lds_read16<(j) * kHalfTile + ((r) & 3) * 2048>(f[j][r], (ad)[(r) >> 2])
  each<8>([&](auto r) __attribute__((always_inline)) { PPMOE_RD(0, r.value, a_base); });
  each<4>([&](auto r) __attribute__((always_inline)) { PPMOE_RD(1, r.value, b_base); });
  // MFMA x (0..31) of the phase that multiplies half-tiles ja and jb, pinned where it is written (without the
  // sched_barriers the compiler sinks the fragment reads below the MFMAs).  B fragments in a snake, A's held for four.
  auto mfma = [&](auto ja_c, auto jb_c, auto x_c) __attribute__((always_inline)) {
    constexpr int ja = decltype(ja_c)::value, jb = decltype(jb_c)::value, x = decltype(x_c)::value;
    constexpr int ks = x >> 4, i = (x >> 2) & 3, k = (i & 1) ? 3 - (x & 3) : (x & 3);
    constexpr int mi = (ja == 3) * 4 + i, ni = (jb == 2) * 4 + k;
    __builtin_amdgcn_sched_barrier(0);
    acc[mi][ni] = Elem16<DT>::mfma16(f[jb][ks * 4 + k], f[ja][ks * 4 + i], acc[mi][ni]);
    __builtin_amdgcn_sched_barrier(0);
  };
#define PPMOE_LANDED()                                                                               \
  do {                                                                                               \
    asm volatile("s_waitcnt lgkmcnt(0)" : PPMOE_TIE8(f[0]), PPMOE_TIE8(f[1]) : : "memory");          \
    asm volatile("" : PPMOE_TIE8(f[2]), PPMOE_TIE8(f[3]) : : "memory");                              \
  } while (0)
#pragma clang loop unroll(disable)
  for (int t = 0; t < tiles; ++t) {
    const uint32_t nx = kKTile - par;
    const uint32_t at[2] = {a_base[0] + par, a_base[1] + par}, bt[2] = {b_base[0] + par, b_base[1] + par};
    const uint32_t an[2] = {a_base[0] + nx, a_base[1] + nx}, bn[2] = {b_base[0] + nx, b_base[1] + nx};
    // B1 and A1 of this k-tile have landed (younger: the 16 loads of the next one), and every wavefront has read
    // A0 of this one and (but for k-step 1) B0.
    wait_loads<16, 48>(t, behind);
    PPMOE_LANDED();
    __builtin_amdgcn_s_barrier();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<0>{}, IC<1>{}, x);
      if constexpr (X < 4) PPMOE_RD(1, 4 + X, bt);
      if constexpr (X >= 4 && X < 20 && X % 2 == 0) PPMOE_RD(2, (X - 4) / 2, bt);
      // (the four reads of B0's k-step 1 are followed by six others when the MFMAs that need them come up)
      if constexpr (X == 15) asm volatile("s_waitcnt lgkmcnt(6)" : PPMOE_TIE8(f[1]) : : "memory");
      if constexpr (X % 8 == 3) load(IC<0>{}, IC<X / 8>{}, t + 2);
    });
    PPMOE_LANDED();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<0>{}, IC<2>{}, x);
      if constexpr (X < 16 && X % 2 == 0) PPMOE_RD(3, X / 2, at);
    });
    // A0 and B0 of the next k-tile have landed (younger: its B1 and A1 and A0 of the one after), and every
    // wavefront has read all of this one.
    wait_loads<12, 44>(t + 1, behind);
    PPMOE_LANDED();
    __builtin_amdgcn_s_barrier();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<3>{}, IC<2>{}, x);
      if constexpr (X < 16 && X % 2 == 0) PPMOE_RD(0, X / 2, an);
      if constexpr (X < 24 && X % 4 == 3) load(IC<1 + X / 16>{}, IC<(X / 4) & 3>{}, t + 2);
    });
    PPMOE_LANDED();
    each<32>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value;
      mfma(IC<3>{}, IC<1>{}, x);
      if constexpr (X >= 16 && X < 24 && X % 2 == 0) PPMOE_RD(1, (X - 16) / 2, bn);
      if constexpr (X < 24 && X % 4 == 3) load(IC<(X < 8 ? 2 : 3)>{}, IC<(X < 8 ? 2 + X / 4 : X / 4 - 2)>{}, t + 2);
    });
    par = nx;
  }
  // (the fragments read last are not used; they land before the registers die, and the phantom loads before their slots are reused)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  PPMOE_LANDED();
#undef PPMOE_LANDED
#undef PPMOE_RD
}

}  // namespace core
}  // namespace ppmoe
