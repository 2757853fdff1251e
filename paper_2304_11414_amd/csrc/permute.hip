// Dispatching order -> per-expert index lists (the "indices" of Algorithm 1; worked example of
// Section 3.3.3: order 2,3,1,2,0,3,2,0 gives [4,7] [2] [0,3,6] [1,5]).
//
// The position of assignment a = t*k + j in its expert's queue is the number of earlier assignments
// to the same expert.  It is computed without order-dependent atomics, so the permutation is
// identical on every run and on every rank of a tensor-parallel group:
//   1. every wavefront owns a segment of seg_assign consecutive assignments (64 when this file counts
//      them; the tokens of one block when the gating kernel has already counted them on the way)
//      and counts, per local expert, how many of them it holds (ballot + popcount, counts kept in
//      registers);
//   2. the per-segment counts are turned into exclusive prefix sums per expert (by every block of step 3
//      for its own segments; by a launch of its own when there are many segments or experts);
//   3. every wavefront walks its segment again, 64 assignments at a time: rank inside the step by
//      ballot/popcount, plus the running count carried in registers, plus the segment's prefix.
// counts/offsets (capacity-clamped, exclusive scan over the local experts) are rebuilt by every
// wavefront of step 3 from the expert totals, which costs a few shuffles, and written by the first.

#include <mutex>

#include "common.h"

namespace ppmoe {

// Scratch of the allocation-free dispatch call (per-segment counters of the permutation): a
// file-scope array in device memory, kStaticScratchBytes on every device the library runs on, held
// until the process ends.  In host code the name below is only a stand-in for the symbol: its device
// address is looked up once per device (static_scratch_of) and that pointer is what kernels get.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
void* g_scratch_ptr[kMaxScratchDevices] = {};
std::mutex g_scratch_mutex;
}  // namespace

hipError_t static_scratch_of_current_device(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // (this device's copy: the device is current)
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

constexpr int kRegs = kMaxExperts / kWave;  // lane i holds experts i, i+64, i+128, i+192
constexpr int kPlaceThreads = 1024, kPlaceWaves = kPlaceThreads / kWave;   // placing kernel: segments per block

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// For a uniform expert id e: value of run[e / 64] held by lane e % 64.
__device__ __forceinline__ int read_slot(const int (&run)[kRegs], int e) {
  int v = 0;
#pragma unroll
  for (int c = 0; c < kRegs; ++c)
    if ((e >> 6) == c) v = __builtin_amdgcn_readlane(run[c], e & 63);
  return v;
}

__device__ __forceinline__ void add_slot(int (&run)[kRegs], int e, int amount) {
#pragma unroll
  for (int c = 0; c < kRegs; ++c)
    if ((e >> 6) == c && lane_id() == (e & 63)) run[c] += amount;
}

// Step 1.  seg_count[i * n_seg + seg] = number of assignments of segment seg that picked local
// expert i.
__device__ __forceinline__ void count_segment(const int32_t* __restrict__ expert_idx,
                                              int32_t* seg_count, int seg, int64_t n_assign,
                                              int n_seg, int seg_assign, int local_begin, int n_local) {
  const int lane = lane_id();
  int run[kRegs] = {0, 0, 0, 0};
  const int64_t base = static_cast<int64_t>(seg) * seg_assign;
  const int64_t end = min(n_assign, base + seg_assign);
  for (int step = 0; step * kWave < seg_assign; ++step) {
    int64_t a = base + step * kWave + lane;
    int e = -1;
    if (a < end) {
      unsigned le = static_cast<unsigned>(expert_idx[a] - local_begin);
      if (le < static_cast<unsigned>(n_local)) e = static_cast<int>(le);
    }
    unsigned long long todo = __ballot(e >= 0);
    while (todo) {
      int leader = __ffsll(static_cast<long long>(todo)) - 1;
      int e0 = __builtin_amdgcn_readlane(e, leader);
      unsigned long long same = __ballot(e == e0);
      add_slot(run, e0, __popcll(same));
      todo &= ~same;
    }
  }
#pragma unroll
  for (int c = 0; c < kRegs; ++c) {
    int i = c * kWave + lane;
    if (i < n_local) seg_count[static_cast<int64_t>(i) * n_seg + seg] = run[c];
  }
}

__global__ __launch_bounds__(256) void segment_count_kernel(const int32_t* __restrict__ expert_idx,
                                                            int32_t* __restrict__ seg_count,
                                                            int64_t n_assign, int n_seg,
                                                            int seg_assign, int local_begin,
                                                            int n_local) {
  const int seg = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (seg < n_seg)
    count_segment(expert_idx, seg_count, seg, n_assign, n_seg, seg_assign, local_begin, n_local);
}

// The balance loss (Algorithm 1's l_aux; see aux.hip for the formula) from the per-segment partial sums the
// gating kernel left: one block adds them up and writes the loss.  The threads form slices of E (thread
// slice * E + e: neighbouring threads on neighbouring experts of one segment), every slice adds up its
// share of the segments, the slices are added in order: a fixed order, bitwise reproducible.  (One thread
// per expert walking all the segments, two dependent loads at a time, took 80 us for 512 segments; the
// slices finish inside the placing kernel's 10 us.)
__device__ __forceinline__ void finish_balance_loss(const AuxOut& aux) {
  __shared__ float prob[kPlaceThreads];
  __shared__ int32_t cnt[kPlaceThreads];
  __shared__ float term[kMaxExperts];
  const int slices = static_cast<int>(blockDim.x) / aux.E;
  const int slice = threadIdx.x / aux.E, e = threadIdx.x - slice * aux.E;
  if (slice < slices) {
    float p = 0.f;
    int n = 0;
    for (int g0 = slice; g0 < aux.n_part; g0 += slices * 8) {
      float pv[8];
      int nv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int g = g0 + j * slices;
        const size_t at = static_cast<size_t>(min(g, aux.n_part - 1)) * aux.E + e;
        pv[j] = aux.part_prob[at];
        nv[j] = aux.part_cnt[at];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p += g0 + j * slices < aux.n_part ? pv[j] : 0.f;
        n += g0 + j * slices < aux.n_part ? nv[j] : 0;
      }
    }
    prob[threadIdx.x] = p;
    cnt[threadIdx.x] = n;
  }
  __syncthreads();
  if (static_cast<int>(threadIdx.x) < aux.E) {
    float p = 0.f;
    int n = 0;
    for (int sl = 0; sl < slices; ++sl) {
      p += prob[sl * aux.E + threadIdx.x];
      n += cnt[sl * aux.E + threadIdx.x];
    }
    const float mp = aux.T > 0 ? p / static_cast<float>(aux.T) : 0.f;
    if (aux.mean_prob != nullptr) aux.mean_prob[threadIdx.x] = mp;
    if (aux.first_counts != nullptr) aux.first_counts[threadIdx.x] = n;
    term[threadIdx.x] = aux.T > 0 ? mp * (static_cast<float>(n) / static_cast<float>(aux.T)) : 0.f;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = 0.f;
    for (int i = 0; i < aux.E; ++i) sum += term[i];   // ascending expert order
    *aux.l_aux = static_cast<float>(aux.E) * sum;
  }
}

// Step 2 as a launch of its own (see launch_permute).  One block per local expert:
// seg_base = exclusive scan of seg_count over segments (may be done in place), totals[i] = queue length
// of expert i before any capacity clamp.  A thread adds up a run of consecutive segments, the run sums
// are scanned (butterfly inside a wavefront, the wavefront totals in order), and every thread then
// writes the prefixes of its run.
constexpr int kScanThreads = 256;
__global__ __launch_bounds__(kScanThreads) void segment_scan_kernel(const int32_t* seg_count, int32_t* seg_base,
                                                                    int32_t* __restrict__ totals, int n_seg) {
  __shared__ int wave_total[kScanThreads / kWave];
  const int i = blockIdx.x;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int32_t* in = seg_count + static_cast<int64_t>(i) * n_seg;
  int32_t* out = seg_base + static_cast<int64_t>(i) * n_seg;
  const int run = (n_seg + kScanThreads - 1) / kScanThreads;
  const int s0 = threadIdx.x * run, s1 = min(n_seg, s0 + run);
  int sum = 0;
  for (int s = s0; s < s1; ++s) sum += in[s];
  int incl = sum;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    int up = __shfl_up(incl, off, 64);
    if (lane >= off) incl += up;
  }
  if (lane == kWave - 1) wave_total[wave] = incl;
  __syncthreads();
  int before = incl - sum;
  for (int w = 0; w < wave; ++w) before += wave_total[w];
  for (int s = s0; s < s1; ++s) {
    const int v = in[s];
    out[s] = before;
    before += v;
  }
  if (threadIdx.x == kScanThreads - 1) totals[i] = before;
}

// Step 2 folded into step 3: the block's wavefronts share the local experts; for each, a wavefront reads
// the counts of all the segments (64 at a time, the loads independent of each other) and leaves in LDS the
// expert's total and the prefix of each of the block's own segments.
__device__ __forceinline__ void scan_for_block(const int32_t* __restrict__ seg_count, int n_seg, int n_local,
                                               int32_t (&base)[kPlaceWaves][kMaxExperts],
                                               int32_t (&total)[kMaxExperts]) {
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int s0 = blockIdx.x * kPlaceWaves;
  for (int i = wave; i < n_local; i += kPlaceWaves) {
    const int32_t* in = seg_count + static_cast<int64_t>(i) * n_seg;
    const int own = (lane < kPlaceWaves && s0 + lane < n_seg) ? in[s0 + lane] : 0;
    int before = 0, all = 0;
    for (int s = lane; s < n_seg; s += kWave * 8) {
      int v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = s + j * kWave < n_seg ? in[s + j * kWave] : 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        all += v[j];
        before += s + j * kWave < s0 ? v[j] : 0;
      }
    }
    int incl = own;
#pragma unroll
    for (int off = 1; off < kPlaceWaves; off <<= 1) {
      const int up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      before += __shfl_xor(before, off, 64);
      all += __shfl_xor(all, off, 64);
    }
    if (lane < kPlaceWaves) base[lane][i] = before + incl - own;
    if (lane == 0) total[i] = all;
  }
}

// Step 3.  first_pick: expert_idx of this lane's assignment in the segment's first 64.  totals[i]: queue length of
// local expert i; seg_base[i * stride]: assignments to it before this segment.
__device__ __forceinline__ void rank_segment(
    const int32_t* __restrict__ expert_idx, const int32_t* seg_base, int64_t stride, const int32_t* totals,
    int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv_perm, int seg, int64_t n_assign, int seg_assign,
    int local_begin, int n_local, int cap /* INT_MAX when unlimited */, int first_pick) {
  const int lane = lane_id();

  // Kept queue lengths and their exclusive scan over the local experts (ascending expert id).
  int kept[kRegs], off[kRegs], run[kRegs];
  int carry = 0;
#pragma unroll
  for (int c = 0; c < kRegs; ++c) {
    int i = c * kWave + lane;
    kept[c] = off[c] = run[c] = 0;
    if (c * kWave >= n_local) continue;   // (uniform: up to 64 local experts take one pass)
    kept[c] = i < n_local ? min(totals[i], cap) : 0;
    int incl = kept[c];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    off[c] = carry + incl - kept[c];
    carry += __shfl(incl, kWave - 1, 64);
    run[c] = i < n_local ? seg_base[i * stride] : 0;
    if (seg == 0 && i < n_local) {
      counts[i] = kept[c];
      offsets[i] = off[c];
    }
  }
  if (seg == 0 && lane == 0) offsets[n_local] = carry;

  const int64_t base = static_cast<int64_t>(seg) * seg_assign;
  const int64_t end = min(n_assign, base + seg_assign);
  for (int step = 0; step * kWave < seg_assign; ++step) {
    int64_t a = base + step * kWave + lane;
    int e = -1;
    if (a < end) {
      unsigned le = static_cast<unsigned>((step == 0 ? first_pick : expert_idx[a]) - local_begin);
      if (le < static_cast<unsigned>(n_local)) e = static_cast<int>(le);
    }
    int row = -1;
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long todo = __ballot(e >= 0);
    while (todo) {
      int leader = __ffsll(static_cast<long long>(todo)) - 1;
      int e0 = __builtin_amdgcn_readlane(e, leader);
      unsigned long long same = __ballot(e == e0);
      int pos0 = read_slot(run, e0);   // queue position of the first of this group
      int off0 = read_slot(off, e0);
      if (e == e0) {
        int pos = pos0 + __popcll(same & below);
        if (pos < cap) row = off0 + pos;
      }
      add_slot(run, e0, __popcll(same));
      todo &= ~same;
    }
    if (a < end) {
      inv_perm[a] = row;
      if (row >= 0) perm[row] = static_cast<int32_t>(a);
    }
  }
}

// A wavefront per segment.  seg_base != nullptr: the scan has been a launch of its own; else the block does
// it from seg_count.  One more block, when the balance loss is wanted, finishes it.
__global__ __launch_bounds__(kPlaceThreads) void place_kernel(
    const int32_t* __restrict__ expert_idx, const int32_t* __restrict__ seg_count,
    const int32_t* __restrict__ seg_base, const int32_t* __restrict__ totals, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int64_t n_assign,
    int n_seg, int seg_assign, int local_begin, int n_local, int cap, int blocks, AuxOut aux) {
  if (static_cast<int>(blockIdx.x) == blocks) {
    finish_balance_loss(aux);
    return;
  }
  __shared__ int32_t base[kPlaceWaves][kMaxExperts];
  __shared__ int32_t total[kMaxExperts];
  const int wave = threadIdx.x >> 6, seg = blockIdx.x * kPlaceWaves + wave;
  // (this lane's first pick: its load is out before the scan's)
  const int64_t a0 = static_cast<int64_t>(seg) * seg_assign + lane_id();
  const int first_pick = a0 < n_assign ? expert_idx[a0] : -1;
  const bool folded = seg_base == nullptr;
  if (folded) {
    scan_for_block(seg_count, n_seg, n_local, base, total);
    __syncthreads();
  }
  if (seg < n_seg || seg == 0)   // (n_seg == 0: counts and offsets are still defined, all zero)
    rank_segment(expert_idx, folded ? base[wave] : seg_base + seg, folded ? 1 : n_seg, folded ? total : totals, counts,
                 offsets, perm, inv_perm, seg, n_assign, seg_assign, local_begin, n_local, cap, first_pick);
}

constexpr int kFoldExperts = 2 * kPlaceWaves;   // local experts up to which the placing kernel scans

hipError_t launch_permute(const moe_config& c, int64_t cap, const int32_t* expert_idx,
                          int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm,
                          int32_t* seg_scratch, hipStream_t s, int seg_assign, bool counted,
                          const AuxOut* aux) {
  const int64_t n_assign = static_cast<int64_t>(c.T) * c.top_k;
  const int n_seg = static_cast<int>((n_assign + seg_assign - 1) / seg_assign);
  const int N = c.local_count;
  int32_t* seg_count = seg_scratch;
  const int cap_i = (cap < 0 || cap > 0x7fffffff) ? 0x7fffffff : static_cast<int>(cap);
  if (n_seg > 0 && !counted)
    segment_count_kernel<<<(n_seg + 3) / 4, 256, 0, s>>>(expert_idx, seg_count, n_assign, n_seg, seg_assign,
                                                         c.local_begin, N);
  // The scan over the segments is done by every block of the placing kernel while a wavefront has at most 64
  // loads to make for it (8 local experts: up to 4096 segments).  A launch costs 4-5 us whatever it does, those
  // loads 1 us at 512 segments (8192 tokens) and, growing with the segments, about as much as the launch where
  // the line is; beyond it the scan is a launch of its own.  (8192 tokens, 8 experts: scan + rank 4.9 + 6.5 us,
  // this kernel 8.6; 16 tokens: 4.6 + 5.2, 6.4.)  So it is past 32 local experts, whose rows a wavefront takes one
  // after another, a memory latency each (dispatch of 1000 tokens, top-1: 32 experts 18.2 us folded, 19.0 with the
  // launch; 64: 20.4 and 19.0; 128: 25.2 and 20.5; 256, top-8: 31.6 and 20.0).
  const int64_t loads = static_cast<int64_t>((N + kPlaceWaves - 1) / kPlaceWaves) * ((n_seg + kWave - 1) / kWave);
  int32_t *seg_base = nullptr, *totals = nullptr;
  if (loads > 64 || N > kFoldExperts) {
    seg_base = seg_scratch + static_cast<int64_t>(N) * n_seg;
    totals = seg_base + static_cast<int64_t>(N) * n_seg;
    segment_scan_kernel<<<N, kScanThreads, 0, s>>>(seg_count, seg_base, totals, n_seg);
  }
  const bool with_aux = aux != nullptr && aux->l_aux != nullptr;
  const int blocks = n_seg > 0 ? (n_seg + kPlaceWaves - 1) / kPlaceWaves : 1;
  place_kernel<<<blocks + (with_aux ? 1 : 0), kPlaceThreads, 0, s>>>(
      expert_idx, seg_count, seg_base, totals, counts, offsets, perm, inv_perm, n_assign, n_seg, seg_assign,
      c.local_begin, N, cap_i, blocks, with_aux ? *aux : AuxOut{});
  return hipGetLastError();
}

}  // namespace ppmoe
