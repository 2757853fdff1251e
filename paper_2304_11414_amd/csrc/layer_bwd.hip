// Backward of the layer around the expert FFN (the paper prints no backward algorithm -- Section 3.2,
// footnote to Eq. 1, only prices it; this is the chain rule of Algorithm 1's forward, picks held
// fixed):
//   dY[r, :]       = gate_w[t, j] * d_out[t, :]          for the kept local assignment (t, j) in row r
//   d_gate_w[t, j] = <d_out[t, :], y_sliced[r, :]>        (0 for dropped / non-local picks)
//   dlogits        through the (renormalised) top-k weights and the softmax
//   dx[t, :]       = sum over kept local (t, j) of dX_sliced[r, :]  +  dlogits[t, :] Wg
//   dWg            = dlogits^T x,   dbias = column sums of dlogits
// All of it is this device's partial sum, like the forward output.  Row movement kernels are
// HBM-bound; every sum has a fixed order (bitwise reproducible).

#include "common.h"

namespace ppmoe {

namespace {

constexpr int kThreads = 256;

template <int D>
__device__ __forceinline__ void widen8(const void* p, float (&f)[8]) {
  if constexpr (D == MOE_F32) {
    const f32x4 a = reinterpret_cast<const f32x4*>(p)[0], b = reinterpret_cast<const f32x4*>(p)[1];
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  } else {
    const u32x4 v = *reinterpret_cast<const u32x4*>(p);
    Elem16<D>::widen2(v.x, f[0], f[1]);
    Elem16<D>::widen2(v.y, f[2], f[3]);
    Elem16<D>::widen2(v.z, f[4], f[5]);
    Elem16<D>::widen2(v.w, f[6], f[7]);
  }
}

template <int D>
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
  return u32x4{Elem16<D>::pack2(f[0], f[1]), Elem16<D>::pack2(f[2], f[3]), Elem16<D>::pack2(f[4], f[5]),
               Elem16<D>::pack2(f[6], f[7])};
}

// dY[r, :] = gate_w[perm[r]] * d_out[perm[r] / k, :]; a thread moves 8 elements per row.
template <int DOUT, int DT>
__global__ __launch_bounds__(kThreads) void gather_scale_kernel(const void* __restrict__ d_out,
                                                                const int32_t* __restrict__ perm,
                                                                const int32_t* __restrict__ offsets,
                                                                const float* __restrict__ gate_w,
                                                                bf16_t* __restrict__ dY, int n_local, int top_k,
                                                                int d) {
  const int rows = offsets[n_local];
  constexpr int in_bytes = DOUT == MOE_F32 ? 4 : 2;
  const unsigned char* src = static_cast<const unsigned char*>(d_out);
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const int a = perm[r];
    const int t = top_k == 1 ? a : a / top_k;
    const float w = gate_w[a];
    for (int c = threadIdx.x * 8; c < d; c += kThreads * 8) {
      float f[8];
      widen8<DOUT>(src + (static_cast<int64_t>(t) * d + c) * in_bytes, f);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] *= w;
      *reinterpret_cast<u32x4*>(dY + static_cast<int64_t>(r) * d + c) = pack8<DT>(f);
    }
  }
}

// p = softmax(logits);  w_j = p[e_j], or p[e_j] / S with S = sum_j p[e_j] when
// renormalised (gate_w holds the w_j the forward used).  d_gate_w[j] = row_dot[row] / w_j for a kept
// local pick (row_dot = <dY, y_sliced> = w_j <d_out, y_sliced>), else 0.
// Without renormalisation dp[e_j] = dw_j; with it dp[e_j] = (dw_j - sum_i dw_i w_i) / S.
// Softmax: dlogits[e] = p[e] (dp[e] - sum_e' dp[e'] p[e']).
// LPT lanes per token (8 to 64, the smallest power of two >= E; a lane then has one expert, or up to
// four beyond 64), lane j < k of them also owns pick j: the logits come in as whole rows and every sum is a
// butterfly.  Latency bound; at 16384 tokens x 64 experts 10 us, where a thread per
// token walking its row took 45.
template <int LPT>
__global__ __launch_bounds__(kThreads) void gate_backward_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ expert_idx, const float* __restrict__ gate_w,
    const int32_t* __restrict__ inv_perm, const float* __restrict__ row_dot, float* __restrict__ dlogits, int T,
    int E, int k, int renorm) {
  constexpr int NE = LPT == 64 ? kMaxExperts / 64 : 1;   // experts per lane
  const int sub = threadIdx.x % LPT;
  for (int64_t tb = static_cast<int64_t>(blockIdx.x) * (kThreads / LPT); tb < T; tb += static_cast<int64_t>(gridDim.x) * (kThreads / LPT)) {
    const int64_t t = tb + threadIdx.x / LPT;
    const bool live = t < T;   // (lanes past the end stay: the shuffles are the whole wavefront's)
    const float* lg = logits + (live ? t : T - 1) * E;
    float v[NE], m = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = sub + i * LPT;
      v[i] = e < E ? lg[e] : -__builtin_inff();
      m = fmaxf(m, v[i]);
    }
    auto group_sum = [](float x) {
#pragma unroll
      for (int off = LPT / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
      return x;
    };
#pragma unroll
    for (int off = LPT / 2; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      v[i] = sub + i * LPT < E ? expf(v[i] - m) : 0.f;
      sum += v[i];
    }
    sum = group_sum(sum);
    // this lane's pick
    int idx = -1;
    float w = 0.f, dw = 0.f, pj = 0.f;
    if (live && sub < k) {
      const int64_t a = t * k + sub;
      const int row = inv_perm[a];
      w = gate_w[a];
      idx = expert_idx[a];
      dw = row >= 0 ? row_dot[row] / w : 0.f;
      pj = expf(lg[idx] - m) / sum;
    }
    if (renorm) {   // (uniform)
      const float S = group_sum(pj), dww = group_sum(dw * w);
      dw = sub < k ? (dw - dww) / S : 0.f;   // now dp at the picked expert
    }
    const float here = pj * dw;
    const float dot = group_sum(here);   // sum_e dp[e] p[e]
    float o[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) o[i] = -(v[i] / sum) * dot;
    for (int j = 0; j < k; ++j) {   // (a token picks an expert at most once)
      const int ej = __shfl(idx, j, LPT);
      const float add = __shfl(here, j, LPT);
#pragma unroll
      for (int i = 0; i < NE; ++i)
        if (ej == sub + i * LPT) o[i] += add;
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = sub + i * LPT;
      if (live && e < E) dlogits[t * E + e] = o[i];
    }
  }
}

// dx[t, :] = sum over kept local picks of dX_sliced[row, :] + dlogits[t, :] Wg: movement of rows plus a
// contraction over E, which runs on the float32 16x16x4 matrix instruction (dlogits stays float32, Wg is
// widened exactly).  A wavefront owns 16 MT tokens x 128 columns.  The columns are the instruction's M
// index, permuted: in the q-th of eight products M index i is column 8 pi(i) + q, pi(4 g + v) = 4 v + g.
// So a lane's operand for all eight is one 16-byte piece of a router row, and its results for all eight
// are four 16-byte pieces of its token's row, 64 contiguous bytes of a row per store instruction; no LDS.
// Bound: HBM up to about 32 experts, the matrix unit (2 E flop per element at 157 TFLOP/s) beyond.  At
// 16384 x 1024 with 64 experts 38 us, where vector FMAs took 75.
template <int DT, int MT>
__global__ __launch_bounds__(kThreads) void dx_kernel(const bf16_t* __restrict__ dXs,
                                                      const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ dlogits,
                                                      const bf16_t* __restrict__ Wg, bf16_t* __restrict__ dx, int T,
                                                      int d, int E, int k) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = lane & 15, g = lane >> 4;
  const int col0 = (blockIdx.y * 4 + wave) * 128;
  if (col0 >= d) return;   // (no barrier below)
  for (int64_t tg = static_cast<int64_t>(blockIdx.x) * (16 * MT); tg < T; tg += static_cast<int64_t>(gridDim.x) * (16 * MT)) {
    const int t0 = static_cast<int>(tg);
    f32x4 acc[MT][8];        // [q][v]: column col0 + 8 (4 v + g) + q
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[mt][q] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int t = t0 + mt * 16 + j;
      for (int p = 0; t < T && p < k; ++p) {
        const int r = inv_perm[static_cast<int64_t>(t) * k + p];
        if (r < 0) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int c = col0 + 8 * (4 * v + g);
          if (c >= d) continue;
          float f[8];
          widen8<DT>(dXs + static_cast<int64_t>(r) * d + c, f);
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[mt][q][v] += f[q];
        }
      }
    }
    const int wcol = col0 + 8 * (4 * (j & 3) + (j >> 2));   // column piece pi(j)
    // Loads go to clamped addresses (what lies outside is set to zero afterwards): without branches around
    // them the loads of the next steps go out before the products of this one.
    const bf16_t* wg_lane = Wg + min(wcol, d - 8);
    const float* dl_lane[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) dl_lane[mt] = dlogits + static_cast<int64_t>(min(t0 + mt * 16 + j, T - 1)) * E;
    constexpr int U = 4;
    for (int e0 = 0; e0 < E; e0 += 4 * U) {
      u32x4 wr[U];
      float dl[U][MT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(e0 + 4 * u + g, E - 1);
        wr[u] = *reinterpret_cast<const u32x4*>(wg_lane + static_cast<int64_t>(e) * d);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) dl[u][mt] = dl_lane[mt][e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (e0 + 4 * u >= E) break;   // (uniform)
        const bool ok = e0 + 4 * u + g < E;
        const uint32_t w4[4] = {ok ? wr[u].x : 0u, ok ? wr[u].y : 0u, ok ? wr[u].z : 0u, ok ? wr[u].w : 0u};
        float w[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) Elem16<DT>::widen2(w4[q], w[2 * q], w[2 * q + 1]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const float g0 = ok ? dl[u][mt] : 0.f;
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[mt][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q], g0, acc[mt][q], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int t = t0 + mt * 16 + j;
      if (t >= T) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = col0 + 8 * (4 * v + g);
        if (c >= d) continue;
        float f[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) f[q] = acc[mt][q][v];
        *reinterpret_cast<u32x4*>(dx + static_cast<int64_t>(t) * d + c) = pack8<DT>(f);
      }
    }
  }
}

// dWg[e, c] = sum_t dlogits[t, e] x[t, c] on the float32 16x16x4 matrix instruction: a wavefront owns 128
// columns (lane j of a 16-lane group loads 16 bytes, columns 8 j + q feed the q-th of eight products) and up
// to 64 experts (ET groups of 16), over its share of the tokens; the four wavefronts of a block add up
// through LDS in order and a second launch adds the blocks' partial sums in order.  Bound: HBM (x is read
// once per 64 experts), beyond about 32 experts the matrix unit.  At 16384 x 1024 with 64
// experts 32 + 7 us; with vector FMAs, eight experts at a time, x was read E / 8 times and it took 173 + 19.
// The number of token shares: about two wavefronts per SIMD, at least 16 tokens each, and no more than 64 (the partial sums
// are read back once per share): up to 64 experts, columns below 1024 leave SIMDs with one wavefront or none (16384 tokens
// of 256 columns: 128 blocks; layer backward of 8 experts of 256 x 1024 306 us with the vector FMAs, 268 now).
constexpr int kMaxChunks = 64;
inline int dwg_chunks(const moe_config& c) {
  const int col_blocks = (c.d + 127) / 128;
  int n = (512 + col_blocks - 1) / col_blocks;
  const int by_tokens = (c.T + 63) / 64;
  n = n < by_tokens ? n : by_tokens;
  return n < 1 ? 1 : n < kMaxChunks ? n : kMaxChunks;
}
template <int DT, int ET>
__global__ __launch_bounds__(kThreads) void dwg_partial_kernel(const bf16_t* __restrict__ x,
                                                               const float* __restrict__ dlogits,
                                                               float* __restrict__ part, float* __restrict__ part_bias,
                                                               int T, int d, int E) {
  __shared__ float red[4][4 * 8 * 64];
  __shared__ float red_bias[4][ET * 16];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = lane & 15, g = lane >> 4;
  const int chunk = blockIdx.y, e0 = blockIdx.z * (ET * 16);
  const int shares = gridDim.y * 4;
  const int per = ((T + shares - 1) / shares + 3) & ~3;
  const int tb = min(T, (chunk * 4 + wave) * per), te = min(T, tb + per);
  const int col = blockIdx.x * 128 + j * 8;
  f32x4 acc[ET][8];
  float bsum[ET];
#pragma unroll
  for (int et = 0; et < ET; ++et) {
    bsum[et] = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[et][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int U = 4;   // steps of four tokens whose loads go out together
  for (int t0 = tb; t0 < te; t0 += 4 * U) {
    u32x4 xr[U];
    float dl[U][ET];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + 4 * u + g;
      xr[u] = (t < te && col < d) ? *reinterpret_cast<const u32x4*>(x + static_cast<int64_t>(t) * d + col) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int et = 0; et < ET; ++et) {
        const int e = e0 + et * 16 + j;
        dl[u][et] = (t < te && e < E) ? dlogits[static_cast<int64_t>(t) * E + e] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float f[8];
      const uint32_t w4[4] = {xr[u].x, xr[u].y, xr[u].z, xr[u].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) Elem16<DT>::widen2(w4[q], f[2 * q], f[2 * q + 1]);
#pragma unroll
      for (int et = 0; et < ET; ++et) {
        bsum[et] += dl[u][et];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[et][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(dl[u][et], f[q], acc[et][q], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int et = 0; et < ET; ++et) {
    bsum[et] += __shfl_xor(bsum[et], 16, 64);
    bsum[et] += __shfl_xor(bsum[et], 32, 64);
    if (g == 0) red_bias[wave][et * 16 + j] = bsum[et];
  }
  // One group of 16 experts at a time: every wavefront leaves its sums, then wavefront v adds up and stores
  // register v (lane (g, j): expert 4 g + v of the group, columns 8 j + q).
#pragma unroll
  for (int et = 0; et < ET; ++et) {
    if (et > 0) __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int q = 0; q < 8; ++q) red[wave][(v * 8 + q) * 64 + lane] = acc[et][q][v];
    __syncthreads();
    const int e = e0 + et * 16 + 4 * g + wave;
    if (e < E && col < d) {
      float sum[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int at = (wave * 8 + q) * 64 + lane;
        sum[q] = ((red[0][at] + red[1][at]) + red[2][at]) + red[3][at];
      }
      float* o = part + (static_cast<int64_t>(chunk) * E + e) * d + col;
      *reinterpret_cast<f32x4*>(o) = f32x4{sum[0], sum[1], sum[2], sum[3]};
      *reinterpret_cast<f32x4*>(o + 4) = f32x4{sum[4], sum[5], sum[6], sum[7]};
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < ET * 16 && e0 + static_cast<int>(threadIdx.x) < E) {
    const int e = threadIdx.x;
    part_bias[static_cast<int64_t>(chunk) * E + e0 + e] =
        ((red_bias[0][e] + red_bias[1][e]) + red_bias[2][e]) + red_bias[3][e];
  }
}

__global__ __launch_bounds__(kThreads) void dwg_final_kernel(const float* __restrict__ part,
                                                             const float* __restrict__ part_bias,
                                                             float* __restrict__ dWg, float* __restrict__ dbias, int d,
                                                             int E, int chunks) {
  const int64_t n = static_cast<int64_t>(E) * d;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * kThreads) {
    float sum = 0.f;
#pragma unroll 8
    for (int ch = 0; ch < chunks; ++ch) sum += part[ch * n + i];
    dWg[i] = sum;
  }
  if (dbias != nullptr && blockIdx.x == gridDim.x - 1)
    for (int e = threadIdx.x; e < E; e += kThreads) {
      float sum = 0.f;
#pragma unroll 8
      for (int ch = 0; ch < chunks; ++ch) sum += part_bias[ch * E + e];
      dbias[e] = sum;
    }
}

}  // namespace

hipError_t launch_gather_scale(const moe_config& c, const void* d_out, const int32_t* perm,
                               const int32_t* offsets, const float* gate_w, void* dY, int64_t max_rows,
                               hipStream_t s) {
  if (max_rows == 0 || c.T == 0) return hipSuccess;
  const int blocks = static_cast<int>(max_rows < 256 * 16 ? max_rows : 256 * 16);
  bf16_t* dy = static_cast<bf16_t*>(dY);
#define PPMOE_GS(DOUT, DT) \
  gather_scale_kernel<DOUT, DT><<<blocks, kThreads, 0, s>>>(d_out, perm, offsets, gate_w, dy, c.local_count, c.top_k, c.d)
  if (c.in_dtype == MOE_F16) {
    if (c.out_dtype == MOE_F32) PPMOE_GS(MOE_F32, MOE_F16);
    else PPMOE_GS(MOE_F16, MOE_F16);
  } else {
    if (c.out_dtype == MOE_F32) PPMOE_GS(MOE_F32, MOE_BF16);
    else PPMOE_GS(MOE_BF16, MOE_BF16);
  }
#undef PPMOE_GS
  return hipGetLastError();
}

hipError_t launch_gate_backward(const moe_config& c, const float* logits, const int32_t* expert_idx,
                                const float* gate_w, const int32_t* inv_perm, const float* row_dot,
                                float* dlogits, hipStream_t s) {
  if (c.T == 0) return hipSuccess;
  auto blocks_for = [&](int lpt) {
    const int64_t b = (static_cast<int64_t>(c.T) * lpt + kThreads - 1) / kThreads;
    return static_cast<unsigned>(b < (1 << 20) ? b : (1 << 20));
  };
#define PPMOE_GB(LPT)                                                                              \
  gate_backward_kernel<LPT><<<blocks_for(LPT), kThreads, 0, s>>>(                                  \
      logits, expert_idx, gate_w, inv_perm, row_dot, dlogits, c.T, c.E, c.top_k, c.renorm_topk)
  if (c.E <= 8) PPMOE_GB(8);
  else if (c.E <= 16) PPMOE_GB(16);
  else if (c.E <= 32) PPMOE_GB(32);
  else PPMOE_GB(64);
#undef PPMOE_GB
  return hipGetLastError();
}

hipError_t launch_dx(const moe_config& c, const void* dX_sliced, const int32_t* inv_perm,
                     const float* dlogits, const void* Wg, void* dx, hipStream_t s) {
  if (c.T == 0) return hipSuccess;
  // 32 tokens per wavefront halve the router rows' traffic from the L2; with few experts there is little of it
  // and twice the wavefronts are worth more.
  const int mt = c.E > 16 ? 2 : 1;
  const int64_t groups = (static_cast<int64_t>(c.T) + 16 * mt - 1) / (16 * mt);
  const unsigned col_blocks = static_cast<unsigned>((c.d + 511) / 512);
  const bf16_t* dxs = static_cast<const bf16_t*>(dX_sliced);
  const bf16_t* wg = static_cast<const bf16_t*>(Wg);
  bf16_t* out = static_cast<bf16_t*>(dx);
#define PPMOE_DX(DT, MT) \
  dx_kernel<DT, MT><<<dim3(static_cast<unsigned>(groups < (1 << 18) ? groups : (1 << 18)), col_blocks), kThreads, 0, s>>>(dxs, inv_perm, dlogits, wg, out, c.T, c.d, c.E, c.top_k)
  if (c.in_dtype == MOE_F16) {
    if (mt == 2) PPMOE_DX(MOE_F16, 2);
    else PPMOE_DX(MOE_F16, 1);
  } else {
    if (mt == 2) PPMOE_DX(MOE_BF16, 2);
    else PPMOE_DX(MOE_BF16, 1);
  }
#undef PPMOE_DX
  return hipGetLastError();
}

size_t dwg_scratch_bytes(const moe_config& c) {
  return static_cast<size_t>(dwg_chunks(c)) * c.E * (static_cast<size_t>(c.d) + 1) * sizeof(float) + 256;
}

hipError_t launch_dwg(const moe_config& c, const void* x, const float* dlogits, float* dWg, float* dbias,
                      void* scratch, hipStream_t s) {
  const int chunks = dwg_chunks(c);
  float* part = static_cast<float*>(scratch);
  float* part_bias = part + static_cast<size_t>(chunks) * c.E * c.d;
  const bf16_t* xs = static_cast<const bf16_t*>(x);
  const int et = c.E <= 16 ? 1 : c.E <= 32 ? 2 : 4;   // groups of 16 experts per block
  const dim3 grid((c.d + 127) / 128, chunks, (c.E + 16 * et - 1) / (16 * et));
#define PPMOE_DWG(DT, ET) dwg_partial_kernel<DT, ET><<<grid, kThreads, 0, s>>>(xs, dlogits, part, part_bias, c.T, c.d, c.E)
#define PPMOE_DWG_ET(DT)         \
  do {                           \
    if (et == 1) PPMOE_DWG(DT, 1); \
    else if (et == 2) PPMOE_DWG(DT, 2); \
    else PPMOE_DWG(DT, 4);       \
  } while (0)
  if (c.in_dtype == MOE_F16) PPMOE_DWG_ET(MOE_F16);
  else PPMOE_DWG_ET(MOE_BF16);
#undef PPMOE_DWG_ET
#undef PPMOE_DWG
  const int64_t n = static_cast<int64_t>(c.E) * c.d;
  const int blocks = static_cast<int>((n + kThreads - 1) / kThreads < 1024 ? (n + kThreads - 1) / kThreads : 1024);
  dwg_final_kernel<<<blocks, kThreads, 0, s>>>(part, part_bias, dWg, dbias, c.d, c.E, chunks);
  return hipGetLastError();
}

}  // namespace ppmoe
