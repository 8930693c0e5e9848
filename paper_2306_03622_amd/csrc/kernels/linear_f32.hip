// fp32 linear layer y = act(x W^T + b), in full fp32 throughout (products and sums; no
// reduced-precision matrix path). Few rows of x: one wave per output feature n on the vector
// ALUs, lanes striding over k in float4 steps, each lane accumulating its own partial sum in
// order, then a fixed butterfly reduction; rows of x are processed one after another by the
// same wave. More rows: 16 x 16 tiles on the fp32 matrix instructions, the waves of a workgroup
// splitting k.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"
#include "swapin.hpp"

namespace tp {
namespace k {
namespace {

__global__ __launch_bounds__(256) void k_linear_f32(const float* __restrict__ x, int M, int K,
                                                    const float* __restrict__ w, int N,
                                                    const float* __restrict__ bias, int act,
                                                    float* __restrict__ y) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const float* wr = w + (size_t)n * K;
  for (int m = 0; m < M; ++m) {
    const float* xr = x + (size_t)m * K;
    float s = 0.f;
    for (int k = lane * 4; k < K; k += 256) {
      const float4 a = *reinterpret_cast<const float4*>(wr + k);
      const float4 b = *reinterpret_cast<const float4*>(xr + k);
      s = fmaf(a.x, b.x, s);
      s = fmaf(a.y, b.y, s);
      s = fmaf(a.z, b.z, s);
      s = fmaf(a.w, b.w, s);
    }
    s = wave_sum(s);
    if (lane == 0) y[(size_t)m * N + n] = act_apply(s + (bias ? bias[n] : 0.f), act);
  }
}

// y[m][n] for 16 features n by 16 MT rows m per workgroup. Its 8 waves split k into contiguous
// runs of 16-deep chunks; lane (r, q) loads 4 consecutive k of row r at chunk offset 4 q from W
// and from each 16 rows of x, and the i-th elements feed the i-th of four matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums, denormals kept), each with an accumulator
// of its own, even and odd chunks apart. A sum over k is thus split 64 ways (8 waves x 8
// accumulators) and joined pairwise, as the 64 lanes' sums of the kernel above are, so that its
// rounding error is no larger (with 4 accumulators it was: 8.6e-8 against 7.3e-8 for 1000 wide).
// Bound by memory round trips (W and x are read from the caches in 16-row runs of 64 bytes), not by the matrix
// cores. The kernel above re-reads a row of W per row of x in a serial chain: 47 us for 64 x
// 1000 x 1000 with the weights in the caches, this one 5.3 us; 1024 wide, 5 rows 5.2 against
// 4.8 us.
// SWAP: W lies in pinned host memory and is written to w_dev as it is read (see below).
// STAGE: W lies in pinned host memory: a wave's next 8 chunks of the 16 rows are read as runs of 512 bytes, 8 loads in
// flight, and turned into operands through LDS (in the runs of 64 bytes above the host link carried less: 2 x 1000 of 9
// rows 215 us, 184 so, 2 x 2000 of 12 787 and 659). The same sums, so the same bits.
constexpr int kMmWaves = 8;

template <int MT, int U, bool SWAP, bool STAGE>
__device__ __forceinline__ void linear_f32_tile(const float* __restrict__ x, int M, int K, const float* __restrict__ w,
                                                int N, const float* __restrict__ bias, int act,
                                                float* __restrict__ y, float* __restrict__ w_dev, int n0, int m0) {
  __shared__ f32x4 red[kMmWaves][MT][64];
  __shared__ __align__(16) float wst[STAGE ? kMmWaves : 1][STAGE ? 16 : 1][8 * 16 + 4];
  static_assert(!STAGE || 8 % U == 0, "whole rounds of a stage");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const bool nvalid = n0 + r < N;
  const float* wr = w + (size_t)(nvalid ? n0 + r : N - 1) * K;
  const float* xr[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) xr[t] = x + (size_t)min(m0 + 16 * t + r, M - 1) * K;   // rows beyond M: discarded
  static_assert(U % 2 == 0, "chunks in pairs");
  f32x4 acc[8][MT];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nc = (K + 15) >> 4, per = (nc + kMmWaves - 1) / kMmWaves;
  const int c_end = min(nc, (wave + 1) * per);
  for (int c0 = wave * per; c0 < c_end; c0 += U) {
    float4 a[U], b[U][MT];
    const int at = (c0 - wave * per) & 7;        // chunk of the stage
    if (STAGE && at == 0) {
      float4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = 2 * i + (lane >> 5), k = c0 * 16 + (lane & 31) * 4;
        const bool in = k < min(c_end * 16, K);
        v[i] = *reinterpret_cast<const float4*>(w + (size_t)min(n0 + row, N - 1) * K + (in ? k : 0));
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        *reinterpret_cast<float4*>(&wst[wave][2 * i + (lane >> 5)][(lane & 31) * 4]) = v[i];
      __builtin_amdgcn_wave_barrier();           // a wave's LDS operations take effect in order
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u) * 16 + q * 4;
      const bool in = c0 + u < c_end && k < K;
      const int kk = in ? k : 0;
      a[u] = *reinterpret_cast<const float4*>(STAGE ? &wst[wave][r][(at + u) * 16 + q * 4] : wr + kk);
      if (SWAP && in && nvalid) *reinterpret_cast<float4*>(w_dev + (size_t)(n0 + r) * K + kk) = a[u];
#pragma unroll
      for (int t = 0; t < MT; ++t) b[u][t] = *reinterpret_cast<const float4*>(xr[t] + kk);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (both operands zeroed beyond K: the value loaded in their place may be an infinity)
      const bool in = c0 + u < c_end && (c0 + u) * 16 + q * 4 < K;
      const float av[4] = {in ? a[u].x : 0.f, in ? a[u].y : 0.f, in ? a[u].z : 0.f, in ? a[u].w : 0.f};
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const float bv[4] = {in ? b[u][t].x : 0.f, in ? b[u][t].y : 0.f, in ? b[u][t].z : 0.f, in ? b[u][t].w : 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f32x4& c = acc[4 * (u & 1) + i][t];
          c = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[i], c, 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) 
    red[wave][t][lane] = ((acc[0][t] + acc[1][t]) + (acc[2][t] + acc[3][t])) +
                         ((acc[4][t] + acc[5][t]) + (acc[6][t] + acc[7][t]));
  __syncthreads();
  if (wave >= MT) return;
  f32x4 s[kMmWaves];
#pragma unroll
  for (int v = 0; v < kMmWaves; ++v) s[v] = red[v][wave][lane];
#pragma unroll
  for (int h = kMmWaves / 2; h > 0; h /= 2)
#pragma unroll
    for (int v = 0; v < h; ++v) s[v] = s[2 * v] + s[2 * v + 1];
  // lane holds D[n = n0 + 4 q + e][m = m0 + 16 wave + r]
  const int m = m0 + 16 * wave + r, n = n0 + 4 * q;
  if (m >= M) return;
  float* yr = y + (size_t)m * N + n;
  // whole vectors where the caller's output starts at a 16-byte boundary (rows of N % 4 == 0 floats then all do)
  if (n + 3 < N && (N & 3) == 0 && ((uintptr_t)y & 15) == 0) {
    const float4 bb = bias ? *reinterpret_cast<const float4*>(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
    *reinterpret_cast<float4*>(yr) = make_float4(act_apply(s[0][0] + bb.x, act), act_apply(s[0][1] + bb.y, act),
                                                 act_apply(s[0][2] + bb.z, act), act_apply(s[0][3] + bb.w, act));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < N) yr[e] = act_apply(s[0][e] + (bias ? bias[n + e] : 0.f), act);
  }
}

constexpr int kMmU = 2;      // chunks in flight per wave from device memory (4 and 8 measured slower)

constexpr int kMmY = 65536;  // the most row blocks a grid's y takes

// Z: the row blocks continue in the grid's z (always, it cost 4 x 1000 at batch 64 28.0 -> 28.6 us). STAGE:
// weights in host memory.
template <int MT, bool Z = false, bool STAGE = false>
__global__ __launch_bounds__(64 * kMmWaves) void k_linear_f32_mm(const float* __restrict__ x, int M, int K,
                                                                 const float* __restrict__ w, int N,
                                                                 const float* __restrict__ bias, int act,
                                                                 float* __restrict__ y) {
  if constexpr (Z) {
    const long m0 = ((long)blockIdx.z * kMmY + blockIdx.y) * 16 * MT;
    if (m0 >= M) return;
    linear_f32_tile<MT, kMmU, false, STAGE>(x, M, K, w, N, bias, act, y, nullptr, blockIdx.x * 16, (int)m0);
  } else {
    linear_f32_tile<MT, kMmU, false, STAGE>(x, M, K, w, N, bias, act, y, nullptr, blockIdx.x * 16, blockIdx.y * 16 * MT);
  }
}

// Rows of x from which the matrix kernel is the faster one at every width (us per launch, 64 / 256 /
// 1024 / 2000 wide): 5 rows 2.4 / 2.8 / 4.8 / 6.2 against 3.4 / 3.4 / 5.2 / 8.1; 4 rows 2.5 / 2.9 / 4.8 / 6.6
// against 3.0 / 3.1 / 4.5 / 6.9.
constexpr int kMmRows = 5;

// The first layer of an fp32 model whose weights are still in pinned host memory, fused with
// the model's swap-in. Workgroups [0, cwg) compute y = act(x W^T + b): up to kMmRows - 1 rows like
// k_linear_f32, one wave per output feature with its row of W held in registers for every row of
// x, from kMmRows on (MM) as 16 x 16 tiles like k_linear_f32_mm, in either case by the same sequence of operations.
// They read W from the host copy once and write what they read to the device copy; the other workgroups copy every 16-byte vector of
// the image outside W's own [skip0, skip1) host -> device, each thread issuing all its loads
// before its first store. All host reads of the model are thus in flight together.
constexpr int kSwapMaxM = 8, kSwapMaxKV = 4;     // rows of x; float4 per lane and row of W (K <= 1024)
constexpr int kSwapU = 4;                        // 16-byte vectors per gather thread and round

// MM (kMmRows rows and more): workgroups of 512 threads, the first cwg of them 16 x 16 tiles of
// the matrix kernel (the same operations as k_linear_f32_mm's, so the same bits).
template <bool MM>
__global__ __launch_bounds__(MM ? 64 * kMmWaves : 256) void k_linear_f32_swap(const float* __restrict__ x, int M, int K,
                                                         const float* __restrict__ w_host, int N,
                                                         const float* __restrict__ bias_host, int act,
                                                         float* __restrict__ y, float* __restrict__ w_dev,
                                                         const uint4* __restrict__ img_host,
                                                         uint4* __restrict__ img_dev, uint64_t n16, uint64_t skip0,
                                                         uint64_t skip1, int cwg) {
  constexpr int NT = MM ? 64 * kMmWaves : 256;
  if ((int)blockIdx.x < cwg) {
    if constexpr (MM) {
      // all of a row's chunks in flight (K <= 1024): the round trip over the host link is what counts
      linear_f32_tile<1, 8, true, false>(x, M, K, w_host, N, bias_host, act, y, w_dev, blockIdx.x * 16, 0);
      return;
    }
    const int lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    const float* wr = w_host + (size_t)n * K;
    float4 a[kSwapMaxKV];
#pragma unroll
    for (int i = 0; i < kSwapMaxKV; ++i) {
      const int k = lane * 4 + 256 * i;
      if (k < K) a[i] = *reinterpret_cast<const float4*>(wr + k);
    }
#pragma unroll
    for (int i = 0; i < kSwapMaxKV; ++i) {
      const int k = lane * 4 + 256 * i;
      if (k < K) *reinterpret_cast<float4*>(w_dev + (size_t)n * K + k) = a[i];
    }
    const float b = bias_host ? bias_host[n] : 0.f;
    for (int m = 0; m < M; ++m) {
      const float* xr = x + (size_t)m * K;
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < kSwapMaxKV; ++i) {
        const int k = lane * 4 + 256 * i;
        if (k < K) {
          const float4 v = *reinterpret_cast<const float4*>(xr + k);
          s = fmaf(a[i].x, v.x, s);
          s = fmaf(a[i].y, v.y, s);
          s = fmaf(a[i].z, v.z, s);
          s = fmaf(a[i].w, v.w, s);
        }
      }
      s = wave_sum(s);
      if (lane == 0) y[(size_t)m * N + n] = act_apply(s + b, act);
    }
    return;
  }
  // gather: vectors [0, skip0) and [skip1, n16) as one index space of n16 - (skip1 - skip0)
  const uint64_t total = n16 - (skip1 - skip0);
  const uint64_t stride = (uint64_t)(gridDim.x - cwg) * NT;
  for (uint64_t i0 = (uint64_t)(blockIdx.x - cwg) * NT + threadIdx.x; i0 < total; i0 += kSwapU * stride) {
    uint4 v[kSwapU];
#pragma unroll
    for (int u = 0; u < kSwapU; ++u) {
      const uint64_t i = i0 + u * stride;
      const uint64_t j = i < skip0 ? i : i + (skip1 - skip0);
      if (i < total) v[u] = img_host[j];
    }
#pragma unroll
    for (int u = 0; u < kSwapU; ++u) {
      const uint64_t i = i0 + u * stride;
      const uint64_t j = i < skip0 ? i : i + (skip1 - skip0);
      if (i < total) img_dev[j] = v[u];
    }
  }
}

}  // namespace

hipError_t linear_f32_swap(const float* x, int M, int K, int N, int act, float* y, const void* img_host,
                           void* img_dev, uint64_t img_bytes, uint64_t w_off, uint64_t b_off, hipStream_t s) {
  const uint64_t w_bytes = (uint64_t)N * K * 4;
  if (!x || !y || !img_host || !img_dev || M < 1 || M > kSwapMaxM || N < 1 || K < 4 || (K & 3) ||
      K > 256 * kSwapMaxKV || act < 0 || act > 2 || (img_bytes & 15) || (w_off & 15) ||
      w_off + w_bytes > img_bytes || b_off + (uint64_t)N * 4 > img_bytes || (b_off & 3) ||
      ((uintptr_t)img_host & 15) || ((uintptr_t)img_dev & 15))
    return hipErrorInvalidValue;
  const bool mm = M >= kMmRows;
  const int cwg = mm ? (N + 15) / 16 : (N + 3) / 4, nt = mm ? 64 * kMmWaves : 256;
  const uint64_t n16 = img_bytes / 16, skip0 = w_off / 16, skip1 = (w_off + w_bytes + 15) / 16;
  const uint64_t rest = n16 - (skip1 - skip0);
  // every gather thread issues kSwapU loads per round: enough workgroups for one round
  const int gwg = (int)std::min<uint64_t>(1024, std::max<uint64_t>(1, (rest + nt * kSwapU - 1) / (nt * kSwapU)));
  const char* h = static_cast<const char*>(img_host);
  char* d = static_cast<char*>(img_dev);
  auto go = [&](auto kern) {
    (void)launch(kern, dim3(cwg + gwg), dim3(nt), 0, s, x, M, K, reinterpret_cast<const float*>(h + w_off), N,
                 reinterpret_cast<const float*>(h + b_off), act, y, reinterpret_cast<float*>(d + w_off),
                 static_cast<const uint4*>(img_host), static_cast<uint4*>(img_dev), n16, skip0, skip1, cwg);
  };
  if (mm) go(k_linear_f32_swap<true>);
  else go(k_linear_f32_swap<false>);
  return hipGetLastError();
}

hipError_t linear_f32(const float* x, int M, int K, const float* w, int N, const float* bias, int act, float* y,
                      bool w_far, hipStream_t s) {
  if (!x || !w || !y || M < 1 || N < 1 || K < 4 || (K & 3) || act < 0 || act > 2) return hipErrorInvalidValue;
  if (M < kMmRows) {
    (void)launch(k_linear_f32, dim3((N + 3) / 4), dim3(256), 0, s, x, M, K, w, N, bias, act, y);
    return hipGetLastError();
  }
  // Rows per workgroup by how many 16 x 16 tiles there are (us per launch with 16 / 32 / 64 rows, 1000
  // wide): 64 rows [252 tiles] 5.3 / 6.5 / 11.1, 128 [504] 9.2 / 7.2 / 11.2, 256 [1008] 15.3 / 12.6 / 11.8; 512
  // wide, 256 rows [512] 5.9 / 5.2 / 7.4.
  const long nt = (N + 15) / 16, tiles = nt * (((long)M + 15) / 16);
  auto go = [&](auto kern, int rows) {
    const long blocks = ((long)M + rows - 1) / rows;
    // Weights in host memory: as few row blocks as there may be, and a multiple of the 8 XCDs in x (tiles beyond N
    // store nothing), which puts all row blocks of a feature tile on one XCD, so that they share one read of its weights
    // over the link (2 x 1000 read in place, 64 rows 762 us without, 196 so, 256 rows 779 and 196).
    const bool pad = w_far && blocks > 1;
    const dim3 grid((unsigned)(pad ? (nt + 7) / 8 * 8 : nt), (unsigned)std::min<long>(blocks, kMmY),
                    (unsigned)((blocks + kMmY - 1) / kMmY));
    (void)launch(kern, grid, dim3(64 * kMmWaves), 0, s, x, M, K, w, N, bias, act, y);
  };
  if (w_far && M <= 16) go((k_linear_f32_mm<1, false, true>), 16);
  else if (w_far && M <= 32) go((k_linear_f32_mm<2, false, true>), 32);
  else if (w_far && M <= 64L * kMmY) go((k_linear_f32_mm<4, false, true>), 64);
  else if (tiles <= 384 || M <= 16) go(k_linear_f32_mm<1>, 16);
  else if (tiles <= 768 || M <= 32) go(k_linear_f32_mm<2>, 32);
  else if (M <= 64L * kMmY) go(k_linear_f32_mm<4>, 64);
  else go((k_linear_f32_mm<4, true>), 64);
  return hipGetLastError();
}

}  // namespace k
}  // namespace tp
