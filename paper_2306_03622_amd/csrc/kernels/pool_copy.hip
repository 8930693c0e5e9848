// Average pooling (NHWC bf16), the host-to-device gather copy, the copy of an unaligned input, the
// cache touch and the bounded delay kernel.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"
#include "touch.hpp"

namespace tp {
namespace k {
namespace {

// one thread per (sample, channel), positions summed in order in fp32
// One thread per (sample, channel). The HW loads are independent, so they are issued 8 at
// a time into 8 partial sums, which are then added in a fixed order.
__global__ __launch_bounds__(64) void k_avgpool(const uint16_t* __restrict__ x, int B, int HW, int C,
                                                uint16_t* __restrict__ y) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= B * C) return;
  const int b = i / C, c = i - b * C;
  const uint16_t* p = x + (size_t)b * HW * C + c;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int j = 0;
  for (; j + 8 <= HW; j += 8) {
    uint16_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(j + u) * C];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += bf2f(v[u]);
  }
  for (; j < HW; ++j) s[0] += bf2f(p[(size_t)j * C]);
  float t = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) t += s[u];
  y[i] = f2bf(t / (float)HW);
}

// grid-stride copy with U independent 16-byte loads in flight per thread
__global__ __launch_bounds__(256) void k_gather(const uint4* __restrict__ src, uint4* __restrict__ dst, uint64_t n) {
  constexpr int U = 8;
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  for (; i + (U - 1) * stride < n; i += U * stride) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = src[i + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) dst[i + u * stride] = v[u];
  }
  for (; i < n; i += stride) dst[i] = src[i];
}

// Eight bf16 values per thread, loaded one by one (the source starts at any element), stored as one
// vector.
__global__ __launch_bounds__(256) void k_copy_aligned(const uint16_t* __restrict__ src, uint4* __restrict__ dst,
                                                      uint64_t n8) {
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += stride) {
    uint32_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[8 * i + e];
    dst[i] = make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
  }
}

// Loads in flight per thread, workgroups per touch (one per CU). Measured on MI355X, warm
// ResNet-50 / BERT-base requests at batch 1 after a cache flush, with every warm request
// touching: 397 / 534 us untouched; 376 / 528 with 32 workgroups, 373 / 508 with 64, 371 / 498
// with 128, 365 / 501 with 256, 377 / 515 with 2048 of 4 loads each. Back to back (the caches
// already warm) a touch costs BERT-base 8-12 us beside its own kernels (none for ResNet-50),
// so by default only a request that follows another model's touches.
constexpr int kTouchLoads = 8, kTouchWGs = 256;

// Reads n 16-byte vectors (grid-stride, U loads in flight per thread) with ordinary,
// cache-allocating loads and discards them: the bytes end up in the Infinity Cache (and the
// L2s), so that kernels reading them shortly after find them there. Nothing is stored unless
// the XOR of everything a thread read equals `magic`, which the caller makes impossible to
// rely on (the store only keeps the compiler from dropping the loads).
__global__ __launch_bounds__(256) void k_touch(const uint4* __restrict__ p, uint64_t n, uint32_t magic,
                                               uint32_t* __restrict__ sink) {
  constexpr int U = kTouchLoads;
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  uint32_t x = 0;
  for (; i + (U - 1) * stride < n; i += U * stride) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[i + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) x ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n; i += stride) {
    const uint4 v = p[i];
    x ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (x == magic) sink[blockIdx.x & 63] = x;
}

__global__ void k_delay(int iters) {
  for (int i = 0; i < iters; ++i) __builtin_amdgcn_s_sleep(127);
}

}  // namespace

hipError_t avgpool(const uint16_t* x, int B, int HW, int C, uint16_t* y, hipStream_t s) {
  if (!x || !y || B < 1 || HW < 1 || C < 1) return hipErrorInvalidValue;
  (void)launch(k_avgpool, dim3((B * C + 63) / 64), dim3(64), 0, s, x, B, HW, C, y);
  return hipGetLastError();
}

hipError_t copy_aligned(const uint16_t* src, uint64_t n, uint16_t* dst, hipStream_t s) {
  if (!src || !dst || n < 8 || (n & 7) || ((uintptr_t)dst & 15)) return hipErrorInvalidValue;
  const uint64_t wgs = std::min<uint64_t>((n / 8 + 255) / 256, 4096);
  (void)launch(k_copy_aligned, dim3((unsigned)wgs), dim3(256), 0, s, src, reinterpret_cast<uint4*>(dst), n / 8);
  return hipGetLastError();
}

hipError_t gather_copy(const void* src, void* dst, uint64_t bytes, int wgs, hipStream_t s) {
  if (!src || !dst || (bytes & 15) || wgs < 1 || ((uintptr_t)src & 15) || ((uintptr_t)dst & 15))
    return hipErrorInvalidValue;
  if (bytes == 0) return hipSuccess;
  (void)launch(k_gather, dim3(wgs), dim3(256), 0, s, static_cast<const uint4*>(src), static_cast<uint4*>(dst),
                     bytes >> 4);
  return hipGetLastError();
}

hipError_t touch(const void* p, uint64_t bytes, uint32_t* sink, hipStream_t s) {
  if (!p || !sink || (bytes & 15) || ((uintptr_t)p & 15)) return hipErrorInvalidValue;
  if (bytes == 0) return hipSuccess;
  const uint64_t n = bytes >> 4, per_wg = 256 * kTouchLoads;
  const unsigned wgs = (unsigned)std::min<uint64_t>(kTouchWGs, (n + per_wg - 1) / per_wg);
  (void)launch(k_touch, dim3(wgs), dim3(256), 0, s, static_cast<const uint4*>(p), n, 0x9e3779b9u, sink);
  return hipGetLastError();
}

hipError_t delay(int us, hipStream_t s) {
  // s_sleep 127 is about 127 * 64 cycles, ~3.4 us at 2.4 GHz
  const int iters = us <= 3 ? 1 : us / 3;
  (void)launch(k_delay, dim3(1), dim3(64), 0, s, iters);
  return hipGetLastError();
}

}  // namespace k
}  // namespace tp
