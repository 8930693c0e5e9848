// Argument block and row epilogue shared by the bf16 contraction kernels (skinny and
// tiled), and the launcher of the skinny one.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace tp {
namespace k {

// activation loaders: row-major matrix; NHWC im2col with C % 64 == 0 (a 64-deep k-stage
// then lies inside one filter tap)
enum { X_ROWS = 0, X_CONV64 = 3 };

struct GemmArgs {
  const uint16_t* x;
  const uint16_t* w;
  int M, N, K;
  int H, W, C, KW, stride, pad, Ho, Wo;   // convolution geometry (X_CONV*)
  Epilogue ep;
  int kst, splits;                        // k-stages per split, number of splits
  float* partials;                        // [splits][M][N] fp32 when splits > 1
};

template <>
struct PtrFields<GemmArgs> {
  static void add(std::vector<uint32_t>& v, uint32_t at) {
    for (size_t o : {offsetof(GemmArgs, x), offsetof(GemmArgs, w), offsetof(GemmArgs, partials),
                     offsetof(GemmArgs, ep) + offsetof(Epilogue, bias), offsetof(GemmArgs, ep) + offsetof(Epilogue, res),
                     offsetof(GemmArgs, ep) + offsetof(Epilogue, out), offsetof(GemmArgs, ep) + offsetof(Epilogue, ln_g),
                     offsetof(GemmArgs, ep) + offsetof(Epilogue, ln_b), offsetof(GemmArgs, ep) + offsetof(Epilogue, ln_out)})
      v.push_back(at + (uint32_t)o);
  }
};

// The epilogue's inputs for a run of R (4 or 8) consecutive outputs of a row, as raw bits:
// fetched ahead of the values they apply to, so that their loads overlap other loads. `base` is
// m * N + n0; requires n0 % R == 0, n0 + R - 1 < N, N % R == 0.
template <int R>
struct EpRun;
template <>
struct EpRun<4> {
  typedef uint2 Raw;
  Raw bias, res;
};
template <>
struct EpRun<8> {
  typedef uint4 Raw;
  Raw bias, res;
};
typedef EpRun<4> Ep4In;

// RES, when not -1, fixes at compile time whether there is a residual: a kernel that fetches
// these ahead of other loads then has no branch between the loads, which would otherwise make
// the compiler wait for one before issuing the next.
inline int res_kind(const Epilogue& ep) { return ep.res ? 1 : 0; }

template <int RES = -1>
__device__ __forceinline__ Ep4In ep4_fetch(const Epilogue& ep, size_t base, int n0) {
  Ep4In in;   // fields the epilogue does not use stay unset (no copies, no waits)
  if (ep.bias) in.bias = *reinterpret_cast<const uint2*>(ep.bias + n0);
  if (RES >= 0 ? RES == 1 : ep.res != nullptr)
    in.res = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(ep.res) + base);
  return in;
}

__device__ __forceinline__ void add_bf16(float (&v)[4], uint2 w) {
  v[0] += bf2f(w.x & 0xffff); v[1] += bf2f(w.x >> 16); v[2] += bf2f(w.y & 0xffff); v[3] += bf2f(w.y >> 16);
}
__device__ __forceinline__ void add_bf16(float (&v)[8], uint4 w) {
  v[0] += bf2f(w.x & 0xffff); v[1] += bf2f(w.x >> 16); v[2] += bf2f(w.y & 0xffff); v[3] += bf2f(w.y >> 16);
  v[4] += bf2f(w.z & 0xffff); v[5] += bf2f(w.z >> 16); v[6] += bf2f(w.w & 0xffff); v[7] += bf2f(w.w >> 16);
}

// v += bias; v += residual; v = act(v), each step only where the epilogue has it
template <int RES = -1, int R>
__device__ __forceinline__ void ep_apply(const Epilogue& ep, const EpRun<R>& in, float (&v)[R]) {
  if (ep.bias) add_bf16(v, in.bias);
  if (RES >= 0 ? RES == 1 : ep.res != nullptr) add_bf16(v, in.res);
#pragma unroll
  for (int e = 0; e < R; ++e) v[e] = act_apply(v[e], ep.act);
}

template <int R>
__device__ __forceinline__ void ep_store(const Epilogue& ep, size_t base, const float (&v)[R]) {
  if (ep.out_f32) {
#pragma unroll
    for (int e = 0; e < R; e += 4)
      *reinterpret_cast<float4*>(static_cast<float*>(ep.out) + base + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
  } else if constexpr (R == 8) {
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(ep.out) + base) =
        make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
  } else {
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(ep.out) + base) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
  }
}

__device__ __forceinline__ void store_row4(const GemmArgs& a, int m, int n0, f32x4 acc) {
  if (m >= a.M || n0 >= a.N) return;
  const Epilogue& ep = a.ep;
  const size_t base = (size_t)m * a.N + n0;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = acc[e];
  const bool full = (n0 + 3 < a.N) && ((a.N & 3) == 0);
  if (full) {
    const Ep4In in = ep4_fetch(ep, base, n0);
    ep_apply(ep, in, v);
    ep_store(ep, base, v);
    return;
  }
  for (int e = 0; e < 4 && n0 + e < a.N; ++e) {
    float t = v[e];
    if (ep.bias) t += bf2f(ep.bias[n0 + e]);
    if (ep.res) t += bf2f(static_cast<const uint16_t*>(ep.res)[base + e]);
    t = act_apply(t, ep.act);
    if (ep.out_f32) static_cast<float*>(ep.out)[base + e] = t;
    else static_cast<uint16_t*>(ep.out)[base + e] = f2bf(t);
  }
}

// The reduction of a split contraction fused with the row LayerNorm of its result
// (norm.hip); split_reduce_ln_fits tells whether it applies to width N.
// split_group(s): how many split partials a reduction thread loads before it adds any
// (2, 4 or 8: the smallest that covers s, at most 8).
__host__ __device__ constexpr int split_group(int s) { return s <= 2 ? 2 : s <= 4 ? 4 : 8; }
bool split_reduce_ln_fits(int N);
hipError_t split_reduce_ln(const GemmArgs& a, hipStream_t s);

// M <= 32 rows: the skinny kernel (gemv_bf16.hip)
hipError_t launch_skinny(const GemmArgs& a, hipStream_t s);

}  // namespace k
}  // namespace tp
