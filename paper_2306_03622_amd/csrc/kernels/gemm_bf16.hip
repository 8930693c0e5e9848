// bf16 contractions on gfx950 MFMA (v_mfma_f32_16x16x32_bf16), fp32 accumulate, with a
// fused epilogue (bias, optional residual, ReLU/GELU, bf16 or fp32 store).
//
// Convention for every kernel here: the MFMA "A" operand is a 16-row block of the weight
// matrix W[N][K] (rows = output features n) and the "B" operand a 16-row block of the
// activations X[M][K] (rows = tokens / output pixels m). Both are read as 8 consecutive
// k per lane, lane l covering row (l % 16) and k-slot (l / 16), so one accumulator
// register e of lane l holds D[n = 4 (l / 16) + e][m = l % 16]: four consecutive output
// features of one row, which the epilogue stores as one vector.
//
// Kernels here (the skinny M <= 32 case is in gemv_bf16.hip, the 3-channel stem in stem.hip):
//   * k_gemm (gemm_tile.hpp): BN x BM output tiles over a ring of 64-deep k-stages in LDS that
//     loads fill directly, and a deterministic split over k when a deep contraction's tiles
//     cannot fill the chip. The activation loader is either a plain row-major matrix or an
//     NHWC implicit-GEMM (im2col) gather for convolutions, k = (kh * KW + kw) * C + c, matching
//     OHWI weight rows.
#include <algorithm>

#include "gemm_tile.hpp"

namespace tp {
namespace k {

namespace {

// y = epilogue(sum over splits z = 0, 1, ... of P[z]) for four consecutive outputs per thread (N % 8 == 0: other
// widths are not split). A thread fetches the epilogue's inputs and ZG partials before it adds any (a launch that
// waited for each partial in turn spent ~5 us on a few MB: one memory round trip per split);
// the additions keep split order, so results are the same as summing one split at a time.
template <int ZG, int RES>
__global__ __launch_bounds__(256) void k_split_reduce(GemmArgs a) {
  const long q = (long)blockIdx.x * 256 + threadIdx.x;       // index of a group of 4 outputs
  const int groups_per_row = a.N >> 2;
  if (q >= (long)a.M * groups_per_row) return;
  const int m = (int)(q / groups_per_row), n0 = (int)(q - (long)m * groups_per_row) * 4;
  const size_t plane = (size_t)a.M * a.N, base = (size_t)m * a.N + n0;
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  const Ep4In in = ep4_fetch<RES>(a.ep, base, n0);
  for (int z0 = 0; z0 < a.splits; z0 += ZG) {
    float4 t[ZG];
#pragma unroll
    for (int u = 0; u < ZG; ++u)
      if (z0 + u < a.splits) t[u] = *reinterpret_cast<const float4*>(a.partials + (z0 + u) * plane + base);
#pragma unroll
    for (int u = 0; u < ZG; ++u)
      if (z0 + u < a.splits) sum += f32x4{t[u].x, t[u].y, t[u].z, t[u].w};
  }
  float v[4] = {sum[0], sum[1], sum[2], sum[3]};
  ep_apply<RES>(a.ep, in, v);
  ep_store(a.ep, base, v);
}

template <int RES>
void launch_split_reduce_res(const GemmArgs& a, dim3 grid, dim3 block, hipStream_t s) {
  switch (split_group(a.splits)) {
    case 2: (void)launch((k_split_reduce<2, RES>), grid, block, 0, s, a); break;
    case 4: (void)launch((k_split_reduce<4, RES>), grid, block, 0, s, a); break;
    default: (void)launch((k_split_reduce<8, RES>), grid, block, 0, s, a); break;
  }
}

void launch_split_reduce(const GemmArgs& a, dim3 grid, dim3 block, hipStream_t s) {
  switch (res_kind(a.ep)) {
    case 0: launch_split_reduce_res<0>(a, grid, block, s); break;
    default: launch_split_reduce_res<1>(a, grid, block, s); break;
  }
}

// After the contraction: the reduction of a k split (fused with the epilogue's row
// LayerNorm when the width allows), then the LayerNorm of an fp32 result if one is asked for
// and not yet done.
hipError_t finish(const GemmArgs& a, hipStream_t s) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.splits > 1) {
    if (a.ep.ln_g && split_reduce_ln_fits(a.N)) return split_reduce_ln(a, s);
    const long groups = (long)a.M * (a.N / 4);
    const dim3 grid((unsigned)((groups + 255) / 256)), block(256);
    launch_split_reduce(a, grid, block, s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (a.ep.ln_g)
    return layernorm(static_cast<const float*>(a.ep.out), a.M, a.N, a.ep.ln_g, a.ep.ln_b, a.ep.ln_eps, a.ep.ln_out,
                     a.ep.ln_out_f32, s);
  return hipSuccess;
}

template <int BN, int BM, int WGN, int WGM, int NST, int MINW, int MODE, bool VEC = true>
hipError_t launch_tiled(GemmArgs a, int splits, const Split& sp, hipStream_t s) {
  if (!VEC && splits > 1) return hipErrorInvalidValue;       // partials are whole vectors
  const int tn = (a.N + BN - 1) / BN, tm = (a.M + BM - 1) / BM, nst = (a.K + 63) / 64;
  a.kst = (nst + splits - 1) / splits;
  a.splits = (nst + a.kst - 1) / a.kst;        // no empty split
  a.partials = sp.partials;
  const dim3 grid(tn * tm * a.splits), block(64 * WGN * WGM);
  auto go = [&](auto kern) { (void)launch(kern, grid, block, 0, s, a, tn, tm); };
  const bool far = a.ep.w_far;
  if constexpr (MODE == X_ROWS && VEC) {
    if (a.ep.w_packed) {
      far ? go(k_gemm<BN, BM, WGN, WGM, NST, MODE, true, MINW, true, true>)
          : go(k_gemm<BN, BM, WGN, WGM, NST, MODE, true, MINW, true, false>);
      return finish(a, s);
    }
  }
  far ? go(k_gemm<BN, BM, WGN, WGM, NST, MODE, false, MINW, VEC, true>)
      : go(k_gemm<BN, BM, WGN, WGM, NST, MODE, false, MINW, VEC, false>);
  return finish(a, s);
}

template <int MODE>
hipError_t pick_tiled(const GemmArgs& a, const Split& sp, hipStream_t s) {
  const TileShape shape{a.M, a.N, a.K, MODE == X_CONV64, a.ep.act == ACT_GELU, a.ep.ln_g != nullptr,
                        a.ep.w_far != 0};
  const TilePlan p = plan_tiles(shape, sp.partials ? sp.partial_bytes : 0);
  // waves n x m, ring, least waves per SIMD
  if (p.bn == 256 && p.bm == 256) return launch_tiled<256, 256, 4, 2, 2, 1, MODE>(a, p.splits, sp, s);
  if (p.bn == 256) return launch_tiled<256, 128, 4, 2, 3, 1, MODE>(a, p.splits, sp, s);
  if (p.bn == 128 && p.ring == 2) return launch_tiled<128, 128, 4, 2, 2, 4, MODE>(a, p.splits, sp, s);
  if (p.bn == 128) return launch_tiled<128, 128, 4, 2, 3, 2, MODE>(a, p.splits, sp, s);
  if (p.bm == 64 && p.ring == 2) return launch_tiled<64, 64, 2, 2, 2, 4, MODE>(a, p.splits, sp, s);
  if (p.bm == 64) return launch_tiled<64, 64, 2, 2, 4, 2, MODE>(a, p.splits, sp, s);
  if (p.bn == 64) return launch_tiled<64, 32, 2, 2, 5, 2, MODE>(a, p.splits, sp, s);
  if (a.N % 8) return launch_tiled<32, 32, 2, 2, 4, 4, MODE, false>(a, p.splits, sp, s);
  if (p.ring == 4) return launch_tiled<32, 32, 2, 2, 4, 4, MODE>(a, p.splits, sp, s);
  return launch_tiled<32, 32, 2, 2, 6, 3, MODE>(a, p.splits, sp, s);
}

bool ep_ok(const Epilogue& ep) {
  if (ep.ln_g && (!ep.ln_b || !ep.ln_out || !ep.out_f32)) return false;
  return ep.out != nullptr && ep.act >= 0 && ep.act <= 2;
}

}  // namespace

hipError_t linear_bf16(const uint16_t* x, int M, int K, const uint16_t* w, int N, const Epilogue& ep,
                       const Split& sp, hipStream_t s) {
  if (!x || !w || M < 1 || N < 1 || K < 8 || (K & 7) || !ep_ok(ep)) return hipErrorInvalidValue;
  if (ep.w_packed && ((N & 15) || (K & 127))) return hipErrorInvalidValue;
  GemmArgs a{};
  a.x = x; a.w = w; a.M = M; a.N = N; a.K = K; a.ep = ep;
  if (M <= kSkinnyRows) {
    a.splits = 1;
    hipError_t e = launch_skinny(a, s);
    return e == hipSuccess ? finish(a, s) : e;
  }
  // the tiled kernel addresses x and w through 32-bit buffer offsets, and loads them straight into LDS
  // in 16-byte pieces, from 16-byte boundaries only
  if ((size_t)M * K * 2 >= (1u << 31) || (size_t)N * K * 2 >= (1u << 31) || ((uintptr_t)x & 15) || ((uintptr_t)w & 15))
    return hipErrorInvalidValue;
  return pick_tiled<X_ROWS>(a, sp, s);
}

namespace {

// Two contractions share a launch up to this many 32 x 32 tiles: a launch is then mostly its fixed part (some
// 4 us: the launch, the first operands' round trip, the drain and the epilogue), which the pair pays once. Beyond,
// larger tiles in launches of their own win. ResNet-50 at 224 x 224, four pairs, warm us per pass with limits of
// 0 / 512 / 1024 / 2048 / 4096 tiles: batch 1 (240 to 980 tiles) 267 / 262 / 257 / 258 / 259, 2 (480 to 1960) 298 / 298 /
// 296 / 297 / 298, 4 (960 to 3900) 348 / 348 / 347 / 350 / 356, 8 403 / 405 / 402 / 408 / 409.
constexpr long kPairTiles = 1024;

// Checks a convolution and fills its argument block (also a 1x1 stride-1 one's, as a linear layer's).
hipError_t conv_args(const uint16_t* x, int B, int H, int W, int C, const uint16_t* w, int O, int KH, int KW,
                     int stride, int pad, const Epilogue& ep, GemmArgs* out) {
  if (!x || !w || B < 1 || H < 1 || W < 1 || C < 1 || O < 1 || KH < 1 || KW < 1 || stride < 1 || pad < 0 ||
      !ep_ok(ep) || ep.ln_g)
    return hipErrorInvalidValue;
  const int Ho = (H + 2 * pad - KH) / stride + 1, Wo = (W + 2 * pad - KW) / stride + 1;
  if (Ho < 1 || Wo < 1) return hipErrorInvalidValue;
  GemmArgs a{};
  a.x = x; a.w = w; a.M = B * Ho * Wo; a.N = O; a.K = KH * KW * C;
  a.H = H; a.W = W; a.C = C; a.KW = KW; a.stride = stride; a.pad = pad; a.Ho = Ho; a.Wo = Wo;
  a.ep = ep;
  a.ep.w_packed = 0;
  if ((size_t)B * H * W * C * 2 >= (1u << 31) || (size_t)O * KH * KW * C * 2 >= (1u << 31) || ((uintptr_t)x & 15) ||
      ((uintptr_t)w & 15))
    return hipErrorInvalidValue;   // the tiled kernel's 32-bit buffer offsets and 16-byte loads, as above
  if (C & 63) return hipErrorInvalidValue;
  *out = a;
  return hipSuccess;
}

}  // namespace

hipError_t conv_bf16(const uint16_t* x, int B, int H, int W, int C, const uint16_t* w, int O, int KH, int KW,
                     int stride, int pad, const Epilogue& ep, const Split& sp, hipStream_t s) {
  if (KH == 1 && KW == 1 && stride == 1 && pad == 0 && (C & 7) == 0 && !ep.ln_g)
    return linear_bf16(x, B * H * W, C, w, O, ep, sp, s);
  GemmArgs a{};
  const hipError_t e = conv_args(x, B, H, W, C, w, O, KH, KW, stride, pad, ep, &a);
  return e == hipSuccess ? pick_tiled<X_CONV64>(a, sp, s) : e;
}

hipError_t conv1x1_pair(const uint16_t* x, int B, int H, int W, int C, const uint16_t* w0, int O0, const Epilogue& ep0,
                        const uint16_t* w1, int O1, int stride1, const Epilogue& ep1, bool* done, hipStream_t s) {
  *done = false;
  GemmArgs a{}, b{};
  hipError_t e = conv_args(x, B, H, W, C, w0, O0, 1, 1, 1, 0, ep0, &a);
  if (e == hipSuccess) e = conv_args(x, B, H, W, C, w1, O1, 1, 1, stride1, 0, ep1, &b);
  if (e != hipSuccess) return e;
  const int tna = (a.N + 31) / 32, tma = (a.M + 31) / 32, tnb = (b.N + 31) / 32, tmb = (b.M + 31) / 32;
  const long tiles = (long)tna * tma + (long)tnb * tmb;
  // rows past the skinny kernel's, and neither contraction long enough for the plan to split it
  if (tiles > kPairTiles || a.M <= kSkinnyRows || b.M <= kSkinnyRows || C >= 36 * 64 || a.N % 8 || b.N % 8) return hipSuccess;
  a.splits = b.splits = 1;
  a.kst = b.kst = (C + 63) / 64;
  *done = true;
  auto go = [&](auto kern) { (void)launch(kern, dim3((unsigned)tiles), dim3(256), 0, s, a, tna, tma, b, tnb, tmb); };
  if (stride1 == 1) a.ep.w_far ? go(k_gemm_pair<X_ROWS, true>) : go(k_gemm_pair<X_ROWS, false>);
  else a.ep.w_far ? go(k_gemm_pair<X_CONV64, true>) : go(k_gemm_pair<X_CONV64, false>);
  return hipGetLastError();
}

}  // namespace k
}  // namespace tp
