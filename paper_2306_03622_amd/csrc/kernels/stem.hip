// The ResNet stem in one launch: 7 x 7 stride-2 convolution of 3 channels to 64 with bias and ReLU,
// then 3 x 3 stride-2 max-pool. The convolution's output (bf16, rounded as if stored) never leaves the CU: at
// batch 32 its write and the pool's read were 103 MB of HBM traffic.
//
// A workgroup of 4 waves owns kPoolW pooled pixels of up to kPoolR pooled rows of one sample, for all
// channels: 64 convolution pixels (16 per wave) of each of 2 kPoolR + 1 rows, of which a neighbour's share one
// column and one row. All its global loads, the weights and every input row, are issued before the
// first use.
//
// The im2col operand of an MFMA needs 8 consecutive k of a pixel per lane. A filter row of a pixel is
// 21 consecutive elements of a staged input row; with k laid out as 24 per filter row (one unused element before,
// two after, zero in both operands), each lane's 8 are 16 bytes at a 4-byte boundary, two LDS reads instead of
// eight 2-byte gathers and their packing. (That kernel, with the pool a launch of its own, took 67 + 16 us at
// batch 32 and 9.3 + 4.6 us at batch 1; this one 28 and 8.6.) The weights stay in registers (96 of them) for all rows. As for the
// tiled contraction, weight rows are interleaved so that a lane's accumulators hold 8 consecutive channels.
#include <algorithm>

#include "gemm_args.hpp"

namespace tp {
namespace k {
namespace {

constexpr int kPoolW = 31, kPoolR = 8;             // pooled pixels and rows per workgroup
constexpr int kSteps = 6;                          // k-steps of 32: 7 filter rows of 3 chunks of 8, and 3 empty chunks
constexpr int kRowE = 408;                         // elements of a staged input row (51 vectors)
constexpr int kIn = 4 * kPoolR + 7;                // input rows staged at most
constexpr int kWStride = 200;                      // elements of a weight row in LDS (24 chunks and padding)
constexpr int kFlatV = 64 * 147 * 2 / 16;          // 16-byte vectors of the flat weights

// VX: the image is 16-byte aligned and its rows whole 16-byte vectors, else elements are loaded one by one
// (the same values, so the same bits).
template <bool VX>
__global__ __launch_bounds__(256) void k_stem(const uint16_t* __restrict__ x, int H, int W,
                                              const uint16_t* __restrict__ w, const uint16_t* __restrict__ bias,
                                              int Ho, int Wo, int Hp, int Wp, int rows, uint16_t* __restrict__ y) {
  __shared__ __align__(16) uint16_t xl[kIn * kRowE > kFlatV * 8 ? kIn * kRowE : kFlatV * 8];
  __shared__ __align__(16) uint16_t wl[64 * kWStride];         // then the convolution rows on their way to the pool
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int pc0 = blockIdx.x * kPoolW, pr0 = blockIdx.y * rows, b = blockIdx.z;
  const int nrows = min(rows, Hp - pr0);                       // pooled rows; >= 1
  const int oc0 = 2 * pc0 - 1, or0 = 2 * pr0 - 1;              // first convolution column and row
  const int ih0 = 2 * or0 - 3;                                 // first input row
  const int nin = 4 * nrows + 7;                               // input rows: 2 (2 nrows) + 7
  // staged rows start at a vector boundary of the image row, the element before the first window (an
  // even element, as 3 (2 oc0 - 3) is odd) at element sh of it
  const int e0 = (2 * oc0 - 3) * 3 - 1;
  const int v0 = e0 >> 3, sh = e0 - v0 * 8;                    // floor division

  uint4 wv[(kFlatV + 255) / 256], xv[(kIn + 3) / 4];
#pragma unroll
  for (int u = 0; u < (kFlatV + 255) / 256; ++u) {
    const int i = u * 256 + tid;
    wv[u] = i < kFlatV ? reinterpret_cast<const uint4*>(w)[i] : make_uint4(0, 0, 0, 0);
  }
  const int rowv = W * 3 >> 3;                                 // vectors per image row
#pragma unroll
  for (int i = 0; i < (kIn + 3) / 4; ++i) {
    const int rr = wave + 4 * i, ih = ih0 + rr, v = v0 + lane;
    const bool in = rr < nin && ih >= 0 && ih < H && lane < kRowE / 8;
    const uint16_t* row = x + ((size_t)b * H + (in ? ih : 0)) * W * 3;
    if constexpr (VX) {
      xv[i] = in && v >= 0 && v < rowv ? reinterpret_cast<const uint4*>(row)[v] : make_uint4(0, 0, 0, 0);
    } else {
      uint32_t d[4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int j = v * 8 + e;
        const uint32_t t = in && j >= 0 && j < W * 3 ? row[j] : 0;
        d[e >> 1] = e & 1 ? d[e >> 1] | (t << 16) : t;
      }
      xv[i] = make_uint4(d[0], d[1], d[2], d[3]);
    }
  }
  float bf[2][8];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
#pragma unroll
    for (int e = 0; e < 8; ++e) bf[p][e] = 0.f;
    if (bias) add_bf16(bf[p], *reinterpret_cast<const uint4*>(bias + 32 * p + 8 * q));
  }

  // flat weights -> padded chunks: chunk c = 3 kh + j of channel n holds k = 21 kh + 8 j - 1 + (0 .. 7)
#pragma unroll
  for (int u = 0; u < (kFlatV + 255) / 256; ++u) {
    const int i = u * 256 + tid;
    if (i < kFlatV) reinterpret_cast<uint4*>(xl)[i] = wv[u];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    const int c = wave + 4 * u, kh = c / 3, j = c - 3 * kh;    // the same for the whole wave; channel = lane
    uint32_t d[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 8 * j - 1 + e;
      const bool in = c < 21 && k >= 0 && k < 21;
      const uint32_t v = in ? xl[lane * 147 + kh * 21 + k] : 0;
      d[e >> 1] = e & 1 ? d[e >> 1] | (v << 16) : v;
    }
    *reinterpret_cast<uint4*>(&wl[lane * kWStride + 8 * c]) = make_uint4(d[0], d[1], d[2], d[3]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < (kIn + 3) / 4; ++i) {
    const int rr = wave + 4 * i;
    if (rr < nin && lane < kRowE / 8) *reinterpret_cast<uint4*>(&xl[rr * kRowE + lane * 8]) = xv[i];
  }
  uint4 fa[kSteps][4];
  int koff[kSteps];
  uint32_t m0[kSteps], m3[kSteps];             // masks of a chunk's first and last two elements
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int c = 4 * s + q, kh = c / 3, j = c - 3 * kh;
    koff[s] = c < 21 ? kh * kRowE + 8 * j : 0;
    m0[s] = j == 0 ? 0xffff0000u : 0xffffffffu;
    m3[s] = j == 2 ? 0u : 0xffffffffu;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = (g >> 1) * 32 + (r >> 2) * 8 + (g & 1) * 4 + (r & 3);
      fa[s][g] = *reinterpret_cast<const uint4*>(&wl[n * kWStride + 8 * c]);
    }
  }
  __syncthreads();                             // wl is free, xl holds the input rows

  const int p = wave * 16 + r;                 // this lane's convolution pixel: column oc0 + p
  const uint16_t* xp = xl + sh + 6 * p;
  // the pool: thread = (pooled pixel i, channels 8 cg ..)
  const int pi = tid >> 3, cg = tid & 7, pc = pc0 + pi;
  const bool pool = pi < kPoolW && pc < Wp;
  float m[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = -INFINITY;
  for (int t = 0; t <= 2 * nrows; ++t) {       // convolution row or0 + t
    const bool row = or0 + t >= 0 && or0 + t < Ho;
    uint16_t* cr = wl + (t & 1) * 64 * 64;     // [pixel][64 channels], chunks of 8 swizzled by the pixel
    if (row) {
      f32x4 acc[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const uint32_t* bp = reinterpret_cast<const uint32_t*>(xp + 2 * t * kRowE + koff[s]);
        uint4 v = make_uint4(bp[0] & m0[s], bp[1], bp[2], bp[3] & m3[s]);
        if (s == kSteps - 1 && q > 0) v = make_uint4(0, 0, 0, 0);    // the empty chunks
#pragma unroll
        for (int g = 0; g < 4; ++g)
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[s][g]), as_bf16x8(v), acc[g], 0, 0, 0);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = act_apply(acc[2 * h + (e >> 2)][e & 3] + bf[h][e], ACT_RELU);
        *reinterpret_cast<uint4*>(cr + p * 64 + (((4 * h + q) ^ (p & 7)) << 3)) =
            make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
      }
    }
    __syncthreads();
    float hm[8];                               // the row's maximum over the pooled pixel's three columns
#pragma unroll
    for (int e = 0; e < 8; ++e) hm[e] = -INFINITY;
    if (row && pool) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int px = 2 * pi + d, col = oc0 + px;
        if (col >= 0 && col < Wo) {
          const uint4 v = *reinterpret_cast<const uint4*>(cr + px * 64 + ((cg ^ (px & 7)) << 3));
          const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            hm[2 * e] = fmaxf(hm[2 * e], bf2f(vw[e] & 0xffff));
            hm[2 * e + 1] = fmaxf(hm[2 * e + 1], bf2f(vw[e] >> 16));
          }
        }
      }
    }
    if (t & 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) m[e] = fmaxf(m[e], hm[e]);
    } else {                                   // the last row of one pooled row and the first of the next
      if (t > 0 && pool) {
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = fmaxf(m[e], hm[e]);
        *reinterpret_cast<uint4*>(y + (((size_t)b * Hp + pr0 + t / 2 - 1) * Wp + pc) * 64 + 8 * cg) =
            make_uint4(f2bf2(m[0], m[1]), f2bf2(m[2], m[3]), f2bf2(m[4], m[5]), f2bf2(m[6], m[7]));
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) m[e] = hm[e];
    }
  }
}

}  // namespace

hipError_t stem_pool(const uint16_t* x, int B, int H, int W, const uint16_t* w, const uint16_t* bias, uint16_t* y,
                     hipStream_t s) {
  if (!x || !w || !y || B < 1 || H < 1 || W < 1 || ((uintptr_t)w & 15) || ((uintptr_t)bias & 15) || ((uintptr_t)y & 15))
    return hipErrorInvalidValue;
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1, Hp = (Ho - 1) / 2 + 1, Wp = (Wo - 1) / 2 + 1;
  // Pooled rows per workgroup: as few as make at most two workgroups per CU (the registers' limit), up to kPoolR;
  // a workgroup's weights and staging cost about as much as three pooled rows (224 x 224 images, us with 1 / 2 / 4 / 7 / 8
  // rows: batch 1 8.6 / 10.5 / 14.5 / 20.3 / 22.2, 8 19.8 / 13.5 / 15.2 / 21.1 / 23.2, 16 34 / 25 / 19.5 / 21.8 / 23.7, 32 60 / 41 /
  // 34.9 / 28.0 / 30.0).
  const int segs = (Wp + kPoolW - 1) / kPoolW;
  const int rows = (int)std::min<long>(kPoolR, ((long)segs * Hp * B + 511) / 512);
  auto go = [&](auto kern) {
    (void)launch(kern, dim3(segs, (Hp + rows - 1) / rows, B), dim3(256), 0, s, x, H, W, w, bias, Ho, Wo, Hp, Wp, rows, y);
  };
  if (W * 3 % 8 == 0 && ((uintptr_t)x & 15) == 0) go(k_stem<true>);
  else go(k_stem<false>);
  return hipGetLastError();
}

}  // namespace k
}  // namespace tp
