// Multi-head self-attention for head dim 64 and short sequences (S <= 256, S % 32 == 0),
// one workgroup per (sample, head, 16 NW queries); each wave owns 16 queries.
//
// K and V of the head are staged row-major in LDS ([key][d]). Scores are
// computed as S^T = K Q^T on MFMA (A = 16 keys, B = 16 queries), so lane l holds the
// scores of query l % 16 against keys 16 t + 4 (l / 16) + e. The softmax reductions
// over keys therefore stay inside a lane plus two cross-lane exchanges (lanes l ^ 16,
// l ^ 32), in fp32. The exponentials exp(s - max), rounded to bf16, are used directly as
// the A operand of O = P V, and the output is multiplied by 1 / their fp32 sum: a 32-key MFMA
// k-block takes the lane's own values from two consecutive score tiles, and the matching V
// entries are read with gfx950's transposing LDS load (ds_read_b64_tr_b16) in the same key order,
// so no data moves between lanes.
#include "common.hpp"
#include "kernels.hpp"

namespace tp {
namespace k {
namespace {

// The sequence length is a template argument, so every key tile is known at compile time (with a
// run-time tile count the conditional MFMA accumulators compiled to hundreds of register copies:
// S 96, 5 samples of 12 heads, 4.8 us against 4.0 us for S 128).
template <int S, int NW>
__global__ __launch_bounds__(64 * NW) void k_attention(const uint16_t* __restrict__ qkv, int H,
                                                       uint16_t* __restrict__ out) {
  constexpr int LDK = 72, LDV = 80, NT = S / 16, NTHR = 64 * NW;
  static_assert(S % 32 == 0, "whole 32-key blocks");
  __shared__ __attribute__((aligned(16))) uint16_t Ks[S * LDK];
  __shared__ __attribute__((aligned(16))) uint16_t Vs[S * LDV];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z;
  const int D = H * 64, ld = 3 * D;
  const uint16_t* base = qkv + (size_t)b * S * ld;

  // this wave's queries first (independent of the staging); a wave past the sequence end
  // loads row 0 and does nothing with it
  const int q0 = blockIdx.x * (16 * NW) + wave * 16;
  const bool active = q0 < S;
  const uint16_t* qrow = base + (size_t)(active ? q0 + r : 0) * ld + h * 64 + (g << 3);
  const uint4 qf0 = *reinterpret_cast<const uint4*>(qrow);
  const uint4 qf1 = *reinterpret_cast<const uint4*>(qrow + 32);

  // K and V of the head: every load of this thread issued before the first LDS store, so
  // the round trips overlap. Both are read as key = 32 i + tid / 8, 8 dims at (tid % 8) * 8,
  // a key's 128 bytes per 8 lanes, so one wave's load covers 8 whole rows; both are stored
  // as whole 16-byte pieces. (V stored transposed 2 bytes at a time, read as 8-byte pieces,
  // took 5.6 / 5.5 us per launch at BERT-base batch 1 / 8 with the best padding of several;
  // other transposes, by lanes holding 64 consecutive keys or by an 8 x 8 exchange among
  // lanes, 6.7-7.4 us; all the same bits.)
  constexpr int NV = (S * 8 + NTHR - 1) / NTHR;
  uint4 kv[NV], vv[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int key = (i * NTHR + tid) >> 3, d8 = (tid & 7) << 3;
    const uint16_t* row = base + (size_t)(key < S ? key : 0) * ld + h * 64 + d8;
    kv[i] = *reinterpret_cast<const uint4*>(row + D);
    vv[i] = *reinterpret_cast<const uint4*>(row + 2 * D);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int key = (i * NTHR + tid) >> 3, d8 = (tid & 7) << 3;
    if (key < S) {
      *reinterpret_cast<uint4*>(&Ks[key * LDK + d8]) = kv[i];
      *reinterpret_cast<uint4*>(&Vs[key * LDV + d8]) = vv[i];
    }
  }
  __syncthreads();

  if (!active) return;
  f32x4 sc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t* krow = &Ks[(16 * t + r) * LDK + (g << 3)];
    sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(*reinterpret_cast<const uint4*>(krow)),
                                                    as_bf16x8(qf0), sc[t], 0, 0, 0);
    sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(*reinterpret_cast<const uint4*>(krow + 32)),
                                                    as_bf16x8(qf1), sc[t], 0, 0, 0);
  }
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[t][e]);
  mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  float sum = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // exp((s - max) / sqrt(64)) as one hardware base-2 exponential
      const float p = __builtin_amdgcn_exp2f((sc[t][e] - mx) * (0.125f * 1.44269504088896341f));
      sc[t][e] = p;
      sum += p;
    }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  const float inv = 1.f / sum;

  f32x4 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < NT / 2; ++u) {
    const f32x4 p0 = sc[2 * u], p1 = sc[2 * u + 1];
    uint4 pa;
    pa.x = f2bf2(p0[0], p0[1]);
    pa.y = f2bf2(p0[2], p0[3]);
    pa.z = f2bf2(p1[0], p1[1]);
    pa.w = f2bf2(p1[2], p1[3]);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      // V^T fragment of keys 32 u + 4 g + 0..3 (lo) and 16 further (hi), dim 16 dt + r, read
      // transposed from row-major V: within a 16-lane group, lane l receives element l % 4 of
      // the 8-byte pieces the group's lanes l / 4 + 4 j (j = 0..3) address, so lane s of the
      // group addresses key row (s % 16) / 4 at dims 16 dt + 4 (s % 4)
      const uint16_t* vr = &Vs[(32 * u + 4 * g + (r >> 2)) * LDV + 16 * dt + 4 * (r & 3)];
      typedef short v4s __attribute__((ext_vector_type(4)));
      const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)vr);
      const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(vr + 16 * LDV));
      const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(pa), as_bf16x8(make_uint4(l2.x, l2.y, h2.x, h2.y)),
                                                      o[dt], 0, 0, 0);
    }
  }
  // lane holds O[query q0 + 4 g + e][d = 16 dt + r]; the query's 1 / sum is with lane 4 g + e
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float scale = __shfl(inv, 4 * g + e, 64);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      out[((size_t)b * S + q0 + 4 * g + e) * D + h * 64 + 16 * dt + r] = f2bf(o[dt][e] * scale);
  }
}

}  // namespace

hipError_t attention(const uint16_t* qkv, int B, int S, int H, uint16_t* out, hipStream_t s) {
  if (!qkv || !out || B < 1 || H < 1 || S < 32 || (S & 31) || S > 256) return hipErrorInvalidValue;
  // Waves (16 queries each) per workgroup, each of which stages K and V once: up to 128 keys four
  // (with one or two, staging costs more than the extra workgroups gain: BERT-base at batch 8, whole
  // warm pass 0.790 ms with four, 0.839 with two, 0.915 with one). Longer sequences take four while
  // that leaves CUs idle (S 256, 60 sample-heads: 5.1 us against 6.1 with eight), else eight, which fill
  // a CU that the staged K and V leave room for two workgroups on (96 / 384 sample-heads: 6.5 / 19.0 us
  // against 7.5 / 26.4), or from 192 sample-heads on a wave for every 16 queries of a sequence of up to
  // 192, of which the second workgroup of eight would have few (S 160, 192 / 384: 6.5 / 9.9 us against 7.6 / 12.4).
  const long heads = (long)H * B;
  const int nw = S <= 128 || 2 * heads < 192 ? 4 : S <= 192 && heads >= 192 ? S / 16 : 8;
  const dim3 grid((S + 16 * nw - 1) / (16 * nw), H, B), block(64 * nw);
  auto go = [&](auto kern) { (void)launch(kern, grid, block, 0, s, qkv, H, out); };
  switch (S) {
    case 32: go(k_attention<32, 4>); break;
    case 64: go(k_attention<64, 4>); break;
    case 96: go(k_attention<96, 4>); break;
    case 128: go(k_attention<128, 4>); break;
    case 160: nw == 4 ? go(k_attention<160, 4>) : nw == 8 ? go(k_attention<160, 8>) : go(k_attention<160, 10>); break;
    case 192: nw == 4 ? go(k_attention<192, 4>) : nw == 8 ? go(k_attention<192, 8>) : go(k_attention<192, 12>); break;
    case 224: nw == 4 ? go(k_attention<224, 4>) : go(k_attention<224, 8>); break;
    default: nw == 4 ? go(k_attention<256, 4>) : go(k_attention<256, 8>); break;
  }
  return hipGetLastError();
}

}  // namespace k
}  // namespace tp
