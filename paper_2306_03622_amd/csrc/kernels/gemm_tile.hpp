// The tiled bf16 contraction of gfx950 (k_gemm) as a device template; gemm_bf16.hip chooses its
// shape. Operand convention as everywhere here: the MFMA "A" operand is 16 weight rows n, the
// "B" operand 16 activation rows m.
#pragma once
#include "gemm_args.hpp"
#include "tile_plan.hpp"

namespace tp {
namespace k {

// Buffer loads of an operand: one buffer resource per matrix (base, size in bytes < 2^31), a
// 32-bit byte offset per lane; a lane at or beyond the size reads zero, so an operand outside
// the matrix or the image costs an offset select.
constexpr uint32_t kOffNone = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// A run's bias or residual, 16 (R = 8) or 8 bytes
template <int R>
__device__ __forceinline__ typename EpRun<R>::Raw ep_run_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (R == 8) return buffer_load16(r, off);
  else return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// Loads 16 bytes per lane straight into LDS: lane l's bytes land at LDS byte `dst` + 16 l (dst
// is wave-uniform). In assembly because the compiler, which knows the builtin as a write to
// LDS, waits for every such load in flight before each LDS read that follows in program order:
// the ring below then hides nothing (~0.47 us a stage whatever the tile and the ring's depth,
// against 0.12 us). No register is written but m0, the LDS base; the waits are lds_wait_barrier's.
// OPERAND: m0 is an operand that the compiler sets, else the block sets it (the s_nop is the wait state between
// that and the load either way). The compiler's schedules differ: small tiles lose up to 1.1% where the block sets
// it (six encoder layers of 1024 x 4096, 1024 rows, 385 us against 381; ResNet-50 at batch 8 406 against 404), large ones where
// the compiler does (ResNet-50 at batch 32 837 against 830).
template <bool OPERAND>
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, uint32_t dst, uint32_t voff, int soff) {
  if constexpr (OPERAND)
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 ::"{m0}"(dst), "v"(voff), "s"(r), "s"(soff));
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 ::"s"(dst), "v"(voff), "s"(r), "s"(soff) : "m0");
}

// Waits until at most N of this wave's vector-memory operations are in flight and its LDS reads
// have returned, then for every wave of the workgroup to do the same.
template <int N>
__device__ __forceinline__ void lds_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}

// One BN x BM output tile over the 64-deep k-stages [s0, s0 + n) of this split.
//
// A ring of NST stages in LDS, filled by loads that go straight there (no staging registers, no
// LDS stores). Stage j is read while stages j+1 .. j+NST-1 are in flight; one barrier per stage:
// each wave waits until its own loads of the next stage have landed (all but the (NST - 2) LPS
// youngest: loads return in order, and every wave issues LPS per stage) and its reads of this
// stage have returned, so that behind the barrier the next stage is whole and this stage's slot
// free, into which stage j + NST is then loaded, by large tiles a few
// loads per group of multiplications (8 waves' 8 loads at once queue for the load path, 16 cycles
// each, and hold up the multiplications behind them: 8192 x 4096 x 4096, 236 -> 220 us; small tiles lose
// by it). The barrier stands before the stage's last group of
// multiplications, which therefore covers the first LDS reads of the next stage; within a stage
// the fragments of a group are read one group ahead.
//
// LDS layout: row-major operands as rows of 128 bytes, the 16-byte chunk c of a row at position
// c ^ key(row), with a key that gives the 8 rows read together 8 different positions (no bank
// conflicts); a lane loads the chunk that belongs at its place. Blocked weights (PK, 16 rows x 128 k per
// block) are 1 KB runs already in fragment order; the second 8 rows of a run swap their halves
// for the same reason.
//
// Where a wave owns an even number NB of 16-row weight blocks, the rows of two consecutive
// fragments are interleaved so that a lane's accumulators hold 8 consecutive output features:
// the epilogue then works on 16-byte runs in registers, without a turn through LDS.
//
// EPF: the epilogue's bias and residual are loaded before the first operands, so that their
// round trip overlaps the main loop (small tiles; large ones have no registers to spare).
// VEC: N is a multiple of 8 (4 for a single block per wave), runs of outputs are whole vectors; others are not split.
// The body of workgroup `id` of `total`; lds: gemm_lds bytes.
constexpr size_t gemm_lds(int bn, int bm, int nst) { return (size_t)nst * (bn + bm) * 128; }

template <int BN, int BM, int WGN, int WGM, int NST, int MODE, bool PK, bool VEC, bool FAR>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, int tn, int tm, int id, int total, char* lds) {
  constexpr int NW = WGN * WGM;
  constexpr int TA = BN / 8 / NW, TB = BM / 8 / NW, LPS = TA + TB;   // 1 KB loads per wave and stage
  constexpr int WN = BN / WGN, WM = BM / WGM, NB = WN / 16, MB = WM / 16;
  constexpr bool PAIR = NB % 2 == 0;
  constexpr int IG = PAIR ? 2 : 1;       // weight fragments per group
  constexpr int GP = NB / IG, T = 2 * GP;              // groups per 32-deep half stage, per stage
  constexpr int SP = LPS <= 4 ? 1 : NST > 2 ? T : T / 2;   // groups over which a stage's loads are spread
  constexpr int PER = (LPS + SP - 1) / SP;             // loads per group
  constexpr int RUN = PAIR ? 8 : 4, NR = NB * 4 / RUN; // outputs per run, runs per lane and row block
  constexpr bool EPF = VEC && NR * MB <= 4;
  constexpr bool M0_OPERAND = BN <= 64;
  static_assert(BN % (8 * NW) == 0 && BM % (8 * NW) == 0 && WN % 16 == 0 && WM % 16 == 0 && NB % IG == 0 &&
                    NST >= 2 && NST <= 8 && (VEC || !PAIR), "tile shape");
  constexpr int ABYTES = BN * 128, SBYTES = (BN + BM) * 128;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WGN, wm = wave / WGN;
  const int r = lane & 15, q = lane >> 4;

  const TileAt at = tile_at<FAR>(id, total, tn, tm, a.splits);
  const int z = at.z, n_base = at.tx * BN, m_base = at.ty * BM;
  const int nst = (a.K + 63) >> 6, full = a.K >> 6;
  const int s0 = z * a.kst;
  const int n = min(s0 + a.kst, nst) - s0;      // stages of this split (>= 1: no empty split)

  // per-lane byte offsets of the operand loads (k = 0; X_CONV64: the top-left tap, wrapping modulo
  // 2^32 where the window starts in the padding, which a valid tap brings back inside the image);
  // ta, tb: the lane's chunk of a last stage that is not whole lies beyond K
  const __amdgpu_buffer_rsrc_t rw = buffer_of(a.w, (uint32_t)((size_t)a.N * a.K * 2));
  const __amdgpu_buffer_rsrc_t rx =
      buffer_of(a.x, MODE == X_ROWS ? (uint32_t)((size_t)a.M * a.K * 2)
                                    : (uint32_t)((size_t)(a.M / (a.Ho * a.Wo)) * a.H * a.W * a.C * 2));
  uint32_t offa[TA], offb[TB];
  int ih0[TB], iw0[TB];
  bool ta[TA];
#pragma unroll
  for (int t = 0; t < TA; ++t) {
    const int u = wave * TA + t;
    if constexpr (PK) {
      const int nb = u >> 1, c = lane >> 4, row = (lane & 15) ^ ((lane & 8) >> 1);
      offa[t] = n_base + nb * 16 < a.N
                    ? (uint32_t)(((n_base >> 4) + nb) * (a.K >> 7)) * 4096u + (u & 1) * 1024 + (c * 16 + row) * 16
                    : kOffNone;
      ta[t] = false;
    } else {
      const int row = u * 8 + (lane >> 3);
      const int key = PAIR ? ((row & 3) | (((row >> 3) & 1) << 2)) : (row & 7);
      const int ch = (lane & 7) ^ key;
      offa[t] = n_base + row < a.N ? (uint32_t)(n_base + row) * (uint32_t)(a.K * 2) + ch * 16 : kOffNone;
      ta[t] = full * 64 + ch * 8 >= a.K;
    }
  }
  const int chb = (lane & 7) ^ (lane >> 3);
  const bool tb = full * 64 + chb * 8 >= a.K;
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int m = m_base + (wave * TB + t) * 8 + (lane >> 3);
    const bool valid = m < a.M;
    if constexpr (MODE == X_ROWS) {
      offb[t] = valid ? (uint32_t)m * (uint32_t)(a.K * 2) + chb * 16 : kOffNone;
    } else {
      const int mm = valid ? m : 0, hw = a.Ho * a.Wo, b = mm / hw, rem = mm - b * hw;
      const int oh = rem / a.Wo, ow = rem - oh * a.Wo;
      const int ih = oh * a.stride - a.pad, iw = ow * a.stride - a.pad;
      offb[t] = (uint32_t)((((b * a.H + ih) * a.W + iw) * a.C) * 2 + chb * 16);
      ih0[t] = valid ? ih : -(1 << 20);          // a row beyond M: outside the image at every tap
      iw0[t] = iw;
    }
  }
  // position of the next stage to load; X_CONV64: its filter tap (kh, kw) and channel offset
  int sl = s0, kh = 0, kw = 0, c0 = 0;
  if constexpr (MODE == X_CONV64) {
    const int tap = s0 * 64 / a.C;
    c0 = s0 * 64 - tap * a.C;
    kh = tap / a.KW;
    kw = tap - kh * a.KW;
  }
  // loads [lo, hi) of this wave's LPS loads of the next stage, into ring slot `slot`
  auto issue = [&](int slot, int lo, int hi) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + slot * SBYTES;
    const bool edge = sl >= full;                 // the ragged last stage
#pragma unroll
    for (int u = 0; u < LPS; ++u) {
      if (u < lo || u >= hi) continue;
      if (u < TA) {
        lds_load16<M0_OPERAND>(rw, dst + (wave * TA + u) * 1024, (ta[u] & edge) ? kOffNone : offa[u], sl * (PK ? 2048 : 128));
      } else {
        const int t = u - TA;
        const uint32_t d = dst + ABYTES + (wave * TB + t) * 1024;
        if constexpr (MODE == X_ROWS) {
          lds_load16<M0_OPERAND>(rx, d, (tb & edge) ? kOffNone : offb[t], sl * 128);
        } else {
          const bool ok = ((unsigned)(ih0[t] + kh) < (unsigned)a.H) & ((unsigned)(iw0[t] + kw) < (unsigned)a.W);
          lds_load16<M0_OPERAND>(rx, d, ok ? offb[t] + (uint32_t)(((kh * a.W + kw) * a.C + c0) * 2) : kOffNone, 0);
        }
      }
    }
    if (hi < LPS) return;
    ++sl;
    if constexpr (MODE == X_CONV64) {
      c0 += 64;
      if (c0 == a.C) {
        c0 = 0;
        if (++kw == a.KW) { kw = 0; ++kh; }
      }
    }
  };

  f32x4 acc[NB][MB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fragment i holds weight row 32 (i / 2) + 8 (r / 4) + 4 (i % 2) + r % 4 of the wave's rows at
  // lane row r (PAIR), or row r. Byte addresses inside a stage: of the two 32-deep halves
  // (blocked weights: of even and odd fragments).
  uint32_t aA[2], aB[2];
  if constexpr (PK) {
    const int hb = (r >> 2) & 1;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      aA[i] = PAIR ? (wn * NB + (r >> 3)) * 2048 + q * 256 + (hb * 8 + ((i ^ hb) << 2) + (r & 3)) * 16
                   : wn * NB * 2048 + q * 256 + (r ^ ((r & 8) >> 1)) * 16;
  } else {
    const int row = wn * WN + (PAIR ? (r >> 2) * 8 + (r & 3) : r);
    aA[0] = row * 128 + ((q ^ (r & 7)) << 4);
    aA[1] = row * 128 + (((q + 4) ^ (r & 7)) << 4);
  }
  aB[0] = ABYTES + (wm * WM + r) * 128 + ((q ^ (r & 7)) << 4);
  aB[1] = ABYTES + (wm * WM + r) * 128 + (((q + 4) ^ (r & 7)) << 4);

  uint4 fa[2][IG], fb[2][MB];
  // group t of a stage: weight fragments (t % GP) IG .. + IG - 1 of half t / GP
  auto read = [&](const char* base, int t) __attribute__((always_inline)) {
    const int h = t / GP;
    if (t % GP == 0) {
#pragma unroll
      for (int j = 0; j < MB; ++j) fb[h][j] = *reinterpret_cast<const uint4*>(base + aB[h] + j * 2048);
    }
#pragma unroll
    for (int u = 0; u < IG; ++u) {
      const int i = (t % GP) * IG + u;
      if constexpr (PK)
        fa[t & 1][u] = *reinterpret_cast<const uint4*>(base + aA[i & 1] + h * 1024 + (PAIR ? (i >> 1) * 4096 : i * 2048));
      else
        fa[t & 1][u] = *reinterpret_cast<const uint4*>(base + aA[h] + (PAIR ? (i >> 1) * 4096 + (i & 1) * 512 : i * 2048));
    }
  };
  auto multiply = [&](int t) __attribute__((always_inline)) {
    const int h = t / GP;
#pragma unroll
    for (int u = 0; u < IG; ++u)
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        f32x4& c = acc[(t % GP) * IG + u][j];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[t & 1][u]), as_bf16x8(fb[h][j]), c, 0, 0, 0);
      }
  };

  // EPF: run p of row block j covers outputs n_base + wn WN + p 4 RUN + q RUN .. + RUN - 1 of row
  // m_base + wm WM + 16 j + r; an absent bias or residual is a buffer of no bytes, which reads zero
  const int run_n = n_base + wn * WN + q * RUN, run_m = m_base + wm * WM + r;
  EpRun<RUN> pre[EPF ? NR : 1][EPF ? MB : 1];
  if constexpr (EPF) {
    const bool on = a.splits == 1;
    const __amdgpu_buffer_rsrc_t rb = buffer_of(a.ep.bias, on && a.ep.bias ? (uint32_t)(a.N * 2) : 0u);
    const __amdgpu_buffer_rsrc_t rr = buffer_of(a.ep.res, on && a.ep.res ? (uint32_t)((size_t)a.M * a.N * 2) : 0u);
#pragma unroll
    for (int p = 0; p < NR; ++p) {
      const int nn = run_n + p * 4 * RUN;
      const auto b = ep_run_load<RUN>(rb, (uint32_t)(nn * 2));
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        const int m = run_m + 16 * j;
        pre[p][j].bias = b;
        pre[p][j].res = ep_run_load<RUN>(rr, m < a.M ? ((uint32_t)m * (uint32_t)a.N + nn) * 2 : kOffNone);
      }
    }
  }

#pragma unroll
  for (int i = 0; i < NST; ++i)
    if (i < n) issue(i, 0, LPS);
  if (n >= NST) lds_wait_barrier<(NST - 1) * LPS>();
  else lds_wait_barrier<0>();
  const char* cur = lds;
  int slot = 0, j = 0, pend = -1;               // pend: the slot whose stage is not all issued yet
  read(cur, 0);
  // WAIT: loads of stages beyond the next that may be in flight; MORE: a next stage exists;
  // ISSUE: so does stage j + NST
#define TP_STAGE(WAIT, MORE, ISSUE)                                             \
  {                                                                             \
    const int ns = slot + 1 == NST ? 0 : slot + 1;                              \
    const char* nxt = lds + ns * SBYTES;                                        \
    _Pragma("unroll") for (int t = 0; t < T; ++t) {                             \
      if (MORE && t == T - 1) {                                                 \
        lds_wait_barrier<(WAIT)>();                                             \
        if (ISSUE) issue(slot, 0, PER);                                         \
      } else if ((t + 1) * PER < LPS && pend >= 0) {                            \
        issue(pend, (t + 1) * PER, (t + 2) * PER < LPS ? (t + 2) * PER : LPS);  \
      }                                                                         \
      if (t + 1 < T) read(cur, t + 1);                                          \
      else if (MORE) read(nxt, 0);                                              \
      multiply(t);                                                              \
      __builtin_amdgcn_sched_barrier(0);                                        \
    }                                                                           \
    pend = ISSUE && PER < LPS ? slot : -1;                                      \
    cur = nxt;                                                                  \
    slot = ns;                                                                  \
    ++j;                                                                        \
  }
  while (j + NST < n) TP_STAGE((NST - 2) * LPS, true, true)
  // the last stages, R more after each
#define TP_TAIL(R)                                              \
  if constexpr (NST - 1 >= R) {                                 \
    if (n > R) TP_STAGE((R - 1) * LPS, true, false)             \
  }
  TP_TAIL(7) TP_TAIL(6) TP_TAIL(5) TP_TAIL(4) TP_TAIL(3) TP_TAIL(2) TP_TAIL(1)
  TP_STAGE(0, false, false)
#undef TP_TAIL
#undef TP_STAGE

#pragma unroll
  for (int p = 0; p < NR; ++p) {
    const int nn = run_n + p * 4 * RUN;
    EpRun<RUN> in;
    if constexpr (VEC && !EPF) {
      if (a.ep.bias && nn < a.N) in.bias = *reinterpret_cast<const typename EpRun<RUN>::Raw*>(a.ep.bias + nn);
    }
#pragma unroll
    for (int jj = 0; jj < MB; ++jj) {
      const int m = run_m + 16 * jj;
      if (m < a.M && nn < a.N) {
        const size_t base = (size_t)m * a.N + nn;
        float v[RUN];
#pragma unroll
        for (int e = 0; e < RUN; ++e) v[e] = PAIR ? acc[2 * p + (e >> 2)][jj][e & 3] : acc[p][jj][e & 3];
        if (VEC && a.splits > 1) {
          // fp32 partial of this split: P[split][m][n]
          float* o = a.partials + (size_t)z * a.M * a.N + base;
#pragma unroll
          for (int e = 0; e < RUN; e += 4) *reinterpret_cast<float4*>(o + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
        } else if constexpr (VEC) {
          if constexpr (EPF) {
            in = pre[p][jj];
          } else {
            if (a.ep.res) in.res = *reinterpret_cast<const typename EpRun<RUN>::Raw*>(static_cast<const uint16_t*>(a.ep.res) + base);
          }
          ep_apply(a.ep, in, v);
          ep_store(a.ep, base, v);
        } else {
          store_row4(a, m, nn, f32x4{v[0], v[1], v[2], v[3]});
        }
      }
    }
  }
}

template <int BN, int BM, int WGN, int WGM, int NST, int MODE, bool PK, int MINW, bool VEC, bool FAR>
__global__ __launch_bounds__(64 * WGN * WGM, MINW) void k_gemm(GemmArgs a, int tn, int tm) {
  __shared__ __attribute__((aligned(1024))) char lds[gemm_lds(BN, BM, NST)];
  gemm_tile<BN, BM, WGN, WGM, NST, MODE, PK, VEC, FAR>(a, tn, tm, blockIdx.x, gridDim.x, lds);
}

// Two independent contractions in one launch, 32 x 32 tiles: workgroups [0, na) the first, the others the
// second. The same sums in the same order as in launches of their own with any tile (unsplit), so the same bits. Its rule: conv1x1_pair.
template <int MODE_B, bool FAR>
__global__ __launch_bounds__(256, 3) void k_gemm_pair(GemmArgs a, int tna, int tma, GemmArgs b, int tnb, int tmb) {
  __shared__ __attribute__((aligned(1024))) char lds[gemm_lds(32, 32, 6)];
  const int na = tna * tma;
  if ((int)blockIdx.x < na) gemm_tile<32, 32, 2, 2, 6, X_ROWS, false, true, FAR>(a, tna, tma, blockIdx.x, na, lds);
  else gemm_tile<32, 32, 2, 2, 6, MODE_B, false, true, FAR>(b, tnb, tmb, blockIdx.x - na, gridDim.x - na, lds);
}

}  // namespace k
}  // namespace tp
