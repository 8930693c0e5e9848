// Which tiles a bf16 contraction takes, and in which order (no HIP headers: also compiled for the host alone).
#pragma once
#include <algorithm>
#include <cstddef>

#ifdef __HIPCC__
#define TP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define TP_HOST_DEVICE inline
#endif

namespace tp {
namespace k {

// The tile (tx of tn, of features; ty of tm, of rows; k split z) that workgroup `id` of `total` = tn tm splits computes.
// Workgroups go to the 8 XCDs in turn, each with an L2 of its own: XCD x takes the x-th contiguous eighth of
// the tiles. Those are ordered in bands of kBand tile rows, so that the tiles an XCD works on at a time share their
// operands' rows. With weights in host memory (FAR) all rows are one band: an XCD then reads an
// eighth of the weights over the host link, instead of each XCD all of them (a first request of 1000 rows
// to a 2 x 512 model that is read in place: 58 us, in bands 106; four layers of 1024 at 300 rows 230, 332).
constexpr int kBand = 8;

struct TileAt {
  int tx, ty, z;
};

// FAR is a template argument because a choice in the kernel cost its start: ResNet-50 1% (a branch) to 2% (a variable
// band height, whose divisions take longer) at any batch.
template <bool FAR>
TP_HOST_DEVICE TileAt tile_at(int id, int total, int tn, int tm, int splits) {
  const int per = total >> 3, rem = total & 7, xcd = id & 7;
  id = xcd * per + (xcd < rem ? xcd : rem) + (id >> 3);
  TileAt t;
  t.z = splits > 1 ? id / (tn * tm) : 0;
  id -= t.z * tn * tm;
  if (FAR) {
    t.tx = id / tm;
    t.ty = id - t.tx * tm;
    return t;
  }
  const int band = id / (kBand * tn), first = band * kBand, height = kBand < tm - first ? kBand : tm - first;
  const int in = id - first * tn;
  t.tx = in / height;
  t.ty = first + in - t.tx * height;
  return t;
}

// y[M][N] = x[M][K] w[N][K]^T; conv: an implicit-GEMM convolution; gelu, ln: the epilogue has a GELU, a row
// LayerNorm follows; far: the weights are read over the host link
struct TileShape {
  int M, N, K;
  bool conv, gelu, ln, far;
};

// Tile shape (output features x rows), ring depth and k split of a tiled contraction, by how many
// tiles a shape gives the 256 CUs. Measured on MI355X over every contraction of ResNet-50 and
// BERT-base at batch 1, 8 and 32 and MLP layers of 64 to 8192 rows, under graph replay, weights and
// inputs rotating so that they come from beyond the L2s (us; tiles in brackets):
//   128 x 128, two per CU, from 196 tiles and for more than 64 features: 25088 x 128 x 1152 [196] 14.2
//     against 15.9 with 64 x 64, 1568 x 2048 x 512 [208] 8.9 against 10.0; below, 1024 x 3072 x 768 [192]
//     11.8 against 11.4, 6272 x 256 x 2304 [98] 22 against 16; 100352 x 64 x 576 [784] 23 against 17. Up to
//     one tile per CU with three stages in the ring (100352 / 4 x 128 x 512 [196] 8.9, with two 9.8).
//     From 16 stages on, 256 x 256 or 256 x 128 instead where large_tile_us says so.
//   64 x 64 from 192 tiles, with four stages in the ring while two per CU hold all tiles
//     (1024 x 768 x 3072 [192] 12.9, with two stages 23; 256 x 4096 x 4096 [256] 16.8 against 31), else
//     with two stages and up to five per CU (100352 x 64 x 64 [1568] 7.7 against 10.5 with four).
//     3 x 3 convolutions of 64 stages and more on at most one such tile per CU are split in two
//     (1568 x 512 x 4608 [200] 20.5, unsplit 24).
//   64 x 32 from 176 tiles, two per CU with five stages (480 x 768 x 3072 [180] 10.4 against 10.9 with
//     32 x 32, 1568 x 256 x 1024 [196] 5.3 against 6.1 with three stages).
//   Else 32 x 32, with six stages in the ring where that is at most one tile per CU (196 x 512 x 1024
//     [112] 4.3, with four 4.6) and the contraction deep enough to fill it, else with four (128 x 3072 x
//     768 [384] 5.1 against 5.4).
// A k split costs a reduction, a launch of 2 to 3 us, so otherwise only contractions of 36 stages and
// more whose tiles leave CUs idle are split, each split keeping 9 stages: 64 x 32 tiles from 64 of
// them, up to 448 workgroups (392 x 512 x 4608 [104, 4 splits] 12.3, unsplit 32 x 32 14.7), else
// 32 x 32, up to 256 (49 x 512 x 4608 [32, 8 splits] 7.3, unsplit 16; 196 x 256 x 2304 [56, 4
// splits] 6.9, unsplit 7.6). With a row LayerNorm, which rides on the reduction where the width allows, 32 x 32 tiles
// are split alike (warm passes of three encoder layers, split / unsplit, features x rows x k [tiles]: 64 x 64 x 16384
// [4] 83 / 158, 256 x 128 x 8192 [32] 87 / 126, 768 x 128 x 3072 [96] 103 / 107, 192 x 512 x 2304 [96] 96.6 / 98.2), but
// 64 x 32 tiles, of which each split leaves more to reduce, only from 96 stages on, and from 256 where they are more
// than 96 (512 x 256 x 6144 [64] 112 / 124, x 3072 101 / 104, 64 x 2048 x 3072 [64] 123 / 120; 384 x 512 x 6144 [96]
// 133 / 137, x 3072 121 / 120; 64 x 4096 x 6144 [128] 178 / 166, x 16384 297 / 295, 1024 x 256 x 6144 [128] 141 / 139, x
// 16384 189 / 206).
struct TilePlan {
  int bn, bm, ring, splits;
};

// Time of a contraction with large tiles, a model fitted to the rates measured on MI355X. A round
// of the chip (512 tiles of 128 x 128, two per CU, else 256) costs a rate per stage and a fixed
// part, larger with a GELU; a last round of 128 x 128 tiles that leaves CUs with one tile costs
// 0.66. Rows that are not whole 128-byte lines cost the smallest tiles, which load the most per
// multiplication, 15%. Measured, us, with 128 x 128 / 256 x 128 / 256 x 256 tiles: 8192 x 4096 x 4096 264 / 246 / 220,
// 4096 x 4096 x 4096 129 / 123 / 112, 8192 x 768 x 3072 47 / 43 / 66, 8192 x 1024 x 4096 64 / 60 / 87, 4096 x 1024 x
// 4096 42 / 48 / 80, 6000 x 2000 x 2000 70 / 72 / 62, 8192 x 1536 x 1536 47 / 53 / 48, 8192 x 2304 x 768 44 / 56 / 62.
inline double large_tile_us(int bn, int bm, long tiles, const TileShape& s) {
  const int nst = (s.K + 63) / 64;
  if (bn == 128) {
    const long rem = tiles % 512;
    const double last = rem == 0 ? 0 : rem <= 256 ? 0.66 : std::min(1.0, 0.66 + 0.34 * (rem - 256) / 128);
    return (tiles / 512 + last) * (nst + (s.gelu ? 4.7 : 2.2)) * (s.K % 64 ? 1.15 : 1.0);
  }
  const long rounds = (tiles + 255) / 256;
  return bm == 128 ? rounds * (0.9 * nst + (s.gelu ? 8 : 2)) : rounds * (1.65 * nst + (s.gelu ? 13 : 10));
}

inline TilePlan plan_near(const TileShape& s, size_t scratch_bytes) {
  auto tiles = [&](int bn, int bm) { return (long)((s.N + bn - 1) / bn) * ((s.M + bm - 1) / bm); };
  const int nst = (s.K + 63) / 64;
  if (s.N % 8) return {32, 32, 4, 1};        // outputs in no whole vectors
  // beyond the 32-bit offsets of the epilogue that tiles of four blocks per wave fetch ahead
  if ((size_t)s.M * s.N * 2 >= (1u << 31)) return {256, 128, 3, 1};
  if (tiles(128, 128) >= 196 && s.N > 64) {
    const double us[3] = {large_tile_us(128, 128, tiles(128, 128), s), large_tile_us(256, 128, tiles(256, 128), s),
                          large_tile_us(256, 256, tiles(256, 256), s)};
    if (nst < 16 || (us[0] <= us[1] && us[0] <= us[2])) return {128, 128, tiles(128, 128) <= 256 ? 3 : 2, 1};
    return us[1] <= us[2] ? TilePlan{256, 128, 3, 1} : TilePlan{256, 256, 2, 1};
  }
  const size_t per_split = (size_t)s.M * s.N * 4;
  const long most = (long)(scratch_bytes / per_split);    // splits that fit the scratch
  if (tiles(64, 64) >= 192) {
    const bool deep_conv = s.conv && nst >= 64 && tiles(64, 64) <= 256 && most >= 2;
    return {64, 64, tiles(64, 64) <= 512 ? 4 : 2, deep_conv ? 2 : 1};
  }
  if (tiles(64, 32) >= 176) return {64, 32, 5, 1};
  if (nst >= 36) {
    const bool wide = tiles(64, 32) >= 64;
    const long nt = wide ? tiles(64, 32) : tiles(32, 32);
    const int z = (int)std::min<long>({(wide ? 448 : 256) / nt, nst / 9, most});
    const bool pays = !(s.ln && wide) || nst >= (nt <= 96 ? 96 : 256);
    if (z > 1 && pays) return wide ? TilePlan{64, 32, 5, z} : TilePlan{32, 32, 6, z};
  }
  return {32, 32, tiles(32, 32) <= 256 && nst >= 8 ? 6 : 4, 1};
}

// With the weights in host memory and fewer columns of tiles than XCDs, several XCDs read the same weights over the link:
// 32 x 32 tiles then, which add their sums in the same order, for weights of 256 KB and more and up to 2048 of
// them (read in place, us with the tiles above / these: ResNet-50 at 224 x 224, batch 8 2190 / 1782, 12 2116 / 1882, 32 2475 /
// 2370; beyond, two encoder layers of 768 at 8192 rows, 6144 tiles, 1913 / 2460).
inline TilePlan plan_tiles(const TileShape& s, size_t scratch_bytes) {
  const TilePlan p = plan_near(s, scratch_bytes);
  const long columns = (s.N + p.bn - 1) / p.bn, small = (long)((s.N + 31) / 32) * ((s.M + 31) / 32);
  if (s.far && p.splits == 1 && p.bn > 32 && columns < 8 && (long)s.N * s.K >= 1 << 17 && small <= 2048)
    return {32, 32, small <= 256 ? 6 : 4, 1};
  return p;
}

}  // namespace k
}  // namespace tp
