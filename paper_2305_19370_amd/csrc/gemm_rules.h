// Which tile form a product takes, by estimated time. Host arithmetic only.
#pragma once

#include <cmath>
#include <cstdint>
#include <initializer_list>

namespace bpt {

// The bf16 tile forms: 256 x 256 (8 waves), 128 x 128 and 64 x 64 (4 waves), 64 x 64 with four
// groups of 4 waves sharing K.
enum Tile { T256, T128, T64, T64K4 };

// What the estimate of a tile form depends on besides the number of tiles and stages
struct TileJob {
  int64_t nper = 0;      // columns of three matrices keep a tile inside one of them
  int in_order = 0;      // no form that shares K
  int both_kmajor = 0;   // both operands are transposed on their way from LDS
  int epi2 = 0;          // the epilogue reads a second operand or writes a second result
};

// Estimated microseconds of n tiles of `stages` k stages. Fitted to measurements of the layer's 14
// products, operands in HBM and in the caches: 64..32768 rows, D = 256..5120 (multiples of 256 and others),
// F = 4 D, in every form (a part of them in profiles/gemm_tile_forms.md). The choice costs 1.5 to 2 % over
// the best form in the mean. A full round of 256 x 256 tiles takes 0.65 per stage (0.48 while few CUs
// work) and 13 for prologue and epilogue, whose stores all CUs issue at once, 4 more with a second
// operand or result there: 24000 x 1024 x 1024 stored in bf16 takes 60, with 128 x 128 tiles 69; with a
// residual 88 and 82. 128 x 128 tiles take 0.26 with one workgroup on a CU and 0.56 with two (they share
// the LDS, which is what bounds them), from 0.40 on where only some CUs have two; 64 x 64 tiles 0.108
// alone and 0.13 each up to five on a CU; the K-sharing form a quarter of the stages at 0.25 (few CUs) to
// 0.5. Beyond 8192 k the operands no longer stay in the L2s and the smaller tiles, which read them more
// often, slow down. With both operands K-major a stage of 64 x 64 tiles takes longer and one of the
// K-sharing and 256 x 256 forms less: dWo of 4000 tokens at D = 768 takes 30 with 64 x 64 tiles, 22
// where they share K.
inline double tile_us(Tile t, int64_t n, double stages, const TileJob& j) {
  const double full = t == T128 ? 512 : t == T64 ? 1280 : 256;
  const double rounds = std::floor((double)n / full), rem = (double)n - rounds * full;
  if (stages > 256 && t != T256) stages *= 1.1;
  if (j.both_kmajor) stages *= t == T256 ? 0.9 : t == T64 ? 1.15 : t == T64K4 ? 0.8 : 1;
  switch (t) {
    case T256: {
      const double fixed = j.epi2 ? 17 : 13;
      return rounds * (stages * 0.65 + fixed) + (rem > 0 ? stages * (0.48 + 0.17 * rem / 256) + fixed : 0);
    }
    case T128:
      return rounds * (stages * 0.56 + 5) +
             (rem > 256 ? stages * (0.40 + 0.16 * (rem - 256) / 256) + 5 : rem > 0 ? stages * 0.26 + 5 : 0);
    case T64:
      return rounds * (stages * 0.65 + 4) + (rem > 256 ? stages * 0.13 * rem / 256 + 4 : rem > 0 ? stages * 0.108 + 4 : 0);
    case T64K4: {
      const double it = std::ceil(stages / 4);
      return rounds * (it * 0.5 + 6) + (rem > 0 ? it * (0.25 + 0.25 * rem / 256) + 6 : 0);
    }
  }
  return 0;
}

// The cheapest tile form for M x ncols over nz batch entries or K slices of `stages` stages
inline Tile best_tile(int64_t M, int64_t ncols, int64_t nz, double stages, const TileJob& j, double* us) {
  Tile best = T128;
  double t = -1;
  for (Tile c : {T128, T256, T64, T64K4}) {
    const int64_t b = c == T256 ? 256 : c == T128 ? 128 : 64;
    if (j.nper % b != 0 || (j.in_order && c == T64K4)) continue;
    const double u = tile_us(c, ((M + b - 1) / b) * ((ncols + b - 1) / b) * nz, stages, j);
    if (t < 0 || u < t) {
      t = u;
      best = c;
    }
  }
  if (us) *us = t;
  return best;
}

// The fp32 tile forms: squares of 128, 64 and 32, and 32 with four groups sharing K.
enum F32Tile { F128, F64, F32T, F32K4 };

// Estimated microseconds of n tiles of `stages` k stages of 16, as tile_us, for 64..2000 rows and
// K = 64..4096 (the choice costs 1 % over the best form of 280 measured products in the mean): w
// workgroups per CU take their share of the matrix cores (0.98, 0.24, 0.06 per stage at the full
// rate) or, alone, the latency of a stage.
inline double f32_us(F32Tile t, int64_t n, double stages) {
  const double w = (double)n / 256;
  switch (t) {
    case F128: return std::ceil(w) * 1.07 * stages + 6;
    case F64: return std::fmax(0.40, 0.355 * std::ceil(w)) * stages + 3.3;
    case F32T: return (w <= 1 ? 0.216 : 0.1 + 0.108 * w) * stages + 2.5;
    case F32K4: return std::ceil(stages / 4) * std::fmax(0.48, 0.5 * w) + 3.5;
  }
  return 0;
}

inline F32Tile best_f32_tile(int64_t M, int64_t ncols, int64_t nz, double stages, int64_t nper, int in_order, double* us) {
  F32Tile best = F32T;
  double t = -1;
  for (F32Tile c : {F64, F128, F32T, F32K4}) {
    const int64_t b = c == F128 ? 128 : c == F64 ? 64 : 32;
    if (nper % b != 0 || (in_order && c == F32K4)) continue;
    const double u = f32_us(c, ((M + b - 1) / b) * ((ncols + b - 1) / b) * nz, stages);
    if (t < 0 || u < t) {
      t = u;
      best = c;
    }
  }
  if (us) *us = t;
  return best;
}

// Slices of K (at most cap, whole stages, no fewer than 8 each) of an M x N product stored in fp32:
// the least estimated time of the tiles and, at 4 TB/s, of writing and adding the slices.
inline int best_ksplit(bool f32, int64_t M, int64_t N, int64_t K, int cap, int64_t nper, int both_kmajor, double* us) {
  int best = 1;
  double tbest = 0;
  TileJob j;
  j.nper = nper;
  j.both_kmajor = both_kmajor;
  const int64_t bk = f32 ? 16 : 32, nk = (K + bk - 1) / bk;
  for (int z = 1; z <= cap; ++z) {
    const int64_t stages = (nk + z - 1) / z;
    if (z > 1 && stages < 8) break;
    double t;
    if (f32) best_f32_tile(M, N, z, (double)stages, nper, 0, &t);
    else best_tile(M, N, z, (double)stages, j, &t);
    if (z > 1) t += 3.0 + (2.0 * z + 1) * 4.0 * M * N / 4.0e6;
    if (z == 1 || t < tbest) {
      tbest = t;
      best = z;
    }
  }
  if (us) *us = tbest;
  return best;
}

// Whether three products of M x nper with one left operand (Q, K, V; dWq, dWk, dWv) run as one of
// M x 3 nper: unless its tiles, each inside one of the three, are estimated clearly slower than three
// launches (by an eighth: 128 x 128 tiles with warm operands do better than estimated). A bf16 width that is
// an odd multiple of 128 has no 256 x 256 tiles as one: dWq, dWk, dWv of 9152 tokens at D = 3968 take 1084 us,
// 711 one by one; of 4000 tokens at D = 640 39 and 65. Over 160 products of 100..30000 tokens, D = 384..4992, cold,
// the choice costs 0.7 % over the better of the two in the mean, always one launch 5.9 %.
inline bool three_as_one(bool f32, int64_t M, int64_t nper, int64_t K, int cap3, int cap1) {
  double one, each;
  best_ksplit(f32, M, 3 * nper, K, cap3, nper, 0, &one);
  best_ksplit(f32, M, nper, K, cap1, 0, 0, &each);
  return one <= 1.125 * 3 * each;
}

}  // namespace bpt
