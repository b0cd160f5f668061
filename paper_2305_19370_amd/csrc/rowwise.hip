// Row-wise and layout kernels of the BPT layer: LayerNorm forward / backward and
// its parameter gradients, bias gradients (row / column sums), the softmax
// backward's per-row Delta = rowsum(dO * O), and the sum of K slices. All are HBM-bound; each
// reads and writes every element once (LayerNorm re-reads its row from cache).
#include <algorithm>

#include "common.h"
#include "drop.h"
#include "internal.h"

namespace bpt {

template <typename T> struct Vec4;
template <> struct Vec4<float> {
  static BPT_DEV void load(const float* p, float v[4]) {
    const f32x4 x = *(const f32x4*)p;
    v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
  }
  static BPT_DEV void store(float* p, const float v[4]) { *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]}; }
};
template <> struct Vec4<bf16> {
  static BPT_DEV void load(const bf16* p, float v[4]) {
    const bf16x4 x = *(const bf16x4*)p;
    v[0] = (float)x[0]; v[1] = (float)x[1]; v[2] = (float)x[2]; v[3] = (float)x[3];
  }
  static BPT_DEV void store(bf16* p, const float v[4]) {
    bf16x4 x;
    x[0] = (bf16)v[0]; x[1] = (bf16)v[1]; x[2] = (bf16)v[2]; x[3] = (bf16)v[3];
    *(bf16x4*)p = x;
  }
};

// 8 consecutive elements <-> 8 floats, with 16-byte accesses
template <typename T> struct Vec8;
template <> struct Vec8<float> {
  static BPT_DEV void load(const float* p, float v[8]) {
    const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
    v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3]; v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  }
  static BPT_DEV void store(float* p, const float v[8]) {
    *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]};
    *(f32x4*)(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
  }
};
template <> struct Vec8<bf16> {
  static BPT_DEV void load(const bf16* p, float v[8]) {
    const bf16x8 x = *(const bf16x8*)p;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)x[e];
  }
  static BPT_DEV void store(bf16* p, const float v[8]) {
    bf16x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (bf16)v[e];
    *(bf16x8*)p = x;
  }
};

// ------------------------------------------------------------------ LayerNorm forward
// Rows of D <= 512 NC (D % 8 == 0): one wave per row holds the whole row in registers (NC
// chunks of 8 consecutive elements per lane, chunk c of lane l at columns 8 (l + 64 c)), so
// every element is read once and written once. Two-pass mean / variance over the registers.
template <typename TI, typename TO, int NC>
__global__ __launch_bounds__(256) void ln_fwd_reg_kernel(const TI* x, int64_t ldx, const float* g,
                                                         const float* bb, TO* out, int64_t ldo, float* mu,
                                                         float* rstd, int64_t rows, int D, float eps, int use_stats) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= rows) return;
  const TI* xr = x + row * ldx;
  float v[NC][8];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int d = 8 * (lane + 64 * c);
    if (d < D) Vec8<TI>::load(xr + d, v[c]);
  }
  float mean, rs;
  if (!use_stats) {
    float sm = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) sm += 8 * (lane + 64 * c) < D ? v[c][e] : 0.0f;
    mean = warp_sum(sm) / (float)D;
    float q = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dv = 8 * (lane + 64 * c) < D ? v[c][e] - mean : 0.0f;
        q = fmaf(dv, dv, q);
      }
    rs = 1.0f / sqrtf(warp_sum(q) / (float)D + eps);
    if (lane == 0) {
      mu[row] = mean;
      rstd[row] = rs;
    }
  } else {
    mean = mu[row];
    rs = rstd[row];
  }
  TO* orow = out + row * ldo;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int d = 8 * (lane + 64 * c);
    if (d >= D) continue;
    float gv[8], bv[8];
    if (g) Vec8<float>::load(g + d, gv);
    if (bb) Vec8<float>::load(bb + d, bv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float y = (v[c][e] - mean) * rs;
      if (g) y *= gv[e];
      if (bb) y += bv[e];
      v[c][e] = y;
    }
    Vec8<TO>::store(orow + d, v[c]);
  }
}

// Any D (a multiple of 4): one wave per row; each lane walks groups of 4 columns and
// re-reads the row (from cache) for the variance and the output. Two-pass mean / variance.
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const TI* x, int64_t ldx, const float* g,
                                                     const float* bb, TO* out, int64_t ldo, float* mu,
                                                     float* rstd, int64_t rows, int64_t D, float eps,
                                                     int use_stats) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const TI* xr = x + row * ldx;
  float mean, rs;
  if (!use_stats) {
    float s = 0.0f;
    for (int64_t d = 4 * lane; d < D; d += 256) {
      float v[4];
      Vec4<TI>::load(xr + d, v);
      s += (v[0] + v[1]) + (v[2] + v[3]);
    }
    mean = warp_sum(s) / (float)D;
    float q = 0.0f;
    for (int64_t d = 4 * lane; d < D; d += 256) {
      float v[4];
      Vec4<TI>::load(xr + d, v);
#pragma unroll
      for (int e = 0; e < 4; ++e) q = fmaf(v[e] - mean, v[e] - mean, q);
    }
    const float var = warp_sum(q) / (float)D;
    rs = 1.0f / sqrtf(var + eps);
    if (lane == 0) {
      mu[row] = mean;
      rstd[row] = rs;
    }
  } else {
    mean = mu[row];
    rs = rstd[row];
  }
  TO* orow = out + row * ldo;
  for (int64_t d = 4 * lane; d < D; d += 256) {
    float v[4];
    Vec4<TI>::load(xr + d, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float y = (v[e] - mean) * rs;
      if (g) y *= g[d + e];
      if (bb) y += bb[d + e];
      v[e] = y;
    }
    Vec4<TO>::store(orow + d, v);
  }
}

// ------------------------------------------------------------------ LayerNorm backward
// Storage row of dout's row r (seg > 0: a pitch of `pitch` rows per seg rows)
struct RowMap {
  int64_t seg = 0, gap = 0;                          // gap = pitch - seg
  BPT_DEV int64_t at(int64_t r) const {
    if (gap == 0) return r;
    return r + (r >> 31 ? r / seg : (int64_t)((uint32_t)r / (uint32_t)seg)) * gap;
  }
};
// dz = rstd * (gd - mean(gd) - xhat * mean(gd * xhat)), gd = dout * gamma; out = resid + dz.
// Rows of D <= 512 NC WPR (D % 8 == 0): WPR waves per row hold the row of x and of dout in
// registers, wave w its chunks NC w .. NC w + NC - 1 of 512 columns.
//
// PARAM also sums the parameter gradients in the same pass: a workgroup walks rows
// blockIdx.x, + gridDim.x, ... (four at a time with WPR = 1), its lanes keep the sums of
// their columns, and the block's sums go to partial [2][gridDim.x][D] for chunk_reduce.
// HBM-bound: x and dout are read once for all three gradients. Final LayerNorm of 16384 x
// 2048 bf16 rows, dX and parameters: 45 us (4.5 TB/s) and 6.6 for the reduction, against
// 124 us in four passes (dout widened to fp32, dX, partial sums, reduction).
template <typename TI, typename TD, typename TR, typename TO, typename T2, int NC, int WPR, bool PARAM, bool DROP>
__global__ __launch_bounds__(256) void ln_bwd_reg_kernel(const TI* x, const float* mu, const float* rstd,
                                                         const float* g, const TD* dout, const TR* resid,
                                                         TO* out, T2* out2, float* partial, int64_t rows, int D,
                                                         RowMap map, DropArgs drop) {
  static_assert(WPR == 1 || WPR == 4, "waves per row");
  static_assert(WPR == 4 || !PARAM || NC <= 4, "LDS of the block sums");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // row in scalar registers
  const int col0 = 8 * (lane + (WPR == 4 ? 64 * NC * wave : 0));
  __shared__ float red[2][4][2];
  __shared__ __attribute__((aligned(16))) float sums[PARAM && WPR == 1 ? 2 * 512 * NC : 1];
  float ag[PARAM ? NC : 1][8], ab[PARAM ? NC : 1][8];
  if constexpr (PARAM) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) ag[c][e] = ab[c][e] = 0.0f;
  }
  const int64_t step = (int64_t)gridDim.x * (WPR == 4 ? 1 : 4);
  int par = 0;
  for (int64_t row = WPR == 4 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave; row < rows; row += step) {
    const float m = mu[row], rs = rstd[row];
    const int64_t drow = map.at(row);
    float xh[NC][8], gd[NC][8];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = col0 + 512 * c;
      if (d < D) {
        Vec8<TI>::load(x + row * D + d, xh[c]);
        Vec8<TD>::load(dout + drow * D + d, gd[c]);
      }
    }
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = col0 + 512 * c;
      if (d < D) {
        float gv[8];
        if (g) Vec8<float>::load(g + d, gv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          xh[c][e] = (xh[c][e] - m) * rs;
          if constexpr (PARAM) {
            ag[c][e] = fmaf(gd[c][e], xh[c][e], ag[c][e]);
            ab[c][e] += gd[c][e];
          }
          if (g) gd[c][e] *= gv[e];
          s1 += gd[c][e];
          s2 = fmaf(gd[c][e], xh[c][e], s2);
        }
      }
    }
    s1 = warp_sum(s1);
    s2 = warp_sum(s2);
    if constexpr (WPR == 4) {                 // two buffers in turn: one barrier per row
      if (lane == 0) {
        red[par][wave][0] = s1;
        red[par][wave][1] = s2;
      }
      __syncthreads();
      s1 = ((red[par][0][0] + red[par][1][0]) + red[par][2][0]) + red[par][3][0];
      s2 = ((red[par][0][1] + red[par][1][1]) + red[par][2][1]) + red[par][3][1];
      par ^= 1;
    }
    s1 /= (float)D;
    s2 /= (float)D;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = col0 + 512 * c;
      if (d < D) {
        float rv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (resid) Vec8<TR>::load(resid + row * D + d, rv);
#pragma unroll
        for (int e = 0; e < 8; ++e) rv[e] += rs * (gd[c][e] - s1 - xh[c][e] * s2);
        Vec8<TO>::store(out + row * D + d, rv);
        if constexpr (DROP) {
          float f[8];
          drop_factors(drop, drop.row0 + row, d, f);
          drop_factors(drop, drop.row0 + row, d + 4, f + 4);
#pragma unroll
          for (int e = 0; e < 8; ++e) rv[e] *= f[e];
        }
        if (out2) Vec8<T2>::store(out2 + row * D + d, rv);
      }
    }
  }
  if constexpr (PARAM) {
    if constexpr (WPR == 1) {                 // the four waves' sums, in wave order
      for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            float* sg = sums + 512 * c + 8 * lane;
            float* sb = sg + 512 * NC;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              sg[e] = w ? sg[e] + ag[c][e] : ag[c][e];
              sb[e] = w ? sb[e] + ab[c][e] : ab[c][e];
            }
          }
        }
        __syncthreads();
      }
      for (int d = 4 * threadIdx.x; d < D; d += 4 * 256) {
        *(f32x4*)(partial + (int64_t)blockIdx.x * D + d) = *(const f32x4*)(sums + d);
        *(f32x4*)(partial + ((int64_t)gridDim.x + blockIdx.x) * D + d) = *(const f32x4*)(sums + 512 * NC + d);
      }
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int d = col0 + 512 * c;
        if (d < D) {
          Vec8<float>::store(partial + (int64_t)blockIdx.x * D + d, ag[c]);
          Vec8<float>::store(partial + ((int64_t)gridDim.x + blockIdx.x) * D + d, ab[c]);
        }
      }
    }
  }
}

// Any D (a multiple of 4).
template <typename TI, typename TR, typename TO, typename T2>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const TI* x, const float* mu, const float* rstd,
                                                     const float* g, const float* dout, const TR* resid,
                                                     TO* out, T2* out2, int64_t rows, int64_t D, RowMap map) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const TI* xr = x + row * D;
  const float* dr = dout + map.at(row) * D;
  const float m = mu[row], rs = rstd[row];
  float s1 = 0.0f, s2 = 0.0f;
  for (int64_t d = 4 * lane; d < D; d += 256) {
    float xv[4], dv[4];
    Vec4<TI>::load(xr + d, xv);
    Vec4<float>::load(dr + d, dv);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gd = g ? dv[e] * g[d + e] : dv[e];
      s1 += gd;
      s2 = fmaf(gd, (xv[e] - m) * rs, s2);
    }
  }
  s1 = warp_sum(s1) / (float)D;
  s2 = warp_sum(s2) / (float)D;
  for (int64_t d = 4 * lane; d < D; d += 256) {
    float xv[4], dv[4], rv[4] = {0, 0, 0, 0};
    Vec4<TI>::load(xr + d, xv);
    Vec4<float>::load(dr + d, dv);
    if (resid) Vec4<TR>::load(resid + row * D + d, rv);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gd = g ? dv[e] * g[d + e] : dv[e];
      const float xh = (xv[e] - m) * rs;
      rv[e] += rs * (gd - s1 - xh * s2);
    }
    Vec4<TO>::store(out + row * D + d, rv);
    if (out2) Vec4<T2>::store(out2 + row * D + d, rv);
  }
}

// ------------------------------------------------------------------ column / row sums
static constexpr int kChunks = 128;

// Second stage: out0[d] (+)= sum_c partial[c D + d] and out1[d] (+)= sum_c partial[(nch + c) D + d],
// c < nch. A block per 16 columns: 16 lanes of 64 bytes, 16 groups of chunks; group k sums
// chunks k, k + 16, ... (eight loads in flight) and the group sums are added through LDS in
// group order.
__global__ __launch_bounds__(256) void chunk_reduce_kernel(const float* partial, int nch, float* out0,
                                                           float* out1, int64_t D, int accumulate) {
  __shared__ float red[2][16][17];
  const int cl = threadIdx.x & 15, k = threadIdx.x >> 4;
  const int64_t d = (int64_t)blockIdx.x * 16 + cl;
  float s0 = 0.0f, s1 = 0.0f;
  if (d < D) {
    for (int c0 = k; c0 < nch; c0 += 64) {
      float v0[4], v1[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = c0 + 16 * u;
        v0[u] = c < nch ? partial[(int64_t)c * D + d] : 0.0f;
        v1[u] = (out1 && c < nch) ? partial[(int64_t)(nch + c) * D + d] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { s0 += v0[u]; s1 += v1[u]; }
    }
  }
  red[0][k][cl] = s0;
  red[1][k][cl] = s1;
  __syncthreads();
  if (k < 2 && d < D) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += red[k][i][cl];
    float* out = k ? out1 : out0;
    if (out) out[d] = accumulate ? out[d] + s : s;
  }
}

// Column sums, first stage: a block of four waves per (512-column group, row chunk of `per`
// rows), wave w its rows w, w + 4, ... (8 consecutive columns per lane with 16-byte loads,
// four rows in flight); the wave sums are added through LDS in wave order.
template <typename T>
__global__ __launch_bounds__(256) void col_partial8_kernel(const T* in, int64_t ld, int64_t rows, int64_t per, int64_t cols,
                                                           float* partial) {
  __shared__ __attribute__((aligned(16))) float red[3][512];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t c = ((int64_t)blockIdx.x * 64 + lane) * 8;
  const int64_t r0 = blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (c < cols) {
    int64_t r = r0 + wave;
    for (; r + 12 < r1; r += 16) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) Vec8<T>::load(in + (r + 4 * u) * ld + c, v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += v[u][e];
    }
    for (; r < r1; r += 4) {
      float v[8];
      Vec8<T>::load(in + r * ld + c, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] += v[e];
    }
  }
  if (wave > 0) Vec8<float>::store(&red[wave - 1][8 * lane], s);
  __syncthreads();
  if (wave == 0 && c < cols) {
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] += red[w][8 * lane + e];
    Vec8<float>::store(partial + (int64_t)blockIdx.y * cols + c, s);
  }
}

// LayerNorm parameter partials, wide form: a block of four waves per (512-column group, row
// chunk); wave w sums the w-th quarter of the chunk's rows (8 columns per lane, 16-byte
// loads, two rows in flight), and the four quarter sums are added through LDS in wave order.
template <typename TI>
__global__ __launch_bounds__(256) void ln_param_partial8_kernel(const TI* x, const float* mu, const float* rstd,
                                                                const float* dout, float* partial, int64_t rows,
                                                                int64_t D, RowMap map) {
  __shared__ float red[2][4][64 * 8];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t d = ((int64_t)blockIdx.x * 64 + lane) * 8;
  const bool ok = d < D;
  const int64_t per = (rows + kChunks - 1) / kChunks;
  const int64_t c0 = blockIdx.y * per, c1 = c0 + per < rows ? c0 + per : rows;
  const int64_t q = (per + 3) / 4;
  const int64_t r0 = c0 + wv * q, r1 = r0 + q < c1 ? r0 + q : c1;
  float sg[8] = {0, 0, 0, 0, 0, 0, 0, 0}, sb[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (ok) {
    int64_t r = r0;
    for (; r + 2 <= r1; r += 2) {
      float xv[2][8], dv[2][8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        Vec8<TI>::load(x + (r + u) * D + d, xv[u]);
        Vec8<float>::load(dout + map.at(r + u) * D + d, dv[u]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float m = mu[r + u], rs = rstd[r + u];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          sg[e] = fmaf(dv[u][e], (xv[u][e] - m) * rs, sg[e]);
          sb[e] += dv[u][e];
        }
      }
    }
    for (; r < r1; ++r) {
      float xv[8], dv[8];
      Vec8<TI>::load(x + r * D + d, xv);
      Vec8<float>::load(dout + map.at(r) * D + d, dv);
      const float m = mu[r], rs = rstd[r];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sg[e] = fmaf(dv[e], (xv[e] - m) * rs, sg[e]);
        sb[e] += dv[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    red[0][wv][lane * 8 + e] = sg[e];
    red[1][wv][lane * 8 + e] = sb[e];
  }
  __syncthreads();
  if (wv == 0 && ok) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sg[e] = ((red[0][0][lane * 8 + e] + red[0][1][lane * 8 + e]) + red[0][2][lane * 8 + e]) + red[0][3][lane * 8 + e];
      sb[e] = ((red[1][0][lane * 8 + e] + red[1][1][lane * 8 + e]) + red[1][2][lane * 8 + e]) + red[1][3][lane * 8 + e];
    }
    Vec8<float>::store(partial + (int64_t)blockIdx.y * D + d, sg);
    Vec8<float>::store(partial + (int64_t)(kChunks + blockIdx.y) * D + d, sb);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void row_sum_kernel(const T* in, int64_t ld, int64_t rows, int64_t cols,
                                                      float* out, int accumulate) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  float s = 0.0f;
  for (int64_t c = lane; c < cols; c += 64) s += to_f32<T>(in[row * ld + c]);
  s = warp_sum(s);
  if (lane == 0) out[row] = accumulate ? out[row] + s : s;
}

// The same for 16-byte-aligned rows (ld a multiple of 8): each lane adds 8 consecutive
// columns per 16-byte load, with four loads in flight per lane; a scalar pass adds the
// columns past the last whole group of 8.
template <typename T>
__global__ __launch_bounds__(256) void row_sum8_kernel(const T* in, int64_t ld, int64_t rows, int64_t cols,
                                                       float* out, int accumulate) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const T* r = in + row * ld;
  const int64_t c8 = cols & ~(int64_t)7;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  int64_t c = 8 * lane;
  for (; c + 3 * 512 < c8; c += 4 * 512) {
    float v[4][8];
#pragma unroll
    for (int u = 0; u < 4; ++u) Vec8<T>::load(r + c + 512 * u, v[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[u] += v[u][e];
  }
  for (; c < c8; c += 512) {
    float v[8];
    Vec8<T>::load(r + c, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[0] += v[e];
  }
  float s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  for (int64_t t = c8 + lane; t < cols; t += 64) s += to_f32<T>(r[t]);
  s = warp_sum(s);
  if (lane == 0) out[row] = accumulate ? out[row] + s : s;
}

// ------------------------------------------------------------------ softmax-backward Delta
// One wave per token (b, s): Delta[b, h, s] = sum_d dO[t, h*dh + d] O[t, h*dh + d] for every
// head, from 16-byte loads of the token's two rows; the lanes of one head reduce by
// shuffles; stored negated (the backward kernels start dP from -Delta). Also
// nlse2 = -lse * log2(e), the negated base-2 log-sum-exp. Padding tokens s in [S, Sp) get
// zeros.
template <typename T>
__global__ __launch_bounds__(256) void delta_kernel(const T* dO, const T* O, int64_t ld, const float* lse,
                                                    float* ndelta, float* nlse2, int B, int64_t S, int64_t Sp,
                                                    int H, int dh) {
  constexpr int EPL = 16 / sizeof(T);                // elements per lane and load
  const int lane = threadIdx.x & 63;
  const int64_t tok = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // over B * Sp
  if (tok >= (int64_t)B * Sp) return;
  const int b = (int)(tok / Sp);
  const int64_t s = tok % Sp;
  const int D = H * dh, lpg = dh / EPL;             // lanes per head in one load step
  for (int e0 = 0; e0 < D; e0 += 64 * EPL) {
    const int e = e0 + lane * EPL;                  // the lanes of one head are all in or all out
    float acc = 0.0f;
    if (s < S && e < D) {
      const int64_t off = ((int64_t)b * S + s) * ld + e;
      float x[EPL], y[EPL];
#pragma unroll
      for (int k = 0; k < EPL; k += 4) {
        Vec4<T>::load(dO + off + k, x + k);
        Vec4<T>::load(O + off + k, y + k);
      }
#pragma unroll
      for (int k = 0; k < EPL; ++k) acc = fmaf(x[k], y[k], acc);
    }
    for (int o = lpg / 2; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane % lpg == 0 && e < D) {
      const int h = e / dh;
      const int64_t i = ((int64_t)b * H + h) * Sp + s;
      ndelta[i] = -acc;
      nlse2[i] = s < S ? -lse[i] * 1.4426950408889634f : 0.0f;
    }
  }
}

// ------------------------------------------------------------------ cross-entropy rows
// (m, l) summarises exp over a set of logits as l * exp(m); two summaries combine
// exactly. m = -inf, l = 0 is the empty set.
BPT_DEV void lse_merge(float& m, float& l, float m2, float l2) {
  const float mm = fmaxf(m, m2);
  if (mm == -__builtin_inff()) return;
  l = l * __expf(m - mm) + l2 * __expf(m2 - mm);
  m = mm;
}

// One workgroup per row t of a block of logits z (fp32, row stride ld, 16-byte aligned
// rows): each thread summarises its columns of [0, V) online, the summaries combine by
// shuffles and through LDS, and thread 0 writes lse[t] = m + log l and the token loss
// lse[t] - z[t, y_t], or NaN when the target is outside [0, V).
__global__ __launch_bounds__(256) void xent_rows_kernel(const float* z, int64_t ld, int64_t V,
                                                        const int32_t* tgt, float* lse, float* tok) {
  const int64_t t = blockIdx.x;
  const float* zr = z + t * ld;
  const int tid = threadIdx.x;
  float m = -__builtin_inff(), l = 0.0f;
  for (int64_t v = 4 * (int64_t)tid; v < V; v += 4 * 256) {
    float x[4];
    if (v + 4 <= V) {
      const f32x4 q = *(const f32x4*)(zr + v);
      x[0] = q[0]; x[1] = q[1]; x[2] = q[2]; x[3] = q[3];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = v + e < V ? zr[v + e] : -__builtin_inff();
    }
    const float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) s += __expf(x[e] - mx);
    lse_merge(m, l, mx, s);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float m2 = __shfl_xor(m, o, 64), l2 = __shfl_xor(l, o, 64);
    lse_merge(m, l, m2, l2);
  }
  __shared__ float sm[4], sl[4];
  if ((tid & 63) == 0) {
    sm[tid >> 6] = m;
    sl[tid >> 6] = l;
  }
  __syncthreads();
  if (tid == 0) {
    m = sm[0];
    l = sl[0];
    for (int w = 1; w < 4; ++w) lse_merge(m, l, sm[w], sl[w]);
    const float r = m + __logf(l);
    lse[t] = r;
    const int y = tgt[t];
    tok[t] = (y >= 0 && y < V) ? r - zr[y] : __builtin_nanf("");
  }
}

// One wave per row: lane i merges summaries i, i + 64, ..., the lanes' merge by exchanges.
__global__ __launch_bounds__(256) void xent_merge_kernel(const float* part, int64_t ng, int64_t rows, int64_t V,
                                                         const int32_t* tgt, const float* tlogit, float* lse, float* tok) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= rows) return;
  float m = -__builtin_inff(), l = 0.0f;
  for (int64_t j = lane; j < ng; j += 64) {
    const u32x2 q = *(const u32x2*)(part + 2 * (t * ng + j));
    lse_merge(m, l, __uint_as_float(q[0]), __uint_as_float(q[1]));
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float m2 = __shfl_xor(m, o, 64), l2 = __shfl_xor(l, o, 64);
    lse_merge(m, l, m2, l2);
  }
  if (lane == 0) {
    const float r = m + __logf(l);
    lse[t] = r;
    const int y = tgt[t];
    tok[t] = (y >= 0 && y < V) ? r - tlogit[t] : __builtin_nanf("");
  }
}

// out[0] = (sum of x[0..n)) / n, summed in a fixed order by one workgroup.
__global__ __launch_bounds__(1024) void mean_kernel(const float* x, int64_t n, float* out) {
  __shared__ float part[1024];
  float s = 0.0f;
  for (int64_t i = threadIdx.x; i < n; i += 1024) s += x[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = part[0] / (float)n;
}

// ------------------------------------------------------------------ host launchers
#define BPT_T(dt, T, ...) \
  do {                   \
    if ((dt) == F32) {   \
      using T = float;   \
      __VA_ARGS__;       \
    } else {             \
      using T = bf16;    \
      __VA_ARGS__;       \
    }                    \
  } while (0)

hipError_t layer_norm(Dt ti, Dt to, const void* x, int64_t ldx, const float* g, const float* b, void* out,
                      int64_t ldo, float* mu, float* rstd, int64_t rows, int64_t D, float eps,
                      int use_stats, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 3) / 4));
  // register-resident rows when D % 8 == 0, D <= 8192 and every row starts 16-byte aligned
  const bool vec = D % 8 == 0 && D <= 8192 && ldx % 8 == 0 && ldo % 8 == 0 && ((uintptr_t)x & 15) == 0 &&
                   ((uintptr_t)out & 15) == 0 && ((uintptr_t)g & 15) == 0 && ((uintptr_t)b & 15) == 0;
#define BPT_LN_FWD(NCV)                                                                                  \
  BPT_T(ti, TI, BPT_T(to, TO,                                                                            \
        hipLaunchKernelGGL((ln_fwd_reg_kernel<TI, TO, NCV>), grid, dim3(256), 0, s, (const TI*)x, ldx, g, \
                           b, (TO*)out, ldo, mu, rstd, rows, (int)D, eps, use_stats)));                  \
  return hipGetLastError()
  if (vec) {                                // the least chunk count that holds the row
    const int64_t nc = (D + 511) / 512;
    if (nc <= 1) { BPT_LN_FWD(1); }
    if (nc <= 2) { BPT_LN_FWD(2); }
    if (nc <= 3) { BPT_LN_FWD(3); }
    if (nc <= 4) { BPT_LN_FWD(4); }
    if (nc <= 6) { BPT_LN_FWD(6); }
    if (nc <= 8) { BPT_LN_FWD(8); }
    if (nc <= 10) { BPT_LN_FWD(10); }
    BPT_LN_FWD(16);
  }
#undef BPT_LN_FWD
  BPT_T(ti, TI, BPT_T(to, TO,
        hipLaunchKernelGGL((ln_fwd_kernel<TI, TO>), grid, dim3(256), 0, s, (const TI*)x, ldx, g, b,
                           (TO*)out, ldo, mu, rstd, rows, D, eps, use_stats)));
  return hipGetLastError();
}

// Workgroups of a PARAM launch, each leaving one partial row per sum: about two per CU
// (8 waves, enough loads in flight for HBM), never fewer than 8 rows each (4 where a workgroup
// takes one row at a time), and no more than the partial buffer holds. fp32 dY: 16384 x 4096 bf16 rows
// in 128 workgroups 321 us, in 512 117; 500 x 5120 rows in 63 workgroups 26.3 us, in 125 19.5.
static int ln_param_blocks(int64_t rows, int64_t D, int64_t partial_floats) {
  const int64_t fit = partial_floats / (2 * D), least = D <= 2048 ? 8 : 4;
  return (int)std::max<int64_t>(1, std::min<int64_t>({512, (rows + least - 1) / least, fit}));
}
int64_t layer_norm_bwd_partials(int64_t rows, int64_t D) { return 2 * D * ln_param_blocks(rows, D, INT64_MAX); }

template <typename TI, typename TD, typename TR, typename TO, typename T2, bool DROP>
static hipError_t ln_bwd_typed(const void* x, const float* mu, const float* rstd, const float* g, const void* dout,
                               const void* resid, void* out, void* out2, float* dgamma, float* dbeta, float* partial,
                               int64_t partial_floats, int64_t rows, int64_t D, RowMap map, const DropArgs& drop,
                               hipStream_t s) {
  const bool param = dgamma || dbeta;
  const int nblk = param ? ln_param_blocks(rows, D, partial_floats) : 0;
#define BPT_LN_BWD(NCV, WPRV)                                                                                     \
  do {                                                                                                            \
    if (param)                                                                                                    \
      hipLaunchKernelGGL((ln_bwd_reg_kernel<TI, TD, TR, TO, T2, NCV, WPRV, true, DROP>), dim3(nblk), dim3(256), 0, s, \
                         (const TI*)x, mu, rstd, g, (const TD*)dout, (const TR*)resid, (TO*)out, (T2*)out2,       \
                         partial, rows, (int)D, map, drop);                                                       \
    else                                                                                                          \
      hipLaunchKernelGGL((ln_bwd_reg_kernel<TI, TD, TR, TO, T2, NCV, WPRV, false, DROP>),                         \
                         dim3((unsigned)(WPRV == 4 ? rows : (rows + 3) / 4)), dim3(256), 0, s, (const TI*)x, mu,  \
                         rstd, g, (const TD*)dout, (const TR*)resid, (TO*)out, (T2*)out2, (float*)nullptr, rows,  \
                         (int)D, map, drop);                                                                      \
  } while (0)
  const int64_t nc = (D + 511) / 512;       // up to 2048 columns a wave holds the row, beyond that four waves do
  if (nc <= 1) BPT_LN_BWD(1, 1);
  else if (nc <= 2) BPT_LN_BWD(2, 1);
  else if (nc <= 4) BPT_LN_BWD(4, 1);
  else if (nc <= 8) BPT_LN_BWD(2, 4);
  else if (nc <= 12) BPT_LN_BWD(3, 4);
  else BPT_LN_BWD(4, 4);
#undef BPT_LN_BWD
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !param) return e;
  hipLaunchKernelGGL(chunk_reduce_kernel, dim3((unsigned)((D + 15) / 16)), dim3(256), 0, s, partial, nblk, dgamma,
                     dbeta, D, 0);
  return hipGetLastError();
}

static hipError_t layer_norm_param_grad(Dt ti, const void* x, const float* mu, const float* rstd, const float* dout,
                                        float* dgamma, float* dbeta, float* partial, int64_t rows, int64_t D,
                                        RowMap map, hipStream_t s);

bool layer_norm_bwd_fused(int64_t D) { return D % 8 == 0 && D <= 8192; }

hipError_t layer_norm_bwd(Dt ti, const void* x, const float* mu, const float* rstd, const float* g, Dt td,
                          const void* dout, Dt tr, const void* resid, Dt to, void* out, Dt t2, void* out2,
                          float* dgamma, float* dbeta, float* partial, int64_t partial_floats, int64_t rows, int64_t D,
                          int64_t seg, int64_t pitch, const DropArgs* drop, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  RowMap map;
  if (seg > 0) map.seg = seg, map.gap = pitch - seg;
  const bool param = dgamma || dbeta;
  const uintptr_t all = (uintptr_t)x | (uintptr_t)dout | (uintptr_t)resid | (uintptr_t)out | (uintptr_t)out2 |
                        (uintptr_t)g | (uintptr_t)partial;
  if (layer_norm_bwd_fused(D) && (all & 15) == 0) {
    // the type combinations in use: LN2 (dh and its rounded copy), LN1 (dX), the final LayerNorm
#define BPT_LN_IF(A, TD_, R, O, O2, TI, TD, TR, TO, T2)                                                          \
  if (ti == A && td == TD_ && (!resid || tr == R) && to == O && (!out2 || t2 == O2))                             \
    return ln_bwd_typed<TI, TD, TR, TO, T2, false>(x, mu, rstd, g, dout, resid, out, out2, dgamma, dbeta,        \
                                                   partial, partial_floats, rows, D, map, DropArgs(), s)
    if (drop) {                             // LN2 with dropout: the copy into the output projection
      if (ti != F32 || td != F32 || to != F32 || !out2 || tr != t2) return hipErrorInvalidValue;
      return t2 == BF16 ? ln_bwd_typed<float, float, bf16, float, bf16, true>(x, mu, rstd, g, dout, resid, out, out2, dgamma,
                                                                              dbeta, partial, partial_floats, rows, D, map,
                                                                              *drop, s)
                        : ln_bwd_typed<float, float, float, float, float, true>(x, mu, rstd, g, dout, resid, out, out2,
                                                                                dgamma, dbeta, partial, partial_floats,
                                                                                rows, D, map, *drop, s);
    }
    BPT_LN_IF(F32, F32, F32, F32, F32, float, float, float, float, float);
    BPT_LN_IF(F32, F32, BF16, F32, BF16, float, float, bf16, float, bf16);
    BPT_LN_IF(F32, F32, F32, BF16, BF16, float, float, float, bf16, bf16);
    BPT_LN_IF(BF16, F32, F32, F32, F32, bf16, float, float, float, float);
    BPT_LN_IF(BF16, F32, F32, BF16, BF16, bf16, float, float, bf16, bf16);
    BPT_LN_IF(F32, BF16, F32, F32, F32, float, bf16, float, float, float);
    BPT_LN_IF(BF16, BF16, F32, BF16, BF16, bf16, bf16, float, bf16, bf16);
#undef BPT_LN_IF
  }
  if (td != F32 || drop) return hipErrorInvalidValue;   // the caller widens dout and masks rows this long
  const dim3 grid((unsigned)((rows + 3) / 4));
  BPT_T(ti, TI, BPT_T(tr, TR, BPT_T(to, TO, BPT_T(t2, T2,
        hipLaunchKernelGGL((ln_bwd_kernel<TI, TR, TO, T2>), grid, dim3(256), 0, s, (const TI*)x, mu,
                           rstd, g, (const float*)dout, (const TR*)resid, (TO*)out, (T2*)out2, rows, D, map)))));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !param) return e;
  return layer_norm_param_grad(ti, x, mu, rstd, (const float*)dout, dgamma, dbeta, partial, rows, D, map, s);
}

size_t layer_norm_param_grad_ws(int64_t D) { return (size_t)2 * kChunks * (size_t)D; }

static hipError_t layer_norm_param_grad(Dt ti, const void* x, const float* mu, const float* rstd, const float* dout,
                                        float* dgamma, float* dbeta, float* partial, int64_t rows, int64_t D,
                                        RowMap map, hipStream_t s) {
  const dim3 grid8((unsigned)((D + 511) / 512), kChunks);
  BPT_T(ti, TI, hipLaunchKernelGGL((ln_param_partial8_kernel<TI>), grid8, dim3(256), 0, s, (const TI*)x,
                                   mu, rstd, dout, partial, rows, D, map));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chunk_reduce_kernel, dim3((unsigned)((D + 15) / 16)), dim3(256), 0, s, partial, kChunks,
                     dgamma, dbeta, D, 0);
  return hipGetLastError();
}

hipError_t col_sum(Dt t, const void* in, int64_t ld, int64_t rows, int64_t cols, float* out, float* partial,
                   int64_t partial_floats, hipStream_t s) {
  if (cols % 8 || ld % 8 || ((uintptr_t)in & 15) || ((uintptr_t)partial & 15) || partial_floats < cols)
    return hipErrorInvalidValue;
  // about 1024 blocks (four per CU), of at least 16 rows each
  const int64_t gx = (cols + 511) / 512;
  const int64_t nch = std::max<int64_t>(1, std::min<int64_t>({1024 / gx, (rows + 15) / 16, partial_floats / cols, 512}));
  const int64_t per = (rows + nch - 1) / nch;
  BPT_T(t, T, hipLaunchKernelGGL((col_partial8_kernel<T>), dim3((unsigned)gx, (unsigned)nch), dim3(256), 0, s, (const T*)in,
                                 ld, rows, per, cols, partial));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chunk_reduce_kernel, dim3((unsigned)((cols + 15) / 16)), dim3(256), 0, s, partial, (int)nch,
                     out, (float*)nullptr, cols, 0);
  return hipGetLastError();
}

hipError_t row_sum(Dt t, const void* in, int64_t ld, int64_t rows, int64_t cols, float* out,
                   int accumulate, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 3) / 4));
  if (ld % 8 == 0 && ((uintptr_t)in & 15) == 0)
    BPT_T(t, T, hipLaunchKernelGGL((row_sum8_kernel<T>), grid, dim3(256), 0, s, (const T*)in, ld, rows, cols, out,
                                   accumulate));
  else
    BPT_T(t, T, hipLaunchKernelGGL((row_sum_kernel<T>), grid, dim3(256), 0, s, (const T*)in, ld, rows, cols, out,
                                   accumulate));
  return hipGetLastError();
}

hipError_t attn_delta(Dt t, const void* dout, const void* o, int64_t ld, const float* lse, float* ndelta,
                      float* nlse2, int B, int64_t S, int64_t Sp, int H, int dh, hipStream_t s) {
  // one wave per token; a head spans whole 16-byte loads
  const int64_t n = (int64_t)B * Sp;
  if (dh % (t == F32 ? 4 : 8) != 0) return hipErrorInvalidValue;
  BPT_T(t, T, hipLaunchKernelGGL((delta_kernel<T>), dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s,
                                 (const T*)dout, (const T*)o, ld, lse, ndelta, nlse2, B, S, Sp, H, dh));
  return hipGetLastError();
}

hipError_t xent_rows(const float* z, int64_t ld, int64_t rows, int64_t V, const int32_t* tgt, float* lse,
                     float* tok, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (ld % 4 != 0 || ((uintptr_t)z & 15) != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(xent_rows_kernel, dim3((unsigned)rows), dim3(256), 0, s, z, ld, V, tgt, lse, tok);
  return hipGetLastError();
}

hipError_t xent_merge(const float* part, int64_t ng, int64_t rows, int64_t V, const int32_t* tgt, const float* tlogit,
                      float* lse, float* tok, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(xent_merge_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, part, ng, rows, V, tgt, tlogit,
                     lse, tok);
  return hipGetLastError();
}

hipError_t mean_of(const float* x, int64_t n, float* out, hipStream_t s) {
  if (n <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(1024), 0, s, x, n, out);
  return hipGetLastError();
}

// Slices of K are added in order, four columns per thread; columns of up to three outputs.
__global__ __launch_bounds__(256) void sum_slices_kernel(const float* part, int nz, int64_t n, int64_t cols4, float* o0,
                                                         float* o1, float* o2, int64_t nper4, int accumulate) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;      // group of four
  if (4 * q >= n) return;
  float* out = o0;
  int64_t at = q;
  if (nper4 > 0) {
    const int64_t m = q / cols4, c = q - m * cols4;
    const int w = c >= 2 * nper4 ? 2 : c >= nper4 ? 1 : 0;
    out = w == 2 ? o2 : w ? o1 : o0;
    at = m * nper4 + c - w * nper4;
  }
  f32x4 acc = accumulate ? ((const f32x4*)out)[at] : f32x4{0, 0, 0, 0};
  int z = 0;
  for (; z + 4 <= nz; z += 4) {                                   // four loads in flight
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = ((const f32x4*)(part + (z + u) * n))[q];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += v[u];
  }
  for (; z < nz; ++z) acc += ((const f32x4*)(part + z * n))[q];
  ((f32x4*)out)[at] = acc;
}

template <typename TR, typename TO>
__global__ __launch_bounds__(256) void sum_slices_add_kernel(const float* part, int nz, int64_t n, int64_t cols, const TR* R,
                                                             const float* bias, TO* out) {
  const int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);      // group of four
  if (i >= n) return;
  f32x4 acc = *(const f32x4*)(part + i);
#pragma unroll 4
  for (int z = 1; z < nz; ++z) acc += *(const f32x4*)(part + z * n + i);
  float v[4] = {acc[0], acc[1], acc[2], acc[3]};
  if (R) {
    float r[4];
    Vec4<TR>::load(R + i, r);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += r[e];
  }
  if (bias) {
    float b[4];
    Vec4<float>::load(bias + i % cols, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += b[e];
  }
  Vec4<TO>::store(out + i, v);
}

hipError_t sum_slices_add(const float* part, int nz, int64_t rows, int64_t cols, Dt tr, const void* R, const float* bias,
                          Dt to, void* out, hipStream_t s) {
  const int64_t n = rows * cols;
  if (n <= 0) return hipSuccess;
  if (cols % 4 != 0) return hipErrorInvalidValue;
  BPT_T(tr, TR, BPT_T(to, TO,
        hipLaunchKernelGGL((sum_slices_add_kernel<TR, TO>), dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, part,
                           nz, n, cols, (const TR*)R, bias, (TO*)out)));
  return hipGetLastError();
}

hipError_t sum_slices(const float* part, int nz, int64_t rows, int64_t cols, float* const outs[3], int64_t nper,
                      int accumulate, hipStream_t s) {
  const int64_t n = rows * cols;
  if (n <= 0) return hipSuccess;
  if (cols % 4 != 0 || nper % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sum_slices_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, part, nz, n, cols / 4,
                     outs[0], nper > 0 ? outs[1] : nullptr, nper > 0 ? outs[2] : nullptr, nper / 4, accumulate);
  return hipGetLastError();
}

}  // namespace bpt
