// Kernels of a GPT training step around the layer (the models of Section 5): the
// token + position embedding and its gradients, an elementwise conversion to fp32,
// and the AdamW update. All are HBM-bound streams: every element is read once and
// written once, 16-byte accesses where the layout allows.
#include "common.h"
#include "internal.h"

namespace bpt {

namespace {

// 8 consecutive elements as floats (16-byte loads for bf16, 2 x 16 for fp32)
BPT_DEV void ld8(const float* p, float v[8]) {
  const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}
BPT_DEV void ld8(const bf16* p, float v[8]) {
  const bf16x8 x = *(const bf16x8*)p;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)x[e];
}
BPT_DEV void st8(float* p, const float v[8]) {
  *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]};
  *(f32x4*)(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
}
BPT_DEV void st8(bf16* p, const float v[8]) {
  bf16x8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (bf16)v[e];
  *(bf16x8*)p = x;
}

}  // namespace

// X[t] = Wte[tok[t]] + Wpe[t mod S]: one wave per token row, 8 columns per lane and
// step; the sum is formed in fp32 and rounded once. NaN row for a token outside [0, V).
template <typename T>
__global__ __launch_bounds__(256) void embed_fwd_kernel(const int32_t* tok, const T* Wte, const T* Wpe, T* X,
                                                        int64_t rows, int64_t S, int64_t D, int64_t V) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= rows) return;
  const int64_t y = tok[t];
  const bool ok = y >= 0 && y < V;
  const T* er = Wte + (ok ? y : 0) * D;
  const T* pr = Wpe ? Wpe + (t % S) * D : nullptr;
  for (int64_t d = 8 * lane; d < D; d += 512) {
    float a[8], b[8];
    ld8(er + d, a);
    if (pr) {
      ld8(pr + d, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] += b[e];
    }
    if (!ok) {
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = __builtin_nanf("");
    }
    st8(X + t * D + d, a);
  }
}

// dWte[v] = sum of dX[t] over the tokens t equal to v, in a fixed order (the parts of a list per
// wave, each in token order, then the lists); 0 for a row no token names. Owner computes: workgroup (x, y) owns the rows v = x + r NV (NV a power of two, at
// most kRows rows) in columns [512 y, 512 y + 512). It scans the token ids (which stay in
// L2), lists the tokens of its rows in LDS, ordered by row and token, and each of its waves
// adds up an eighth of the list, many rows of dX in flight whatever rows they belong to. A list
// holds kList tokens of a chunk of kChunk ids; the first writes every row of its workgroup, each
// further one the rows it names, on top of what is there: dWte needs neither clearing nor atomics.
//
// Bound by the V D fp32 stores and the latency of the dX reads; the interleaved rows spread
// the frequent (low) ids over the workgroups, the even parts over their waves.
// 16384 tokens by a 1/rank law, D = 2048, V = 50257: 156 us (fp32 atomics, 8 strided
// adds per lane: 984 us, and 59 us of clearing). An id that dominates is added up by one workgroup
// per 512 columns: 32768 tokens, 90 % of them one id: 1.02 ms (atomics 6.5), fp32 2.3 (6.5).
constexpr int kChunk = 16384, kList = 2048, kRows = 512, kWaves = 8;

// 4 elements as loaded
template <typename T> struct Raw4;
template <> struct Raw4<float> {
  f32x4 q;
  BPT_DEV void load(const float* p) { q = *(const f32x4*)p; }
  BPT_DEV f32x4 get() const { return q; }
};
template <> struct Raw4<bf16> {
  u32x2 q;
  BPT_DEV void load(const bf16* p) { q = *(const u32x2*)p; }
  BPT_DEV f32x4 get() const {
    return f32x4{__uint_as_float(q[0] << 16), __uint_as_float(q[0] & 0xFFFF0000u), __uint_as_float(q[1] << 16),
                 __uint_as_float(q[1] & 0xFFFF0000u)};
  }
};

template <typename T>
__global__ __launch_bounds__(64 * kWaves) void embed_dwte_kernel(const int32_t* tok, const T* dX, float* dWte, int64_t rows,
                                                         int64_t D, int64_t V, int lnv) {
  __shared__ uint32_t list[kList], sorted[kList];   // row << 16 | token index in the chunk
  __shared__ int cnt[kRows], start[kRows], wtot[kWaves], headrow[kWaves];
  __shared__ __attribute__((aligned(16))) float red[kWaves][512];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = blockIdx.x, nv = 1 << lnv;
  const int nr = (int)((V - grp + nv - 1) >> lnv);  // rows of this workgroup
  // two groups of 4 columns per lane, 256 apart: every store of a wave is 1 KiB in a row
  const int64_t col0 = (int64_t)blockIdx.y * 512 + 4 * lane, col1 = col0 + 256;
  const bool in0 = col0 < D, in1 = col1 < D;        // D % 8 == 0
  const int64_t lc0 = in0 ? col0 : 0, lc1 = in1 ? col1 : 0;
  constexpr int PER = kChunk / (64 * kWaves);                 // tokens per lane and chunk
  bool first = true;                                // no list has been added yet
  int64_t c0 = 0;
  int base = 0;                                     // entries of this chunk in earlier lists
  while (true) {
    for (int i = tid; i < kRows; i += 64 * kWaves) cnt[i] = 0;
    // this wave's share of the chunk's token ids
    const int64_t w0 = c0 + wave * (kChunk / kWaves);
    // segment i of it: tokens w0 + 256 i + 4 lane .. + 3; bit j: token j names a row of ours
    auto match = [&](int i, int (&r)[4]) {
      const int64_t t = w0 + 256 * i + 4 * lane;
      int y[4] = {-1, -1, -1, -1};
      if (t + 4 <= rows) {
        const u32x4 q = *(const u32x4*)(tok + t);   // t % 4 == 0, tok 16-byte aligned
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = (int)q[j];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (t + j < rows) y[j] = tok[t + j];
      }
      uint32_t hit = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        hit |= (uint32_t)y[j] < (uint32_t)V && (y[j] & (nv - 1)) == grp ? 1u << j : 0u;
        r[j] = y[j] >> lnv;
      }
      return hit;
    };
    int n = 0;
#pragma unroll 4
    for (int i = 0; i < PER / 4; ++i) {
      int r[4];
      n += __popc(match(i, r));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0) wtot[wave] = n;
    __syncthreads();
    int pos = -base, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) pos += wtot[w];
      total += wtot[w];
    }
#pragma unroll 4
    for (int i = 0; i < PER / 4; ++i) {
      int r[4];
      const uint32_t hit = match(i, r);
      if (!__ballot(hit != 0)) continue;
      const uint64_t below = (1ull << lane) - 1;    // matches of the lanes before this one
      const int c = __popc(hit);
      const uint64_t b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4);
      int at = pos + __popcll(b0 & below) + 2 * __popcll(b1 & below) + 4 * __popcll(b2 & below);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (hit >> j & 1) {
          if (at >= 0 && at < kList) {
            list[at] = (uint32_t)r[j] << 16 | (uint32_t)(wave * (kChunk / kWaves) + 256 * i + 4 * lane + j);
            atomicAdd(&cnt[r[j]], 1);
          }
          ++at;
        }
      pos += __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
    }
    const int len = total - base < kList ? total - base : kList;
    __syncthreads();
    // order the list by row, tokens of a row in order: start[r] = first place of row r, then
    // one wave deals the entries out, 64 at a time and one row of those at a time
    if (len > 0) {
      if (wave == 0) {
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kRows / 64; ++i) {
          const int c = cnt[64 * i + lane];
          int x = c;                                // inclusive prefix over the lanes
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
          }
          start[64 * i + lane] = sum + x - c;
          sum += __shfl(x, 63, 64);
        }
        for (int i = 0; i < len; i += 64) {
          const bool have = i + lane < len;
          const uint32_t e = have ? list[i + lane] : 0u;
          uint64_t left = __ballot(have);
          while (left) {
            const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)e, __builtin_ctzll(left)) >> 16;
            const uint64_t same = __ballot(have && e >> 16 == r);
            const int at = start[r];
            if (same >> lane & 1) sorted[at + __popcll(same & ((1ull << lane) - 1))] = e;
            if (lane == 0) start[r] = at + __popcll(same);
            left &= ~same;
          }
        }
      }
      __syncthreads();
    }
    auto load_row = [&](int r, f32x4& a0, f32x4& a1) {
      const float* out = dWte + ((int64_t)grp + ((int64_t)r << lnv)) * D;
      if (in0) a0 += *(const f32x4*)(out + col0);
      if (in1) a1 += *(const f32x4*)(out + col1);
    };
    auto store_row = [&](int r, const f32x4& a0, const f32x4& a1) {
      float* out = dWte + ((int64_t)grp + ((int64_t)r << lnv)) * D;
      if (in0) *(f32x4*)(out + col0) = a0;
      if (in1) *(f32x4*)(out + col1) = a1;
    };
    // A wave adds an equal part of the sorted list, UF dX rows in flight. A row that begins in
    // its part is its own to store; the part of a row that began in an earlier one goes to LDS.
    const int q = (len + kWaves - 1) / kWaves, i0 = wave * q < len ? wave * q : len, i1 = i0 + q < len ? i0 + q : len;
    int row = -1;                                   // the row being added
    bool head = false;                              // it began in an earlier part
    f32x4 a0 = {}, a1 = {};
    if (lane == 0) headrow[wave] = -1;
    auto flush = [&]() {
      if (row < 0) return;
      if (head) {
        *(f32x4*)&red[wave][4 * lane] = a0;
        *(f32x4*)&red[wave][256 + 4 * lane] = a1;
        if (lane == 0) headrow[wave] = row;
      } else {
        if (!first) load_row(row, a0, a1);
        store_row(row, a0, a1);
      }
      row = -1;
    };
    constexpr int UF = sizeof(T) == 2 ? 16 : 8;      // dX rows in flight
    if (i0 < i1) {
      head = i0 > 0 && sorted[i0 - 1] >> 16 == sorted[i0] >> 16;
      for (int i = i0; i < i1; i += UF) {
        const int k = i1 - i < UF ? i1 - i : UF;
        const uint32_t el = lane < k ? sorted[i + lane] : 0u;
        uint32_t e[UF];
        Raw4<T> v0[UF], v1[UF];
#pragma unroll
        for (int u = 0; u < UF; ++u)
          if (u < k) {
            e[u] = (uint32_t)__builtin_amdgcn_readlane((int)el, u);
            const T* p = dX + (c0 + (int64_t)(e[u] & 0xFFFF)) * D;
            v0[u].load(p + lc0);
            v1[u].load(p + lc1);
          }
#pragma unroll
        for (int u = 0; u < UF; ++u)
          if (u < k) {
            if (row != (int)(e[u] >> 16)) {
              if (row >= 0) {
                flush();
                head = false;
              }
              row = (int)(e[u] >> 16);
              a0 = a1 = f32x4{};
            }
            a0 += v0[u].get();
            a1 += v1[u].get();
          }
      }
      if (head) flush();                            // the whole part belongs to one row
    }
    if (first)                                      // rows no token of the first list names
      for (int r = wave; r < nr; r += kWaves)
        if (cnt[r] == 0) store_row(r, f32x4{}, f32x4{});
    if (len > 0) {
      __syncthreads();
      if (row >= 0) {                               // the last row of the part, with what follows it
        for (int w = wave + 1; w < kWaves; ++w) {
          if (headrow[w] != row) break;
          a0 += *(const f32x4*)&red[w][4 * lane];
          a1 += *(const f32x4*)&red[w][256 + 4 * lane];
        }
        flush();
      }
    }
    first = false;
    base += kList;
    if (base >= total) {                            // the next chunk of token ids
      base = 0;
      c0 += kChunk;
      if (c0 >= rows) return;
    }
    __syncthreads();                                // the next list takes this one's place
  }
}

// dWpe[s] = sum_b dX[b S + s], summed in batch order: 8 columns per thread.
template <typename T>
__global__ __launch_bounds__(256) void embed_dwpe_kernel(const T* dX, float* dWpe, int64_t B, int64_t S,
                                                         int64_t D) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= S * D) return;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t b = 0; b < B; ++b) {
    float g[8];
    ld8(dX + b * S * D + i, g);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += g[e];
  }
  st8(dWpe + i, acc);
}

// out[i] = (float)in[i], 8 elements per thread (n a multiple of 8)
__global__ __launch_bounds__(256) void bf16_to_f32_kernel(const bf16* in, float* out, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  float v[8];
  ld8(in + i, v);
  st8(out + i, v);
}

// One AdamW step. c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t) (formed in double on the
// host). Four elements per thread with 16-byte accesses; the last n mod 4 elements
// one by one. Grid-stride over the groups of four.
template <typename TL>
__global__ __launch_bounds__(256) void adamw_kernel(float* p, const float* g, float* m, float* v, TL* pl,
                                                    int64_t n, float lr, float b1, float b2, float eps,
                                                    float wd, float c1, float c2) {
  const float decay = 1.0f - lr * wd;
  auto one = [&](float& pp, float gg, float& mm, float& vv) {
    mm = b1 * mm + (1.0f - b1) * gg;
    vv = b2 * vv + (1.0f - b2) * gg * gg;
    pp = pp * decay - lr * (mm * c1) / (sqrtf(vv * c2) + eps);
  };
  const int64_t n4 = n / 4;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n4; q += stride) {
    f32x4 pp = ((const f32x4*)p)[q], mm = ((const f32x4*)m)[q], vv = ((const f32x4*)v)[q];
    const f32x4 gg = ((const f32x4*)g)[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float a = pp[e], b = mm[e], c = vv[e];
      one(a, gg[e], b, c);
      pp[e] = a; mm[e] = b; vv[e] = c;
    }
    ((f32x4*)p)[q] = pp;
    ((f32x4*)m)[q] = mm;
    ((f32x4*)v)[q] = vv;
    if (pl) {
      if constexpr (sizeof(TL) == 2) {
        bf16x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (bf16)pp[e];
        ((bf16x4*)pl)[q] = x;
      } else {
        ((f32x4*)pl)[q] = pp;
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)(n - 4 * n4)) {
    const int64_t i = 4 * n4 + threadIdx.x;
    float a = p[i], b = m[i], c = v[i];
    one(a, g[i], b, c);
    p[i] = a; m[i] = b; v[i] = c;
    if (pl) pl[i] = (TL)a;
  }
}

// ------------------------------------------------------------------ launchers
hipError_t embed_fwd(Dt t, const int32_t* tok, const void* Wte, const void* Wpe, void* X, int64_t rows,
                     int64_t S, int64_t D, int64_t V, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 3) / 4));
  if (t == F32)
    hipLaunchKernelGGL(embed_fwd_kernel<float>, grid, dim3(256), 0, s, tok, (const float*)Wte,
                       (const float*)Wpe, (float*)X, rows, S, D, V);
  else
    hipLaunchKernelGGL(embed_fwd_kernel<bf16>, grid, dim3(256), 0, s, tok, (const bf16*)Wte,
                       (const bf16*)Wpe, (bf16*)X, rows, S, D, V);
  return hipGetLastError();
}

hipError_t embed_dwte(Dt t, const int32_t* tok, const void* dX, float* dWte, int64_t rows, int64_t D, int64_t V,
                      hipStream_t s) {
  // Row groups: enough that a group has at most kRows rows, and up to 512 workgroups while
  // rows last: two per CU, all resident at once.
  const int64_t slices = (D + 511) / 512;
  int lnv = 0;
  while (((V + ((int64_t)1 << lnv) - 1) >> lnv) > kRows) ++lnv;
  while (((int64_t)2 << lnv) <= V && (((int64_t)2 << lnv) * slices) <= 512) ++lnv;
  const dim3 grid((unsigned)(1 << lnv), (unsigned)slices);
  if (t == F32)
    hipLaunchKernelGGL(embed_dwte_kernel<float>, grid, dim3(64 * kWaves), 0, s, tok, (const float*)dX, dWte, rows, D, V, lnv);
  else
    hipLaunchKernelGGL(embed_dwte_kernel<bf16>, grid, dim3(64 * kWaves), 0, s, tok, (const bf16*)dX, dWte, rows, D, V, lnv);
  return hipGetLastError();
}

hipError_t embed_dwpe(Dt t, const void* dX, float* dWpe, int64_t B, int64_t S, int64_t D, hipStream_t s) {
  const int64_t n8 = S * D / 8;
  if (n8 <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n8 + 255) / 256));
  if (t == F32)
    hipLaunchKernelGGL(embed_dwpe_kernel<float>, grid, dim3(256), 0, s, (const float*)dX, dWpe, B, S, D);
  else
    hipLaunchKernelGGL(embed_dwpe_kernel<bf16>, grid, dim3(256), 0, s, (const bf16*)dX, dWpe, B, S, D);
  return hipGetLastError();
}

hipError_t bf16_to_f32(const void* in, float* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bf16_to_f32_kernel, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, s,
                     (const bf16*)in, out, n);
  return hipGetLastError();
}

hipError_t adamw(Dt tl, float* p, const float* g, float* m, float* v, void* pl, int64_t n, float lr, float b1,
                 float b2, float eps, float wd, float c1, float c2, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t groups = (n + 3) / 4;
  const unsigned grid = (unsigned)std::min<int64_t>((groups + 255) / 256, 8192);
  if (tl == F32)
    hipLaunchKernelGGL(adamw_kernel<float>, dim3(grid), dim3(256), 0, s, p, g, m, v, (float*)pl, n, lr, b1, b2,
                       eps, wd, c1, c2);
  else
    hipLaunchKernelGGL(adamw_kernel<bf16>, dim3(grid), dim3(256), 0, s, p, g, m, v, (bf16*)pl, n, lr, b1, b2,
                       eps, wd, c1, c2);
  return hipGetLastError();
}

}  // namespace bpt
