// Attention backward, key-outer dK/dV kernel (bf16 and fp32 MFMA variants).
#include <algorithm>

#include "attn_common.h"

namespace bpt {

// ====================================================================== backward dK dV, bf16
// Key-outer: 8 waves (two per SIMD, so one wave's VALU work overlaps the other's
// MFMAs) of 32 keys each, 256 keys per workgroup (or 4 waves, 128: few_blocks), loop over query tiles of 64 (two
// halves of 32). S = Q K^T and dP = dO V^T have the key on the lane axis, so P and dS
// feed dV^T += dO^T P and dK^T += Q^T dS directly as B operands; dO^T and Q^T
// fragments come from the token-major tiles by transposing LDS reads. Q carries
// log2(e)/sqrt(dh), and the score MFMAs start from minus the base-2 log-sum-exp of
// their query rows, so exp2 of the accumulator is P; dK = sqrt(dh)^-1 dS^T Q then
// comes out as ln(2) dS^T (Q log2(e)/sqrt(dh)).
// Query tiles are visited from the last one down, so all workgroups of a head start
// on the same tiles (and share them in L2); the diagonal tiles come last.
template <int DH, int NWAVES>
struct DkvCfg {
  static constexpr int KSTEPS = DH / 16, DT = DH / 32;
  static constexpr int NW = NWAVES;                 // waves per workgroup: 8, or 4 (few_blocks)
  static constexpr int KEYS = 32 * NW;              // keys per workgroup
  static constexpr int TB = RmTile<DH>::BYTES;
  static constexpr int STAGE = 2 * TB + 2 * 64 * 4; // Q, dO tiles; -lse (base 2), -Delta
  static constexpr int NS = NW == 8 || DH == 64 ? 4 : 2;   // stages in the ring
  static constexpr int LDS = NS * STAGE;
  static constexpr int DPS = Ring2<DH, NW>::DPW + 2;  // copies per wave per stage
};

template <int DH, int NWAVES>
__global__ __launch_bounds__(64 * NWAVES, NWAVES == 8 ? 1 : 2) void attn_bwd_dkdv_bf16_kernel(AttnArgs a) {
  using C = DkvCfg<DH, NWAVES>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = (int)a.S;
  int hh, blk;
  xcd_map_heads((int)blockIdx.x, a.H * a.B, (S + C::KEYS - 1) / C::KEYS, hh, blk);
  const int h = hh % a.H, b = hh / a.H;
  const int k0 = blk * C::KEYS;                     // causal: low key blocks have the most queries
  const int kw = k0 + 32 * wave;                    // first key of this wave
  const int key = kw + (lane & 31);

  const bf16* Qb = (const bf16*)a.q + (int64_t)b * a.S * a.ld_q + h * DH;
  const bf16* Kb = (const bf16*)a.k + (int64_t)b * a.S * a.ld_k + h * DH;
  const bf16* Vb = (const bf16*)a.v + (int64_t)b * a.S * a.ld_v + h * DH;
  const bf16* dOb = (const bf16*)a.dout + (int64_t)b * a.S * a.ld_do + h * DH;
  const float* nlse2 = a.nlse2 + ((int64_t)b * a.H + h) * a.Sp;
  const float* ndelta = a.ndelta + ((int64_t)b * a.H + h) * a.Sp;

  bf16x8 kf[C::KSTEPS], vf[C::KSTEPS];
  {
    const int kr = key < S ? key : S - 1;
#pragma unroll
    for (int kk = 0; kk < C::KSTEPS; ++kk) {
      kf[kk] = __builtin_bit_cast(bf16x8, ld16(Kb + (int64_t)kr * a.ld_k + 16 * kk + 8 * (lane >> 5)));
      vf[kk] = __builtin_bit_cast(bf16x8, ld16(Vb + (int64_t)kr * a.ld_v + 16 * kk + 8 * (lane >> 5)));
      settle(kf[kk]);
      settle(vf[kk]);
    }
  }

  const int qstart = a.causal ? k0 : 0;             // a multiple of 64
  const int ntiles = qstart < S ? (S - qstart + 63) / 64 : 0;
  const int n_diag = a.causal ? C::KEYS / 64 : 0;   // tiles jt < n_diag straddle the keys
  // iteration it visits query tile jt = ntiles - 1 - it
  auto issue = [&](int it) {
    const int qt0 = qstart + 64 * (ntiles - 1 - it);
    char* st = smem + (it % C::NS) * C::STAGE;
    ring_issue<DH, C::NW>(st, Qb, (int)a.ld_q, qt0, dOb, (int)a.ld_do, qt0, S - 1, wave, lane);
    // -lse (base 2) and -Delta of the 64 queries (indices < Sp: in bounds; rows >= S are
    // masked); every wave copies them, so that all waves count the same copies
    dma4s(nlse2 + qt0, 4u * lane, st + 2 * C::TB);
    dma4s(ndelta + qt0, 4u * lane, st + 2 * C::TB + 256);
  };

  f32x16 adv[C::DT], adk[C::DT];
#pragma unroll
  for (int t = 0; t < C::DT; ++t) adv[t] = adk[t] = f32x16{};

  auto tile = [&](int it, auto MASK) {
    const int qt0 = qstart + 64 * (ntiles - 1 - it);
    const char* qs = smem + (it % C::NS) * C::STAGE;
    const char* ds = qs + C::TB;
    const float* ls = (const float*)(qs + 2 * C::TB);
    // query offset inside the tile of register r: 32*mt + acc_row(r, lane); visible
    // iff lo <= offset <= hi
    const int lo = a.causal ? key - qt0 : 0;
    const int hi = key < S ? S - 1 - qt0 : -1;
    // the lane part of the offset moves into the bounds, so that every comparison is
    // against a constant
    const int lo4 = lo - 4 * (lane >> 5), hi4 = hi - 4 * (lane >> 5);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      // S starts from -lse and dP from -Delta of their query rows, so the MFMAs leave
      // the exponent of P and dP - Delta
      f32x16 s, dp;
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int qi = 32 * mt + 8 * rg + 4 * (lane >> 5);
        const f32x4 l4 = *(const f32x4*)(ls + qi);
        const f32x4 d4 = *(const f32x4*)(ls + 64 + qi);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[4 * rg + e] = l4[e];
          dp[4 * rg + e] = d4[e];
        }
      }
#pragma unroll
      for (int kk = 0; kk < C::KSTEPS; ++kk) {
        s = mfma32x32x16(frag_rows<DH>(qs, 32 * mt, 2 * kk, lane), kf[kk], s);
        dp = mfma32x32x16(frag_rows<DH>(ds, 32 * mt, 2 * kk, lane), vf[kk], dp);
        __builtin_amdgcn_sched_barrier(0);        // bound the fragments read ahead
      }
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * rg + e;
          float p = fast_exp2(s[r]);
          if constexpr (decltype(MASK)::value) {
            const int off = 32 * mt + 8 * rg + e;
            p = (off >= lo4 && off <= hi4) ? p : 0.0f;
          }
          s[r] = p;
          dp[r] = p * dp[r];                           // dS
        }
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bf16x8 pb = acc_to_b(s, hf), sb = acc_to_b(dp, hf);
#pragma unroll
        for (int t = 0; t < C::DT; ++t) {
          adv[t] = mfma32x32x16(frag_tr<DH>(ds, 32 * mt + 16 * hf, 32 * t, lane), pb, adv[t]);
          adk[t] = mfma32x32x16(frag_tr<DH>(qs, 32 * mt + 16 * hf, 32 * t, lane), sb, adk[t]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };

  // Phases, each a loop over one tile body (uniform over the workgroup, so every
  // barrier is reached by all waves): the ragged last query tile (masked), the tiles
  // every key of the workgroup fully sees (unmasked), and the tiles that straddle the
  // workgroup's keys (masked); a wave skips the arithmetic of tiles entirely before
  // its keys.
  const bool ragged = ntiles > 0 && qstart + 64 * (ntiles - 1) + 63 >= S;
  const int it_a = ragged ? 1 : 0;
  const int it_b = k0 + C::KEYS > S ? it_a : std::max(it_a, ntiles - n_diag);
  auto step = [&](int it) {
    if (C::NS == 4 && it + 2 < ntiles) wait_vmcnt<2 * C::DPS>();
    else if (C::NS == 4 && it + 1 < ntiles) wait_vmcnt<C::DPS>();
    else wait_vmcnt<0>();
    __syncthreads();                  // stage it visible; every wave is done with stage it-1
    if (it + C::NS - 1 < ntiles) issue(it + C::NS - 1);  // into the slot of stage it-1
  };
  auto visible = [&](int it) { return !(a.causal && qstart + 64 * (ntiles - 1 - it) + 63 < kw); };
#pragma unroll
  for (int st = 0; st < C::NS - 1; ++st)
    if (st < ntiles) issue(st);
  int it = 0;
  for (; it < it_a; ++it) {
    step(it);
    if (visible(it)) tile(it, std::true_type{});
  }
  for (; it < it_b; ++it) {
    step(it);
    tile(it, std::false_type{});
  }
  for (; it < ntiles; ++it) {
    step(it);
    if (visible(it)) tile(it, std::true_type{});
  }

  if (key < a.Sp) {
    const int64_t col = (int64_t)b * a.Sp + key;
    bf16* dKt = (bf16*)a.dkt + (int64_t)h * DH * a.ld_dt + col;
    bf16* dVt = (bf16*)a.dvt + (int64_t)h * DH * a.ld_dt + col;
#pragma unroll
    for (int t = 0; t < C::DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t d = 32 * t + acc_row(r, lane);
        dKt[d * a.ld_dt] = (bf16)(adk[t][r] * LN2);
        dVt[d * a.ld_dt] = (bf16)adv[t][r];
      }
  }
}

// ====================================================================== backward dK dV, fp32
// 16 keys per workgroup; wave w takes the query tiles of 16 w, w + 4, ... S and dP have the
// key on the lane axis, so P and dS are the B operands of dV^T += dO^T P, dK^T += Q^T dS.
template <int DH>
__global__ __launch_bounds__(256) void attn_bwd_dkdv_f32_kernel(AttnArgs a) {
  constexpr int NC = DH / 16;
  __shared__ __attribute__((aligned(16))) float red[4][DH][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c16 = lane & 15;
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t S = a.S, k0 = (int64_t)blockIdx.x * 16, kv = k0 + c16;   // causal: low blocks have the most queries
  const float scale = rsqrtf((float)DH);
  const float* Qb = (const float*)a.q + (int64_t)b * S * a.ld_q + (int64_t)h * DH;
  const float* Kb = (const float*)a.k + (int64_t)b * S * a.ld_k + (int64_t)h * DH;
  const float* Vb = (const float*)a.v + (int64_t)b * S * a.ld_v + (int64_t)h * DH;
  const float* dOb = (const float*)a.dout + (int64_t)b * S * a.ld_do + (int64_t)h * DH;
  const float* lse = a.lse + ((int64_t)b * a.H + h) * a.Sp;
  const float* ndelta = a.ndelta + ((int64_t)b * a.H + h) * a.Sp;
  const int64_t kr = kv < S ? kv : S - 1;
  const RowFrag<DH> kf = row_frag<DH>(Kb + kr * a.ld_k, g), vf = row_frag<DH>(Vb + kr * a.ld_v, g);
  f32x4 dk[NC], dv[NC];
#pragma unroll
  for (int t = 0; t < NC; ++t) dk[t] = dv[t] = f32x4{};
  const int64_t qstart = a.causal ? k0 : 0;
  if (k0 < S)
    for (int64_t q0 = qstart + 16 * wave; q0 < S; q0 += 64) {
      const int64_t qr = q0 + c16 < S ? q0 + c16 : S - 1;
      const RowFrag<DH> qf = row_frag<DH>(Qb + qr * a.ld_q, g), of = row_frag<DH>(dOb + qr * a.ld_do, g);
      const f32x4 l4 = *(const f32x4*)(lse + q0 + 4 * g), d4 = *(const f32x4*)(ndelta + q0 + 4 * g);   // rows < Sp
      const ColFrag<DH> oc = col_frag<DH>(dOb, a.ld_do, q0, S - 1, g, c16);
      f32x4 p = dot_frags<DH>(qf, kf), ds = dot_frags<DH>(of, vf);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t q = q0 + 4 * g + r;
        const bool ok = q < S && kv < S && !(a.causal && kv > q);
        p[r] = ok ? fast_exp2((p[r] * scale - l4[r]) * LOG2E) : 0.0f;
        ds[r] = ok ? p[r] * (ds[r] + d4[r]) : 0.0f;
      }
      const ColFrag<DH> qc = col_frag<DH>(Qb, a.ld_q, q0, S - 1, g, c16);
      add_outer<DH>(dv, oc, p);
      add_outer<DH>(dk, qc, ds);
    }
  // add the four waves' parts, dK then dV, and store them feature-major
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NC; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][16 * t + 4 * g + r][c16] = which ? dv[t][r] : dk[t][r];
    __syncthreads();
    float* out = (float*)(which ? a.dvt : a.dkt) + (int64_t)h * DH * a.ld_dt + (int64_t)b * a.Sp + k0;
    const float f = which ? 1.0f : scale;
    for (int i = tid; i < 16 * DH; i += 256) {         // 16 consecutive keys of a feature
      const int d = i >> 4, k = i & 15;
      out[(int64_t)d * a.ld_dt + k] = (((red[0][d][k] + red[1][d][k]) + red[2][d][k]) + red[3][d][k]) * f;
    }
  }
}

template <int DH, int NW>
static hipError_t dkdv_launch_bf16(const AttnArgs& a, hipStream_t s) {
  using C = DkvCfg<DH, NW>;
  auto k = attn_bwd_dkdv_bf16_kernel<DH, NW>;
  hipError_t e = set_lds(k, C::LDS);
  if (e != hipSuccess) return e;
  const int64_t nblk = (a.S + C::KEYS - 1) / C::KEYS;
  hipLaunchKernelGGL(k, dim3((unsigned)(nblk * a.H * a.B)), dim3(64 * NW), C::LDS, s, a);
  return hipGetLastError();
}

template <int DH>
static hipError_t dkdv_launch(Dt dt, const AttnArgs& a, hipStream_t s) {
  if (a.S <= 0 || a.B <= 0) return hipSuccess;
  if (dt == BF16) {
    return few_blocks(a.S, (int64_t)a.H * a.B, a.causal) ? dkdv_launch_bf16<DH, 4>(a, s) : dkdv_launch_bf16<DH, 8>(a, s);
  } else {
    hipLaunchKernelGGL(attn_bwd_dkdv_f32_kernel<DH>, dim3((unsigned)(a.Sp / 16), a.H, a.B), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t attn_bwd_dkdv(Dt dt, const AttnArgs& a, hipStream_t s) {
  if (a.dh == 64) return dkdv_launch<64>(dt, a, s);
  if (a.dh == 128) return dkdv_launch<128>(dt, a, s);
  return hipErrorInvalidValue;
}

}  // namespace bpt
