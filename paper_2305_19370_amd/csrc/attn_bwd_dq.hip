// Attention backward, query-outer dQ kernel (bf16 and fp32 MFMA variants).
#include <algorithm>

#include "attn_common.h"

namespace bpt {

// ====================================================================== backward dQ, bf16
// Query-outer: 8 waves (two per SIMD, so one wave's VALU work overlaps the other's
// MFMAs) of 32 queries each, 256 per workgroup (or 4 waves, 128: few_blocks), loop over key tiles of 64:
// S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T. K^T
// fragments come from the K tile by transposing LDS reads. Q carries log2(e)/sqrt(dh),
// and the score MFMAs start from minus the base-2 log-sum-exp of the lane's query, so
// exp2 of the accumulator is P.
template <int DH, int NWAVES>
struct DqCfg {
  static constexpr int KSTEPS = DH / 16, DT = DH / 32;
  static constexpr int NW = NWAVES;                 // waves per workgroup: 8, or 4 (few_blocks)
  static constexpr int QROWS = 32 * NW;             // queries per workgroup
  static constexpr int TB = RmTile<DH>::BYTES;
  static constexpr int STAGE = 2 * TB;              // K and V tiles of 64 keys
  static constexpr int NS = NW == 8 || DH == 64 ? 4 : 2;   // stages in the ring
  static constexpr int LDS = NS * STAGE;
  static constexpr int DPS = Ring2<DH, NW>::DPW;    // copies per wave per stage
};

template <int DH, int NWAVES>
__global__ __launch_bounds__(64 * NWAVES, NWAVES == 8 ? 1 : 2) void attn_bwd_dq_bf16_kernel(AttnArgs a) {
  using C = DqCfg<DH, NWAVES>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = (int)a.S;
  const int nblk = (S + C::QROWS - 1) / C::QROWS;
  int hh, blk;
  xcd_map_heads((int)blockIdx.x, a.H * a.B, nblk, hh, blk);
  const int h = hh % a.H, b = hh / a.H;
  const int qt = a.causal ? nblk - 1 - blk : blk;   // causal: the blocks with the most keys first
  const int q0 = qt * C::QROWS;
  const int qw = q0 + 32 * wave;
  const int qrow = qw + (lane & 31);
  const float scale = rsqrtf((float)DH);

  const bf16* Qb = (const bf16*)a.q + (int64_t)b * a.S * a.ld_q + h * DH;
  const bf16* Kb = (const bf16*)a.k + (int64_t)b * a.S * a.ld_k + h * DH;
  const bf16* Vb = (const bf16*)a.v + (int64_t)b * a.S * a.ld_v + h * DH;
  const bf16* dOb = (const bf16*)a.dout + (int64_t)b * a.S * a.ld_do + h * DH;

  bf16x8 qf[C::KSTEPS], dof[C::KSTEPS];
  const bool qok = qrow < S;
  const int qr = qok ? qrow : S - 1;
#pragma unroll
  for (int kk = 0; kk < C::KSTEPS; ++kk) {
    qf[kk] = __builtin_bit_cast(bf16x8, ld16(Qb + (int64_t)qr * a.ld_q + 16 * kk + 8 * (lane >> 5)));
    dof[kk] = __builtin_bit_cast(bf16x8, ld16(dOb + (int64_t)qr * a.ld_do + 16 * kk + 8 * (lane >> 5)));
    settle(qf[kk]);
    settle(dof[kk]);
  }
  const int64_t sidx = ((int64_t)b * a.H + h) * a.Sp + qr;
  const float nlse2 = qok ? a.nlse2[sidx] : 0.0f;
  const float ndl = qok ? a.ndelta[sidx] : 0.0f;   // -Delta
  settle(nlse2);
  settle(ndl);
  const int kv_last = !qok ? -1 : (a.causal ? qrow : S - 1);   // last key this query may see

  const int kv_end = a.causal ? (q0 + C::QROWS < S ? q0 + C::QROWS : S) : S;
  const int ntiles = (kv_end + 63) / 64;
  const RingOff<DH, C::NW> roff = ring_offsets<DH, C::NW>((int)a.ld_k, (int)a.ld_v, wave, lane);
  auto issue = [&](int j) {
    char* st = smem + (j % C::NS) * C::STAGE;
    if (64 * j + 63 < S) ring_issue_full<DH, C::NW>(st, Kb, (int)a.ld_k, 64 * j, Vb, (int)a.ld_v, 64 * j, roff, wave);
    else ring_issue<DH, C::NW>(st, Kb, (int)a.ld_k, 64 * j, Vb, (int)a.ld_v, 64 * j, S - 1, wave, lane);
  };

  f32x16 acc[C::DT];                                // dQ^T of the wave's queries
#pragma unroll
  for (int t = 0; t < C::DT; ++t) acc[t] = f32x16{};

  auto tile = [&](int j, auto MASK) {
    const int kv0 = 64 * j;
    const char* kt = smem + (j % C::NS) * C::STAGE;
    const char* vt = kt + C::TB;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = nlse2;                                // the MFMAs leave the exponent of P
        dp[r] = ndl;                                 // and dP^T - Delta
      }
#pragma unroll
      for (int kk = 0; kk < C::KSTEPS; ++kk) {
        s = mfma32x32x16(frag_rows<DH>(kt, 32 * mt, 2 * kk, lane), qf[kk], s);
        dp = mfma32x32x16(frag_rows<DH>(vt, 32 * mt, 2 * kk, lane), dof[kk], dp);
      }
      // key offset of register r: acc_row(r, lane); the lane part moves into the limit
      // so that every comparison is against a constant
      const int lim = kv_last - kv0 - 32 * mt - 4 * (lane >> 5);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float p = fast_exp2(s[r]);
        if constexpr (decltype(MASK)::value) p = (8 * (r >> 2) + (r & 3) <= lim) ? p : 0.0f;
        s[r] = p * dp[r];                           // dS^T
      }
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bf16x8 sb = acc_to_b(s, hf);
#pragma unroll
        for (int t = 0; t < C::DT; ++t)
          acc[t] = mfma32x32x16(frag_tr<DH>(kt, 32 * mt + 16 * hf, 32 * t, lane), sb, acc[t]);
      }
    }
  };

  // Key tiles every query of the workgroup fully sees take the unmasked body; the
  // diagonal and ragged tiles (and every tile of a block with queries past the end)
  // take the masked one. Every barrier is reached by all waves; a wave skips the
  // arithmetic of tiles entirely after its queries.
  int n_full;
  if constexpr (C::NW == 4) {   // std::min selects between references, which kept ntiles in scratch memory here
    n_full = a.causal && (q0 + 1) / 64 < ntiles ? (q0 + 1) / 64 : ntiles;
    n_full = n_full < S / 64 ? n_full : S / 64;
  } else {                      // (and the 8-wave form is 1 % faster with it)
    n_full = a.causal ? std::min(ntiles, (q0 + 1) / 64) : ntiles;
    n_full = std::min(n_full, S / 64);
  }
  if (q0 + C::QROWS > S) n_full = 0;
#pragma unroll
  for (int st = 0; st < C::NS - 1; ++st)
    if (st < ntiles) issue(st);
  auto step = [&](int j) {
    // stage j has landed once at most the stages issued after it are pending
    if (C::NS == 4 && j + 2 < ntiles) wait_vmcnt<2 * C::DPS>();
    else if (C::NS == 4 && j + 1 < ntiles) wait_vmcnt<C::DPS>();
    else wait_vmcnt<0>();
    __syncthreads();                  // stage j visible; every wave is done with stage j-1
    if (j + C::NS - 1 < ntiles) issue(j + C::NS - 1);   // into the slot of stage j-1
  };
  int j = 0;
  for (; j < n_full; ++j) {
    step(j);
    tile(j, std::false_type{});
  }
  for (; j < ntiles; ++j) {
    step(j);
    if (!(a.causal && 64 * j > qw + 31)) tile(j, std::true_type{});
  }

  if (qrow < a.Sp) {
    bf16* dQt = (bf16*)a.dqt + (int64_t)h * DH * a.ld_dt + (int64_t)b * a.Sp + qrow;
#pragma unroll
    for (int t = 0; t < C::DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int d = 32 * t + acc_row(r, lane);
        dQt[(int64_t)d * a.ld_dt] = (bf16)(qok ? acc[t][r] * scale : 0.0f);
      }
  }
}

// ====================================================================== backward dQ, fp32
// 16 queries per workgroup; wave w takes the key tiles of 16 w, w + 4, ... S^T and dP^T
// have the query on the lane axis, so dS^T is the B operand of dQ^T += K^T dS^T.
template <int DH>
__global__ __launch_bounds__(256) void attn_bwd_dq_f32_kernel(AttnArgs a) {
  constexpr int NC = DH / 16;
  __shared__ __attribute__((aligned(16))) float red[4][DH][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c16 = lane & 15;
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t S = a.S;
  const int64_t blk = a.causal ? gridDim.x - 1 - blockIdx.x : blockIdx.x;   // causal: most keys first
  const int64_t q0 = blk * 16, q = q0 + c16, qr = q < S ? q : S - 1;
  const float scale = rsqrtf((float)DH);
  const float* Qb = (const float*)a.q + (int64_t)b * S * a.ld_q + (int64_t)h * DH;
  const float* Kb = (const float*)a.k + (int64_t)b * S * a.ld_k + (int64_t)h * DH;
  const float* Vb = (const float*)a.v + (int64_t)b * S * a.ld_v + (int64_t)h * DH;
  const float* dOb = (const float*)a.dout + (int64_t)b * S * a.ld_do + (int64_t)h * DH;
  const RowFrag<DH> qf = row_frag<DH>(Qb + qr * a.ld_q, g), of = row_frag<DH>(dOb + qr * a.ld_do, g);
  const int64_t sidx = ((int64_t)b * a.H + h) * a.Sp + qr;
  const float lq = a.lse[sidx], ndl = a.ndelta[sidx];
  f32x4 dq[NC];
#pragma unroll
  for (int t = 0; t < NC; ++t) dq[t] = f32x4{};
  const int64_t kv_end = q0 >= S ? 0 : a.causal ? (q0 + 16 < S ? q0 + 16 : S) : S;
  const int64_t kv_lim = q >= S ? 0 : a.causal && q + 1 < kv_end ? q + 1 : kv_end;   // keys this lane's query may see
  for (int64_t kv0 = 16 * wave; kv0 < kv_end; kv0 += 64) {
    const int64_t kr = kv0 + c16 < S ? kv0 + c16 : S - 1;
    const RowFrag<DH> kf = row_frag<DH>(Kb + kr * a.ld_k, g), vf = row_frag<DH>(Vb + kr * a.ld_v, g);
    const ColFrag<DH> kc = col_frag<DH>(Kb, a.ld_k, kv0, S - 1, g, c16);
    const f32x4 s = dot_frags<DH>(kf, qf);
    f32x4 ds = dot_frags<DH>(vf, of);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      ds[r] = kv0 + 4 * g + r < kv_lim ? fast_exp2((s[r] * scale - lq) * LOG2E) * (ds[r] + ndl) : 0.0f;
    add_outer<DH>(dq, kc, ds);
  }
#pragma unroll
  for (int t = 0; t < NC; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][16 * t + 4 * g + r][c16] = dq[t][r];
  __syncthreads();
  float* out = (float*)a.dqt + (int64_t)h * DH * a.ld_dt + (int64_t)b * a.Sp + q0;
  for (int i = tid; i < 16 * DH; i += 256) {           // 16 consecutive queries of a feature
    const int d = i >> 4, k = i & 15;
    out[(int64_t)d * a.ld_dt + k] = (((red[0][d][k] + red[1][d][k]) + red[2][d][k]) + red[3][d][k]) * scale;
  }
}

template <int DH, int NW>
static hipError_t dq_launch_bf16(const AttnArgs& a, hipStream_t s) {
  using C = DqCfg<DH, NW>;
  auto k = attn_bwd_dq_bf16_kernel<DH, NW>;
  hipError_t e = set_lds(k, C::LDS);
  if (e != hipSuccess) return e;
  const int64_t nblk = (a.S + C::QROWS - 1) / C::QROWS;
  hipLaunchKernelGGL(k, dim3((unsigned)(nblk * a.H * a.B)), dim3(64 * NW), C::LDS, s, a);
  return hipGetLastError();
}

template <int DH>
static hipError_t dq_launch(Dt dt, const AttnArgs& a, hipStream_t s) {
  if (a.S <= 0 || a.B <= 0) return hipSuccess;
  if (dt == BF16) {
    return few_blocks(a.S, (int64_t)a.H * a.B, a.causal) ? dq_launch_bf16<DH, 4>(a, s) : dq_launch_bf16<DH, 8>(a, s);
  } else {
    hipLaunchKernelGGL(attn_bwd_dq_f32_kernel<DH>, dim3((unsigned)(a.Sp / 16), a.H, a.B), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t attn_bwd_dq(Dt dt, const AttnArgs& a, hipStream_t s) {
  if (a.dh == 64) return dq_launch<64>(dt, a, s);
  if (a.dh == 128) return dq_launch<128>(dt, a, s);
  return hipErrorInvalidValue;
}

}  // namespace bpt
