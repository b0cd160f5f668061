// Host-side launchers shared between libbpt's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bpt {

// F16 is used for one tensor only: GELU'(z) saved by the FFN recompute of the bf16 path.
enum Dt { F32 = 0, BF16 = 1, F16 = 2 };

// ---------------------------------------------------------------- GEMM
// C[M, N] = A[M, K] * B[N, K]^T ("NT": both operands K-contiguous), fp32 accumulation,
// optional batch (grid z) with element strides, followed by a fused epilogue.
enum Epi {
  EPI_STORE = 0,   // C = acc            (fp32 C may accumulate: C += acc)
  EPI_RESID = 1,   // C = acc + R[m, n] (+ bias[n])
  EPI_GELU = 2,    // z = acc (+ bias[n] or bias[m]); C = GELU(z); C2 = GELU'(z) if C2
  EPI_MUL = 3,     // C = acc * R[m, n]  (R fp32 or fp16)
  EPI_RELU = 5,    // as EPI_GELU with max(0, z) and its derivative (0 at z = 0)
  EPI_XENT_T = 6,  // cross-entropy gradient of transposed logits acc (rows m = vocabulary, columns
                   // n = tokens): for m < nvalid C = alpha (exp(acc - rowv[n]) - [m == tgt[n]]),
                   // rowv a token's log-sum-exp; C = 0 for nvalid <= m
  EPI_LSE = 7,     // bf16 operands; row summaries of the logits acc instead of the logits: for
                   // every 64 columns j, C[m, j] = (max, sum of exp(acc - max)) over columns
                   // below nvalid, as two floats; tlogit[m] = acc[m, tgt[m]] for 0 <= tgt[m] < nvalid
};

struct GemmArgs {
  const void* A = nullptr;
  const void* B = nullptr;
  void* C = nullptr;
  const void* R = nullptr;     // residual (EPI_RESID) or multiplier (EPI_MUL)
  const float* bias = nullptr;
  void* C2 = nullptr;          // second output of EPI_GELU / EPI_RELU, element type c2t (F32 or F16)
  Dt c2t = F32;
  int64_t M = 0, N = 0, K = 0;
  int64_t Nstore = 0;          // columns [N, Nstore) of C (and C2) are written with 0
  int64_t lda = 0, ldb = 0, ldc = 0, ldr = 0, ldc2 = 0;
  int64_t sA = 0, sB = 0, sC = 0, sR = 0, sC2 = 0;   // batch strides in elements
  int batch = 1;
  int accumulate = 0;          // fp32 C only: C += acc
  float alpha = 1.0f;          // EPI_STORE: acc is multiplied by alpha before it is stored;
                               // EPI_XENT_T: the gradient's scale
  const float* rowv = nullptr; // EPI_XENT_T: per-column log-sum-exp (natural log), [N]
  const int32_t* tgt = nullptr;// EPI_XENT_T: per-column target row, [N]
  int64_t nvalid = 0;          // EPI_XENT_T: rows from nvalid on are not logits; EPI_LSE: columns
  float* tlogit = nullptr;     // EPI_LSE: the target's logit of each row (tgt per row there), [M]
  int in_order = 0;            // every element adds its products in the order of k, so that it is
                               // the same for any M and N (no tile form that shares K)
  int bias_on_m = 0;           // EPI_GELU / EPI_RELU: bias indexed by row instead of column
  // Transposed operands (which ones go with which epilogue: gemm.hip's lists): trans_a means A is stored K-major, element
  // (m, k) at A[k * lda + m]; likewise trans_b for B (element (n, k) at B[k * ldb + n]).
  // For such an operand, x_rows is the number of k rows that may be read (rows from
  // x_rows up to K are not read, and the other operand must be zero at those k), and
  // x_cols the number of columns that may be read from the pointer (>= M or N; a
  // multiple of 8). 0 means K and M (or N).
  // With both operands K-major, K may be any length: rows past it are read as zeros.
  int trans_a = 0, trans_b = 0;
  int64_t a_rows = 0, b_rows = 0, a_cols = 0, b_cols = 0;
  // A K-major (and B not): k counts rows in segments of seg_pitch of which the first seg_rows
  // exist, stored one after the other (sequences padded in B but not in A); rows past a
  // segment's end are not read, and B must be zero there. seg_pitch % 64 == 0; 0: none.
  int64_t seg_rows = 0, seg_pitch = 0;
  // ksplit > 1 (EPI_STORE, batch 1): grid z is a slice of K, a run of whole k stages, whose
  // partial product goes to C + z * sC
  int ksplit = 1;
  // nper > 0: columns [w nper, (w + 1) nper), w = 0, 1, 2, take B from Bx[w] (B K-major) and go
  // to Cx[w] where those are given; alpha applies to w = 0 only. A column tile lies in one w
  // (gemm_takes_nper).
  int64_t nper = 0;
  // kper > 0 (A K-major, B not): B's columns k in [w kper, (w + 1) kper) come from Bx[w]
  int64_t kper = 0;
  const void* Bx[3] = {nullptr, nullptr, nullptr};
  void* Cx[3] = {nullptr, nullptr, nullptr};
};

// Whether a GEMM of M x 3 nper may be given as one with nper > 0
bool gemm_takes_nper(Dt ab, int64_t nper);
// Whether it should, rather than as three of M x nper (at most cap3, cap1 slices of K)
bool gemm_three_as_one(Dt ab, int64_t M, int64_t nper, int64_t K, int cap3, int cap1);
// Slices of K (at most cap) for an M x N product stored in fp32 whose tiles alone would leave
// CUs idle. both_kmajor: trans_a and trans_b.
int gemm_ksplit(Dt ab, int64_t M, int64_t N, int64_t K, int cap, int both_kmajor = 0);

// ab: element type of A and B. ct: type of C; rt: type of R.
hipError_t gemm(Dt ab, Epi epi, Dt ct, Dt rt, const GemmArgs& a, hipStream_t s);

// ---------------------------------------------------------------- attention
// The bf16 kernels take Q multiplied by log2(e)/sqrt(dh), so that Q K^T are the scores in
// base-2 units (exp2 of them is the unnormalised probability); the fp32 kernels take Q
// as the projection produced it.
struct AttnArgs {
  // token-major tensors: token (b, s) is row b*S + s
  const void* q = nullptr;  int64_t ld_q = 0;    // pointer already at head 0's first column
  const void* k = nullptr;  int64_t ld_k = 0;
  const void* v = nullptr;  int64_t ld_v = 0;
  const void* dout = nullptr; int64_t ld_do = 0;
  void* o = nullptr;        int64_t ld_o = 0;
  // feature-major outputs: element (b, s, f) at row f, column b*Sp + s
  void* dqt = nullptr; void* dkt = nullptr; void* dvt = nullptr; int64_t ld_dt = 0;
  float* lse = nullptr;        // [B, H, Sp] natural log
  const float* ndelta = nullptr;// [B, H, Sp] -Delta, Delta = rowsum(dO * O)
  const float* nlse2 = nullptr;// [B, H, Sp] minus the log-sum-exp in base 2 (bf16 backward)
  int64_t S = 0, Sp = 0;
  int B = 0, H = 0, dh = 0;
  int causal = 0;
  int64_t q_begin = 0, q_end = 0;  // forward: query rows [q_begin, q_end) of batch b_begin
  int b_begin = 0, nb = 0;
};

// Whether `rows` rows of each of `heads` heads make too few blocks of 256 rows for one per CU,
// so that the bf16 kernels run blocks of 128 (4 waves, two workgroups on a CU): with the causal
// mask they even out blocks of unequal work (forward / dK dV / dQ of 4 x 1000 tokens, 12 heads
// of 64: 24 / 41 / 33 -> 20 / 37 / 30 us; one of 4096 tokens, 16 heads of 128: 106 / 224 / 149
// -> 98 / 204 / 125 us; with 512 blocks of 256 they lose up to 15 %). Without it all blocks
// are alike and sharing tiles among 8 waves wins earlier (256 blocks: 127 -> 146 us forward).
// The results are the same bit for bit.
inline bool few_blocks(int64_t rows, int64_t heads, int causal) {
  return (rows + 255) / 256 * heads <= (causal ? 256 : 128);
}

hipError_t attn_fwd(Dt dt, const AttnArgs& a, hipStream_t s);
// backward: dK and dV (key-outer kernel), dQ (query-outer kernel)
hipError_t attn_bwd_dkdv(Dt dt, const AttnArgs& a, hipStream_t s);
hipError_t attn_bwd_dq(Dt dt, const AttnArgs& a, hipStream_t s);

// ---------------------------------------------------------------- residual-branch dropout
// Element (t, n) of branch `site` is kept iff word n % 4 of Philox4x32-10 at counter
// (n / 4, t, site, 0), key (k0, k1), is >= threshold; kept values are multiplied by scale.
struct DropArgs {
  uint32_t k0 = 0, k1 = 0, site = 0, threshold = 0;
  float scale = 1.0f;
  int64_t row0 = 0;            // token index t of the first row passed
};

// ---------------------------------------------------------------- row-wise / layout kernels
// LayerNorm over D per row. x: [rows, D] (ti); out [rows, D] (to).
// mode 0: compute and write mu/rstd; mode 1: use the given mu/rstd.
hipError_t layer_norm(Dt ti, Dt to, const void* x, int64_t ldx, const float* g, const float* b,
                      void* out, int64_t ldo, float* mu, float* rstd, int64_t rows, int64_t D,
                      float eps, int use_stats, hipStream_t s);

// out = resid + LN^T(dout), per row (resid may be null: 0); out2 (optional, type t2) gets
// the same values. Unless both are null, dgamma[d] = sum_r dout[r,d] * xhat[r,d] and
// dbeta[d] = sum_r dout[r,d] (overwrite; either may be null), through `partial`, workspace of
// at least layer_norm_param_grad_ws(D) floats (more are used if there). dout is fp32, or bf16
// where layer_norm_bwd_fused(D). With seg > 0, dout has a row pitch of `pitch` rows per seg
// rows: row r is stored at r + r / seg * (pitch - seg). drop (null: none; only where
// layer_norm_bwd_fused(D)): out2 gets the values through that dropout.
size_t layer_norm_param_grad_ws(int64_t D);
int64_t layer_norm_bwd_partials(int64_t rows, int64_t D);   // floats of `partial` it can use, if layer_norm_bwd_fused(D)
bool layer_norm_bwd_fused(int64_t D);
hipError_t layer_norm_bwd(Dt ti, const void* x, const float* mu, const float* rstd, const float* g, Dt td,
                          const void* dout, Dt tr, const void* resid, Dt to, void* out, Dt t2, void* out2,
                          float* dgamma, float* dbeta, float* partial, int64_t partial_floats, int64_t rows, int64_t D,
                          int64_t seg, int64_t pitch, const DropArgs* drop, hipStream_t s);

// out[c] = sum_r in[r, c]  (in: [rows, cols] of type t, rows 16-byte aligned, cols % 8 == 0), through
// `partial` of at least cols floats (more are used if there)
hipError_t col_sum(Dt t, const void* in, int64_t ld, int64_t rows, int64_t cols, float* out, float* partial,
                   int64_t partial_floats, hipStream_t s);
// out[r] (+)= sum_c in[r, c]
hipError_t row_sum(Dt t, const void* in, int64_t ld, int64_t rows, int64_t cols, float* out,
                   int accumulate, hipStream_t s);

// ndelta[b, h, s] = -sum_d dO[b*S+s, h*dh+d] * O[b*S+s, h*dh+d]; nlse2 = -lse * log2(e);
// both are 0 for the padding positions s >= S
hipError_t attn_delta(Dt t, const void* dout, const void* o, int64_t ld, const float* lse, float* ndelta,
                      float* nlse2, int B, int64_t S, int64_t Sp, int H, int dh, hipStream_t s);

// ---------------------------------------------------------------- cross-entropy of an LM head
// Per row t of a block of fp32 logits z [rows, ld]: lse[t] over the first V columns and
// the token loss lse[t] - z[t, tgt[t]] (NaN for a target outside [0, V)).
hipError_t xent_rows(const float* z, int64_t ld, int64_t rows, int64_t V, const int32_t* tgt, float* lse,
                     float* tok, hipStream_t s);
// The same from EPI_LSE's summaries part [rows, ng] (two floats each, merged in order) and the
// targets' logits.
hipError_t xent_merge(const float* part, int64_t ng, int64_t rows, int64_t V, const int32_t* tgt, const float* tlogit,
                      float* lse, float* tok, hipStream_t s);
// out[0] = mean of x[0..n), summed in a fixed order
hipError_t mean_of(const float* x, int64_t n, float* out, hipStream_t s);
// ---------------------------------------------------------------- GPT step pieces
// X[t] = Wte[tok[t]] + Wpe[t mod S] (Wpe may be null); NaN row for tok outside [0, V). D % 8 == 0.
hipError_t embed_fwd(Dt t, const int32_t* tok, const void* Wte, const void* Wpe, void* X, int64_t rows,
                     int64_t S, int64_t D, int64_t V, hipStream_t s);
// dWte[v] = sum of dX[t] over the tokens t with tok[t] = v, in a fixed order (overwrite)
hipError_t embed_dwte(Dt t, const int32_t* tok, const void* dX, float* dWte, int64_t rows, int64_t D, int64_t V,
                      hipStream_t s);
// dWpe[s] = sum_b dX[b S + s] (overwrite)
hipError_t embed_dwpe(Dt t, const void* dX, float* dWpe, int64_t B, int64_t S, int64_t D, hipStream_t s);
// out[i] = in[i] (bf16 -> fp32), n % 8 == 0
hipError_t bf16_to_f32(const void* in, float* out, int64_t n, hipStream_t s);
// one AdamW step over n fp32 elements; pl (type tl) gets the updated p when not null
hipError_t adamw(Dt tl, float* p, const float* g, float* m, float* v, void* pl, int64_t n, float lr, float b1,
                 float b2, float eps, float wd, float c1, float c2, hipStream_t s);

// out[m, c] (+)= sum over z < nz of part[z, m, c], rows x cols each, added in slice order; with
// nper > 0 column c goes to outs[c / nper][m, c % nper], else all to outs[0] (cols, nper % 4 == 0)
hipError_t sum_slices(const float* part, int nz, int64_t rows, int64_t cols, float* const outs[3], int64_t nper,
                      int accumulate, hipStream_t s);
// out[m, c] = R[m, c] + bias[c] + sum over z < nz of part[z, m, c] in slice order, rounded once to
// `to` (R of type tr or null, bias fp32 or null; rows x cols, cols % 4 == 0)
hipError_t sum_slices_add(const float* part, int nz, int64_t rows, int64_t cols, Dt tr, const void* R, const float* bias,
                          Dt to, void* out, hipStream_t s);
// out = R + f * (acc + bias) over rows x D (acc fp32 [rows, D]; bias fp32 [D] or null)
hipError_t dropout_add(const float* acc, Dt tr, const void* R, const float* bias, Dt to, void* out, int64_t rows,
                       int64_t D, const DropArgs& a, hipStream_t s);
// out = f * in over rows x D
hipError_t dropout_scale(Dt ti, const void* in, Dt to, void* out, int64_t rows, int64_t D, const DropArgs& a,
                         hipStream_t s);

}  // namespace bpt
