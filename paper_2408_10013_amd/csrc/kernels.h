// Internal: launchers of the layer's HIP kernels.  All pointers are device pointers, all
// matrices row-major; element type is float or bf16 (SSDT_F32 / SSDT_BF16) with fp32
// arithmetic and accumulation throughout.  Every reduction runs in a fixed order, so results
// do not depend on addresses or timing.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ssdt.h"

namespace ssdt {
namespace k {

enum Epi {
  EPI_NONE = 0,    // C = acc
  EPI_BIAS,        // C = acc + bias
  EPI_BIAS_ACT,    // u = acc + bias; C = u (skipped when C is null); C2 = act(u)
  EPI_BIAS_RESID,  // C = acc + bias + resid
  EPI_ACTBWD       // C = acc * act'(aux)   (aux = pre-activation for GELU, activation output for ReLU)
};

// C[M,N] = sum_k A(m,k) B(k,n)   with   A(m,k) = transA ? A[k*lda+m] : A[m*lda+k]
//                                       B(k,n) = transB ? B[n*ldb+k] : B[k*ldb+n]
struct Gemm {
  int M = 0, N = 0, K = 0;
  const void *A = nullptr;
  long lda = 0;
  bool transA = false;
  const void *B = nullptr;
  long ldb = 0;
  bool transB = false;
  void *C = nullptr;
  long ldc = 0;
  int epi = EPI_NONE;
  const void *bias = nullptr;   // [N] or null (then treated as 0)
  const void *resid = nullptr;  // [M, ldr]
  long ldr = 0;
  void *C2 = nullptr;           // [M, ldc]
  const void *aux = nullptr;    // [M, ldc]
  int act = SSDT_ACT_GELU;
  int dtype = SSDT_F32;
  void *colsum = nullptr;       // [N] or null: sum over k of B(k, n), taken from the operand fragments while they pass
                                // through the registers.  Only the kernels that read k-major operands as stored can
                                // do this; every other path returns hipErrorNotSupported (nothing launched).
  bool colsum_accumulate = false;  // add to what colsum holds
  void *scratch = nullptr;      // optional: room for transposed copies of operands, or for partial products (bf16)
  size_t scratch_bytes = 0;
  bool split = false;           // the contraction may be split over workgroups (another order of the fp32 additions)
  // The forward products of layers with ReLU, bf16.  A pre-activation near zero changes sides with the last bit of what it was
  // summed from, and with it a whole column of the gradients.  A product whose result is rounded to bf16 on the way there
  // makes a difference of 2^-24 into one of 2^-9 wherever a rounding tips over, and every further rounding spreads it: two
  // orders of addition, equally far from the exact result (4 to 5 %), lie up to 4 % apart at width 4096.
  // one_order: all of them.  Among the bf16 kernels only those that add like gemm_tile_k's tiles with 64 k a stage, so that the
  // bits do not hang on the choice of a tile.  (The 256 x 256 kernels add like them too, but where gemm_km256_k staggers its
  // loop over k, N >= 16384 and K <= 8192: there each XCD starts elsewhere.)
  bool one_order = false;
  // ordered: the ones in front of the pre-activation's own.  At every size that is not whole tiles of 128 x 128 x 64: k ascending,
  // whatever kernel runs.  The pre-activation's product tips one sign in 10^7 and the one behind it none: with these two in
  // any order the gradients of a layer move by 0.3 % at most (22 layers, widths 128 to 4096, 45 to 2800 tokens).
  bool ordered = false;
};
hipError_t gemm(const Gemm &g, hipStream_t s);
hipError_t gemm_generic(const Gemm &g, hipStream_t s);  // the FMA kernel, any shape (gemm() falls back to it)
hipError_t gemm_f32(const Gemm &g, hipStream_t s);      // fp32 on the matrix cores
extern int g_f32_tile;                                  // test hook: 64 or 32 pins that kernel's tile
extern int g_force_waves;                               // 0 = choose; > 0 pins the tile rows per workgroup-order group
extern int g_force_tile;                                // 0 = choose; 128 / 256 pin the matrix-core tile
// scratch bytes gemm() can make use of for this problem (0 for fp32)
// Leading dimension of the K-contiguous scratch copy of a GEMM operand: rows that are a multiple of 32 KiB
// long get 128 bytes of padding (measured 4-6 % on the N = 8192, K = 32768 shapes of the layer, where unpadded
// rows raised the kernel's L2 miss rate from 20 % to 34 %; neutral on the other shapes).
inline long nt_copy_ld(int K) { return ((long)K * 2) % 32768 == 0 ? (long)K + 64 : (long)K; }
size_t gemm_scratch_bytes(int M, int N, int K, bool transA, bool transB, int dtype);
size_t gemm_nt_scratch_bytes(int M, int N, int K, bool transA, bool transB, int dtype);  // gemm_mfma_bf16's own need

// An axis of a grid holds fewer than 2^32 threads: the launch of more is not refused, the upper bits of their number are dropped.
// Whether workgroups of 256 threads fit one axis.  (Attention beyond that, short sequences and very many heads, goes from the tile
// kernels to the row kernels, whose grid has three axes.)
inline bool one_axis(long workgroups) { return workgroups < (1l << 24); }
// The norm backward's workgroups, those of the column sums and those of dx: go(sums, dx_blocks) launches both kinds, or one.
template <typename F>
inline void norm_bwd_launch(F go, int chunks, int col_blocks, int rows) {
  const int dx_blocks = (rows + 3) / 4;
  if (one_axis((long)chunks * col_blocks + dx_blocks)) return go(chunks, dx_blocks);
  go(chunks, 0);
  go(0, dx_blocks);
}

// Row norm over H.  kind = SSDT_NORM_*.  mean may be null for RMSNorm.
hipError_t norm_fwd(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int rows,
                    int H, float eps, int kind, int dtype, hipStream_t s);
// dx = (resid ? resid : 0) + norm-backward(dy); dgamma/dbeta by a two-stage column reduction
// through `partial` (fp32, `room` elements: 2 H or more).
hipError_t norm_bwd(const void *dy, const void *x, const float *mean, const float *rstd, const void *gamma,
                    const void *resid, void *dx, void *dgamma, void *dbeta, float *partial, size_t room, int rows, int H,
                    int kind, int dtype, bool accumulate, hipStream_t s);
// out[n] = sum_m a[m, n]  (bias gradients), same two-stage scheme
hipError_t colsum(const void *a, long lda, void *out, float *partial, size_t room, int rows, int cols, int dtype,
                  bool accumulate, hipStream_t s);
// w <- w - lr * g, elementwise in fp32, stored in the tensors' type
hipError_t sgd_update(void *w, const void *g, size_t n, float lr, int dtype, hipStream_t s);
size_t colreduce_partial_floats(int rows, int cols);

struct Attn {
  int B = 0, A = 0, Sq = 0, Sk = 0, d = 0;
  float scale = 1.f;
  int mask = SSDT_MASK_NONE;
  const int32_t *kv_len = nullptr;  // [B], key-padding mask only
  int dtype = SSDT_F32;
  const void *q = nullptr, *k = nullptr, *v = nullptr;  // rows b*S + i, head h at columns h*d
  long ldq = 0, ldk = 0, ldv = 0;
  void *o = nullptr;
  long ldo = 0;
  float *lse = nullptr;  // [B, A, Sq]
  bool ordered = false;  // forward, as in Gemm: the row kernels' order and fp32 probabilities unless tiles are whole
  // backward only
  const void *dout = nullptr;
  long lddo = 0;
  void *dq = nullptr, *dk = nullptr, *dv = nullptr;
  long lddq = 0, lddk = 0, lddv = 0;
  float *delta = nullptr;  // scratch, 2 x [B, A, Sq] floats (the second half holds lse in base-2 units for the matrix-core backward)
};
// calls F(D) for the smallest D that holds the head
#define SSDT_BY_HEAD(d, F)                                                                                 \
  do {                                                                                                     \
    if ((d) <= 32) F(32); else if ((d) <= 64) F(64); else if ((d) <= 96) F(96); else F(128);                \
  } while (0)
hipError_t attn_fwd(const Attn &a, hipStream_t s);
hipError_t attn_bwd(const Attn &a, hipStream_t s);
// the one-wavefront-per-row kernels (attn_rows.h), any shape: where they are faster, and for what the tile kernels do not take
hipError_t attn_fwd_generic(const Attn &a, hipStream_t s);
hipError_t attn_bwd_generic(const Attn &a, hipStream_t s);
// delta[b,h,i] = sum_c o[i,c] dout[i,c]; with lse2 also lse in base-2 units, +inf for a row without keys
hipError_t attn_delta(const Attn &a, float *lse2, hipStream_t s);

// out[c, r] = in[r, c]
hipError_t transpose(const void *in, long ldi, void *out, long ldo, int rows, int cols, int dtype, hipStream_t s);
// y += x  (elementwise, n elements)
hipError_t add_inplace(void *y, const void *x, size_t n, int dtype, hipStream_t s);

// 16-byte-vectorised row kernels; return hipErrorNotSupported when the shape / alignment does not fit
hipError_t norm_fwd_vec(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int rows,
                        int H, float eps, int kind, int dtype, hipStream_t s);
hipError_t norm_bwd_vec(const void *dy, const void *x, const float *mean, const float *rstd, const void *gamma,
                        const void *resid, void *dx, float *partial, int rows, int H, int kind, int chunks, int dtype, hipStream_t s);
hipError_t attn_delta_vec(const void *o, long ldo, const void *dout, long lddo, float *delta, const float *lse, float *lse2,
                          int B, int Sq, int A, int d, int dtype, hipStream_t s);
hipError_t colreduce1_vec(const void *a, long lda, float *partial, int rows, int cols, int chunks, hipStream_t s);  // (bf16)

// fast paths (bf16 on the matrix cores); return hipErrorNotSupported when the shape does not fit
hipError_t gemm_mfma_bf16(const Gemm &g, hipStream_t s);
hipError_t gemm_mfma_km_bf16(const Gemm &g, hipStream_t s);  // reads k-major operands as stored; no scratch
hipError_t gemm_mfma_tile_bf16(const Gemm &g, hipStream_t s);  // any number of rows; may split the contraction into scratch
bool gemm_tile_fits(int M, int N, int K, bool transA, bool transB, int dtype);   // shape conditions of that kernel
bool gemm_large_fits(int M, int N, int K, bool transA, bool transB, int dtype);  // the 256 x 256 kernels should take it
// A linear's weight gradient w (transA) and input gradient d (transB) in one launch; hipErrorNotSupported (nothing launched)
// where two launches are better.  Neither may write what the other reads.  With w.colsum the bias sums fall out of w's kernel, in
// fp32 here only (gemm() leaves them to colsum() there).  plan: what gemm_linear_bwd_scratch_bytes chose, or null.
struct PairPlan {
  int rows = 0, in = 0, out = 0;  // the linear
  bool pair = false;              // one launch
  int cfg = 0, sw = 1, sd = 1;    // its tile, the splits of w and d
};
hipError_t gemm_pair_bf16(const Gemm &w, const Gemm &d, const PairPlan *plan, hipStream_t s);
hipError_t gemm_pair_f32(const Gemm &w, const Gemm &d, hipStream_t s);
size_t gemm_linear_bwd_scratch_bytes(int rows, int in, int out, int dtype, PairPlan *plan);  // partial products of a linear's backward
extern int g_tile_cfg, g_tile_splits;  // test hooks of that kernel: >= 0 pins the tile, > 0 the number of splits
bool gemm_km_fits(int M, int N, int K, bool transA, bool transB, int dtype);  // shape conditions of that kernel
extern int g_km_stagger;  // stages between the K-loop starts of neighbouring XCDs (-100 = by shape)
extern int g_km_pf;       // stages that the L2 prefetch runs ahead (-1 = by shape, 0 = none)
extern int g_km_mode;  // 0 = off, 1 = for problems with a k-major operand (default), 2 = also for the NT form
hipError_t attn_fwd_mfma_bf16(const Attn &a, hipStream_t s);
hipError_t attn_bwd_mfma_bf16(const Attn &a, hipStream_t s);
bool attn_few_keys(const Attn &a, long items);  // which of the forward's two kernels for whole tiles, by its blocks of 128 queries
hipError_t attn_fwd_f32(const Attn &a, hipStream_t s);  // fp32 on the matrix cores, likewise
hipError_t attn_bwd_f32(const Attn &a, hipStream_t s);

}  // namespace k
}  // namespace ssdt
