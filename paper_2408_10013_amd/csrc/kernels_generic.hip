// Generic kernels of the layer, templated on the storage type (float / bf16), fp32 math.
//
//  - gemm_generic: LDS-tiled FMA matrix multiply for any transposition and any shape: the fallback for what
//    no matrix-core kernel takes (bf16 widths that are no multiple of 8, operands that are not aligned).
//  - attn_*_generic: one wavefront per query (or key) row with an online softmax (attn_rows.h); exact -inf
//    masking; for a few tokens, where they are faster, and for head sizes and alignments the tile kernels do not take.
//  - norm forward/backward (one wavefront per row), deterministic two-stage column
//    reductions for bias and gain gradients, transpose, add.
//
// The operations are the textbook definitions of the transformer layer the paper's
// Sec. 2.1 names (attention block, MLP block, norms, residuals).
#include <algorithm>

#include "attn_rows.h"
#include "dev.h"
#include "kernels.h"
#include "prof.h"

namespace ssdt {
namespace k {

#define SSDT_LAUNCH_CHECK() do { hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return e_; } while (0)

// ------------------------------------------------------------------------------------------
// GEMM
// ------------------------------------------------------------------------------------------
struct GemmP {
  int M, N, K;
  const void *A, *B;
  void *C, *C2;
  const void *bias, *resid, *aux;
  long lda, ldb, ldc, ldr;
  int transA, transB, epi, act;
};

template <typename T>
__global__ __launch_bounds__(256) void gemm_generic_k(GemmP p) {
  __shared__ float As[16][64 + 4];
  __shared__ float Bs[16][64 + 4];
  const T *A = (const T *)p.A, *B = (const T *)p.B;
  int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < p.K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int idx = tid + i * 256, m, kk;
      if (!p.transA) { kk = idx & 15; m = idx >> 4; } else { m = idx & 63; kk = idx >> 6; }
      int gm = m0 + m, gk = k0 + kk;
      float v = 0.f;
      if (gm < p.M && gk < p.K) v = ld(A + (p.transA ? (long)gk * p.lda + gm : (long)gm * p.lda + gk));
      As[kk][m] = v;
      int n;
      if (!p.transB) { n = idx & 63; kk = idx >> 6; } else { kk = idx & 15; n = idx >> 4; }
      int gn = n0 + n;
      gk = k0 + kk;
      v = 0.f;
      if (gn < p.N && gk < p.K) v = ld(B + (p.transB ? (long)gn * p.ldb + gk : (long)gk * p.ldb + gn));
      Bs[kk][n] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  T *C = (T *)p.C, *C2 = (T *)p.C2;
  const T *bias = (const T *)p.bias, *resid = (const T *)p.resid, *aux = (const T *)p.aux;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = m0 + ty * 4 + i;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = n0 + tx * 4 + j;
      if (n >= p.N) continue;
      float v = acc[i][j];
      if (bias && p.epi != EPI_NONE && p.epi != EPI_ACTBWD) v += ld(bias + n);
      long o = (long)m * p.ldc + n;
      switch (p.epi) {
        case EPI_BIAS_ACT:
          if (C) st(C + o, v);
          st(C2 + o, p.act == SSDT_ACT_GELU ? gelu_f(v) : fmaxf(v, 0.f));
          break;
        case EPI_BIAS_RESID:
          st(C + o, v + ld(resid + (long)m * p.ldr + n));
          break;
        case EPI_ACTBWD: {
          float u = ld(aux + o);
          st(C + o, v * (p.act == SSDT_ACT_GELU ? gelu_grad_f(u) : (u > 0.f ? 1.f : 0.f)));
          break;
        }
        default:
          st(C + o, v);
      }
    }
  }
}

hipError_t gemm_generic(const Gemm &g, hipStream_t s) {
  GemmP p{g.M, g.N, g.K, g.A, g.B, g.C, g.C2, g.bias, g.resid, g.aux, g.lda, g.ldb, g.ldc, g.ldr,
          g.transA, g.transB, g.epi, g.act};
  dim3 grid((g.N + 63) / 64, (g.M + 63) / 64);
  prof::Scope ps(prof::GEMM_GENERIC, 2.0 * g.M * g.N * g.K, 0, s);
  if (g.dtype == SSDT_F32) hipLaunchKernelGGL(gemm_generic_k<float>, grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL(gemm_generic_k<bf16>, grid, dim3(256), 0, s, p);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

hipError_t gemm(const Gemm &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
  const bool ordered = g.ordered && g.dtype == SSDT_BF16 && (g.M % 128 || g.N % 128 || g.K % 64);
  if (g.dtype == SSDT_BF16 && !ordered) {
    hipError_t e = hipErrorNotSupported;
    const bool large = gemm_large_fits(g.M, g.N, g.K, g.transA, g.transB, g.dtype);
    if (large) e = gemm_mfma_km_bf16(g, s);  // 256 x 256 tiles, operands taken as stored
    if (e != hipErrorNotSupported) return e;
    if (!large) e = gemm_mfma_tile_bf16(g, s);  // smaller tiles, any number of rows, operands taken as stored
    if (e != hipErrorNotSupported) return e;
    e = gemm_mfma_bf16(g, s);  // K-contiguous form, other operands through transposed copies
    if (e != hipErrorNotSupported) return e;
  }
  if (g.colsum) return hipErrorNotSupported;
  hipError_t e = gemm_f32(g, s);  // fp32, and bf16 forward products of any width and alignment
  if (e != hipErrorNotSupported) return e;
  return gemm_generic(g, s);
}

// ------------------------------------------------------------------------------------------
// norms
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void norm_fwd_k(const T *x, const T *gamma, const T *beta, T *y, float *mean,
                                                  float *rstd, int rows, int H, float eps, int kind) {
  int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const T *xr = x + (long)row * H;
  float mu = 0.f;
  if (kind == SSDT_NORM_LAYERNORM) {
    float sum = 0.f;
    for (int c = lane; c < H; c += 64) sum += ld(xr + c);
    mu = wave_sum(sum) / (float)H;
  }
  float sq = 0.f;
  for (int c = lane; c < H; c += 64) {
    float dlt = ld(xr + c) - mu;
    sq += dlt * dlt;
  }
  float r = 1.f / sqrtf(wave_sum(sq) / (float)H + eps);
  T *yr = y + (long)row * H;
  for (int c = lane; c < H; c += 64) {
    float v = (ld(xr + c) - mu) * r * ld(gamma + c);
    if (beta) v += ld(beta + c);
    st(yr + c, v);
  }
  if (lane == 0) {
    if (mean) mean[row] = mu;
    rstd[row] = r;
  }
}

hipError_t norm_fwd(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int rows,
                    int H, float eps, int kind, int dtype, hipStream_t s) {
  hipError_t e = norm_fwd_vec(x, gamma, beta, y, mean, rstd, rows, H, eps, kind, dtype, s);
  if (e != hipErrorNotSupported) return e;
  dim3 grid((rows + 3) / 4);
  prof::Scope ps(prof::NORM_FWD, 0, 2.0 * rows * H * (dtype == SSDT_F32 ? 4 : 2), s);
  if (dtype == SSDT_F32)
    hipLaunchKernelGGL(norm_fwd_k<float>, grid, dim3(256), 0, s, (const float *)x, (const float *)gamma,
                       (const float *)beta, (float *)y, mean, rstd, rows, H, eps, kind);
  else
    hipLaunchKernelGGL(norm_fwd_k<bf16>, grid, dim3(256), 0, s, (const bf16 *)x, (const bf16 *)gamma,
                       (const bf16 *)beta, (bf16 *)y, mean, rstd, rows, H, eps, kind);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

template <typename T>
__device__ __forceinline__ void norm_bwd_dx(const T *dy, const T *x, const float *mean, const float *rstd, const T *gamma,
                                            const T *resid, T *dx, int rows, int H, int kind, int block) {
  int lane = threadIdx.x & 63, row = block * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const T *xr = x + (long)row * H, *dyr = dy + (long)row * H;
  float mu = (kind == SSDT_NORM_LAYERNORM) ? mean[row] : 0.f, r = rstd[row];
  float s1 = 0.f, s2 = 0.f;
  for (int c = lane; c < H; c += 64) {
    float dh = ld(dyr + c) * ld(gamma + c);
    float xh = (ld(xr + c) - mu) * r;
    s1 += dh;
    s2 += dh * xh;
  }
  float c1 = (kind == SSDT_NORM_LAYERNORM) ? wave_sum(s1) / (float)H : 0.f;
  float c2 = wave_sum(s2) / (float)H;
  for (int c = lane; c < H; c += 64) {
    float dh = ld(dyr + c) * ld(gamma + c);
    float xh = (ld(xr + c) - mu) * r;
    float v = r * (dh - c1 - xh * c2);
    if (resid) v += ld(resid + (long)row * H + c);
    st(dx + (long)row * H + c, v);
  }
}

// Rows are dealt to chunks of 32 and more, at most 128 of them: short enough that the few column blocks of a narrow
// matrix still fill the machine and a wavefront's eight rows are all on their way at once (chunks of 128 rows: 18 us
// on 4096 x 2048 with both sums).
// `room`: chunks whose sums the caller's buffer holds (at least one).  The buffer is sized for two sums of the widest matrix in
// chunks of 128 rows, at most 64: what a norm, a third or a quarter as wide, puts into it is three to four times as many.
static inline int colreduce_chunks(int rows, size_t room) {
  const int c = std::min(std::max(rows / 32, 1), 128);
  return (int)std::min((size_t)c, room);
}
size_t colreduce_partial_floats(int rows, int cols) { return (size_t)2 * std::min(std::max(rows / 128, 1), 64) * cols; }

// Stage 1: block (cx, chunk) sums 128 columns over its chunk of rows.  NORM: g += a*xhat, b += a.
template <typename T, bool NORM>
__device__ __forceinline__ void colreduce1(const T *a, long lda, const T *x, const float *mean, const float *rstd, int kind,
                                           float *partial, int rows, int cols, int rows_per_chunk, int chunks, int cx, int chunk) {
  __shared__ float sg[4][128], sb[4][128];
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int c0 = cx * 128 + lane * 2;
  int r0 = chunk * rows_per_chunk, r1 = min(rows, r0 + rows_per_chunk);
  float g0 = 0.f, g1 = 0.f, b0 = 0.f, b1 = 0.f;
#pragma unroll 4
  for (int r = r0 + w; r < r1; r += 4) {
    float mu = 0.f, rs = 1.f;
    if (NORM) {
      mu = (kind == SSDT_NORM_LAYERNORM) ? mean[r] : 0.f;
      rs = rstd[r];
    }
    if (c0 < cols) {
      float v = ld(a + (long)r * lda + c0);
      b0 += v;
      if (NORM) g0 += v * (ld(x + (long)r * lda + c0) - mu) * rs;
    }
    if (c0 + 1 < cols) {
      float v = ld(a + (long)r * lda + c0 + 1);
      b1 += v;
      if (NORM) g1 += v * (ld(x + (long)r * lda + c0 + 1) - mu) * rs;
    }
  }
  sg[w][lane * 2] = g0; sg[w][lane * 2 + 1] = g1;
  sb[w][lane * 2] = b0; sb[w][lane * 2 + 1] = b1;
  __syncthreads();
  if (threadIdx.x < 128) {
    int c = cx * 128 + threadIdx.x;
    if (c < cols) {
      float g = ((sg[0][threadIdx.x] + sg[1][threadIdx.x]) + sg[2][threadIdx.x]) + sg[3][threadIdx.x];
      float b = ((sb[0][threadIdx.x] + sb[1][threadIdx.x]) + sb[2][threadIdx.x]) + sb[3][threadIdx.x];
      partial[(size_t)chunk * cols + c] = b;
      if (NORM) partial[(size_t)(chunks + chunk) * cols + c] = g;
    }
  }
}
template <typename T>
__global__ __launch_bounds__(256) void colreduce1_k(const T *a, long lda, float *partial, int rows, int cols, int rows_per_chunk) {
  colreduce1<T, false>(a, lda, nullptr, nullptr, nullptr, 0, partial, rows, cols, rows_per_chunk, gridDim.y, blockIdx.x, blockIdx.y);
}
// both parts of a norm's backward in one launch (see norm_bwd_vec_k)
template <typename T>
__global__ __launch_bounds__(256) void norm_bwd_k(const T *dy, const T *x, const float *mean, const float *rstd, const T *gamma,
                                                  const T *resid, T *dx, float *partial, int rows, int H, int kind,
                                                  int rows_per_chunk, int chunks, int col_blocks) {
  const int n1 = chunks * col_blocks, bid = blockIdx.x;
  if (bid < n1) colreduce1<T, true>(dy, H, x, mean, rstd, kind, partial, rows, H, rows_per_chunk, chunks, bid % col_blocks, bid / col_blocks);
  else norm_bwd_dx<T>(dy, x, mean, rstd, gamma, resid, dx, rows, H, kind, bid - n1);
}

// Stage 2: 16 columns per block, sixteen threads per column each adding every sixteenth chunk in turn, their sums in order.  What bounds it
// is trips to memory.  Above 32 chunks eight loads of either sum are on their way at once, the last chunk read again past the end and
// nothing added: a plain loop unrolled by eight leaves fewer than eight to its remainder, one trip each (the layer of 7 x 333, H 1024, 72 chunks: 382 ->
// 380 us, 16 x 512, 128 chunks: 851 -> 847; up to 32 chunks, two trips, the plain loop is level or better by 0.5 us in 114).
// (One thread per column adding all chunks: 20 to 28 us whatever the width; eight threads per column: the layer of 16 x 512, H 1024
// 893 -> 889 us with sixteen, of 7 x 333 411.5 -> 408; level elsewhere.)
template <typename T>
__global__ __launch_bounds__(256) void colreduce2_k(const float *partial, int chunks, int cols, T *out_b, T *out_g, int accumulate) {
  __shared__ float sb[16][16], sg[16][16];
  const int cl = threadIdx.x & 15, grp = threadIdx.x >> 4, c = blockIdx.x * 16 + cl;
  float b = 0.f, g = 0.f;
  if (c < cols) {
    for (int k0 = grp; chunks > 32 && k0 < chunks; k0 += 128) {
      float vb[8], vg[8] = {};
#pragma unroll
      for (int i = 0; i < 8; ++i) vb[i] = partial[(size_t)min(k0 + 16 * i, chunks - 1) * cols + c];
      if (out_g) {
#pragma unroll
        for (int i = 0; i < 8; ++i) vg[i] = partial[(size_t)(chunks + min(k0 + 16 * i, chunks - 1)) * cols + c];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        b += k0 + 16 * i < chunks ? vb[i] : 0.f;
        g += k0 + 16 * i < chunks ? vg[i] : 0.f;
      }
    }
    for (int k = grp; chunks <= 32 && k < chunks; k += 16) {
      b += partial[(size_t)k * cols + c];
      if (out_g) g += partial[(size_t)(chunks + k) * cols + c];
    }
  }
  sb[grp][cl] = b;
  sg[grp][cl] = g;
  __syncthreads();
  if (grp != 0 || c >= cols) return;
#pragma unroll
  for (int k = 1; k < 16; ++k) {
    b += sb[k][cl];
    g += sg[k][cl];
  }
  if (out_b) st(out_b + c, accumulate ? ld(out_b + c) + b : b);
  if (out_g) st(out_g + c, accumulate ? ld(out_g + c) + g : g);
}

template <typename T>
static hipError_t colreduce2(const float *partial, int chunks, int cols, void *out_b, void *out_g, bool accumulate, hipStream_t s) {
  hipLaunchKernelGGL(colreduce2_k<T>, dim3((cols + 15) / 16), dim3(256), 0, s, partial, chunks, cols, (T *)out_b, (T *)out_g,
                     accumulate ? 1 : 0);
  return hipGetLastError();
}

template <typename T>
static hipError_t norm_bwd_t(const T *dy, const T *x, const float *mean, const float *rstd, const T *gamma, const T *resid, T *dx,
                             void *dgamma, void *dbeta, float *partial, size_t room, int rows, int H, int kind, bool accumulate, hipStream_t s) {
  if (room < (size_t)2 * H) return hipErrorInvalidValue;
  const int chunks = colreduce_chunks(rows, room / ((size_t)2 * H));
  hipError_t e = norm_bwd_vec(dy, x, mean, rstd, gamma, resid, dx, partial, rows, H, kind, chunks, sizeof(T) == 4 ? SSDT_F32 : SSDT_BF16, s);
  if (e == hipErrorNotSupported) {
    prof::Scope ps(prof::NORM_BWD, 0, (resid ? 4.0 : 3.0) * rows * H * sizeof(T), s);
    const int col_blocks = (H + 127) / 128;
    auto go = [&](int sums, int dx_blocks) {
      hipLaunchKernelGGL(norm_bwd_k<T>, dim3(sums * col_blocks + dx_blocks), dim3(256), 0, s, dy, x, mean, rstd, gamma, resid, dx,
                         partial, rows, H, kind, (rows + chunks - 1) / chunks, sums, col_blocks);
    };
    norm_bwd_launch(go, chunks, col_blocks, rows);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  prof::Scope ps(prof::COLREDUCE, 0, 8.0 * chunks * H, s);
  return colreduce2<T>(partial, chunks, H, dbeta, dgamma, accumulate, s);
}

hipError_t norm_bwd(const void *dy, const void *x, const float *mean, const float *rstd, const void *gamma,
                    const void *resid, void *dx, void *dgamma, void *dbeta, float *partial, size_t room, int rows, int H,
                    int kind, int dtype, bool accumulate, hipStream_t s) {
  if (dtype == SSDT_F32)
    return norm_bwd_t((const float *)dy, (const float *)x, mean, rstd, (const float *)gamma, (const float *)resid, (float *)dx, dgamma,
                      dbeta, partial, room, rows, H, kind, accumulate, s);
  return norm_bwd_t((const bf16 *)dy, (const bf16 *)x, mean, rstd, (const bf16 *)gamma, (const bf16 *)resid, (bf16 *)dx, dgamma, dbeta,
                    partial, room, rows, H, kind, accumulate, s);
}

template <typename T>
static hipError_t colsum_t(const T *a, long lda, void *out, float *partial, size_t room, int rows, int cols, bool accumulate, hipStream_t s) {
  if (room < (size_t)cols) return hipErrorInvalidValue;
  const int chunks = colreduce_chunks(rows, room / cols);
  prof::Scope ps(prof::COLREDUCE, 0, 1.0 * rows * cols * sizeof(T), s);
  hipError_t e = sizeof(T) == 2 ? colreduce1_vec(a, lda, partial, rows, cols, chunks, s) : hipErrorNotSupported;
  if (e == hipErrorNotSupported) {
    hipLaunchKernelGGL(colreduce1_k<T>, dim3((cols + 127) / 128, chunks), dim3(256), 0, s, a, lda, partial, rows, cols,
                       (rows + chunks - 1) / chunks);
    e = hipGetLastError();
  }
  return e != hipSuccess ? e : colreduce2<T>(partial, chunks, cols, out, nullptr, accumulate, s);
}
hipError_t colsum(const void *a, long lda, void *out, float *partial, size_t room, int rows, int cols, int dtype,
                  bool accumulate, hipStream_t s) {
  if (dtype == SSDT_F32) return colsum_t((const float *)a, lda, out, partial, room, rows, cols, accumulate, s);
  return colsum_t((const bf16 *)a, lda, out, partial, room, rows, cols, accumulate, s);
}

// ------------------------------------------------------------------------------------------
// attention, one wavefront per row
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_generic_k(AttnP p) {
  __shared__ float lds[4][128];
  const int w = threadIdx.x >> 6, i = blockIdx.x * 4 + w;
  if (i < p.Sq) row_fwd<T>(p, blockIdx.z, blockIdx.y, i, threadIdx.x & 63, lds[w]);
}

template <typename T>
__global__ __launch_bounds__(256) void attn_delta_k(AttnP p, float *lse2) {
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int i = blockIdx.x * 4 + w, h = blockIdx.y, b = blockIdx.z;
  if (i >= p.Sq) return;
  const T *o = (const T *)p.o + (long)(b * p.Sq + i) * p.ldo + h * p.d;
  const T *dO = (const T *)p.dout + (long)(b * p.Sq + i) * p.lddo + h * p.d;
  float s = 0.f;
  for (int c = lane; c < p.d; c += 64) s += ld(o + c) * ld(dO + c);
  s = wave_sum(s);
  if (lane == 0) {
    const long at = ((long)b * p.A + h) * p.Sq + i;
    p.delta[at] = s;
    if (lse2) lse2[at] = lse_base2(p.lse[at]);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_generic_k(AttnP p) {
  __shared__ float lds[4][256];
  const int w = threadIdx.x >> 6, i = blockIdx.x * 4 + w;
  if (i < p.Sq) row_dq<T>(p, blockIdx.z, blockIdx.y, i, threadIdx.x & 63, lds[w]);
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_generic_k(AttnP p) {
  __shared__ float lds[4][256];
  const int w = threadIdx.x >> 6, j = blockIdx.x * 4 + w;
  if (j < p.Sk) row_dkv<T>(p, blockIdx.z, blockIdx.y, j, threadIdx.x & 63, lds[w]);
}

static AttnP to_p(const Attn &a) {
  return AttnP{a.B, a.A, a.Sq, a.Sk, a.d, a.mask, a.scale, a.kv_len, a.q, a.k, a.v, a.dout, a.o, a.dq, a.dk, a.dv,
               a.lse, a.delta, a.ldq, a.ldk, a.ldv, a.ldo, a.lddo, a.lddq, a.lddk, a.lddv};
}

hipError_t attn_fwd(const Attn &a, hipStream_t s) {
  if (a.d > 128 || a.d <= 0) return hipErrorInvalidValue;
  if (a.mask == SSDT_MASK_CAUSAL && a.Sq != a.Sk) return hipErrorInvalidValue;
  const bool whole = (a.d == 64 || a.d == 128) && a.Sq % 128 == 0 && a.Sk % 128 == 0;
  if (a.dtype == SSDT_BF16 && (whole || !a.ordered)) {
    hipError_t e = attn_fwd_mfma_bf16(a, s);
    if (e != hipErrorNotSupported) return e;
  } else {
    hipError_t e = attn_fwd_f32(a, s);
    if (e != hipErrorNotSupported) return e;
  }
  return attn_fwd_generic(a, s);
}

static double attn_flops(const Attn &a) {
  return 4.0 * a.B * a.A * (double)a.Sq * a.Sk * a.d * (a.mask == SSDT_MASK_CAUSAL ? 0.5 : 1.0);
}

hipError_t attn_fwd_generic(const Attn &a, hipStream_t s) {
  prof::Scope ps(prof::ATTN_FWD, attn_flops(a), 0, s);
  AttnP p = to_p(a);
  dim3 grid((a.Sq + 3) / 4, a.A, a.B);
  if (a.dtype == SSDT_F32) hipLaunchKernelGGL(attn_fwd_generic_k<float>, grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL(attn_fwd_generic_k<bf16>, grid, dim3(256), 0, s, p);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

hipError_t attn_bwd(const Attn &a, hipStream_t s) {
  if (a.d > 128 || a.d <= 0 || !a.delta) return hipErrorInvalidValue;
  if (a.mask == SSDT_MASK_CAUSAL && a.Sq != a.Sk) return hipErrorInvalidValue;
  if (a.dtype == SSDT_BF16) {
    hipError_t e = attn_bwd_mfma_bf16(a, s);
    if (e != hipErrorNotSupported) return e;
  } else {
    hipError_t e = attn_bwd_f32(a, s);
    if (e != hipErrorNotSupported) return e;
  }
  return attn_bwd_generic(a, s);
}

hipError_t attn_delta(const Attn &a, float *lse2, hipStream_t s) {
  AttnP p = to_p(a);
  hipError_t e = attn_delta_vec(a.o, a.ldo, a.dout, a.lddo, a.delta, a.lse, lse2, a.B, a.Sq, a.A, a.d, a.dtype, s);
  if (e != hipErrorNotSupported) return e;
  dim3 gq((a.Sq + 3) / 4, a.A, a.B);
  if (a.dtype == SSDT_F32) hipLaunchKernelGGL(attn_delta_k<float>, gq, dim3(256), 0, s, p, lse2);
  else hipLaunchKernelGGL(attn_delta_k<bf16>, gq, dim3(256), 0, s, p, lse2);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

hipError_t attn_bwd_generic(const Attn &a, hipStream_t s) {
  prof::Scope ps(prof::ATTN_BWD, 2 * attn_flops(a), 0, s);
  AttnP p = to_p(a);
  dim3 gq((a.Sq + 3) / 4, a.A, a.B), gk((a.Sk + 3) / 4, a.A, a.B);
  if (a.dtype == SSDT_F32) {
    hipLaunchKernelGGL(attn_delta_k<float>, gq, dim3(256), 0, s, p, (float *)nullptr);
    hipLaunchKernelGGL(attn_bwd_dq_generic_k<float>, gq, dim3(256), 0, s, p);
    hipLaunchKernelGGL(attn_bwd_dkv_generic_k<float>, gk, dim3(256), 0, s, p);
  } else {
    hipLaunchKernelGGL(attn_delta_k<bf16>, gq, dim3(256), 0, s, p, (float *)nullptr);
    hipLaunchKernelGGL(attn_bwd_dq_generic_k<bf16>, gq, dim3(256), 0, s, p);
    hipLaunchKernelGGL(attn_bwd_dkv_generic_k<bf16>, gk, dim3(256), 0, s, p);
  }
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

// ------------------------------------------------------------------------------------------
// transpose, add
// ------------------------------------------------------------------------------------------
template <typename U>
__global__ __launch_bounds__(256) void transpose_k(const U *in, long ldi, U *out, long ldo, int rows, int cols) {
  __shared__ U tile[64][65];
  int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  for (int r = ty; r < 64; r += 4)
    if (r0 + r < rows && c0 + tx < cols) tile[r][tx] = in[(long)(r0 + r) * ldi + c0 + tx];
  __syncthreads();
  for (int c = ty; c < 64; c += 4)
    if (c0 + c < cols && r0 + tx < rows) out[(long)(c0 + c) * ldo + r0 + tx] = tile[tx][c];
}

// 16-bit elements, extents multiples of 64, 16-byte aligned rows: each wavefront moves a 64x64 tile with
// 16-byte accesses only and no LDS.  Lane (rb, cb) = (lane / 8, lane % 8) reads the 8x8 block at rows
// 8 rb.., columns 8 cb.. (eight lanes cover one 128-byte line of each row), transposes it in registers and
// writes it as rows 8 cb.., columns 8 rb.. of the output (again eight lanes per 128-byte line).
typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void transpose16_k(const uint16_t *in, long ldi, uint16_t *out, long ldo, int rows, int cols) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = (blockIdx.y * 2 + (wave >> 1)) * 64, c0 = (blockIdx.x * 2 + (wave & 1)) * 64;
  if (r0 >= rows || c0 >= cols) return;
  const int rb = lane >> 3, cb = lane & 7;
  const uint16_t *src = in + (long)(r0 + rb * 8) * ldi + c0 + cb * 8;
  uint32_t v[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const u32x4_nt q = __builtin_nontemporal_load((const u32x4_nt *)(src + i * ldi));
    v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
  }
  uint16_t *dst = out + (long)(c0 + cb * 8) * ldo + r0 + rb * 8;
#pragma unroll
  for (int j = 0; j < 8; ++j) {  // output row j of the block = column j of the input block
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t a = v[2 * k][j >> 1], b = v[2 * k + 1][j >> 1];
      o[k] = (j & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
    }
    const u32x4_nt w = {o[0], o[1], o[2], o[3]};
    __builtin_nontemporal_store(w, (u32x4_nt *)(dst + j * ldo));
  }
}

hipError_t transpose(const void *in, long ldi, void *out, long ldo, int rows, int cols, int dtype, hipStream_t s) {
  dim3 grid((cols + 63) / 64, (rows + 63) / 64);
  prof::Scope ps(prof::TRANSPOSE, 0, 2.0 * rows * cols * (dtype == SSDT_F32 ? 4 : 2), s);
  if (dtype != SSDT_F32 && rows % 64 == 0 && cols % 64 == 0 && ldi % 8 == 0 && ldo % 8 == 0 &&
      ((uintptr_t)in | (uintptr_t)out) % 16 == 0) {
    hipLaunchKernelGGL(transpose16_k, dim3((cols + 127) / 128, (rows + 127) / 128), dim3(256), 0, s, (const uint16_t *)in, ldi,
                       (uint16_t *)out, ldo, rows, cols);
    SSDT_LAUNCH_CHECK();
    return hipSuccess;
  }
  if (dtype == SSDT_F32)
    hipLaunchKernelGGL(transpose_k<uint32_t>, grid, dim3(256), 0, s, (const uint32_t *)in, ldi, (uint32_t *)out, ldo, rows, cols);
  else
    hipLaunchKernelGGL(transpose_k<uint16_t>, grid, dim3(256), 0, s, (const uint16_t *)in, ldi, (uint16_t *)out, ldo, rows, cols);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

template <typename T>
__global__ void sgd_update_k(T *w, const T *g, size_t n, float lr) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) st(w + i, fmaf(-lr, ld(g + i), ld(w + i)));
}
// bf16, 16 bytes per access
__global__ void sgd_update_bf16x8_k(uint4 *w, const uint4 *g, size_t n8, float lr) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n8; i += stride) {
    uint4 a = w[i];
    const uint4 b = g[i];
    uint32_t *pa = (uint32_t *)&a;
    const uint32_t *pb = (const uint32_t *)&b;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float w0 = bf2f((uint16_t)(pa[t] & 0xffff)), w1 = bf2f((uint16_t)(pa[t] >> 16));
      const float g0 = bf2f((uint16_t)(pb[t] & 0xffff)), g1 = bf2f((uint16_t)(pb[t] >> 16));
      pa[t] = pack_bf2(fmaf(-lr, g0, w0), fmaf(-lr, g1, w1));
    }
    w[i] = a;
  }
}

hipError_t sgd_update(void *w, const void *g, size_t n, float lr, int dtype, hipStream_t s) {
  if (n == 0) return hipSuccess;
  prof::Scope ps(prof::ADD, 0, 3.0 * n * (dtype == SSDT_F32 ? 4 : 2), s);
  if (dtype == SSDT_BF16 && n % 8 == 0 && (((uintptr_t)w | (uintptr_t)g) & 15) == 0) {
    size_t blocks = std::min<size_t>((n / 8 + 255) / 256, 16384);
    hipLaunchKernelGGL(sgd_update_bf16x8_k, dim3((unsigned)blocks), dim3(256), 0, s, (uint4 *)w, (const uint4 *)g, n / 8, lr);
  } else {
    size_t blocks = std::min<size_t>((n + 255) / 256, 65536);
    if (dtype == SSDT_F32) hipLaunchKernelGGL(sgd_update_k<float>, dim3((unsigned)blocks), dim3(256), 0, s, (float *)w, (const float *)g, n, lr);
    else hipLaunchKernelGGL(sgd_update_k<bf16>, dim3((unsigned)blocks), dim3(256), 0, s, (bf16 *)w, (const bf16 *)g, n, lr);
  }
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

template <typename T>
__global__ void add_inplace_k(T *y, const T *x, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) st(y + i, ld(y + i) + ld(x + i));
}

hipError_t add_inplace(void *y, const void *x, size_t n, int dtype, hipStream_t s) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) return hipSuccess;
  prof::Scope ps(prof::ADD, 0, 3.0 * n * (dtype == SSDT_F32 ? 4 : 2), s);
  if (dtype == SSDT_F32) hipLaunchKernelGGL(add_inplace_k<float>, dim3((unsigned)blocks), dim3(256), 0, s, (float *)y, (const float *)x, n);
  else hipLaunchKernelGGL(add_inplace_k<bf16>, dim3((unsigned)blocks), dim3(256), 0, s, (bf16 *)y, (const bf16 *)x, n);
  SSDT_LAUNCH_CHECK();
  return hipSuccess;
}

}  // namespace k
}  // namespace ssdt
