// Row kernels, 16 bytes per lane per access: norm forward and backward with the row held in registers (each byte of the row
// is read from memory once), and the first stage of the deterministic column reductions (bias / gain / shift gradients).
// Bound by memory, or on small problems by the trips to it: a row's loads are all on their way at once.  Chosen when the
// width is a multiple of 16 bytes, rows are 16-byte aligned and (for the norms) H <= 8192 in bf16, 4096 in fp32.
// (fp32 against the generic kernels, which walk a row element by element, three times in the forward: both norms of
// 985 rows of 512 forward 17.4 -> 8.2 us, backward 18.9 -> 9.8; of 256 rows of 256 12.4 -> 7.7, 16.2 -> 7.9.)
#include "dev.h"
#include "kernels.h"
#include "prof.h"

namespace ssdt {
namespace k {

// the elements of 16 bytes as floats, and back
template <typename T> struct V16;
template <> struct V16<uint16_t> {
  static constexpr int E = 8;
  static __device__ __forceinline__ void get(const uint4 &v, float *f) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
  static __device__ __forceinline__ uint4 put(const float *f) {
    return make_uint4(pack_bf2(f[0], f[1]), pack_bf2(f[2], f[3]), pack_bf2(f[4], f[5]), pack_bf2(f[6], f[7]));
  }
};
template <> struct V16<float> {
  static constexpr int E = 4;
  static __device__ __forceinline__ void get(const uint4 &v, float *f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  static __device__ __forceinline__ uint4 put(const float *f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
  }
};

template <typename T, int NCH>
__global__ __launch_bounds__(256) void norm_fwd_vec_k(const T *x, const T *gamma, const T *beta,
                                                      T *y, float *mean, float *rstd, int rows, int H, float eps,
                                                      int kind) {
  constexpr int E = V16<T>::E;
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nch = H / E;
  const uint4 *xr = (const uint4 *)(x + (long)row * H);
  uint4 v[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    v[i] = c < nch ? xr[c] : make_uint4(0, 0, 0, 0);
  }
  float mu = 0.f;
  if (kind == SSDT_NORM_LAYERNORM) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      float f[E];
      V16<T>::get(v[i], f);
#pragma unroll
      for (int t = 0; t < E; ++t) sum += f[t];
    }
    mu = wave_sum(sum) / (float)H;
  }
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    if (i * 64 + lane < nch) {
      float f[E];
      V16<T>::get(v[i], f);
#pragma unroll
      for (int t = 0; t < E; ++t) { float d = f[t] - mu; sq += d * d; }
    }
  }
  const float r = 1.f / sqrtf(wave_sum(sq) / (float)H + eps);
  uint4 *yr = (uint4 *)(y + (long)row * H);
  const uint4 *g4 = (const uint4 *)gamma, *b4 = (const uint4 *)beta;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    if (c < nch) {
      float f[E], g[E], o[E];
      V16<T>::get(v[i], f);
      V16<T>::get(g4[c], g);
#pragma unroll
      for (int t = 0; t < E; ++t) o[t] = (f[t] - mu) * r * g[t];
      if (beta) {
        float b[E];
        V16<T>::get(b4[c], b);
#pragma unroll
        for (int t = 0; t < E; ++t) o[t] += b[t];
      }
      yr[c] = V16<T>::put(o);
    }
  }
  if (lane == 0) {
    if (mean) mean[row] = mu;
    rstd[row] = r;
  }
}

template <typename T, int NCH>
__device__ __forceinline__ void norm_bwd_dx(const T *dy, const T *x, const float *mean, const float *rstd,
                                            const T *gamma, const T *resid, T *dx, int rows, int H, int kind,
                                            int block, uint4 *g4) {
  // the gain vector is shared by the block's four rows and read twice per row: staged in LDS once (read from global
  // memory chunk by chunk, every one of its 2 x NCH loads was a full round trip in front of the arithmetic)
  constexpr int E = V16<T>::E;
  const int lane = threadIdx.x & 63, row = block * 4 + (threadIdx.x >> 6);
  const int nch = H / E;
  for (int c = threadIdx.x; c < nch; c += 256) g4[c] = ((const uint4 *)gamma)[c];
  __syncthreads();
  if (row >= rows) return;
  const uint4 *xr = (const uint4 *)(x + (long)row * H), *dyr = (const uint4 *)(dy + (long)row * H);
  const float mu = (kind == SSDT_NORM_LAYERNORM) ? mean[row] : 0.f, r = rstd[row];
  uint4 vx[NCH], vd[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    vx[i] = c < nch ? xr[c] : make_uint4(0, 0, 0, 0);
    vd[i] = c < nch ? dyr[c] : make_uint4(0, 0, 0, 0);
  }
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    if (c < nch) {
      float fx[E], fd[E], g[E];
      V16<T>::get(vx[i], fx);
      V16<T>::get(vd[i], fd);
      V16<T>::get(g4[c], g);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const float dh = fd[t] * g[t], xh = (fx[t] - mu) * r;
        s1 += dh;
        s2 += dh * xh;
      }
    }
  }
  const float c1 = (kind == SSDT_NORM_LAYERNORM) ? wave_sum(s1) / (float)H : 0.f;
  const float c2 = wave_sum(s2) / (float)H;
  uint4 *dxr = (uint4 *)(dx + (long)row * H);
  // the residual-branch gradient: all of its loads go out before the first result is stored (loads issued between
  // stores are waited for one at a time, and this kernel is nothing but memory latency)
  uint4 vr[NCH];
  if (resid) {
    const uint4 *rr = (const uint4 *)(resid + (long)row * H);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = i * 64 + lane;
      vr[i] = c < nch ? rr[c] : make_uint4(0, 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    if (c < nch) {
      float fx[E], fd[E], g[E], o[E];
      V16<T>::get(vx[i], fx);
      V16<T>::get(vd[i], fd);
      V16<T>::get(g4[c], g);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const float dh = fd[t] * g[t], xh = (fx[t] - mu) * r;
        o[t] = r * (dh - c1 - xh * c2);
      }
      if (resid) {
        float q[E];
        V16<T>::get(vr[i], q);
#pragma unroll
        for (int t = 0; t < E; ++t) o[t] += q[t];
      }
      vx[i] = V16<T>::put(o);
    }
  }
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = i * 64 + lane;
    if (c < nch) dxr[c] = vx[i];
  }
}

typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));

// Stage 1 of a column reduction: block (cx, chunk) sums 64 lanes' columns over its chunk of rows, the 4
// wavefronts taking every 4th row, then adds the 4 partial sums in a fixed order.
template <typename T, bool NORM>
__device__ __forceinline__ void colreduce1(const T *a, long lda, const T *x, const float *mean, const float *rstd,
                                           int kind, float *partial, int rows, int cols, int rows_per_chunk, int chunks, int cx,
                                           int chunk, float (*sb)[64 * V16<T>::E], float (*sg)[64 * V16<T>::E]) {
  constexpr int E = V16<T>::E, CB = 64 * E;  // columns of a block
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c0 = cx * CB + lane * E;
  const int r0 = chunk * rows_per_chunk, r1 = min(rows, r0 + rows_per_chunk);
  float g[E], b[E];
#pragma unroll
  for (int t = 0; t < E; ++t) g[t] = b[t] = 0.f;
  if (c0 < cols) {
#pragma unroll 4
    for (int r = r0 + w; r < r1; r += 4) {
      float v[E];
      V16<T>::get(*(const uint4 *)(a + (long)r * lda + c0), v);
#pragma unroll
      for (int t = 0; t < E; ++t) b[t] += v[t];
      if (NORM) {
        const float mu = (kind == SSDT_NORM_LAYERNORM) ? mean[r] : 0.f, rs = rstd[r];
        float xv[E];
        V16<T>::get(*(const uint4 *)(x + (long)r * lda + c0), xv);
#pragma unroll
        for (int t = 0; t < E; ++t) g[t] += v[t] * (xv[t] - mu) * rs;
      }
    }
  }
#pragma unroll
  for (int t = 0; t < E; ++t) {
    sb[w][lane * E + t] = b[t];
    if (NORM) sg[w][lane * E + t] = g[t];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < CB; i += 256) {
    const int c = cx * CB + i;
    if (c < cols) {
      partial[(size_t)chunk * cols + c] = ((sb[0][i] + sb[1][i]) + sb[2][i]) + sb[3][i];
      if (NORM) partial[(size_t)(chunks + chunk) * cols + c] = ((sg[0][i] + sg[1][i]) + sg[2][i]) + sg[3][i];
    }
  }
}
__global__ __launch_bounds__(256) void colreduce1_vec_k(const uint16_t *a, long lda, float *partial, int rows, int cols,
                                                        int rows_per_chunk) {
  __shared__ float sb[4][512];
  colreduce1<uint16_t, false>(a, lda, nullptr, nullptr, nullptr, 0, partial, rows, cols, rows_per_chunk, gridDim.y, blockIdx.x, blockIdx.y, sb, nullptr);
}

// The norm's backward: first the workgroups of the gain and shift gradients' stage 1, then those of dx.  Both read dy and
// x, and neither fills the machine for long: in one launch the second reads what the first has brought into the caches and
// each covers the other's waits.  (A layer's two norms, forward + backward of the layer: 256 tokens of H 256 117.5 -> 111.3 us,
// 256 of H 4096 497.5 -> 488.4, 8192 of H 1024 937 -> 923; level from 4096 tokens of H 4096 on.)
template <typename T, int NCH>
__global__ __launch_bounds__(256) void norm_bwd_vec_k(const T *dy, const T *x, const float *mean, const float *rstd,
                                                      const T *gamma, const T *resid, T *dx, float *partial,
                                                      int rows, int H, int kind, int rows_per_chunk, int chunks, int col_blocks) {
  constexpr int CB = 64 * V16<T>::E, kSums = 2 * 4 * CB * 4, kGain = NCH * 64 * 16;
  __shared__ __attribute__((aligned(16))) char lds[kSums > kGain ? kSums : kGain];  // either kind's: sums, or the gain vector
  float (*sums)[CB] = (float (*)[CB])lds;
  const int n1 = chunks * col_blocks, bid = blockIdx.x;
  if (bid < n1) colreduce1<T, true>(dy, H, x, mean, rstd, kind, partial, rows, H, rows_per_chunk, chunks, bid % col_blocks, bid / col_blocks, sums, sums + 4);
  else norm_bwd_dx<T, NCH>(dy, x, mean, rstd, gamma, resid, dx, rows, H, kind, bid - n1, (uint4 *)lds);
}

// delta[b, h, i] = sum_c o[b, i, h, c] dout[b, i, h, c] for rows that hold the heads side by side (head size a power of two of
// 16 to 1024 bytes): 16-byte loads, d / E lanes per head, whose sums are added together.  With lse2 set, also lse in the units that the
// matrix-core backward recomputes probabilities in (lse_base2).
// Few tokens of up to two KiB: one wavefront per token walks the row.
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_row_k(const T *o, long ldo, const T *dO, long lddo, float *delta,
                                                        const float *lse, float *lse2, long rows, int Sq, int A, int d) {
  constexpr int E = V16<T>::E;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long row = (long)blockIdx.x * 4 + w;  // b * Sq + i
  if (row >= rows) return;
  const int b = (int)(row / Sq), i = (int)(row % Sq), H = A * d, lph = d / E;
  o += row * ldo;
  dO += row * lddo;
  for (int c = lane * E; c < H; c += 64 * E) {
    const u32x4_nt a = __builtin_nontemporal_load((const u32x4_nt *)(o + c));
    const uint4 g = *(const uint4 *)(dO + c);  // read again by the backward kernels that follow
    float x[E], y[E];
    V16<T>::get(make_uint4(a.x, a.y, a.z, a.w), x);
    V16<T>::get(g, y);
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < E; ++t) s = fmaf(x[t], y[t], s);
    for (int m = 1; m < lph; m <<= 1) s += __shfl_xor(s, m, 64);
    if ((lane & (lph - 1)) == 0) {
      const long at = ((long)b * A + c / d) * Sq + i;
      delta[at] = s;
      if (lse2) lse2[at] = lse_base2(lse[at]);
    }
  }
}

// Otherwise a workgroup has one KiB of 16 tokens' rows, each wavefront that of four: all on their way at once, and the sums stored, through
// LDS, with the tokens of a head side by side.  What bounds it is memory: the trip there, which the kernel above makes once for each KiB,
// and, with a store of 4 bytes per token and head, the lines they touch.  1 x 2048, 64 heads of 128: 23.0 -> 13.0 us; 16 x 2048 230 ->
// 175; 4 x 1024, 16 heads 9.3 -> 8.5; 8 x 128, 32 heads of 64 5.7 -> 4.7.  (7 x 333, 16 heads of 64: 4.7, 5.1.)
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_vec_k(const T *o, long ldo, const T *dO, long lddo, float *delta,
                                                        const float *lse, float *lse2, long rows, int parts, int Sq, int A, int d) {
  constexpr int E = V16<T>::E;
  __shared__ float sums[64][17];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, H = A * d, lph = d / E, hp = 64 / lph;
  const int part = blockIdx.x % parts, c = (part * 64 + lane) * E;
  const long r0 = (long)(blockIdx.x / parts) * 16;
  u32x4_nt a[4];
  uint4 g[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const long row = r0 + w * 4 + n;
    a[n] = u32x4_nt{0, 0, 0, 0};
    g[n] = make_uint4(0, 0, 0, 0);
    if (row < rows && c < H) {
      a[n] = __builtin_nontemporal_load((const u32x4_nt *)(o + row * ldo + c));
      g[n] = *(const uint4 *)(dO + row * lddo + c);  // read again by the backward kernels that follow
    }
  }
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    float x[E], y[E], s = 0.f;
    V16<T>::get(make_uint4(a[n].x, a[n].y, a[n].z, a[n].w), x);
    V16<T>::get(g[n], y);
#pragma unroll
    for (int t = 0; t < E; ++t) s = fmaf(x[t], y[t], s);
    for (int m = 1; m < lph; m <<= 1) s += __shfl_xor(s, m, 64);
    if ((lane & (lph - 1)) == 0) sums[lane / lph][w * 4 + n] = s;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < hp * 16; k += 256) {
    const int h = part * hp + k / 16;
    const long row = r0 + k % 16;  // b * Sq + i
    if (row >= rows || h >= A) continue;
    const long at = (row / Sq * A + h) * Sq + row % Sq;
    delta[at] = sums[k / 16][k % 16];
    if (lse2) lse2[at] = lse_base2(lse[at]);
  }
}

static int pick_nch(int H, int E) {
  const int need = (H / E + 63) / 64;
  for (int n : {1, 2, 4, 8, 16})
    if (need <= n) return n;
  return 0;
}
static bool al16(const void *p) { return ((uintptr_t)p & 15) == 0; }
#define SSDT_BY_NCH(nch, F)                                                                                \
  switch (nch) { case 1: F(1); break; case 2: F(2); break; case 4: F(4); break; case 8: F(8); break; default: F(16); }

template <typename T>
static hipError_t norm_fwd_t(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int rows,
                             int H, float eps, int kind, hipStream_t s) {
  const int nch = (H % V16<T>::E == 0) ? pick_nch(H, V16<T>::E) : 0;
  if (!nch || !al16(x) || !al16(y) || !al16(gamma) || (beta && !al16(beta))) return hipErrorNotSupported;
  prof::Scope ps(prof::NORM_FWD, 0, 2.0 * rows * H * sizeof(T), s);
  dim3 grid((rows + 3) / 4);
#define SSDT_GO(N) hipLaunchKernelGGL((norm_fwd_vec_k<T, N>), grid, dim3(256), 0, s, (const T *)x, (const T *)gamma, \
                                      (const T *)beta, (T *)y, mean, rstd, rows, H, eps, kind)
  SSDT_BY_NCH(nch, SSDT_GO)
#undef SSDT_GO
  return hipGetLastError();
}
hipError_t norm_fwd_vec(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int rows,
                        int H, float eps, int kind, int dtype, hipStream_t s) {
  return dtype == SSDT_F32 ? norm_fwd_t<float>(x, gamma, beta, y, mean, rstd, rows, H, eps, kind, s)
                           : norm_fwd_t<uint16_t>(x, gamma, beta, y, mean, rstd, rows, H, eps, kind, s);
}

template <typename T>
static hipError_t norm_bwd_t(const void *dy, const void *x, const float *mean, const float *rstd, const void *gamma,
                             const void *resid, void *dx, float *partial, int rows, int H, int kind, int chunks, hipStream_t s) {
  constexpr int CB = 64 * V16<T>::E;
  const int nch = (H % V16<T>::E == 0) ? pick_nch(H, V16<T>::E) : 0;
  if (!nch || !al16(x) || !al16(dy) || !al16(dx) || !al16(gamma) || (resid && !al16(resid))) return hipErrorNotSupported;
  prof::Scope ps(prof::NORM_BWD, 0, (resid ? 4.0 : 3.0) * rows * H * sizeof(T), s);
  const int rpc = (rows + chunks - 1) / chunks, col_blocks = (H + CB - 1) / CB;
  auto go = [&](int sums, int dx_blocks) {
#define SSDT_GO(N) hipLaunchKernelGGL((norm_bwd_vec_k<T, N>), dim3(sums * col_blocks + dx_blocks), dim3(256), 0, s, (const T *)dy, (const T *)x, mean, rstd, \
                                      (const T *)gamma, (const T *)resid, (T *)dx, partial, rows, H, kind, rpc, sums, col_blocks)
    SSDT_BY_NCH(nch, SSDT_GO)
#undef SSDT_GO
  };
  norm_bwd_launch(go, chunks, col_blocks, rows);
  return hipGetLastError();
}
hipError_t norm_bwd_vec(const void *dy, const void *x, const float *mean, const float *rstd, const void *gamma,
                        const void *resid, void *dx, float *partial, int rows, int H, int kind, int chunks, int dtype, hipStream_t s) {
  return dtype == SSDT_F32 ? norm_bwd_t<float>(dy, x, mean, rstd, gamma, resid, dx, partial, rows, H, kind, chunks, s)
                           : norm_bwd_t<uint16_t>(dy, x, mean, rstd, gamma, resid, dx, partial, rows, H, kind, chunks, s);
}

template <typename T>
static hipError_t attn_delta_t(const void *o, long ldo, const void *dout, long lddo, float *delta, const float *lse, float *lse2,
                               int B, int Sq, int A, int d, hipStream_t s) {
  constexpr int E = V16<T>::E;
  const int lph = d / E;
  if (d % E || lph < 1 || lph > 64 || (lph & (lph - 1)) || ldo % E || lddo % E || !al16(o) || !al16(dout)) return hipErrorNotSupported;
  const long rows = (long)B * Sq, blocks = (rows + 15) / 16;
  const int parts = (A * d + 64 * E - 1) / (64 * E);  // KiB of a row
  if ((parts > 2 || rows * parts >= 8192) && one_axis(blocks * parts))
    hipLaunchKernelGGL(attn_delta_vec_k<T>, dim3((unsigned)(blocks * parts)), dim3(256), 0, s, (const T *)o, ldo, (const T *)dout, lddo, delta, lse,
                       lse2, rows, parts, Sq, A, d);
  else
    hipLaunchKernelGGL(attn_delta_row_k<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, (const T *)o, ldo, (const T *)dout, lddo, delta, lse,
                       lse2, rows, Sq, A, d);
  return hipGetLastError();
}
hipError_t attn_delta_vec(const void *o, long ldo, const void *dout, long lddo, float *delta, const float *lse, float *lse2,
                          int B, int Sq, int A, int d, int dtype, hipStream_t s) {
  return dtype == SSDT_F32 ? attn_delta_t<float>(o, ldo, dout, lddo, delta, lse, lse2, B, Sq, A, d, s)
                           : attn_delta_t<uint16_t>(o, ldo, dout, lddo, delta, lse, lse2, B, Sq, A, d, s);
}

hipError_t colreduce1_vec(const void *a, long lda, float *partial, int rows, int cols, int chunks, hipStream_t s) {
  if (cols % 8 || lda % 8 || !al16(a)) return hipErrorNotSupported;
  hipLaunchKernelGGL(colreduce1_vec_k, dim3((cols + 511) / 512, chunks), dim3(256), 0, s, (const uint16_t *)a, lda, partial, rows, cols,
                     (rows + chunks - 1) / chunks);
  return hipGetLastError();
}

}  // namespace k
}  // namespace ssdt
