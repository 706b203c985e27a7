// Attention one row at a time: a wavefront computes one query's output, one query's gradient or one key's two gradients,
// reading exactly the rows that the mask admits.  The row kernels are made of these, and the matrix-core kernels fall
// back on them, see `bad_rows`.
#pragma once
#include "dev.h"
#include "kernels.h"

namespace ssdt {
namespace k {

struct AttnP {
  int B, A, Sq, Sk, d, mask;
  float scale;
  const int32_t *kv_len;
  const void *q, *k, *v, *dout;
  void *o, *dq, *dk, *dv;
  float *lse, *delta;
  long ldq, ldk, ldv, ldo, lddo, lddq, lddk, lddv;
};

__device__ __forceinline__ int key_limit(const AttnP &p, int b, int i) {
  int lim = p.Sk;
  if (p.mask == SSDT_MASK_CAUSAL) lim = min(lim, i + 1);
  if (p.mask == SSDT_MASK_KEYPAD && p.kv_len) lim = min(lim, max(0, p.kv_len[b]));
  return lim;
}

// what the lanes of a wavefront have written to LDS is there for all of them behind this
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The matrix-core kernels multiply a masked row by a probability of zero, and zero times infinity is NaN: an infinity or a
// NaN in a key, value, query or gradient that the mask hides would show in what must not depend on it, and with
// probabilities as sums of bf16 an infinity that may be seen would come out as NaN.  It does show in the accumulators
// (a NaN never leaves them), so a wavefront looks at them once, at its end, and does the rows that are not finite again
// by the functions below.
// Zero if all of x is finite, else NaN; `seen` is what earlier calls returned.
template <int N, typename V>
__device__ __forceinline__ float not_finite(const V (&x)[N], float seen = 0.f) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (unsigned r = 0; r < sizeof(V) / 4; ++r) seen = fmaf(x[i][r], 0.f, seen);
  return seen;
}
// The wavefront's rows, one per lane modulo ROWS (16 or 32), that some lane calls bad.
template <int ROWS>
__device__ __forceinline__ unsigned bad_rows(bool bad) {
  unsigned long long m = __builtin_amdgcn_ballot_w64(bad);
  m |= m >> 32;
  if (ROWS == 16) m |= m >> 16;
  return (unsigned)m & (unsigned)((1ull << ROWS) - 1);
}

// Calls row(r, lane, w) for the rows r of the workgroup (ROWS of them per wavefront w) that bad_rows has found; what the
// wavefronts share in LDS is free by then.
template <int ROWS, typename F>
__device__ __forceinline__ void redo(unsigned again, F row) {
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  for (; again; again &= again - 1) row(w * ROWS + __builtin_ctz(again), lane, w);
}

// The same for a caller that has no register left for the thread's index: it gives the wavefront and the lane.
template <int ROWS, typename F>
__device__ __forceinline__ void redo(unsigned again, int w, int lane, F row) {
  __syncthreads();
  for (; again; again &= again - 1) row(w * ROWS + __builtin_ctz(again), lane, w);
}

// The kernel's first argument, read again: what only the rare path needs then takes no registers before it.
template <typename P>
using late_args_t = const __attribute__((address_space(4))) P *;
template <typename P>
__device__ __forceinline__ late_args_t<P> late_args() {
  late_args_t<P> p = (late_args_t<P>)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// output and log-sum-exp of query i; `sq`: 128 floats of LDS of the wavefront's own
template <typename T>
__device__ __forceinline__ void row_fwd(const AttnP &p, int b, int h, int i, int lane, float *sq) {
  const T *q = (const T *)p.q + (long)(b * p.Sq + i) * p.ldq + h * p.d;
  const T *kb = (const T *)p.k + (long)b * p.Sk * p.ldk + h * p.d;
  const T *vb = (const T *)p.v + (long)b * p.Sk * p.ldv + h * p.d;
  wave_sync();
  for (int c = lane; c < p.d; c += 64) sq[c] = ld(q + c);
  wave_sync();
  int lim = key_limit(p, b, i);
  float m = -INFINITY, l = 0.f, acc0 = 0.f, acc1 = 0.f;
  for (int j0 = 0; j0 < lim; j0 += 64) {
    int j = j0 + lane;
    float s = -INFINITY;
    if (j < lim) {
      const T *kr = kb + (long)j * p.ldk;
      float dot = 0.f;
      for (int c = 0; c < p.d; ++c) dot = fmaf(sq[c], ld(kr + c), dot);
      s = dot * p.scale;
    }
    float mn = fmaxf(m, wave_max(s));
    float pj = (j < lim) ? expf(s - mn) : 0.f;
    float corr = (m == -INFINITY) ? 0.f : expf(m - mn);
    l = l * corr + wave_sum(pj);
    acc0 *= corr;
    acc1 *= corr;
    int cnt = min(64, lim - j0);
    for (int jj = 0; jj < cnt; ++jj) {
      float pp = __shfl(pj, jj, 64);
      const T *vr = vb + (long)(j0 + jj) * p.ldv;
      if (lane < p.d) acc0 = fmaf(pp, ld(vr + lane), acc0);
      if (lane + 64 < p.d) acc1 = fmaf(pp, ld(vr + lane + 64), acc1);
    }
    m = mn;
  }
  T *o = (T *)p.o + (long)(b * p.Sq + i) * p.ldo + h * p.d;
  float inv = l > 0.f ? 1.f / l : 0.f;
  if (lane < p.d) st(o + lane, acc0 * inv);
  if (lane + 64 < p.d) st(o + lane + 64, acc1 * inv);
  if (lane == 0) p.lse[((long)b * p.A + h) * p.Sq + i] = l > 0.f ? m + logf(l) : -INFINITY;
}

// gradient of query i; `lds`: 256 floats
template <typename T>
__device__ __forceinline__ void row_dq(const AttnP &p, int b, int h, int i, int lane, float *lds) {
  float *sq = lds, *sdo = lds + 128;
  long row = (long)b * p.Sq + i;
  const T *q = (const T *)p.q + row * p.ldq + h * p.d;
  const T *dO = (const T *)p.dout + row * p.lddo + h * p.d;
  const T *kb = (const T *)p.k + (long)b * p.Sk * p.ldk + h * p.d;
  const T *vb = (const T *)p.v + (long)b * p.Sk * p.ldv + h * p.d;
  wave_sync();
  for (int c = lane; c < p.d; c += 64) {
    sq[c] = ld(q + c);
    sdo[c] = ld(dO + c);
  }
  wave_sync();
  int lim = key_limit(p, b, i);
  long si = ((long)b * p.A + h) * p.Sq + i;
  float lse = p.lse[si], dl = p.delta[si];
  float acc0 = 0.f, acc1 = 0.f;
  for (int j0 = 0; j0 < lim; j0 += 64) {
    int j = j0 + lane;
    float ds = 0.f;
    if (j < lim && lse != -INFINITY) {
      const T *kr = kb + (long)j * p.ldk, *vr = vb + (long)j * p.ldv;
      float dot = 0.f, dp = 0.f;
      for (int c = 0; c < p.d; ++c) {
        dot = fmaf(sq[c], ld(kr + c), dot);
        dp = fmaf(sdo[c], ld(vr + c), dp);
      }
      ds = expf(dot * p.scale - lse) * (dp - dl);
    }
    int cnt = min(64, lim - j0);
    for (int jj = 0; jj < cnt; ++jj) {
      float dd = __shfl(ds, jj, 64);
      const T *kr = kb + (long)(j0 + jj) * p.ldk;
      if (lane < p.d) acc0 = fmaf(dd, ld(kr + lane), acc0);
      if (lane + 64 < p.d) acc1 = fmaf(dd, ld(kr + lane + 64), acc1);
    }
  }
  T *dq = (T *)p.dq + row * p.lddq + h * p.d;
  if (lane < p.d) st(dq + lane, acc0 * p.scale);
  if (lane + 64 < p.d) st(dq + lane + 64, acc1 * p.scale);
}

// gradients of key j and its value; `lds`: 256 floats
template <typename T>
__device__ __forceinline__ void row_dkv(const AttnP &p, int b, int h, int j, int lane, float *lds) {
  float *sk = lds, *sv = lds + 128;
  long row = (long)b * p.Sk + j;
  const T *kr = (const T *)p.k + row * p.ldk + h * p.d;
  const T *vr = (const T *)p.v + row * p.ldv + h * p.d;
  wave_sync();
  for (int c = lane; c < p.d; c += 64) {
    sk[c] = ld(kr + c);
    sv[c] = ld(vr + c);
  }
  wave_sync();
  bool key_valid = !(p.mask == SSDT_MASK_KEYPAD && p.kv_len && j >= p.kv_len[b]);
  int istart = (p.mask == SSDT_MASK_CAUSAL) ? j : 0;
  float dk0 = 0.f, dk1 = 0.f, dv0 = 0.f, dv1 = 0.f;
  const T *qb = (const T *)p.q + (long)b * p.Sq * p.ldq + h * p.d;
  const T *dob = (const T *)p.dout + (long)b * p.Sq * p.lddo + h * p.d;
  if (key_valid) {
    for (int i0 = istart; i0 < p.Sq; i0 += 64) {
      int i = i0 + lane;
      float pp = 0.f, ds = 0.f;
      if (i < p.Sq) {
        long si = ((long)b * p.A + h) * p.Sq + i;
        float lse = p.lse[si];
        if (lse != -INFINITY) {
          const T *qr = qb + (long)i * p.ldq, *dr = dob + (long)i * p.lddo;
          float dot = 0.f, dp = 0.f;
          for (int c = 0; c < p.d; ++c) {
            dot = fmaf(ld(qr + c), sk[c], dot);
            dp = fmaf(ld(dr + c), sv[c], dp);
          }
          pp = expf(dot * p.scale - lse);
          ds = pp * (dp - p.delta[si]);
        }
      }
      int cnt = min(64, p.Sq - i0);
      for (int ii = 0; ii < cnt; ++ii) {
        float p1 = __shfl(pp, ii, 64), d1 = __shfl(ds, ii, 64);
        const T *qr = qb + (long)(i0 + ii) * p.ldq, *dr = dob + (long)(i0 + ii) * p.lddo;
        if (lane < p.d) {
          dv0 = fmaf(p1, ld(dr + lane), dv0);
          dk0 = fmaf(d1, ld(qr + lane), dk0);
        }
        if (lane + 64 < p.d) {
          dv1 = fmaf(p1, ld(dr + lane + 64), dv1);
          dk1 = fmaf(d1, ld(qr + lane + 64), dk1);
        }
      }
    }
  }
  T *dk = (T *)p.dk + row * p.lddk + h * p.d, *dv = (T *)p.dv + row * p.lddv + h * p.d;
  if (lane < p.d) {
    st(dk + lane, dk0 * p.scale);
    st(dv + lane, dv0);
  }
  if (lane + 64 < p.d) {
    st(dk + lane + 64, dk1 * p.scale);
    st(dv + lane + 64, dv1);
  }
}

}  // namespace k
}  // namespace ssdt
