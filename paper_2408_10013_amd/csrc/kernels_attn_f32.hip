// fp32 attention (forward also on bf16 storage, see Attn::ordered) on the matrix cores (v_mfma_f32_16x16x4_f32): forward with
// an online softmax and the backward with both sides in one launch, any sequence length, head sizes that are multiples of 4.
//
// The one-wavefront-per-row kernels it replaces read every key and value once per query and add the scores element by
// element; they were bound by those loads (64 sequences-times-heads of 512 x 512 x 64, causal: 532 us forward, 1670 backward; 16 of
// 1024 x 1024 x 128: 1085 and 3591).  Here 16 queries share each tile of 64 keys out of LDS: 55 and 174, 131 and 343 (the
// matrix pipe's fp32 rate, 157 TFLOP/s, is the bound; a quarter of it is reached on the first, a sixth to a fifth on the second).  The backward
// at head sizes above 64 does not fit its registers: 8 vector registers are spilled at 96 and 60 at 128, some of them inside
// the tile loop.  The results are the same bits: the
// instruction adds its four products one after the other, k ascending, and everything else is done in the same order
// (scores over columns, exponentials of the same differences, the sum of a tile's 64 probabilities as the same tree,
// outputs over keys, gradients over keys or queries, one rescale per tile).
//
// Layouts.  A wavefront owns 16 queries (key side: keys), one per lane l % 16 of each quarter q = l / 16.  Scores come out
// as (tile rows) x (own column): the tile's rows are fed permuted, row 4 (i % 4) + i / 4 of a 16-row block as row i, so that
// register r of quarter q holds tile row 4 r + q -- exactly what the next product wants as its k-th operand element
// in its r-th instruction, without a transposition.  Tiles lie in LDS as 64 rows of D floats; within a group of
// 16 columns, column 4 t + q is stored at position 4 q + t, so that one 16-byte read gives quarter q its operands of four
// instructions; the 16-byte chunks of a row are XOR-ed with swz(row), which keeps both the 16-byte reads (16 rows, one chunk)
// and the 4-byte reads of the transposed use (4 rows, 4 chunks) free of bank conflicts.
#include "attn_rows.h"
#include "dev.h"
#include "kernels.h"
#include "prof.h"

namespace ssdt {
namespace k {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct FaF {
  int B, A, Sq, Sk, d, mask;
  float scale;
  const int32_t *kv_len;
  const float *q, *k, *v, *dout, *delta;
  float *o, *dq, *dk, *dv, *lse;
  long ldq, ldk, ldv, ldo, lddo, lddq, lddk, lddv;
};

// the same call for the row functions
__device__ __forceinline__ AttnP by_rows() {
  const late_args_t<FaF> p = late_args<FaF>();
  return AttnP{p->B, p->A, p->Sq, p->Sk, p->d, p->mask, p->scale, p->kv_len, p->q, p->k, p->v, p->dout, p->o, p->dq, p->dk, p->dv,
               p->lse, const_cast<float *>(p->delta), p->ldq, p->ldk, p->ldv, p->ldo, p->lddo, p->lddq, p->lddk, p->lddv};
}

constexpr int kT = 64;  // tile rows
// floats between rows of a tile with D columns (D a multiple of 32 that holds the head): whole multiples of the 64 banks
__device__ __host__ constexpr int row_of(int D) { return (D + 63) / 64 * 64; }

__device__ __forceinline__ int swz16(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// 64 rows x D columns of a matrix into an LDS tile, through registers: each thread one or two groups of 16 columns of a row.
// Rows from `rows` on (counted from the matrix's start) and columns from d on are zeros: the buffer descriptor ends behind
// the last row.
template <int D, typename T = float>
struct TileF {
  static constexpr int NG = row_of(D) / 64;
  __amdgpu_buffer_rsrc_t rsrc;
  static constexpr int E = sizeof(T);
  int ldb, d, row, grp0;
  uint32_t v[NG][4 * E];
  __device__ __forceinline__ void start(const T *base, long ld, int rows, int d_, int tid) {
    const int n = rows <= 0 ? 0 : (int)(((long)(rows - 1) * ld + d_) * E);  // (below 2^31: checked by the launcher)
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, n, 0x00020000);
    ldb = (int)ld * E;
    d = d_;
    row = tid & 63;
    grp0 = __builtin_amdgcn_readfirstlane(tid >> 6);
  }
  __device__ __forceinline__ void load(int r0) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int off = (r0 + row) * ldb + (grp0 + 4 * i) * 16 * E;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + j * 16, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[i][j * 4 + t] = x[t];
      }
    }
  }
  __device__ __forceinline__ void put(float *s) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const int g = grp0 + 4 * i;
      if (g >= D / 16) continue;
      float x[16];
#pragma unroll
      for (int c = 0; c < 16; ++c)
        x[c] = __uint_as_float(E == 4 ? v[i][c] : c & 1 ? v[i][c >> 1] & 0xffff0000u : v[i][c >> 1] << 16);
      if (g * 16 + 16 > d) {
#pragma unroll
        for (int c = 0; c < 16; ++c) x[c] = g * 16 + c < d ? x[c] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(f32x4_t *)(s + row * row_of(D) + (((g * 4 + q) ^ swz16(row)) << 2)) = f32x4_t{x[q], x[4 + q], x[8 + q], x[12 + q]};
    }
  }
};

// Heads up to 64: the next tile's loads fly under the current tile's products.  Wider ones have no registers for that (they
// would spill); two workgroups share a compute unit and cover for each other.
template <int D>
constexpr bool kAhead = D <= 64;

// the own row of a wavefront's lane as operands: element t of group g = column 16 g + 4 t + quarter
template <int D, typename T>
__device__ __forceinline__ void own_row(const T *src, bool valid, int d, int lq, f32x4_t (&f)[D / 16]) {
#pragma unroll
  for (int g = 0; g < D / 16; ++g)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int c = 16 * g + 4 * t + lq;
      f[g][t] = valid && c < d ? ld(src + c) : 0.f;
    }
}

// (64 tile rows) x (16 own columns): acc[b][r] of quarter q = tile row 16 b + 4 r + q against the lane's own row
template <int D>
__device__ __forceinline__ void rows_by_own(const float *s, const f32x4_t (&f)[D / 16], int lane, f32x4_t (&acc)[4]) {
  const int lr = lane & 15, lq = lane >> 4, pr = (lr & 3) * 4 + (lr >> 2), key = swz16(pr);
#pragma unroll
  for (int b = 0; b < 4; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < D / 16; ++g) {
    f32x4_t a[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) a[b] = *(const f32x4_t *)(s + (b * 16 + pr) * row_of(D) + (((g * 4 + lq) ^ key) << 2));
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][t], f[g][t], acc[b], 0, 0, 0);
  }
}

// out[c][own] += sum over tile rows of s[row][c] x w[row][own]: out[g][r] of quarter q = column 16 g + 4 q + r
template <int D>
__device__ __forceinline__ void cols_by_weights(const float *s, const f32x4_t (&w)[4], int lane, f32x4_t (&out)[D / 16]) {
  const int lr = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = b * 16 + 4 * t + lq, key = swz16(4 * t + lq);
#pragma unroll
      for (int g = 0; g < D / 16; ++g) {
        const float x = s[row * row_of(D) + (((g * 4 + (lr & 3)) ^ key) << 2) + (lr >> 2)];
        out[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w[b][t], out[g], 0, 0, 0);
      }
    }
}

template <int D, typename T>
__device__ __forceinline__ void store_row(T *dst, const f32x4_t (&v)[D / 16], float mul, int d, int lq) {
#pragma unroll
  for (int g = 0; g < D / 16; ++g)
    if (16 * g + 4 * lq < d) {
#pragma unroll
      for (int t = 0; t < 4; ++t) st(dst + 16 * g + 4 * lq + t, v[g][t] * mul);
    }
}

__device__ __forceinline__ int fa_limit(const FaF &p, int b) {
  int lim = p.Sk;
  if (p.mask == SSDT_MASK_KEYPAD && p.kv_len) lim = min(lim, max(0, p.kv_len[b]));
  return lim;
}

// forward: 64 queries per workgroup, 16 per wavefront
template <int D, typename T>
__global__ __launch_bounds__(256, 2) void fa_f32_fwd_k(FaF p) {
  __shared__ __attribute__((aligned(16))) float sK[kT * row_of(D)], sV[kT * row_of(D)];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lq = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z, q0 = blockIdx.x * 64, qi = q0 + w * 16 + lr;
  int limit = fa_limit(p, b);
  const int own_lim = p.mask == SSDT_MASK_CAUSAL ? min(limit, qi + 1) : limit;  // this lane's query sees keys below it
  if (p.mask == SSDT_MASK_CAUSAL) limit = min(limit, q0 + 64);
  f32x4_t qf[D / 16], acc[D / 16];
  own_row<D>((const T *)p.q + ((long)b * p.Sq + qi) * p.ldq + h * p.d, qi < p.Sq, p.d, lq, qf);
#pragma unroll
  for (int g = 0; g < D / 16; ++g) acc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  TileF<D, T> tk, tv;
  tk.start((const T *)p.k + (long)b * p.Sk * p.ldk + h * p.d, p.ldk, limit, p.d, tid);
  tv.start((const T *)p.v + (long)b * p.Sk * p.ldv + h * p.d, p.ldv, limit, p.d, tid);
  if (kAhead<D>) {
    tk.load(0);
    tv.load(0);
  }
  for (int j0 = 0; j0 < limit; j0 += kT) {
    __syncthreads();  // everyone is done with the previous tile
    if (!kAhead<D>) {
      tk.load(j0);
      tv.load(j0);
    }
    tk.put(sK);
    tv.put(sV);
    __syncthreads();
    if (kAhead<D>) {  // (beyond the limit: zeros, not used)
      tk.load(j0 + kT);
      tv.load(j0 + kT);
    }
    f32x4_t s[4];
    rows_by_own<D>(sK, qf, lane, s);
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[kb][r] = j0 + kb * 16 + 4 * r + lq < own_lim ? s[kb][r] * p.scale : -INFINITY;
        mx = fmaxf(mx, s[kb][r]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), corr = m == -INFINITY ? 0.f : expf(m - mn);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[kb][r] = j0 + kb * 16 + 4 * r + lq < own_lim ? expf(s[kb][r] - mn) : 0.f;
    // the sum of the 64 probabilities as a butterfly over 64 lanes adds them: distance 32, 16, 8, 4, 2, 1
    float t4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) t4[r] = (s[0][r] + s[2][r]) + (s[1][r] + s[3][r]);
    float sum = (t4[0] + t4[2]) + (t4[1] + t4[3]);
    sum += __shfl_xor(sum, 32, 64);
    sum += __shfl_xor(sum, 16, 64);
    l = l * corr + sum;
#pragma unroll
    for (int g = 0; g < D / 16; ++g) acc[g] *= corr;
    m = mn;
    cols_by_weights<D>(sV, s, lane, acc);
  }
  const unsigned again = bad_rows<16>(qi < p.Sq && not_finite(acc) != 0.f);
  if (qi < p.Sq && !(again >> lr & 1)) {
    store_row<D>((T *)p.o + ((long)b * p.Sq + qi) * p.ldo + h * p.d, acc, l > 0.f ? 1.f / l : 0.f, p.d, lq);
    if (lq == 0) p.lse[((long)b * p.A + h) * p.Sq + qi] = l > 0.f ? m + logf(l) : -INFINITY;
  }
  redo<16>(again, [&](int r, int l64, int wv) { row_fwd<T>(by_rows(), b, h, q0 + r, l64, sK + wv * 128); });
}

// backward, query side: dQ[i] = scale sum_j dS_ij k_j, 64 queries per workgroup
template <int D>
__device__ __forceinline__ void f32_dq(const FaF &p, int bx, int h, int b, float *sK, float *sV) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lq = lane >> 4;
  const int q0 = bx * 64, qi = q0 + w * 16 + lr;
  int limit = fa_limit(p, b);
  const int own_lim = p.mask == SSDT_MASK_CAUSAL ? min(limit, qi + 1) : limit;
  if (p.mask == SSDT_MASK_CAUSAL) limit = min(limit, q0 + 64);
  f32x4_t qf[D / 16], dof[D / 16], acc[D / 16];
  own_row<D>(p.q + ((long)b * p.Sq + qi) * p.ldq + h * p.d, qi < p.Sq, p.d, lq, qf);
  own_row<D>(p.dout + ((long)b * p.Sq + qi) * p.lddo + h * p.d, qi < p.Sq, p.d, lq, dof);
#pragma unroll
  for (int g = 0; g < D / 16; ++g) acc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const long si = ((long)b * p.A + h) * p.Sq + qi;
  const float lse = qi < p.Sq ? p.lse[si] : -INFINITY, delta = qi < p.Sq ? p.delta[si] : 0.f;
  TileF<D> tk, tv;
  tk.start(p.k + (long)b * p.Sk * p.ldk + h * p.d, p.ldk, limit, p.d, tid);
  tv.start(p.v + (long)b * p.Sk * p.ldv + h * p.d, p.ldv, limit, p.d, tid);
  if (kAhead<D>) {
    tk.load(0);
    tv.load(0);
  }
  for (int j0 = 0; j0 < limit; j0 += kT) {
    __syncthreads();
    if (!kAhead<D>) {
      tk.load(j0);
      tv.load(j0);
    }
    tk.put(sK);
    tv.put(sV);
    __syncthreads();
    if (kAhead<D>) {
      tk.load(j0 + kT);
      tv.load(j0 + kT);
    }
    f32x4_t s[4], dp[4];
    rows_by_own<D>(sK, qf, lane, s);
    rows_by_own<D>(sV, dof, lane, dp);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool in = j0 + kb * 16 + 4 * r + lq < own_lim && lse != -INFINITY;
        const float e = expf(in ? s[kb][r] * p.scale - lse : -INFINITY);
        s[kb][r] = in ? e * (dp[kb][r] - delta) : 0.f;
      }
    cols_by_weights<D>(sK, s, lane, acc);
  }
  const unsigned again = bad_rows<16>(qi < p.Sq && not_finite(acc) != 0.f);
  if (qi < p.Sq && !(again >> lr & 1)) store_row<D>(p.dq + ((long)b * p.Sq + qi) * p.lddq + h * p.d, acc, p.scale, p.d, lq);
  redo<16>(again, [&](int r, int l64, int wv) { row_dq<float>(by_rows(), b, h, q0 + r, l64, sK + wv * 256); });
}

// backward, key side: dK[j] = scale sum_i dS_ij q_i, dV[j] = sum_i P_ij dO_i, 64 keys per workgroup
template <int D>
__device__ __forceinline__ void f32_dkv(const FaF &p, int bx, int h, int b, float *sQ, float *sdO, float *sLse, float *sDelta) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lq = lane >> 4;
  const int k0 = bx * 64, kj = k0 + w * 16 + lr;
  const int limit = fa_limit(p, b);
  f32x4_t kf[D / 16], vf[D / 16], dk[D / 16], dv[D / 16];
  own_row<D>(p.k + ((long)b * p.Sk + kj) * p.ldk + h * p.d, kj < limit, p.d, lq, kf);
  own_row<D>(p.v + ((long)b * p.Sk + kj) * p.ldv + h * p.d, kj < limit, p.d, lq, vf);
#pragma unroll
  for (int g = 0; g < D / 16; ++g) dk[g] = dv[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float *lse_g = p.lse + ((long)b * p.A + h) * p.Sq, *delta_g = p.delta + ((long)b * p.A + h) * p.Sq;
  TileF<D> tq, tdo;
  tq.start(p.q + (long)b * p.Sq * p.ldq + h * p.d, p.ldq, p.Sq, p.d, tid);
  tdo.start(p.dout + (long)b * p.Sq * p.lddo + h * p.d, p.lddo, p.Sq, p.d, tid);
  // a block whose keys are all beyond the limit has nothing to add up
  const int first = k0 >= limit ? p.Sq : p.mask == SSDT_MASK_CAUSAL ? k0 : 0;  // k0 is a multiple of the tile
  if (kAhead<D>) {
    tq.load(first);
    tdo.load(first);
  }
  for (int i0 = first; i0 < p.Sq; i0 += kT) {
    __syncthreads();
    if (!kAhead<D>) {
      tq.load(i0);
      tdo.load(i0);
    }
    tq.put(sQ);
    tdo.put(sdO);
    if (tid < kT) sLse[tid] = i0 + tid < p.Sq ? lse_g[i0 + tid] : -INFINITY;
    else if (tid < 2 * kT) sDelta[tid - kT] = i0 + tid - kT < p.Sq ? delta_g[i0 + tid - kT] : 0.f;
    __syncthreads();
    if (kAhead<D>) {
      tq.load(i0 + kT);
      tdo.load(i0 + kT);
    }
    f32x4_t s[4], dp[4];
    rows_by_own<D>(sQ, kf, lane, s);
    rows_by_own<D>(sdO, vf, lane, dp);
#pragma unroll
    for (int ib = 0; ib < 4; ++ib)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = ib * 16 + 4 * r + lq;
        const float lse = sLse[i];
        const bool in = kj < limit && lse != -INFINITY && !(p.mask == SSDT_MASK_CAUSAL && kj > i0 + i);
        s[ib][r] = expf(in ? s[ib][r] * p.scale - lse : -INFINITY);  // (not `in ? expf(..) : 0`: that is a branch per element)
        dp[ib][r] = in ? s[ib][r] * (dp[ib][r] - sDelta[i]) : 0.f;
      }
    cols_by_weights<D>(sdO, s, lane, dv);
    cols_by_weights<D>(sQ, dp, lane, dk);
  }
  const unsigned again = bad_rows<16>(kj < p.Sk && not_finite(dv, not_finite(dk)) != 0.f);
  if (kj < p.Sk && !(again >> lr & 1)) {
    store_row<D>(p.dk + ((long)b * p.Sk + kj) * p.lddk + h * p.d, dk, p.scale, p.d, lq);
    store_row<D>(p.dv + ((long)b * p.Sk + kj) * p.lddv + h * p.d, dv, 1.f, p.d, lq);
  }
  redo<16>(again, [&](int r, int l64, int wv) { row_dkv<float>(by_rows(), b, h, k0 + r, l64, sQ + wv * 256); });
}

// The two sides of the backward do not depend on each other and share a launch: the key side's workgroups first, which
// take longer (two launches: 37 us on 8 of 128 x 128 x 64, 28 in one).
template <int D>
__global__ __launch_bounds__(256, 2) void fa_f32_bwd_k(FaF p, int nkb, int nqb) {
  __shared__ __attribute__((aligned(16))) float s0[kT * row_of(D)], s1[kT * row_of(D)], sLse[kT], sDelta[kT];
  const int heads = p.A * p.B, nk = nkb * heads;
  const int bid = (int)blockIdx.x < nk ? blockIdx.x : blockIdx.x - nk, n = (int)blockIdx.x < nk ? nkb : nqb;
  const int bx = bid % n, h = bid / n % p.A, b = bid / n / p.A;
  if ((int)blockIdx.x < nk) f32_dkv<D>(p, bx, h, b, s0, s1, sLse, sDelta);
  else f32_dq<D>(p, bx, h, b, s0, s1);
}

// Whether they are worth it: a tile of 64 takes its time however little of it is used (forward + backward of 1 x 1: 10 us
// by the other kernels, 20 here; 37 x 37 x 32: 27 and 21; 70 x 70 x 100: backward 47 and 53; 130 x 130 x 128: 105 and 87).
static bool f32_worth(const Attn &a, bool bwd) { return (long)a.Sq * a.Sk >= (bwd && a.d > 64 ? 8192 : 1024); }

// What the kernels address with 32-bit byte offsets from a sequence's first row must stay below 2^31 (a tile beyond the
// last row included); 16-byte loads want whole ones per head.
static bool f32_supported(const Attn &a, bool bwd) {
  if (a.d % 4 || a.d > 128) return false;
  if (a.dtype == SSDT_BF16 && (bwd || a.ldk % 2 || a.ldv % 2 || (uintptr_t)a.k % 4 || (uintptr_t)a.v % 4)) return false;
  auto fits = [](long rows, long ld) { return (rows + 2 * kT + 64) * ld * 4 < 0x7fffffffL; };
  if (!fits(a.Sk, a.ldk) || !fits(a.Sk, a.ldv)) return false;
  return !bwd || (fits(a.Sq, a.ldq) && fits(a.Sq, a.lddo));
}
static FaF to_f32(const Attn &a) {
  return FaF{a.B, a.A, a.Sq, a.Sk, a.d, a.mask, a.scale, a.kv_len, (const float *)a.q, (const float *)a.k, (const float *)a.v,
             (const float *)a.dout, a.delta, (float *)a.o, (float *)a.dq, (float *)a.dk, (float *)a.dv, a.lse,
             a.ldq, a.ldk, a.ldv, a.ldo, a.lddo, a.lddq, a.lddk, a.lddv};
}
static double f32_flops(const Attn &a) { return 4.0 * a.B * a.A * (double)a.Sq * a.Sk * a.d * (a.mask == SSDT_MASK_CAUSAL ? 0.5 : 1.0); }

hipError_t attn_fwd_f32(const Attn &a, hipStream_t s) {
  if (!f32_supported(a, false) || !f32_worth(a, false)) return hipErrorNotSupported;
  prof::Scope ps(prof::ATTN_FWD, f32_flops(a), 0, s);
  const FaF p = to_f32(a);
  const dim3 grid((a.Sq + 63) / 64, a.A, a.B);
#define SSDT_GO(D)                                                                                              \
  if (a.dtype == SSDT_F32) hipLaunchKernelGGL((fa_f32_fwd_k<D, float>), grid, dim3(256), 0, s, p);                \
  else hipLaunchKernelGGL((fa_f32_fwd_k<D, bf16>), grid, dim3(256), 0, s, p)
  SSDT_BY_HEAD(a.d, SSDT_GO);
#undef SSDT_GO
  return hipGetLastError();
}

hipError_t attn_bwd_f32(const Attn &a, hipStream_t s) {
  const int nkb = (a.Sk + 63) / 64, nqb = (a.Sq + 63) / 64;
  const long workgroups = (long)(nkb + nqb) * a.A * a.B;
  if (!f32_supported(a, true) || !f32_worth(a, true) || !one_axis(workgroups)) return hipErrorNotSupported;
  prof::Scope ps(prof::ATTN_BWD, 2 * f32_flops(a), 0, s);
  hipError_t e = attn_delta(a, nullptr, s);
  if (e != hipSuccess) return e;
  const FaF p = to_f32(a);
  const dim3 grid((unsigned)workgroups);
#define SSDT_GO(D) hipLaunchKernelGGL(fa_f32_bwd_k<D>, grid, dim3(256), 0, s, p, nkb, nqb)
  SSDT_BY_HEAD(a.d, SSDT_GO);
#undef SSDT_GO
  return hipGetLastError();
}

}  // namespace k
}  // namespace ssdt
