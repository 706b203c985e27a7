// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32), any shape, any transposition, any alignment.
//
// bf16 storage, forward form only: for products whose order of additions is kept (Gemm::ordered), and for widths and
// alignments that the bf16 kernels do not take.
// The instruction multiplies and adds in fp32 with one rounding per step, k ascending (checked against a chain of fmaf on
// the host), and a tile's contraction is never split, so every output is the same sum in the same order, and the same
// bits, as a thread of the FMA kernel this replaces would produce.  That kernel was bound by its LDS reads (two bytes
// per flop: 46 us on 256 x 768 x 256, 374 on 985 x 512 x 2048, 538 on 4096 x 3072 x 1024; here 6, 33 and 266); here a wavefront reads 16 bytes per lane for four
// instructions of 32 cycles, and the matrix pipe (157 TFLOP/s) or, on small problems, the latency of a stage bounds it.
//
// Operands that are aligned to 16 bytes, the usual ones, come by direct global-to-LDS loads (gemm_f32_direct_k, further down);
// bf16 storage, odd contractions and other alignments go through registers (gemm_f32_k):
// 256 threads = 4 wavefronts in 2 x 2; tiles of 64 or 32 squared (128 was never better: with two stages on their way its
// accumulators leave room for two wavefronts per SIMD).  A stage is 16 k times (128 / tile), so that each
// thread brings in eight k of a row of either operand whatever the tile: through registers, loaded two stages ahead (a stage
// is shorter than a load takes: 985 x 512 x 2048 38 us one stage ahead, 33 two), into one of two LDS buffers.
// In LDS the 16 k of a row are stored with k = 4 t + q at position 4 q + t: the lanes of quarter q of a wavefront need
// k = q, 4 + q, 8 + q, 12 + q for four successive instructions and get them in one 16-byte read.  Rows are 80 bytes apart:
// 16 rows then start in 16 different four-bank groups.
#include <algorithm>
#include <type_traits>

#include "dev.h"
#include "kernels.h"
#include "mfma_common.h"
#include "prof.h"

namespace ssdt {
namespace k {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_a4_t __attribute__((ext_vector_type(4), aligned(4)));

struct F32P {
  int M, N, K;
  const void *A, *B;  // float or bf16, like everything up to aux
  void *C, *C2;
  const void *bias, *resid, *aux;
  long lda, ldb, ldc, ldr;
  int epi, act, tiles_m;
  float *colsum;  // sum over k of B(k, n), or null (k-major operands only)
  int colsum_acc;
};

constexpr int kRow = 20;  // floats between rows of a 16-k group in LDS

// How an operand is stored: k-major (element (k, r) at k * ld + r), K-contiguous rows read 16 bytes at a time (extents a
// multiple of 16 bytes), or K-contiguous rows read element by element.
enum { KMAJOR = 0, KVEC = 1, KSCALAR = 2 };

// One operand's loader: this thread's eight k of row `row` of every stage.  Buffer loads whose descriptor ends with the
// operand: what lies behind the last row arrives as zero, without a branch (a branch around the loads makes the
// compiler wait for them at its end).
template <typename T>
struct F32Raw { uint32_t w[8]; };  // eight elements as loaded: floats, or bf16 one to a register (read by 16 bytes: two, in the first four)
template <int MODE, typename T>
struct F32Side {
  static constexpr int E = sizeof(T);
  uint64_t at;
  long left, step;
  unsigned voff, ldb;
  int k;
  __device__ __forceinline__ void start(const T *base, long ld, int r0, int ext, int K, int row, int k8, int stage_k) {
    at = (uint64_t)(uintptr_t)(MODE == KMAJOR ? base + r0 : base + (long)r0 * ld);
    left = E * (MODE == KMAJOR ? (long)(K - 1) * ld + ext - r0 : (long)(ext - 1 - r0) * ld + K);
    step = E * (MODE == KMAJOR ? (long)stage_k * ld : (long)stage_k);
    ldb = (unsigned)ld * E;
    voff = MODE == KMAJOR ? (unsigned)k8 * 8 * ldb + row * E : (unsigned)row * ldb + k8 * 8 * E;
    k = k8 * 8;
  }
  __device__ __forceinline__ void load(F32Raw<T> &v) {
    const int hi = (int)(left >> 32), lo = (int)left;
    const int n = hi < 0 ? 0 : ((hi | (lo & (int)0x80000000)) ? 0x7fffffff : lo);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)at, 0, n, 0x00020000);
    if (MODE == KVEC) {
#pragma unroll
      for (int i = 0; i < E / 2; ++i) {
        const auto q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(voff + i * 16), 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) v.w[i * 4 + t] = q[t];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int off = (int)(MODE == KMAJOR ? voff + i * ldb : voff + i * E);
        if constexpr (E == 4) v.w[i] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        else v.w[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
      }
    }
    at += step;
    left -= step;
  }
  // as floats; the tail of a K-contiguous row continues in the next row and is masked, k0: the stage's first k
  __device__ __forceinline__ void get(const F32Raw<T> &v, float (&o)[8], int k0, int K) const {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      o[i] = __uint_as_float(E == 4 ? v.w[i] : MODE == KVEC ? (i & 1 ? v.w[i >> 1] & 0xffff0000u : v.w[i >> 1] << 16) : v.w[i] << 16);
    if (MODE == KMAJOR || k0 + k + 8 <= K) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = k0 + k + i < K ? o[i] : 0.f;
  }
};

template <int BT>
struct F32Lds { float s[2][2][128 / BT][BT * kRow]; };  // [buffer][operand][16-k group][row]

// tile `bid` of the problem
template <int BT, int AM, int BM, typename T>
__device__ __forceinline__ void f32_body(const F32P &p, int bid, F32Lds<BT> &lds) {
  constexpr int G = 128 / BT, TB = BT / 32, SK = 16 * G;  // 16-k groups per stage; 16 x 16 blocks per wavefront and dimension
  auto &s = lds.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1, lr = lane & 15, lq = lane >> 4;
  const int m0 = bid % p.tiles_m * BT, n0 = bid / p.tiles_m * BT;
  const int row = tid & (BT - 1), k8 = tid / BT;  // this thread's part of a stage, of either operand
  F32Side<AM, T> sa;
  F32Side<BM, T> sb;
  sa.start((const T *)p.A, p.lda, m0, p.M, p.K, row, k8, SK);
  sb.start((const T *)p.B, p.ldb, n0, p.N, p.K, row, k8, SK);
  f32x4_t acc[TB][TB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  F32Raw<T> va[2], vb[2];  // the next two stages, on their way
  // k = 8 (k8 % 2) + e of a group, e = 0..7, goes to position 4 (e % 4) + 2 (k8 % 2) + e / 4
  auto put = [&](int buf, int st) {
    float a[8], b[8];
    sa.get(va[buf], a, st * SK, p.K);
    sb.get(vb[buf], b, st * SK, p.K);
    float *da = &s[buf][0][k8 >> 1][row * kRow + 2 * (k8 & 1)], *db = &s[buf][1][k8 >> 1][row * kRow + 2 * (k8 & 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      *(float2 *)(da + 4 * q) = make_float2(a[q], a[4 + q]);
      *(float2 *)(db + 4 * q) = make_float2(b[q], b[4 + q]);
    }
  };
  auto load = [&](int buf) {  // (behind the last stage: out of range, or the start of the next rows, and not used)
    sa.load(va[buf]);
    sb.load(vb[buf]);
  };
  // Column sums of B: every workgroup of a weight gradient adds its fragments up (16 or 8 additions per lane and stage beside
  // matrix instructions of 512 cycles; a branch here would cost more), the first row of tiles stores them.  A stage's sum
  // is added with compensation, so the error does not grow with the number of stages.  (What is lost of an infinite sum is
  // no number: without the test the next stage would turn the infinity into NaN.)
  constexpr bool SUM = AM == KMAJOR && BM == KMAJOR;
  float tot[TB], low[TB];
#pragma unroll
  for (int j = 0; j < TB; ++j) tot[j] = low[j] = 0.f;
  const int ns = (p.K + SK - 1) / SK;
  // stage st out of buffer st % 2; stage st + 2 sets out for the registers that stage st left
  auto stage = [&](int st, int buf) {
    load(buf);
    float part[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) part[j] = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      f32x4_t a[TB], b[TB];
#pragma unroll
      for (int i = 0; i < TB; ++i) a[i] = *(const f32x4_t *)&s[buf][0][g][((wm * TB + i) * 16 + lr) * kRow + 4 * lq];
#pragma unroll
      for (int j = 0; j < TB; ++j) b[j] = *(const f32x4_t *)&s[buf][1][g][((wn * TB + j) * 16 + lr) * kRow + 4 * lq];
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][t], a[i][t], acc[i][j], 0, 0, 0);
      if (SUM)
#pragma unroll
        for (int j = 0; j < TB; ++j) part[j] += (b[j][0] + b[j][1]) + (b[j][2] + b[j][3]);
    }
    if (SUM)
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const float y = part[j] - low[j], t = tot[j] + y;
        low[j] = fabsf(t) < INFINITY ? (t - tot[j]) - y : 0.f;
        tot[j] = t;
      }
    put(buf ^ 1, st + 1);
    __syncthreads();
  };
  load(0);
  load(1);
  put(0, 0);
  __syncthreads();
  for (int st = 0; st < ns; st += 2) {
    stage(st, 0);
    if (st + 1 < ns) stage(st + 1, 1);
  }
  if (SUM && p.colsum && m0 == 0 && wm == 0) {
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      float x = tot[j];
      x += __shfl_xor(x, 16, 64);
      x += __shfl_xor(x, 32, 64);
      const int n = n0 + (wn * TB + j) * 16 + lr;
      if (lq == 0 && n < p.N) p.colsum[n] = p.colsum_acc ? p.colsum[n] + x : x;
    }
  }
  // this lane: row m, columns n .. n + 3 of each block
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    const int m = m0 + (wm * TB + i) * 16 + lr;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int n = n0 + (wn * TB + j) * 16 + lq * 4;
      const long o = (long)m * p.ldc + n;
      const bool whole = n + 4 <= p.N;
      float c[4], c2[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float x = acc[i][j][t], y = 0.f;
        if (n + t < p.N) {
          if (p.bias && p.epi != EPI_NONE && p.epi != EPI_ACTBWD) x += ld((const T *)p.bias + n + t);
          if (p.epi == EPI_BIAS_ACT) y = p.act == SSDT_ACT_GELU ? gelu_f(x) : fmaxf(x, 0.f);
          else if (p.epi == EPI_BIAS_RESID) x += ld((const T *)p.resid + (long)m * p.ldr + n + t);
          else if (p.epi == EPI_ACTBWD) {
            const float u = ld((const T *)p.aux + o + t);
            x *= p.act == SSDT_ACT_GELU ? gelu_grad_f(u) : (u > 0.f ? 1.f : 0.f);
          }
        }
        c[t] = x;
        c2[t] = y;
      }
      T *C = (T *)p.C + o, *C2 = (T *)p.C2 + o;
      if (sizeof(T) == 4 && whole) {
        if (p.C) *(f32x4_a4_t *)C = f32x4_a4_t{c[0], c[1], c[2], c[3]};
        if (p.epi == EPI_BIAS_ACT) *(f32x4_a4_t *)C2 = f32x4_a4_t{c2[0], c2[1], c2[2], c2[3]};
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (n + t < p.N) {
            if (p.C) st(C + t, c[t]);
            if (p.epi == EPI_BIAS_ACT) st(C2 + t, c2[t]);
          }
      }
    }
  }
}

template <int BT, int AM, int BM, typename T>
__global__ __launch_bounds__(256) void gemm_f32_k(F32P p) {
  __shared__ __attribute__((aligned(16))) F32Lds<BT> lds;
  f32_body<BT, AM, BM, T>(p, blockIdx.x, lds);
}
// The two products of a linear's backward in one launch (see gemm_tile_pair_k): the first `first` workgroups are the weight
// gradient's if w_first, else the input gradient's, MODE how the latter's operands are read.
template <int BT, int MODE>
__global__ __launch_bounds__(256) void gemm_f32_pair_k(F32P w, F32P d, int first, int w_first) {
  __shared__ __attribute__((aligned(16))) F32Lds<BT> lds;
  const int bid = blockIdx.x;
  const bool head = bid < first;
  if (head == (w_first != 0)) f32_body<BT, KMAJOR, KMAJOR, float>(w, head ? bid : bid - first, lds);
  else f32_body<BT, MODE, MODE, float>(d, head ? bid : bid - first, lds);
}

// ---- operands aligned to 16 bytes -----------------------------------------------------------------------------------
// A small problem is one or two workgroups per compute unit, one wavefront per SIMD, and what bounds it is everything that such a
// wavefront issues beside its matrix instructions (32 cycles each, a stage's chain 512): staging through registers, 450 ns a
// stage of 64 k, spends half of them on waits, conversions and LDS stores.  Here a stage has neither, its loads' descriptor moves
// on by six scalar instructions (recomputed in 64 bits it cost 50 ns of a stage), its LDS reads are dealt out between the matrix
// instructions, and the ring is three stages deep: 300 ns.  256 x 256 x 1024 14.1 -> 8.9 us, 985 x 512 x 2048 34 -> 25,
// 4096 x 3072 x 1024 220 -> 205 (127 TFLOP/s; 145 is what the matrix instructions alone reach at the clock they leave), both products of
// 985 x 2048 -> 512's backward 45 -> 42, of 256 x 256 -> 1024's 14.7 -> 10.0.
typedef __attribute__((address_space(3))) float lds_f32_t;

// One operand's side of the loader and of the fragment reads: a stage of SK k comes by direct global-to-LDS loads (two of
// 16 bytes per thread) and stays in the order it is stored in.
//   k-major: SK rows of BT floats; 64-byte unit u of k-row k at u ^ key(k), so that the four k-rows of a fragment read
//   lie in different quarters of the 64 banks;
//   K-contiguous: BT rows of SK floats, 16-byte chunk c of row r at c ^ key(r): the 16 rows of a read in 16 chunks.
template <int BT, int MODE>
struct F32Direct {
  static constexpr int SK = 2048 / BT, CPR = (MODE == KMAJOR ? BT : SK) / 4;
  static constexpr unsigned kBytes = BT * SK * 4;
  static __device__ __forceinline__ int key(int r) {
    if (MODE == KMAJOR) return BT == 64 ? r & 3 : (r >> 1) & 1;
    return SK == 64 ? r & 15 : (r >> 1) & 7;
  }
  unsigned voff[2];
  int chunk, k;
  // where the next stage starts; floats from there to the end of the operand (fewer than 2^29: direct_fits) and from stage to stage
  uint64_t at;
  int left, step;
  __device__ __forceinline__ void start(const float *base, long ld, int r0, int ext, int K, int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = j * 256 + tid, row = q / CPR, pos = q % CPR;
      const int c = MODE == KMAJOR ? (((pos >> 2) ^ key(row)) << 2) | (pos & 3) : pos ^ key(row);
      voff[j] = (unsigned)(row * (int)ld + c * 4) * 4u;
      chunk = c;  // (the same for both, K-contiguous)
    }
    at = (uint64_t)(uintptr_t)(MODE == KMAJOR ? base + r0 : base + (long)r0 * ld);
    left = (int)(MODE == KMAJOR ? (long)(K - 1) * ld + ext - r0 : (long)(ext - 1 - r0) * ld + K);
    step = MODE == KMAJOR ? SK * (int)ld : SK;
    k = 0;
  }
  // the next stage; TAIL: it may be the last one
  __device__ __forceinline__ void load(int K, unsigned lds, bool tail) {
    asm volatile("" : "+s"(at), "+s"(left), "+s"(lds));  // (addresses computed ahead would fill the scalar registers)
    v4i_t rsrc;
    rsrc[0] = (int)(unsigned)at;
    rsrc[1] = (int)(unsigned)(at >> 32) & 0xffff;
    rsrc[2] = (left & ~(left >> 31)) << 2;  // (no less than 0)
    rsrc[3] = 0x00020000;
    asm volatile("s_nop 4" : "+s"(rsrc));  // (see Side::desc of gemm_tile_k)
    const bool dead = MODE == KVEC && tail && k + chunk * 4 >= K;  // the tail of a row continues in the next row
#pragma unroll
    for (int j = 0; j < 2; ++j) load_lds16(rsrc, dead ? 0x80000000u : voff[j], lds + j * 4096);
    at += 4l * step;
    left -= step;
    k += SK;
  }
  // element (k = 4 s + lane / 16, own index 16 blk + lane % 16)
  static __device__ __forceinline__ float frag(unsigned lds, int blk, int s, int lane) {
    const int lr = lane & 15, lq = lane >> 4;
    const unsigned a = MODE == KMAJOR ? lds + (4 * s + lq) * (BT * 4) + ((blk ^ key(lq)) * 64 + lr * 4)
                                      : lds + (blk * 16 + lr) * (SK * 4) + ((s ^ key(lr)) * 16 + lq * 4);
    return *(const lds_f32_t *)(uintptr_t)a;
  }
};

// What the epilogue adds to or multiplies four columns of a row with
__device__ __forceinline__ f32x4_t in4(const float *src, int n, int N) {
  if (n + 4 <= N) return *(const f32x4_a4_t *)src;
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (n + t < N) v[t] = src[t];
  return v;
}

// Tile `bid` of the problem, stages in a ring of R: the same sums in the same order as f32_body, bias sums included.
// A stage is two halves; the fragments of a half are read while the matrix instructions of the half before run, and the one
// barrier of a stage sits between its halves: behind it the next stage is read and the stage R further on loaded over this one.
template <int BT, int R, int AM, int BM>
__device__ __forceinline__ void f32_direct_body(const F32P &p, int bid, char *smem) {
  typedef F32Direct<BT, AM> SA;
  typedef F32Direct<BT, BM> SB;
  constexpr int TB = BT / 32, SK = SA::SK, HS = SK / 8, L = 4;  // HS: matrix instructions deep, a half; L: a thread's loads, a stage
  constexpr unsigned kStage = SA::kBytes + SB::kBytes;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const int m0 = bid % p.tiles_m * BT, n0 = bid / p.tiles_m * BT, nk = (p.K + SK - 1) / SK;
  SA sa;
  SB sb;
  sa.start((const float *)p.A, p.lda, m0, p.M, p.K, tid);
  sb.start((const float *)p.B, p.ldb, n0, p.N, p.K, tid);
  const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_t *)smem;
  f32x4_t acc[TB][TB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  constexpr bool SUM = AM == KMAJOR && BM == KMAJOR;  // column sums of B, as in f32_body
  float tot[TB], low[TB], part[TB];
#pragma unroll
  for (int j = 0; j < TB; ++j) tot[j] = low[j] = part[j] = 0.f;
  float af[2][HS][TB], bf[2][HS][TB];
  auto load_a = [&](int buf, bool tail) { sa.load(p.K, lds0 + buf * kStage + wave * 1024, tail); };
  auto load_b = [&](int buf, bool tail) { sb.load(p.K, lds0 + buf * kStage + SA::kBytes + wave * 1024, tail); };
  auto read_step = [&](int buf, int h, int s) {
#pragma unroll
    for (int j = 0; j < TB; ++j) bf[h][s][j] = SB::frag(lds0 + buf * kStage + SA::kBytes, wn * TB + j, h * HS + s, lane);
#pragma unroll
    for (int i = 0; i < TB; ++i) af[h][s][i] = SA::frag(lds0 + buf * kStage, wm * TB + i, h * HS + s, lane);
  };
  // Half h out of the registers, half h ^ 1 of the stage in buffer `next` read meanwhile (MORE), two steps behind each matrix
  // step: a read takes the LDS four cycles and four wavefronts share it, issued in one group they held up the matrix pipe
  // for 600 cycles a stage.
  auto half = [&](int h, int next, bool load, bool tail) {
#pragma unroll
    for (int s = 0; s < HS; ++s) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[h][s][j], af[h][s][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (s < HS / 2) {
        read_step(next, h ^ 1, 2 * s);
        read_step(next, h ^ 1, 2 * s + 1);
      }
      if (h == 1 && load) {
        if (s == HS / 2) load_a((next + R - 1) % R, tail);
        if (s == HS / 2 + HS / 4) load_b((next + R - 1) % R, tail);
      }
      if (SUM && s % 4 == 3)
#pragma unroll
        for (int j = 0; j < TB; ++j) part[j] += (bf[h][s - 3][j] + bf[h][s - 2][j]) + (bf[h][s - 1][j] + bf[h][s][j]);
    }
    if (SUM && h == 1)
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const float y = part[j] - low[j], t = tot[j] + y;
        low[j] = fabsf(t) < INFINITY ? (t - tot[j]) - y : 0.f;
        tot[j] = t;
        part[j] = 0.f;
      }
  };
  // the epilogue's operands, requested at the start of the last stage: this lane has row m, columns n .. n + 3 of each block
  f32x4_t ein[TB][TB], ebias[TB];
  auto fetch = [&]() {
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int n = n0 + (wn * TB + j) * 16 + lq * 4;
      ebias[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (p.bias && p.epi != EPI_NONE && p.epi != EPI_ACTBWD) ebias[j] = in4((const float *)p.bias + n, n, p.N);
#pragma unroll
      for (int i = 0; i < TB; ++i) {
        const int m = m0 + (wm * TB + i) * 16 + lr;
        ein[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (m < p.M && p.epi == EPI_BIAS_RESID) ein[i][j] = in4((const float *)p.resid + (long)m * p.ldr + n, n, p.N);
        if (m < p.M && p.epi == EPI_ACTBWD) ein[i][j] = in4((const float *)p.aux + (long)m * p.ldc + n, n, p.N);
      }
    }
  };
  // waits for every LDS read and for all of the loads on their way but those of the last `later` stages, CAP at most
  auto wait_stages = [&](int later, auto cap) {
    constexpr int CAP = decltype(cap)::value;
    if (CAP >= 3 && later >= 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * L) : "memory");
    else if (CAP >= 2 && later >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * L) : "memory");
    else if (CAP >= 1 && later >= 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(L) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  typedef std::integral_constant<int, R - 1> InFlight;
  typedef std::integral_constant<int, R - 2> InFlight2;
  auto stage = [&](int st, int buf, auto inner) {  // INNER: stage st + R exists and is not the last
    constexpr bool INNER = decltype(inner)::value;
    if (!INNER && st + 1 == nk) fetch();
    half(0, buf, false, false);
    if (INNER || st + 1 < nk) wait_stages(INNER ? R : nk - 2 - st, InFlight2());
    half(1, (buf + 1) % R, INNER || st + R < nk, !INNER);  // (behind the last stage: reads whatever is there, not used)
  };
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (i < nk) { load_a(i, true); load_b(i, true); }
  wait_stages(nk - 1, InFlight());
#pragma unroll
  for (int s = 0; s < HS; ++s) read_step(0, 0, s);
  int st = 0;
  for (; st + 2 * R < nk; st += R) {
#pragma unroll
    for (int i = 0; i < R; ++i) stage(st + i, i, std::true_type());
  }
  for (; st < nk; st += R) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (st + i < nk) stage(st + i, i, std::false_type());
  }
  if (SUM && p.colsum && m0 == 0 && wm == 0) {
    float *sums = (float *)p.colsum;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      float x = tot[j];
      x += __shfl_xor(x, 16, 64);
      x += __shfl_xor(x, 32, 64);
      const int n = n0 + (wn * TB + j) * 16 + lr;
      if (lq == 0 && n < p.N) sums[n] = p.colsum_acc ? sums[n] + x : x;
    }
  }
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    const int m = m0 + (wm * TB + i) * 16 + lr;
    if (m >= p.M) continue;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int n = n0 + (wn * TB + j) * 16 + lq * 4;
      const long o = (long)m * p.ldc + n;
      f32x4_t c = acc[i][j], c2;
      if (p.bias && p.epi != EPI_NONE && p.epi != EPI_ACTBWD)
#pragma unroll
        for (int t = 0; t < 4; ++t) c[t] += ebias[j][t];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        c2[t] = c[t];
        if (p.epi == EPI_BIAS_ACT) c2[t] = p.act == SSDT_ACT_GELU ? gelu_f(c[t]) : fmaxf(c[t], 0.f);
        else if (p.epi == EPI_BIAS_RESID) c[t] += ein[i][j][t];
        else if (p.epi == EPI_ACTBWD) c[t] *= p.act == SSDT_ACT_GELU ? gelu_grad_f(ein[i][j][t]) : (ein[i][j][t] > 0.f ? 1.f : 0.f);
      }
      float *C = (float *)p.C + o, *C2 = (float *)p.C2 + o;
      if (n + 4 <= p.N) {
        if (p.C) *(f32x4_a4_t *)C = c;
        if (p.epi == EPI_BIAS_ACT) *(f32x4_a4_t *)C2 = c2;
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (n + t < p.N) {
            if (p.C) C[t] = c[t];
            if (p.epi == EPI_BIAS_ACT) C2[t] = c2[t];
          }
      }
    }
  }
}

template <int BT, int R>
constexpr unsigned f32_direct_lds() { return R * 2 * BT * (2048 / BT) * 4; }
template <int BT, int R, int AM, int BM>
__global__ __launch_bounds__(256) void gemm_f32_direct_k(F32P p) {
  __shared__ __attribute__((aligned(1024))) char smem[f32_direct_lds<BT, R>()];
  f32_direct_body<BT, R, AM, BM>(p, blockIdx.x, smem);
}
template <int BT, int R>
__global__ __launch_bounds__(256) void gemm_f32_direct_pair_k(F32P w, F32P d, int first, int w_first) {
  __shared__ __attribute__((aligned(1024))) char smem[f32_direct_lds<BT, R>()];
  const int bid = blockIdx.x;
  const bool head = bid < first;
  if (head == (w_first != 0)) f32_direct_body<BT, R, KMAJOR, KMAJOR>(w, head ? bid : bid - first, smem);
  else f32_direct_body<BT, R, KVEC, KVEC>(d, head ? bid : bid - first, smem);
}

int g_f32_tile = 0, g_f32_ring = 0;  // test hooks: 64 or 32 pins the tile, 2 or 3 the ring of the direct kernels

static long f32_tiles(int M, int N, int bt) { return (long)((M + bt - 1) / bt) * ((N + bt - 1) / bt); }

// Whether the direct kernels take a problem: rows and columns start at 16 bytes, a row of k ends with 16 whole bytes (a
// chunk must not reach into the next row's data), and an operand is less than 2 GiB.  Everything else goes through registers.
static bool direct_fits(const Gemm &g) {
  if (g.dtype != SSDT_F32 || (uintptr_t)g.A % 16 || (uintptr_t)g.B % 16 || g.lda % 4 || g.ldb % 4) return false;
  if ((!g.transA || g.transB) && g.K % 4) return false;
  const long ea = g.transA ? (long)(g.K - 1) * g.lda + g.M : (long)(g.M - 1) * g.lda + g.K;
  const long eb = g.transB ? (long)(g.N - 1) * g.ldb + g.K : (long)(g.K - 1) * g.ldb + g.N;
  return ea < (1L << 29) && eb < (1L << 29);
}

// Through registers: tile by predicted time per k, in nanoseconds, for n tiles per compute unit: 7 each for 32 squared, 22.5 each
// and 7.5 more for 64 (512 x 2048 x 985, n = 4 or 1: 27 against 29 us; 985 x 2048 x 512, n = 8 or 2: 34 against 33;
// 4096 x 3072 x 1024, n = 48 or 12: 346 against 266).
template <typename F>
static int pick_tile(F tiles_per_unit) {
  if (g_f32_tile) return g_f32_tile;
  return 7.0 * tiles_per_unit(32) <= 7.5 + 22.5 * tiles_per_unit(64) ? 32 : 64;
}
// Direct: a launch takes z us and, for n tiles per compute unit, a + b n nanoseconds per k, never less than c n.  Measured (32
// squared with a ring of 2 and of 3, 64 with 3): 256 x 256 x 1024 11.2, 8.9, 22.4 us; 985 x 1536 x 512 19.0, 20.1, 22.0;
// 985 x 2048 x 512 26.5, 28.0, 25.3; 4096 x 3072 x 1024 221, 229, 205.  `tail` k of a shorter tile run beside nothing at the end.
struct F32Cfg { int bt, ring; double a, b, c, z; };
static const F32Cfg kF32[] = {{32, 2, 4.0, 3.4, 4.75, 3.3}, {32, 3, 1.0, 4.5, 5.1, 3.3}, {64, 3, 0.0, 17.3, 16.2, 4.6}};
template <typename F>
static const F32Cfg &pick_direct(F tiles_per_unit, double k, double tail) {
  const F32Cfg *best = nullptr;
  double least = 0;
  for (const F32Cfg &c : kF32) {
    if ((g_f32_tile && c.bt != g_f32_tile) || (g_f32_ring && c.ring != g_f32_ring)) continue;
    const double n = tiles_per_unit(c.bt), t = c.z + 1e-3 * (k * std::max(c.a + c.b * n, c.c * n) + tail * (c.a + c.b));
    if (!best || t < least) { best = &c; least = t; }
  }
  return best ? *best : kF32[1];
}

template <int BT, int R>
static void launch_direct(const Gemm &g, F32P p, hipStream_t s) {
  p.tiles_m = (p.M + BT - 1) / BT;
  const dim3 grid((unsigned)((long)p.tiles_m * ((p.N + BT - 1) / BT)));
  if (g.transA) hipLaunchKernelGGL((gemm_f32_direct_k<BT, R, KMAJOR, KMAJOR>), grid, dim3(256), 0, s, p);
  else if (!g.transB) hipLaunchKernelGGL((gemm_f32_direct_k<BT, R, KVEC, KMAJOR>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_direct_k<BT, R, KVEC, KVEC>), grid, dim3(256), 0, s, p);
}
template <int BT>
static void launch_f32(const Gemm &g, F32P p, hipStream_t s) {
  p.tiles_m = (p.M + BT - 1) / BT;
  const dim3 grid((unsigned)((long)p.tiles_m * ((p.N + BT - 1) / BT)));
  if (g.dtype == SSDT_BF16) {
    const bool vec = g.K % 8 == 0 && g.lda % 2 == 0 && (uintptr_t)g.A % 4 == 0;
    if (vec) hipLaunchKernelGGL((gemm_f32_k<BT, KVEC, KMAJOR, bf16>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((gemm_f32_k<BT, KSCALAR, KMAJOR, bf16>), grid, dim3(256), 0, s, p);
    return;
  }
  const bool vec = g.K % 4 == 0;
  if (g.transA) hipLaunchKernelGGL((gemm_f32_k<BT, KMAJOR, KMAJOR, float>), grid, dim3(256), 0, s, p);
  else if (!g.transB && vec) hipLaunchKernelGGL((gemm_f32_k<BT, KVEC, KMAJOR, float>), grid, dim3(256), 0, s, p);
  else if (!g.transB) hipLaunchKernelGGL((gemm_f32_k<BT, KSCALAR, KMAJOR, float>), grid, dim3(256), 0, s, p);
  else if (vec) hipLaunchKernelGGL((gemm_f32_k<BT, KVEC, KVEC, float>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_k<BT, KSCALAR, KSCALAR, float>), grid, dim3(256), 0, s, p);
}

static hipError_t prepare(const Gemm &g, F32P *p) {
  if ((g.dtype == SSDT_BF16 && (g.transA || g.transB)) || (g.transA && g.transB) || (g.colsum && (!g.transA || g.transB))) return hipErrorNotSupported;
  // (a tile's rows are addressed with 32-bit byte offsets, and a row ends inside its own leading dimension)
  if (g.lda >= (1L << 21) || g.ldb >= (1L << 21) || g.lda < (g.transA ? g.M : g.K) || g.ldb < (g.transB ? g.K : g.N)) return hipErrorNotSupported;
  *p = F32P{g.M, g.N, g.K, g.A, g.B, g.C, g.C2, g.bias, g.resid, g.aux, g.lda, g.ldb, g.ldc, g.ldr, g.epi, g.act, 0,
            (float *)g.colsum, g.colsum_accumulate ? 1 : 0};
  return hipSuccess;
}

hipError_t gemm_f32(const Gemm &g, hipStream_t s) {
  F32P p;
  hipError_t e = prepare(g, &p);
  if (e != hipSuccess) return e;
  prof::Scope ps(prof::GEMM_F32, 2.0 * g.M * g.N * g.K, 0, s);
  const auto per_unit = [&](int bt) { return (double)((f32_tiles(g.M, g.N, bt) + 255) / 256); };
  if (direct_fits(g)) {
    const F32Cfg &c = pick_direct(per_unit, g.K, 0);
    if (c.bt == 64) launch_direct<64, 3>(g, p, s);
    else if (c.ring == 3) launch_direct<32, 3>(g, p, s);
    else launch_direct<32, 2>(g, p, s);
    return hipGetLastError();
  }
  switch (pick_tile(per_unit)) {
    case 64: launch_f32<64>(g, p, s); break;
    default: launch_f32<32>(g, p, s);
  }
  return hipGetLastError();
}

// R: the direct kernels with a ring of R, 0: through registers
template <int BT, int R>
static void launch_f32_pair(F32P w, F32P d, hipStream_t s) {
  w.tiles_m = (w.M + BT - 1) / BT;
  d.tiles_m = (d.M + BT - 1) / BT;
  const unsigned nw = (unsigned)f32_tiles(w.M, w.N, BT), nd = (unsigned)f32_tiles(d.M, d.N, BT);
  const int w_first = w.K >= d.K, first = (int)(w_first ? nw : nd);
  const dim3 grid(nw + nd);
  if constexpr (R > 0) hipLaunchKernelGGL((gemm_f32_direct_pair_k<BT, R>), grid, dim3(256), 0, s, w, d, first, w_first);
  else if (d.K % 4 == 0) hipLaunchKernelGGL((gemm_f32_pair_k<BT, KVEC>), grid, dim3(256), 0, s, w, d, first, w_first);
  else hipLaunchKernelGGL((gemm_f32_pair_k<BT, KSCALAR>), grid, dim3(256), 0, s, w, d, first, w_first);
}

hipError_t gemm_pair_f32(const Gemm &w, const Gemm &d, hipStream_t s) {
  F32P pw, pd;
  if (w.dtype != SSDT_F32 || !w.transA || w.transB || d.transA || !d.transB) return hipErrorNotSupported;
  hipError_t e = prepare(w, &pw);
  if (e == hipSuccess) e = prepare(d, &pd);
  if (e != hipSuccess) return e;
  prof::Scope ps(prof::GEMM_F32, 2.0 * w.M * w.N * w.K + 2.0 * d.M * d.N * d.K, 0, s);
  const double longest = std::max(w.K, d.K);
  const auto per_unit = [&](int t) {
    return std::max(1.0, ((double)f32_tiles(w.M, w.N, t) * w.K + (double)f32_tiles(d.M, d.N, t) * d.K) / longest / 256.0);
  };
  if (direct_fits(w) && direct_fits(d)) {
    const F32Cfg &c = pick_direct(per_unit, longest, 0.7 * std::min(w.K, d.K));
    if (c.bt == 64) launch_f32_pair<64, 3>(pw, pd, s);
    else if (c.ring == 3) launch_f32_pair<32, 3>(pw, pd, s);
    else launch_f32_pair<32, 2>(pw, pd, s);
  } else if (pick_tile(per_unit) == 64) launch_f32_pair<64, 0>(pw, pd, s);
  else launch_f32_pair<32, 0>(pw, pd, s);
  return hipGetLastError();
}

}  // namespace k
}  // namespace ssdt
