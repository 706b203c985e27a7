// bf16 GEMM on the CDNA4 matrix cores, fp32 accumulation, for every problem that gemm_nt256_k / gemm_km256_k
// (256 x 256 tiles, at least one per compute unit, whole stages) do not take: fewer tiles, any number of rows or
// tokens, any width that is a multiple of 8.
//
// What bounds such a problem is how many compute units have a tile and how many wavefronts share one, not the matrix
// pipe, so the tile comes in three sizes, the contraction can be split over workgroups, and the
// two products of a linear's backward can share a launch (see DISPATCH).  Where a compute unit has one or two tiles, a
// stage is shorter than the trip to memory that fills it: there the stages stand in a ring of three or four instead of two
// buffers (128 x 1280 x 5120 42 -> 23 us, 1024 x 2048 x 2048 24 -> 17, both products of 256 x 256 -> 1024's backward 12.4 -> 8.9).
// Operands are read as they are stored, K-contiguous or k-major, as in gemm_km256_k: a stage of 64 k goes to LDS by
// direct global-to-LDS loads, k-major fragments are fetched with the transposing LDS read.  The loads are buffer
// loads whose descriptor ends where the operand ends: what lies beyond the last row arrives as zero, so ragged
// extents need no second code path and no masks, except the tail of a K-contiguous row (see the loader).
//
// For the smallest problems the four wavefronts of a workgroup stand side by side along k instead (kwave_body).
//
// Against the form this replaces (128 x 128 tiles, register-staged, operands brought to the K-contiguous form by
// transposed copies): 4096 x 2048 x 8192 211 -> 137 us, 1024 x 2048 x 2048 45 -> 17, 1024 x 1024 x 8192 150 -> 33.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "dev.h"
#include "kernels.h"
#include "mfma_common.h"
#include "prof.h"

namespace ssdt {
namespace k {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) v4i_t lds_v4i_t;
typedef __attribute__((address_space(3))) char lds_char_t;

struct TileP {
  int M, N, K;
  const uint16_t *A, *B;
  long lda, ldb, ldc, ldr;
  uint16_t *C, *C2;
  const uint16_t *bias, *resid, *aux;
  int act, epi, tiles_m, tiles_n, gm;
  int splits, stages_per_split;  // the contraction in `splits` parts of that many stages; 1 = whole
  float *part;                   // splits > 1: fp32 partial products [splits][M][N], then column sums [splits][N]
  uint16_t *colsum;              // as in NtP: sum over k of B(k, n)
  int colsum_acc;
};

#define SSDT_FENCE __builtin_amdgcn_sched_barrier(0)

constexpr int kSK = 64;  // k per stage (SK below: 64, or 128 where the wavefronts share a stage's k)

// One operand's side of the loader and of the fragment reads.  ROWS: the tile's extent in this operand's own
// dimension; KM: stored k-major.
//   K-contiguous: a stage is ROWS rows of 128 bytes, 16-byte chunk c of row r at slot c ^ ((r >> 1) & 7);
//   k-major: 64 k-rows of 2 ROWS bytes, 32-byte unit u of k-row k at u ^ key(k), key = (k & 3) | ((k >> 3) & 1) << 2 for
//   rows of 256 bytes and more; with rows of 128 bytes the row's parity already picks the half of the 64 banks and the key
//   is ((k >> 1) & 1) | ((k >> 3) & 1) << 1.  Either way the eight k-rows {0..3, 8..11} that 32 lanes of a transposing read
//   touch at one unit lie in eight different groups of eight banks.
//   A stage of 128 k: K-contiguous rows have 256 bytes, chunk c of row r at c ^ (r & 15); k-major rows of 64 bytes, four of
//   which make up the 64 banks, have key (k >> 3) & 1.
//   BIG: an operand of 2^34 elements and more, whose end is kept in 64 bits.
template <int ROWS, bool KM, int NT, int SK, bool BIG = false>
struct Side {
  typedef typename std::conditional<BIG, long, int>::type Ext;
  static constexpr int LJ = ROWS * SK / 8 / NT, CPR = (KM ? ROWS : SK) / 8;
  static constexpr unsigned kBytes = ROWS * SK * 2;
  static __device__ __forceinline__ int key(int i) {
    if (!KM) return SK == 128 ? i & 15 : (i >> 1) & 7;
    return ROWS >= 128 ? ((i & 3) | (((i >> 3) & 1) << 2)) : ROWS >= 64 ? (((i >> 1) & 1) | (((i >> 3) & 1) << 1)) : ((i >> 3) & 1);
  }
  unsigned voff[LJ];
  int chunk;  // K-contiguous: this thread's 8-wide chunk of the stage (the same for every j: NT / CPR is a multiple of 16)
  __device__ __forceinline__ void init(int tid, long ld) {
#pragma unroll
    for (int j = 0; j < LJ; ++j) {
      const int q = j * NT + tid, row = q / CPR, pos = q % CPR;
      chunk = KM ? (((pos >> 1) ^ key(row)) << 1) | (pos & 1) : pos ^ key(row);
      voff[j] = (unsigned)(row * (int)ld + chunk * 8) * 2u;
    }
  }
  // Where the next stage starts, units of 16 bytes from there to the end of the operand (everything is a whole number of them;
  // prepare() sees whether 31 bits hold it) and from stage to stage, the k it starts at.  (Scalar instructions count: a small
  // problem is one wavefront per SIMD, bound by what it issues.  With 64-bit extents a stage took 30 to 50 ns longer.)
  uint64_t at;
  Ext left;
  int step, k;
  // `ext` = the operand's extent in its own dimension, r0 / k0 = the tile's origin
  __device__ __forceinline__ void start(const uint16_t *base, long ld, int r0, int ext, int k0, int K) {
    at = (uint64_t)(uintptr_t)(KM ? base + (long)k0 * ld + r0 : base + (long)r0 * ld + k0);
    left = (Ext)((KM ? (long)(K - 1 - k0) * ld + ext - r0 : (long)(ext - 1 - r0) * ld + K - k0) / 8);
    step = KM ? SK / 8 * (int)ld : SK / 8;
    k = k0;
  }
  // The next stage piece by piece: its descriptor, piece j (tail: the stage may be the last one), and on to the stage behind it.
  __device__ __forceinline__ v4i_t desc() {
    asm volatile("" : "+s"(at), "+s"(left));  // (addresses computed ahead would fill the scalar registers)
    v4i_t rsrc;
    rsrc[0] = (int)(unsigned)at;
    rsrc[1] = (int)(unsigned)(at >> 32) & 0xffff;
    const Ext rest = left & ~(left >> (8 * sizeof(Ext) - 1));
    rsrc[2] = (rest >> 27) ? 0x7fffffff : (int)rest << 4;  // (2^31 is out of range)
    rsrc[3] = 0x00020000;
    // a scalar register written by a vector instruction (readfirstlane) needs five wait states before a vector memory
    // instruction reads it; the compiler does not look into the loads' assembly for that
    asm volatile("s_nop 4" : "+s"(rsrc));
    return rsrc;
  }
  // (Two wait states: in a kernel that spills no scalar registers nothing writes the descriptor between desc() and here.  With five
  // each, rings of four took 1.6 % longer.)
  __device__ __forceinline__ void piece(const v4i_t &rsrc, int j, int K, unsigned dst, bool tail) {
    // the tail of a K-contiguous row continues in the next row: such chunks are sent out of range
    const bool dead = !KM && tail && k + chunk * 8 >= K;
    load_lds16(rsrc, dead ? 0x80000000u : voff[j], dst + j * NT * 16);
  }
  __device__ __forceinline__ void next() {
    at += 16l * step;
    left -= step;
    k += SK;
  }
  __device__ __forceinline__ void load(int K, unsigned lds, int wave, bool tail) {
    unsigned dst = __builtin_amdgcn_readfirstlane(lds + wave * 1024);
    asm volatile("" : "+s"(dst));
    const v4i_t rsrc = desc();
#pragma unroll
    for (int j = 0; j < LJ; ++j) piece(rsrc, j, K, dst, tail);
    next();
  }
  // The same fragments from a lane's base of a step (k-major, a row of 256 bytes and more: the block is XOR-ed into it): one address
  // register instead of one for each block.
  static __device__ __forceinline__ unsigned base(int step, int lane) {
    const int lr = lane & 15, lq = lane >> 4;
    if (KM) return (unsigned)((step * 32 + 8 * lq + (lr >> 2)) * (ROWS * 2) + key(8 * lq + (lr >> 2)) * 32 + 8 * (lr & 3));
    return (unsigned)(lr * (SK * 2) + ((4 * step + lq) ^ key(lr)) * 16);
  }
  static __device__ __forceinline__ bf16x8_t frag_from(unsigned base, unsigned lds, int blk) {
    static_assert(!KM || ROWS >= 128, "a block's 32 bytes must be bits of their own");
    if (KM) {
      const lds_char_t *at = (const lds_char_t *)(uintptr_t)((base ^ (unsigned)(blk * 32)) + lds);
      union { struct { s16x4_t a, b; } s; bf16x8_t v; } u;
      u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)at);
      u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(at + 4 * ROWS * 2));
      return u.v;
    }
    union { v4i_t a; bf16x8_t v; } u;
    u.a = *(const lds_v4i_t *)(uintptr_t)(base + lds + (unsigned)(blk * 16 * SK * 2));
    return u.v;
  }
  // fragment of the 16-row block `blk`, 32-wide step `step`: 8 consecutive k of row (lane & 15) per lane
  static __device__ __forceinline__ bf16x8_t frag(unsigned lds, int blk, int step, int lane) {
    const int lr = lane & 15, lq = lane >> 4;
    if (KM) {
      const int kr = step * 32 + 8 * lq + (lr >> 2);
      const unsigned a = lds + kr * (ROWS * 2) + (unsigned)((blk ^ key(8 * lq + (lr >> 2))) * 32 + 8 * (lr & 3));
      const lds_char_t *at = (const lds_char_t *)(uintptr_t)a;
      union { struct { s16x4_t a, b; } s; bf16x8_t v; } u;
      u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)at);
      u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(at + 4 * ROWS * 2));
      return u.v;
    }
    const unsigned a = lds + (blk * 16 + lr) * (SK * 2) + (((4 * step + lq) ^ key(lr)) * 16);
    union { v4i_t a; bf16x8_t v; } u;
    u.a = *(const lds_v4i_t *)(uintptr_t)a;
    return u.v;
  }
};

// eight bf16 of a row whose address is a multiple of 8 (the tensors of the epilogue need no more)
typedef unsigned int u32x4_a8_t __attribute__((ext_vector_type(4), aligned(8)));
__device__ __forceinline__ void load8(const uint16_t *src, float *f) {
  const u32x4_a8_t q = *(const u32x4_a8_t *)src;
  unpack8f(make_uint4(q.x, q.y, q.z, q.w), f);
}
__device__ __forceinline__ void store8(uint16_t *dst, const float *v) {
  const u32x4_a8_t q = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
  __builtin_nontemporal_store(q, (u32x4_a8_t *)dst);
}

// the residual or activation input of 8 consecutive columns of one row, as stored (zeros where the epilogue has none)
__device__ __forceinline__ u32x4_a8_t epilogue_in8(const TileP &p, int m, int n) {
  if (p.epi == EPI_BIAS_RESID) return *(const u32x4_a8_t *)(p.resid + (long)m * p.ldr + n);
  if (p.epi == EPI_ACTBWD) return *(const u32x4_a8_t *)(p.aux + (long)m * p.ldc + n);
  return u32x4_a8_t{0, 0, 0, 0};
}
__device__ __forceinline__ u32x4_a8_t bias8(const TileP &p, int n) {
  if (p.epi != EPI_NONE && p.epi != EPI_ACTBWD && p.bias) return *(const u32x4_a8_t *)(p.bias + n);
  return u32x4_a8_t{0, 0, 0, 0};
}
// the epilogue on 8 consecutive columns of one row, given the two above
__device__ __forceinline__ void tile_epilogue8(const TileP &p, float *v, int m, int n, u32x4_a8_t bias, u32x4_a8_t in) {
  const long o = (long)m * p.ldc + n;
  if (p.epi != EPI_NONE && p.epi != EPI_ACTBWD && p.bias) {
    float b[8];
    unpack8f(make_uint4(bias.x, bias.y, bias.z, bias.w), b);
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] += b[t];
  }
  if (p.epi == EPI_BIAS_ACT) {
    if (p.C) store8(p.C + o, v);
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = p.act == SSDT_ACT_GELU ? gelu_f(v[t]) : fmaxf(v[t], 0.f);
    store8(p.C2 + o, v);
    return;
  }
  if (p.epi == EPI_BIAS_RESID) {
    float r[8];
    unpack8f(make_uint4(in.x, in.y, in.z, in.w), r);
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] += r[t];
  } else if (p.epi == EPI_ACTBWD) {
    float u[8];
    unpack8f(make_uint4(in.x, in.y, in.z, in.w), u);
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] *= p.act == SSDT_ACT_GELU ? gelu_grad_f(u[t]) : (u[t] > 0.f ? 1.f : 0.f);
  }
  store8(p.C + o, v);
}

// Waits for every LDS read and for all of the loads on their way but those of the last `later` stages (of L loads a thread; CAP
// stages at most), then for the other wavefronts.
template <int L, typename Cap>
__device__ __forceinline__ void wait_stages(int later, Cap) {
  constexpr int CAP = Cap::value;
  if (CAP >= 3 && later >= 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * L) : "memory");
  else if (CAP >= 2 && later >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * L) : "memory");
  else if (CAP >= 1 && later >= 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(L) : "memory");
  else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// four column sums, or partial sums of a split
__device__ __forceinline__ void store_colsum(const TileP &p, int n, int split, float (&v)[4]) {
  if (p.splits > 1) {
    *(float4 *)(p.part + (long)p.splits * p.M * p.N + (long)split * p.N + n) = make_float4(v[0], v[1], v[2], v[3]);
    return;
  }
  if (p.colsum_acc) {
    float old[4];
    unpack4(*(const uint2 *)(p.colsum + n), old);
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] += old[t];
  }
  *(uint2 *)(p.colsum + n) = pack4(v);
}

// Wavefronts that share a tile, in two rows.  A ring of three or more has one or two workgroups on a compute unit: four wavefronts, one to
// a SIMD, leave nothing to cover their waits for fragments and barriers, and the epilogue is theirs alone.  Eight: 128 x 128, ring of 4, 2331 x
// 1024 x 4096 37.7 -> 31.1 us; 64 x 128, ring of 3, 1024 x 2048 x 5120 30.3 -> 29.3, 1024 x 5120 x 2048 with GELU 37.6 -> 34.5, 1024 x 2048 x 2048
// 15.0 -> 14.4.  Among a layer's other products it saves 20 % of a product's time at 0.6 PFLOP/s by 128 x 128 (1330 of them), 9 % by 64 x 128 (2700).
// (Wavefronts that do nothing but load, one, two or four of them: no faster.)
constexpr int waves_of(int BM, int BN, int R) { return R >= 3 && BN == 128 ? 8 : 4; }
constexpr int threads_of(bool KW, int NW) { return KW ? 256 : 64 * NW; }

// One tile: workgroup `bid` of the problem's tiles_m * tiles_n * splits (tiles of a split after each other).
// R: stages in the ring.  These kernels differ in nothing but tile, ring and speed: every output is the same sum in the same order.
template <int BM, int BN, int R, bool AKM, bool BKM, bool BIG = false, int NW = waves_of(BM, BN, R)>
__device__ __forceinline__ void tile_body(const TileP &p, int bid, uint16_t *smem) {
  constexpr int NT = 64 * NW, WGN = NW / 2, WTM = BM / 2, WTN = BN / WGN, TM = WTM / 16, TN = WTN / 16;
  typedef Side<BM, AKM, NT, kSK, BIG> SA;
  typedef Side<BN, BKM, NT, kSK, BIG> SB;
  constexpr unsigned kStage = SA::kBytes + SB::kBytes;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
  const int tiles = p.tiles_m * p.tiles_n, split = bid / tiles;
  NtP q;  // tile_of looks at these only
  q.tiles_m = p.tiles_m; q.tiles_n = p.tiles_n; q.gm = p.gm;
  int tile_m, tile_n;
  tile_of(q, bid - split * tiles, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk_all = (p.K + kSK - 1) / kSK, s0 = split * p.stages_per_split, nk = min(nk_all - s0, p.stages_per_split);
  SA sa;
  SB sb;
  sa.init(tid, p.lda);
  sb.init(tid, p.ldb);
  const unsigned lds0 = (unsigned)(uintptr_t)smem;
  f32x4_t acc[TM][TN], accs[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < TN; ++j) accs[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // column sums of B (bias gradient of a weight-gradient product): a block of ones multiplied in by the wavefronts of
  // the first tile row that hold distinct fragments, as in gemm_km256_k
  const bool sum = AKM && BKM && p.colsum && tile_m == 0 && wm == 0;
  union { unsigned w[4]; bf16x8_t v; } ones;
  ones.w[0] = ones.w[1] = ones.w[2] = ones.w[3] = 0x3F803F80u;

  // A stage is two 32-wide steps.  The fragments of a step are read while the MFMAs of the step before run; the reads
  // of a stage's second step are the last of that stage, so its one barrier sits between the two steps: behind it the
  // next stage is read and the stage R further on is loaded over this one.  (Both steps of the next stage read behind the
  // barrier, into a second set of registers: 10 % slower.)
  // DEALT: eight wavefronts' reads and loads stand one by one between the matrix instructions, the loads spread over both steps; in front of
  // them, as the compiler has it, they keep the tile waiting.  Four wavefronts are better off in the compiler's order: 64-row tiles by 2 to
  // 6 %, 128 x 128 in a ring of two by 1 to 2 % of its time among a layer's other products, 10 % and more with up to 24 stages (3500 products of 1170 layers; by
  // themselves some are 10 % faster with everything dealt out, 1024 x 6144 x 2048 32.4 -> 29.6 us, and make their layer slower all the same).
  constexpr bool DEALT = NW == 8;
  sa.start(p.A, p.lda, m0, p.M, s0 * kSK, p.K);
  sb.start(p.B, p.ldb, n0, p.N, s0 * kSK, p.K);
  bf16x8_t af[2][TM], bf[2][TN];
  auto load_stage = [&](int buf, bool tail) {
    sa.load(p.K, lds0 + buf * kStage, wave, tail);
    sb.load(p.K, lds0 + buf * kStage + SA::kBytes, wave, tail);
  };
  // fragment r of a step, in the order in which the matrix instructions want them
  auto read_one = [&](int buf, int step, int r) {
    if (r == 1) af[step][0] = SA::frag(lds0 + buf * kStage, wm * TM, step, lane);
    else if (r <= TN) bf[step][r ? r - 1 : 0] = SB::frag(lds0 + buf * kStage + SA::kBytes, wn * TN + (r ? r - 1 : 0), step, lane);
    else af[step][r - TN] = SA::frag(lds0 + buf * kStage, wm * TM + r - TN, step, lane);
  };
  auto read_step = [&](int buf, int step) {
#pragma unroll
    for (int r = 0; r < TM + TN; ++r) read_one(buf, step, r);
  };
  auto add_sums = [&](int step) {
    if (AKM && BKM && sum) {
#pragma unroll
      for (int j = 0; j < TN; ++j) accs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[step][j], ones.v, accs[j], 0, 0, 0);
    }
  };
  auto mfma_step = [&](int step) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[step][j], af[step][i], acc[i][j], 0, 0, 0);
    add_sums(step);
  };
  constexpr int L = SA::LJ + SB::LJ;  // a thread's loads per stage
  // What the epilogue reads is requested at the start of the last stage, when no load of a stage is on its way any more: read
  // row by row between the stores, every pass was a round trip to memory (4096 x 2048 x 2048 with a residual 50 -> 44 us).
  constexpr int LPR = WTN / 8, RPP = 64 / LPR, PASSES = 32 / RPP;
  const int c8 = (lane % LPR) * 8, n = n0 + wn * WTN + c8;
  u32x4_a8_t ein[TM / 2][PASSES], ebias = {0, 0, 0, 0};
  auto fetch = [&]() {
    if (n < p.N && p.splits == 1) ebias = bias8(p, n);
#pragma unroll
    for (int I = 0; I < TM / 2; ++I)
#pragma unroll
      for (int pass = 0; pass < PASSES; ++pass) {
        const int m = m0 + wm * WTM + I * 32 + pass * RPP + lane / LPR;
        ein[I][pass] = u32x4_a8_t{0, 0, 0, 0};
        if (m < p.M && n < p.N && p.splits == 1) ein[I][pass] = epilogue_in8(p, m, n);
      }
  };
  typedef std::integral_constant<int, R - 1> InFlight;
  typedef std::integral_constant<int, R - 2> InFlight2;
  // The matrix instructions of a step, between them the reads of step `rstep` of buffer `rbuf` and pieces [l0, l1) of the next
  // stage to load, which goes to buffer `lbuf`.
  v4i_t ra, rb;
  auto load_one = [&](int q, int lbuf, bool tail) {
    const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + lbuf * kStage + wave * 1024);
    if (q == 0) ra = sa.desc();
    if (q < SA::LJ) sa.piece(ra, q, p.K, dst, tail);
    if (q == SA::LJ - 1) sa.next();
    if (q == SA::LJ) rb = sb.desc();
    if (q >= SA::LJ) sb.piece(rb, q - SA::LJ, p.K, dst + SA::kBytes, tail);
    if (q == L - 1) sb.next();
  };
  auto phase = [&](int step, bool read, int rbuf, int rstep, bool load, int lbuf, bool tail, auto first, auto last) {
    constexpr int N = TM * TN, L0 = decltype(first)::value, L1 = decltype(last)::value;
#pragma unroll
    for (int t = 0; t < N; ++t) {
      SSDT_FENCE;
      acc[t / TN][t % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[step][t % TN], af[step][t / TN], acc[t / TN][t % TN], 0, 0, 0);
      SSDT_FENCE;
      if (read) {
#pragma unroll
        for (int r = t; r < TM + TN; r += N) read_one(rbuf, rstep, r);
      }
      if (load) {
#pragma unroll
        for (int q = L0; q < L1; ++q)
          if ((q - L0) * N / (L1 - L0) == t) load_one(q, lbuf, tail);
      }
    }
    add_sums(step);
    SSDT_FENCE;
  };
  typedef std::integral_constant<int, 0> None;
  typedef std::integral_constant<int, R == 2 ? L : (L + 1) / 2> Some;
  typedef std::integral_constant<int, L> All;
  // INNER: stage st + R exists and is not the last
  auto stage = [&](int st, int buf, auto inner) {
    constexpr bool INNER = decltype(inner)::value;
    const bool more = INNER || st + 1 < nk, load = INNER || st + R < nk;
    if (!INNER && st + 1 == nk) fetch();
    if (DEALT) {
      phase(0, true, buf, 1, st > 0 && (INNER || st - 1 + R < nk), (buf + R - 1) % R, !INNER, Some(), All());
      if (more) wait_stages<L>(INNER ? R : nk - 2 - st, InFlight2());
      phase(1, more, (buf + 1) % R, 0, load, buf, !INNER, None(), Some());
      return;
    }
    read_step(buf, 1);
    mfma_step(0);
    if (more) {
      wait_stages<L>(INNER ? R : nk - 2 - st, InFlight2());
      if (load) load_stage(buf, !INNER);
      read_step((buf + 1) % R, 0);
    }
    mfma_step(1);
  };
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (i < nk) load_stage(i, true);
  wait_stages<L>(nk - 1, InFlight());
  read_step(0, 0);
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
  const int lr = lane & 15, lq = lane >> 4;
  if (AKM && BKM && sum && lr == 0) {  // this lane: columns j*16 + lq*4 + 0..3
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WTN + j * 16 + lq * 4;
      if (n >= p.N) continue;
      float v[4] = {accs[j][0], accs[j][1], accs[j][2], accs[j][3]};
      store_colsum(p, n, split, v);
    }
  }
  // epilogue through LDS, 32 rows of the wavefront's part at a time: lane l of block (i, j) holds row i*16 + (l & 15),
  // columns j*16 + (l >> 4)*4 + 0..3; read back row by row so that an access is 16 bytes and rows are contiguous
  __syncthreads();
  constexpr int LD = WTN + 4;
  float *stg = (float *)smem + wave * (32 * LD);
#pragma unroll
  for (int I = 0; I < TM / 2; ++I) {
#pragma unroll
    for (int il = 0; il < 2; ++il)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4_t a = acc[I * 2 + il][j];
        *(float4 *)(stg + (il * 16 + lr) * LD + j * 16 + lq * 4) = make_float4(a[0], a[1], a[2], a[3]);
      }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int row = pass * RPP + lane / LPR, m = m0 + wm * WTM + I * 32 + row;
      const float4 lo = *(const float4 *)(stg + row * LD + c8), hi = *(const float4 *)(stg + row * LD + c8 + 4);
      if (m >= p.M || n >= p.N) continue;
      if (p.splits > 1) {
        float *o = p.part + ((long)split * p.M + m) * p.N + n;
        *(float4 *)o = lo;
        *(float4 *)(o + 4) = hi;
      } else {
        float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        tile_epilogue8(p, v, m, n, ebias, ein[I][pass]);
      }
    }
  }
}

// The same with the wavefronts side by side along k: a stage is 128 k, wavefront w takes its 32-wide step w on the whole tile,
// and the four partial tiles are added through LDS at the end, in the order of the wavefronts (another order of additions than
// tile_body's: not where that one is to be kept, see Gemm::one_order).
template <int BM, int BN, int R, bool AKM, bool BKM>
__device__ __forceinline__ void kwave_body(const TileP &p, int bid, uint16_t *smem) {
  constexpr int NT = 256, SK = 128, TM = BM / 16, TN = BN / 16;
  typedef Side<BM, AKM, NT, SK> SA;
  typedef Side<BN, BKM, NT, SK> SB;
  constexpr unsigned kStage = SA::kBytes + SB::kBytes;
  constexpr int L = SA::LJ + SB::LJ;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = p.tiles_m * p.tiles_n, split = bid / tiles;
  NtP q;  // tile_of looks at these only
  q.tiles_m = p.tiles_m; q.tiles_n = p.tiles_n; q.gm = p.gm;
  int tile_m, tile_n;
  tile_of(q, bid - split * tiles, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nk_all = (p.K + SK - 1) / SK, s0 = split * p.stages_per_split, nk = min(nk_all - s0, p.stages_per_split);
  SA sa;
  SB sb;
  sa.init(tid, p.lda);
  sb.init(tid, p.ldb);
  sa.start(p.A, p.lda, m0, p.M, s0 * SK, p.K);
  sb.start(p.B, p.ldb, n0, p.N, s0 * SK, p.K);
  const unsigned lds0 = (unsigned)(uintptr_t)smem;
  f32x4_t acc[TM][TN], accs[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    accs[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  const bool sum = AKM && BKM && p.colsum && tile_m == 0;  // column sums of B, as in tile_body
  union { unsigned w[4]; bf16x8_t v; } ones;
  ones.w[0] = ones.w[1] = ones.w[2] = ones.w[3] = 0x3F803F80u;
  bf16x8_t af[2][TM], bf[2][TN];
  auto load_stage = [&](int buf, bool tail) {
    sa.load(p.K, lds0 + buf * kStage, wave, tail);
    sb.load(p.K, lds0 + buf * kStage + SA::kBytes, wave, tail);
  };
  auto read_stage = [&](int buf, int set) {
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[set][j] = SB::frag(lds0 + buf * kStage + SA::kBytes, j, wave, lane);
#pragma unroll
    for (int i = 0; i < TM; ++i) af[set][i] = SA::frag(lds0 + buf * kStage, i, wave, lane);
  };
  auto mfma_stage = [&](int set) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[set][j], af[set][i], acc[i][j], 0, 0, 0);
    if (AKM && BKM && sum) {
#pragma unroll
      for (int j = 0; j < TN; ++j) accs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[set][j], ones.v, accs[j], 0, 0, 0);
    }
  };
  // the epilogue's rows: thread t has 8 columns of rows t / (BN / 8) + it * RPP
  constexpr int CPT = BN / 8, RPP = NT / CPT, PASSES = (BM + RPP - 1) / RPP;
  const int c8 = (tid % CPT) * 8, n = n0 + c8, r0 = tid / CPT;
  u32x4_a8_t ein[PASSES], ebias = {0, 0, 0, 0};
  auto fetch = [&]() {
    if (n < p.N && p.splits == 1) ebias = bias8(p, n);
#pragma unroll
    for (int it = 0; it < PASSES; ++it) {
      const int row = r0 + it * RPP, m = m0 + row;
      ein[it] = u32x4_a8_t{0, 0, 0, 0};
      if (row < BM && m < p.M && n < p.N && p.splits == 1) ein[it] = epilogue_in8(p, m, n);
    }
  };
  typedef std::integral_constant<int, R - 1> InFlight;
  typedef std::integral_constant<int, R - 2> InFlight2;
  // Interval st: stage st is in the registers (set st & 1), the next one is read while its matrix instructions run, and behind
  // the barrier, where everyone has read stage st, the one R further on is loaded over it.  INNER as in tile_body.
  auto interval = [&](int st, int buf, int set, auto inner) {
    constexpr bool INNER = decltype(inner)::value;
    if (INNER || st + 1 < nk) {
      wait_stages<L>(INNER ? R : nk - 2 - st, InFlight2());
      read_stage((buf + 1) % R, set ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      if (INNER || st + R < nk) load_stage(buf, !INNER);
    } else {
      fetch();
    }
    mfma_stage(set);
  };
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (i < nk) load_stage(i, true);
  wait_stages<L>(nk - 1, InFlight());
  read_stage(0, 0);
  constexpr int U = R % 2 ? 2 * R : R;
  int st = 0;
  for (; st + U + R < nk; st += U) {
#pragma unroll
    for (int i = 0; i < U; ++i) interval(st + i, i % R, i & 1, std::true_type());
  }
  for (; st < nk; st += U) {
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (st + i < nk) interval(st + i, i % R, i & 1, std::false_type());
  }
  // partial tiles [wavefront][row][BN + 4], partial sums [wavefront][BN] behind them
  constexpr int LD = BN + 4;
  float *parts = (float *)smem, *psum = parts + 4 * BM * LD;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *(float4 *)(parts + (wave * BM + i * 16 + lr) * LD + j * 16 + lq * 4) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
  if (AKM && BKM && sum && lr == 0)
#pragma unroll
    for (int j = 0; j < TN; ++j) *(float4 *)(psum + wave * BN + j * 16 + lq * 4) = make_float4(accs[j][0], accs[j][1], accs[j][2], accs[j][3]);
  __syncthreads();
  if (AKM && BKM && sum && tid < BN / 4 && n0 + tid * 4 < p.N) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] += psum[w * BN + tid * 4 + t];
    store_colsum(p, n0 + tid * 4, split, v);
  }
#pragma unroll
  for (int it = 0; it < PASSES; ++it) {
    const int row = r0 + it * RPP, m = m0 + row;
    if (row >= BM || m >= p.M || n >= p.N) continue;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float *src = parts + (w * BM + row) * LD + c8;
      const float4 lo = *(const float4 *)src, hi = *(const float4 *)(src + 4);
      v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
      v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
    }
    if (p.splits > 1) {
      float *o = p.part + ((long)split * p.M + m) * p.N + n;
      *(float4 *)o = make_float4(v[0], v[1], v[2], v[3]);
      *(float4 *)(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else {
      tile_epilogue8(p, v, m, n, ebias, ein[it]);
    }
  }
}

// ---- 256 x 128 -----------------------------------------------------------------------------------------------------
// For one to a few tiles of 256 x 128 per compute unit, fewer than 256 tiles of 256 x 256.  Such a problem by 128 x 128 tiles, two
// workgroups on a unit, is bound by LDS: a wavefront's 64 x 64 part reads 8 KiB of fragments for sixteen matrix instructions, 128
// bytes a cycle for the unit, all there is, and the loads write as much again as half of that.  Here eight wavefronts share a
// tile and each has 128 x 64, a quarter less to read per instruction: four side by side on one half of a stage's k, four on the
// other, and the two sums are added through LDS at the end (another order of additions than tile_body's: not where that one is
// to be kept).  The schedule is that of gemm_km256_k: the first operand's fragments refilled block by block, the second's in two
// sets, one barrier a stage behind the first block, no two LDS reads back to back; the loads are buffer loads, six a
// wavefront, dealt out between the blocks, three stages in a ring.
// 4096 x 2048 x 8192 156 -> 136 us with a residual, K-contiguous 150 -> 129 (1.07 PFLOP/s; 145 at best by four-deep rings of 128 x
// 128), 8192 x 1024 x 4096 81 -> 67, 4096 x 2048 x 2048 47 -> 39.  Both operands k-major only 103 -> 99: every fragment is two reads there.
template <bool AKM, bool BKM>
__device__ __forceinline__ void wide_body(const TileP &p, int bid, uint16_t *smem) {
  constexpr int BM = 256, BN = 128, NT = 512, R = 3, MB = 8, NB = 4;
  typedef Side<BM, AKM, NT, kSK> SA;
  typedef Side<BN, BKM, NT, kSK> SB;
  constexpr unsigned kStage = SA::kBytes + SB::kBytes;
  constexpr int L = SA::LJ + SB::LJ;  // 4 + 2
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
  NtP q;  // tile_of looks at these only
  q.tiles_m = p.tiles_m; q.tiles_n = p.tiles_n; q.gm = p.gm;
  int tile_m, tile_n;
  tile_of(q, bid, &tile_m, &tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN, nk = (p.K + kSK - 1) / kSK;
  SA sa;
  SB sb;
  sa.init(tid, p.lda);
  sb.init(tid, p.ldb);
  sa.start(p.A, p.lda, m0, p.M, 0, p.K);
  sb.start(p.B, p.ldb, n0, p.N, 0, p.K);
  const unsigned lds0 = (unsigned)(uintptr_t)smem;
  f32x4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t Af[MB], Bf[2][NB];
  // column sums of B, as in tile_body: the wavefronts of the first tile row with distinct fragments, in a loop of their own
  const bool sum = AKM && BKM && p.colsum && tile_m == 0 && wm == 0;
  float *psum = (float *)((char *)smem + R * kStage) + wn * 64;  // [half of k][wn][64] behind the stages
  auto load_all = [&](unsigned at, bool tail) {
    const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + at + wave * 1024);
    const v4i_t ra = sa.desc(), rb = sb.desc();
#pragma unroll
    for (int j = 0; j < SA::LJ; ++j) sa.piece(ra, j, p.K, dst, tail);
#pragma unroll
    for (int j = 0; j < SB::LJ; ++j) sb.piece(rb, j, p.K, dst + SA::kBytes, tail);
    sa.next();
    sb.next();
  };
  unsigned ba = SA::base(kg, lane), bb = SB::base(kg, lane);
  auto rdA = [&](int i, unsigned at) { return SA::frag_from(ba, lds0 + at, wm * MB + i); };
  auto rdB = [&](int j, unsigned at) { return SB::frag_from(bb, lds0 + at + SA::kBytes, wn * NB + j); };
  auto mfma_block = [&](int i, int set, int j0, int j1) {
    SSDT_FENCE;
#pragma unroll
    for (int j = j0; j < j1; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bf[set][j], Af[i], acc[i][j], 0, 0, 0);
    SSDT_FENCE;
  };
  unsigned rd = kStage, wr = 0;  // where the next stage is, where the stage R further on goes: bytes of LDS
  auto advance = [&](unsigned x) { return x == (R - 1) * kStage ? 0u : x + kStage; };
  // stage st, in the registers but for what its own reads still bring; behind the barrier the next one is read
  auto stage = [&](int st, int set, auto inner, auto sum_block) {
    constexpr bool INNER = decltype(inner)::value;
    mfma_block(0, set, 0, NB);
    sum_block(set);
    const bool more = INNER || st + 1 < nk, load = INNER || st + R < nk;
    if (more) wait_stages<L>(INNER ? R : nk - 2 - st, std::integral_constant<int, R - 2>());
    SSDT_FENCE;
    asm volatile("" : "+v"(ba), "+v"(bb));  // (the blocks' addresses, kept from stage to stage, would not leave enough registers)
    v4i_t ra, rb;
    const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + wr + wave * 1024);
#pragma unroll
    for (int i = 1; i < MB; ++i) {
      mfma_block(i, set, 0, 1);
      if (more && i <= NB) Bf[set ^ 1][i - 1] = rdB(i - 1, rd);
      mfma_block(i, set, 1, 3);
      if (more && i == 1) Af[0] = rdA(0, rd);
      if (load) {
        if (i == 1) ra = sa.desc();
        if (i >= 1 && i <= 4) sa.piece(ra, i - 1, p.K, dst, !INNER);
        if (i == 5) rb = sb.desc();
        if (i >= 5 && i <= 6) sb.piece(rb, i - 5, p.K, dst + SA::kBytes, !INNER);
      }
      mfma_block(i, set, 3, NB);
      if (more) Af[i] = rdA(i, rd);
    }
    sa.next();
    sb.next();
    rd = advance(rd);
    wr = advance(wr);
  };
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (i < nk) load_all(i * kStage, true);
  wait_stages<L>(nk - 1, std::integral_constant<int, R - 1>());
#pragma unroll
  for (int j = 0; j < NB; ++j) Bf[0][j] = rdB(j, 0);
#pragma unroll
  for (int i = 0; i < MB; ++i) Af[i] = rdA(i, 0);
  auto stages = [&](auto sum_block) {
    int st = 0;
    for (; st + 2 + R < nk; st += 2) {
      stage(st, 0, std::true_type(), sum_block);
      stage(st + 1, 1, std::true_type(), sum_block);
    }
    for (; st < nk; st += 2) {
      stage(st, 0, std::false_type(), sum_block);
      if (st + 1 < nk) stage(st + 1, 1, std::false_type(), sum_block);
    }
  };
  if (AKM && BKM && sum) {
    f32x4_t accs[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) accs[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    stages([&](int set) {
      union { unsigned w[4]; bf16x8_t v; } ones;
      ones.w[0] = ones.w[1] = ones.w[2] = ones.w[3] = 0x3F803F80u;
#pragma unroll
      for (int j = 0; j < NB; ++j) accs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bf[set][j], ones.v, accs[j], 0, 0, 0);
    });
    if (lr == 0)
#pragma unroll
      for (int j = 0; j < NB; ++j) *(float4 *)(psum + kg * 128 + j * 16 + lq * 4) = make_float4(accs[j][0], accs[j][1], accs[j][2], accs[j][3]);
  } else {
    stages([](int) {});
  }
  // The two halves of the contraction: each wavefront keeps 64 of its 128 rows and hands the others to the wavefront that has the
  // other half of k, through that one's part of LDS; from there row by row, 16 bytes per lane.
  constexpr int LD = 68;
  u32x4_a8_t ein[8], ebias = {0, 0, 0, 0};
  const int c8 = (lane & 7) * 8, n = n0 + wn * 64 + c8, mb = m0 + wm * 128 + kg * 64;
  if (n < p.N) ebias = bias8(p, n);
#pragma unroll
  for (int pass = 0; pass < 8; ++pass) {
    const int m = mb + pass * 8 + (lane >> 3);
    ein[pass] = u32x4_a8_t{0, 0, 0, 0};
    if (m < p.M && n < p.N) ein[pass] = epilogue_in8(p, m, n);
  }
  float *own = (float *)smem + wave * (64 * LD), *other = (float *)smem + (wave ^ 4) * (64 * LD);
  __syncthreads();
#pragma unroll
  for (int il = 0; il < 4; ++il)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32x4_t a = kg ? acc[il][j] : acc[4 + il][j];
      *(float4 *)(other + (il * 16 + lr) * LD + j * 16 + lq * 4) = make_float4(a[0], a[1], a[2], a[3]);
    }
  __syncthreads();
  if (AKM && BKM && sum && !kg && lane < 16 && n0 + wn * 64 + lane * 4 < p.N) {
    const float4 lo = *(const float4 *)(psum + lane * 4), hi = *(const float4 *)(psum + 128 + lane * 4);
    float v[4] = {lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w};
    store_colsum(p, n0 + wn * 64 + lane * 4, 0, v);
  }
#pragma unroll
  for (int il = 0; il < 4; ++il)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32x4_t a = kg ? acc[4 + il][j] : acc[il][j];
      float4 *at = (float4 *)(own + (il * 16 + lr) * LD + j * 16 + lq * 4);
      const float4 o = *at;
      *at = make_float4(a[0] + o.x, a[1] + o.y, a[2] + o.z, a[3] + o.w);
    }
#pragma unroll
  for (int pass = 0; pass < 8; ++pass) {
    const int row = pass * 8 + (lane >> 3), m = mb + row;
    const float4 lo = *(const float4 *)(own + row * LD + c8), hi = *(const float4 *)(own + row * LD + c8 + 4);
    if (m >= p.M || n >= p.N) continue;
    float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    tile_epilogue8(p, v, m, n, ebias, ein[pass]);
  }
}

template <bool AKM, bool BKM>
__global__ __launch_bounds__(512) void gemm_wide_k(TileP p) {
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  wide_body<AKM, BKM>(p, blockIdx.x, smem);
}
// as gemm_tile_pair_k
__global__ __launch_bounds__(512) void gemm_wide_pair_k(TileP w, TileP d, int first, int w_first) {
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  const int bid = blockIdx.x;
  const bool head = bid < first;
  if (head == (w_first != 0)) wide_body<true, true>(w, head ? bid : bid - first, smem);
  else wide_body<false, false>(d, head ? bid : bid - first, smem);
}

// KW: wavefronts along k
template <int BM, int BN, int R, bool KW, bool AKM, bool BKM, bool BIG = false, int NW = waves_of(BM, BN, R)>
__device__ __forceinline__ void any_body(const TileP &p, int bid, uint16_t *smem) {
  if constexpr (KW) kwave_body<BM, BN, R, AKM, BKM>(p, bid, smem);
  else tile_body<BM, BN, R, AKM, BKM, BIG, NW>(p, bid, smem);
}
template <int BM, int BN, int R, bool KW, bool AKM, bool BKM, bool BIG>
__global__ __launch_bounds__(threads_of(KW, waves_of(BM, BN, R)), 2) void gemm_tile_k(TileP p) {
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  any_body<BM, BN, R, KW, AKM, BKM, BIG>(p, blockIdx.x, smem);
}

// The two products of a linear's backward in one launch: the weight gradient (both operands k-major) and the input
// gradient (both K-contiguous) read the same dY and do not depend on each other.  Launched one after the other, the
// second waits until the last workgroup of the first has finished; here the one with the longer tiles goes first and the
// other fills the machine behind it.
template <int BM, int BN, int R, bool KW, int NW>
__global__ __launch_bounds__(threads_of(KW, NW), 2) void gemm_tile_pair_k(TileP w, TileP d, int first, int w_first) {
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  const int bid = blockIdx.x;
  const bool head = bid < first;
  if (head == (w_first != 0)) any_body<BM, BN, R, KW, true, true, false, NW>(w, head ? bid : bid - first, smem);
  else any_body<BM, BN, R, KW, false, false, false, NW>(d, head ? bid : bid - first, smem);
}

// Second half of a split product: adds the partial products in the order of the splits and applies the epilogue;
// the blocks behind the ones that cover C do the same for the column sums.
__global__ __launch_bounds__(256) void tile_reduce_k(TileP p) {
  const long n8 = p.N / 8, i = (long)blockIdx.x * 256 + threadIdx.x, plane = (long)p.M * p.N;
  if (i >= p.M * n8) {
    const long c = i - p.M * n8;
    if (!p.colsum || c >= n8) return;
    const float *s = p.part + p.splits * plane + c * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < p.splits; ++k)
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] += s[(long)k * p.N + t];
    if (p.colsum_acc) {
      float old[8];
      load8(p.colsum + c * 8, old);
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] += old[t];
    }
    store8(p.colsum + c * 8, v);
    return;
  }
  const int m = (int)(i / n8), n = (int)(i % n8) * 8;
  const float *s = p.part + (long)m * p.N + n;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < p.splits; ++k) {
    const float4 lo = *(const float4 *)(s + k * plane), hi = *(const float4 *)(s + k * plane + 4);
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
    v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  tile_epilogue8(p, v, m, n, bias8(p, n), epilogue_in8(p, m, n));
}

struct TileCfg { int bm, bn, ring, sk; };  // sk: k per stage, 128 with the wavefronts along k
static const TileCfg kCfg[] = {{128, 128, 2, 64}, {64, 128, 2, 64}, {64, 64, 2, 64}, {64, 128, 3, 64}, {64, 64, 3, 64}, {128, 128, 4, 64},
                                {64, 64, 3, 128}, {32, 64, 3, 128}, {32, 32, 4, 128}, {256, 128, 3, 64}};
constexpr int kCfgs = sizeof kCfg / sizeof kCfg[0];
constexpr int kWide = kCfgs - 1;  // not split
constexpr int kOneOrder = 6;  // the first six add in the same order
// Test hooks: >= 0 pins the tile, > 0 the number of splits (of a pair's input gradient: the tens, if any; workspaces are reported with
// room for them); launches of tile_reduce_k so far.
int g_tile_cfg = -1, g_tile_splits = 0;
std::atomic<int> g_tile_reduces{0};
static int pinned_splits(bool input_grad) { return input_grad && g_tile_splits >= 10 ? g_tile_splits / 10 : g_tile_splits % 10; }

static hipError_t launch_reduce(const TileP &p, hipStream_t s) {
  if (p.splits == 1) return hipSuccess;
  const long items = (long)p.M * (p.N / 8) + (p.colsum ? p.N / 8 : 0);
  hipLaunchKernelGGL(tile_reduce_k, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, p);
  g_tile_reduces.fetch_add(1, std::memory_order_relaxed);
  return hipGetLastError();
}
static unsigned blocks_of(const TileP &p) { return (unsigned)(p.tiles_m * p.tiles_n * p.splits); }

template <int BM, int BN, int R, bool KW>
static constexpr size_t smem_of() {
  constexpr size_t stg = KW ? (size_t)4 * BM * (BN + 4) * 4 + 4 * BN * 4 : (size_t)waves_of(BM, BN, R) * 32 * (BN * 2 / waves_of(BM, BN, R) + 4) * 4;
  constexpr size_t stages = (size_t)R * (BM + BN) * (KW ? 128 : kSK) * 2;
  return stg > stages ? stg : stages;
}
template <int BM, int BN, int R, bool KW, bool AKM, bool BKM, bool BIG = false>
static hipError_t launch_tile(const TileP &p, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_tile_k<BM, BN, R, KW, AKM, BKM, BIG>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_of<BM, BN, R, KW>());
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  prof::Scope ps(prof::GEMM_MFMA_TILE, 2.0 * p.M * p.N * p.K, 0, s);
  hipLaunchKernelGGL((gemm_tile_k<BM, BN, R, KW, AKM, BKM, BIG>), dim3(blocks_of(p)), dim3(threads_of(KW, waves_of(BM, BN, R))), (smem_of<BM, BN, R, KW>()), s, p);
  hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_reduce(p, s);
}
constexpr size_t kWideLds = (size_t)3 * (256 + 128) * kSK * 2 + 4 * 64 * 4;  // stages (the partial tiles need less), column sums
template <bool AKM, bool BKM>
static hipError_t launch_wide(const TileP &p, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_wide_k<AKM, BKM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  prof::Scope ps(prof::GEMM_MFMA_TILE, 2.0 * p.M * p.N * p.K, 0, s);
  hipLaunchKernelGGL((gemm_wide_k<AKM, BKM>), dim3(p.tiles_m * p.tiles_n), dim3(512), kWideLds, s, p);
  return hipGetLastError();
}
static hipError_t launch_wide_pair(const TileP &w, const TileP &d, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_wide_pair_k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideLds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  prof::Scope ps(prof::GEMM_MFMA_TILE, 2.0 * w.M * w.N * w.K + 2.0 * d.M * d.N * d.K, 0, s);
  const bool w_first = w.stages_per_split >= d.stages_per_split;
  hipLaunchKernelGGL(gemm_wide_pair_k, dim3(blocks_of(w) + blocks_of(d)), dim3(512), kWideLds, s, w, d,
                     (int)(w_first ? blocks_of(w) : blocks_of(d)), w_first ? 1 : 0);
  return hipGetLastError();
}
constexpr int kBig = kCfgs;  // 128 x 128 with 64-bit extents
template <bool AKM, bool BKM>
static hipError_t launch_cfg(int cfg, const TileP &p, hipStream_t s) {
  switch (cfg) {
    case kBig: return launch_tile<128, 128, 2, false, AKM, BKM, true>(p, s);
    case 0: return launch_tile<128, 128, 2, false, AKM, BKM>(p, s);
    case 1: return launch_tile<64, 128, 2, false, AKM, BKM>(p, s);
    case 2: return launch_tile<64, 64, 2, false, AKM, BKM>(p, s);
    case 3: return launch_tile<64, 128, 3, false, AKM, BKM>(p, s);
    case 4: return launch_tile<64, 64, 3, false, AKM, BKM>(p, s);
    case 5: return launch_tile<128, 128, 4, false, AKM, BKM>(p, s);
    case 6: return launch_tile<64, 64, 3, true, AKM, BKM>(p, s);
    case 7: return launch_tile<32, 64, 3, true, AKM, BKM>(p, s);
    case 8: return launch_tile<32, 32, 4, true, AKM, BKM>(p, s);
    default: return launch_wide<AKM, BKM>(p, s);
  }
}
template <int BM, int BN, int R, bool KW, int NW = waves_of(BM, BN, R)>
static hipError_t launch_pair(const TileP &w, const TileP &d, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_tile_pair_k<BM, BN, R, KW, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_of<BM, BN, R, KW>());
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  prof::Scope ps(prof::GEMM_MFMA_TILE, 2.0 * w.M * w.N * w.K + 2.0 * d.M * d.N * d.K, 0, s);
  const bool w_first = w.stages_per_split >= d.stages_per_split;
  hipLaunchKernelGGL((gemm_tile_pair_k<BM, BN, R, KW, NW>), dim3(blocks_of(w) + blocks_of(d)), dim3(threads_of(KW, NW)), (smem_of<BM, BN, R, KW>()), s, w, d,
                     (int)(w_first ? blocks_of(w) : blocks_of(d)), w_first ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_reduce(w, s);
  return e != hipSuccess ? e : launch_reduce(d, s);
}

bool gemm_tile_fits(int M, int N, int K, bool transA, bool transB, int dtype) {
  if (dtype != SSDT_BF16 || N % 8) return false;
  if (transA ? M % 8 != 0 : K % 8 != 0) return false;
  if (transB && K % 8) return false;
  return !(transA && transB);  // (the layer has no such product)
}

// DISPATCH.  Predicted time of a problem in microseconds, fitted to what the products of 525 layers took inside the layer: three layers
// in turn, with and without the last-level cache emptied between two passes (MI355X; 32 to 16000 tokens, widths 128 to 4200; 3900 products
// by themselves, 2000 linears' backwards, every tile and split).  A linear's backward took 1.7 % longer than by the best choice, 2.1 on layers that were
// not fitted.  (Fitted to products by themselves, operands in the caches and widths to 2048, it took 5.1 % longer.)
// The two tiles of eight wavefronts, rings of 3 and 4, were fitted anew, to 9700 forward products each among its layer's others (2450 layers, norms in
// between, the weights of 3 to 16 layers in turn).  There the choice costs 1.2 % more than the best tile on average, 7.9 % at the 95th percentile; with
// the entries of the four-wavefront kernels 1.8 and 11.1 %, with those entries' launch cost lowered 1.7 and 10.8 % (384 x 3392 x 13568 took 128 x 128, 121
// us, for 64 x 128, 99).  (Products by themselves say otherwise here too: 768 x 5376 x 1792, 25 us by either, makes its layer 9 us longer by 128 x 128 in
// the ring of 4.)  The other entries and kPairCost are from the 525 layers; pairs of 64 x 128 in a ring of 3 are up to 4 % faster than it says.
// A launch takes z us and e for each tile of a compute unit.  Whole rounds of as many workgroups as fit take c for each of a unit's
// and stage of 64 k; in the last one a stage takes a + b n when n workgroups share a unit, and never less than c for each of
// them, averaged over the machine.  f: us for each megabyte that a stage's panels bring from memory to the XCDs (panels()): small tiles
// read an operand more often than the L2s catch.
//   128 x 128, ring of 2: 0.76 us alone, 0.56 each together (1.0 PFLOP/s on 4096 x 2048 x 8192, 512 tiles);
//              ring of 4, eight wavefronts: 0.47, and alone on its unit always: for one round of tiles and long K (152 tiles of 2331 x 1024
//              x 4096: 31 us against 38 by 64 x 128); 0.60 in whole rounds, where 128 x 128 with two buffers is the better one;
//    64 x 128, ring of 2: 0.33 each from three on: where three share a unit;
//              ring of 3, eight wavefronts: 0.33 alone (384 x 3392 x 13568, 162 tiles: 99 us against 160 and, 128 x 128, 121);
//    64 x 64,  ring of 2: 0.20 each, four to a unit (160 KiB of LDS would hold a fifth, but it waits: 1056 tiles of 33 stages 47 us,
//              1014 of 52 50);
//              ring of 3: 0.20 alone: for the smaller (512 x 2304 x 576: 9 us, by 64 x 128 13).
//   wavefronts along k (a stage of 128 counts twice): 64 x 64 0.18 alone; 32 x 64 0.14; 32 x 32 0.14: for fewer tiles than
//              compute units, where a stage is bound by the LDS reads of one workgroup: of a 64 x 64 tile four wavefronts side by
//              side read half as much as four quarters of it, and 32 x 32 tiles leave each unit a quarter of the loads.
//              (256 x 256 x 1024 7.4 -> 5.2 us, 128 x 1280 x 5120 22.3 -> 14.6, 256 x 1280 x 5120 25.1 -> 17.7 by 32 x 64, 1024 x 1024
//              x 4096 25.7 -> 21.6 by 64 x 64; both products of 256 x 256 -> 1024's backward 8.5 -> 6.0.)
//  256 x 128: 0.94 us a stage, 0.69 in a last round that leaves much of the machine over.
// Splitting the contraction costs a second launch and the partial products' way out and back, from the caches at about 12 TB/s.
struct TileCost { double a, b, c, e, f, z; int fit; };  // fit: workgroups that share a compute unit at most
static const TileCost kCost[kCfgs] = {{0.746, 0.01, 0.562, 2.776, 0, 7.409, 2},      {0.544, 0.078, 0.332, 0.536, 0.042, 5.313, 3},
                                      {0.41, 0.041, 0.195, 0.568, 0.048, 4.39, 4},   {0.108, 0.221, 0.337, 1.31, 0.039, 5.121, 2},
                                      {0.05, 0.153, 0.19, 0.412, 0.066, 4.996, 3},   {0.135, 0.336, 0.599, 4.448, 0.012, 5.435, 1},
                                      {0.134, 0.042, 0.182, 1.33, 0.054, 4.884, 1},  {0.052, 0.089, 0.177, 0.478, 0.045, 4.333, 2},
                                      {0.064, 0.073, 0.117, 0.418, 0.049, 3.756, 2}, {0.663, 0.026, 0.943, 9.984, 0, 6.252, 1}};
constexpr int kMaxSplits = 8;
static int stages_of(int K) { return (K + kSK - 1) / kSK; }
static double reduce_cost(int M, int N, int splits) { return splits > 1 ? 3.1 + 8.0 * splits * M * N / 12e6 : 0.0; }
// A problem in tiles of a kind: rows and columns of tiles, stages of 64 k.  (Everything from here to the launch is on the path of each
// call: a layer's plans, forward and backward, take 1.5 to 5 us, candidates that cannot win are left out early.)
struct Tiling { int tm, tn, stages; long n; };
static Tiling tiling(int M, int N, int K, int cfg) {
  const auto up = [](int x, int by) { return (x + by - 1) >> __builtin_ctz(by); };  // (all powers of two)
  const TileCfg &q = kCfg[cfg];
  Tiling t{up(M, q.bm), up(N, q.bn), up(K, q.sk) * (q.sk / kSK), 0};
  t.n = (long)t.tm * t.tn;
  return t;
}
// Megabytes that the panels of one stage bring to the eight XCDs, each panel once to every XCD that has a tile of it, times the rounds
// of workgroups.  tile_of deals a number of tiles that is a multiple of eight out in eight compact pieces; others go round the XCDs
// one by one, and each XCD reads every panel of B.
static double panels(const Tiling &p, int cfg, int splits, int fit) {
  const double tm = p.tm, tn = p.tn, nt = (double)p.n, n = nt * splits, round = 256.0 * fit;
  const int g = std::min(p.tm >= p.tn ? 4 : 8, p.tm);  // rows of tiles in a group, see choose
  const double at = std::min(n, round), one = std::min(nt, at), beside = at / one, w = std::max(one / 8, 1.0);  // tiles of an XCD
  double rows, cols;
  if (p.n % 8 == 0) {
    rows = std::min(tm, g * std::ceil(w / (g * tn)));
    cols = std::min(tn, std::ceil(w / g));
  } else {
    rows = std::min(std::min(tm, w), g / (g % 8 == 0 ? 8.0 : g % 4 == 0 ? 4.0 : g % 2 == 0 ? 2.0 : 1.0) * std::ceil(one / (g * tn)));
    cols = std::min(tn, w);
  }
  return (rows * kCfg[cfg].bm + cols * kCfg[cfg].bn) * 8 * (2 * kSK) * 1e-6 * std::max(n / round, beside);
}
static size_t split_bytes(int M, int N, int splits) { return splits > 1 ? (size_t)splits * ((size_t)M + 1) * N * 4 : 0; }
static bool split_ok(int K, int splits) { return splits == 1 || splits * 4 <= stages_of(K); }

// How often the contraction can be halved, given `scratch` bytes for partial products.
static int most_halvings(int M, int N, int K, size_t scratch) {
  int h = 0;
  while ((2 << h) <= kMaxSplits && split_ok(K, 2 << h) && split_bytes(M, N, 2 << h) <= scratch) ++h;
  return h;
}

// Small tiles are the likely choice: looked at first, they rule the others out.
static bool few_tiles(int M, int N) { return (long)M * N < 96l * 128 * 128; }

// The choice for a problem given `scratch` bytes for partial products, among the first `cfgs` tiles; returns its predicted time.
// kmajor: both operands are, and a fragment of either is two LDS reads.  128 x 128 alone on a unit feels it most (4096 x 1024 x 8192 87 us
// against 78 by two splits in a ring of two).
static double tile_plan(int M, int N, int K, bool kmajor, size_t scratch, int cfgs, int *cfg, int *splits) {
  const int most = scratch ? most_halvings(M, N, K, scratch) : 0;
  const bool small = few_tiles(M, N);
  double best = 1e30;
  for (int i = 0; i < cfgs; ++i) {
    const int c = small ? cfgs - 1 - i : i;
    const TileCost &q = kCost[c];
    const Tiling p = tiling(M, N, K, c);
    if (q.z + p.n * (q.c * p.stages + q.e) / 256.0 >= best) continue;  // (every unit busy to the end, nothing to reduce)
    for (int h = 0; h <= (c == kWide ? 0 : most); ++h) {
      const long tiles = p.n << h, round = 256l * q.fit, full = tiles < round ? 0 : tiles / round, rest = tiles - full * round;
      const double stages = (p.stages + (1 << h) - 1) >> h;
      const double fixed = q.z + q.e * tiles / 256.0 + reduce_cost(M, N, 1 << h);
      const double stage = full * q.c * q.fit + (rest ? std::max(q.a + q.b * ((rest + 255) / 256), q.c * rest / 256.0) : 0.0);
      if (fixed + stage * stages >= best) continue;
      double t = fixed + (stage + q.f * panels(p, c, 1 << h, q.fit)) * stages;
      if (kmajor && c == 5) t *= 1.05;
      if (t < best) { best = t; *cfg = c; *splits = 1 << h; }
    }
  }
  return best;
}

// The same for two problems in one launch (one tile size, each its own split; half of the scratch for each).  The tiles
// of both share the machine: it is done when the work is (c per tile and stage, and what of the shorter tiles runs beside
// nothing at the end), or when the longest tile is.  Fitted by itself.  (fit 0: no pair, 128 x 128 in a ring of four and 64 x 64 along k
// were never the choice.)
static const TileCost kPairCost[kWide] = {{0.792, 0.014, 0.49, 1.087, 0.023, 4.489, 2}, {0.508, 0.029, 0.284, 0.385, 0.047, 3.035, 3},
                                          {0.291, 0.04, 0.16, 0.296, 0.062, 2.816, 4},  {0.437, 0.005, 0.328, 1.165, 0.014, 2.865, 2},
                                          {0.215, 0.01, 0.189, 0.389, 0.03, 2.72, 3},   {},
                                          {},                                           {0.146, 0.008, 0.151, 0.463, 0.017, 2.706, 2},
                                          {0.045, 0.032, 0.12, 0.39, 0.015, 2.908, 2}};
// When `slots` workers are done that take n1 pieces of t1 each and then n2 of t2.
static double deal(long n1, double t1, long n2, double t2, long slots) {
  struct { double at; long n; } g[64] = {{0.0, slots}};  // workers by the time they are free
  int groups = 1;
  double end = 0;
  for (int kind = 0; kind < 2; ++kind)
    for (long rem = kind ? n2 : n1; rem > 0;) {
      int i = 0;
      for (int j = 1; j < groups; ++j)
        if (g[j].at < g[i].at) i = j;
      const double done = g[i].at + (kind ? t2 : t1);
      const long n = std::min(rem, g[i].n);
      rem -= n;
      end = std::max(end, done);
      if (n == g[i].n) g[i].at = done;
      else if (groups < 64) { g[i].n -= n; g[groups].at = done; g[groups++].n = n; }
    }
  return end;
}
struct Shape { int M, N, K; };
static size_t half_of(size_t scratch) { return scratch / 2 / 256 * 256; }
static double pair_plan(const Shape &w, const Shape &d, size_t scratch, PairPlan *out) {
  const size_t half = half_of(scratch);
  const int most_w = most_halvings(w.M, w.N, w.K, half), most_d = most_halvings(d.M, d.N, d.K, half);
  double best = 1e30, rw[4], rd[4];
  for (int h = 0; h <= most_w; ++h) rw[h] = reduce_cost(w.M, w.N, 1 << h);
  for (int h = 0; h <= most_d; ++h) rd[h] = reduce_cost(d.M, d.N, 1 << h);
  const bool small = few_tiles(w.M, w.N) && few_tiles(d.M, d.N);
  for (int i = 0; i < kWide; ++i) {
    const int c = small ? kWide - 1 - i : i;
    const TileCost &q = kPairCost[c];
    if (!q.fit) continue;
    const Tiling pw = tiling(w.M, w.N, w.K, c), pd = tiling(d.M, d.N, d.K, c);
    const double busy = q.z + ((double)(pw.n * pw.stages + pd.n * pd.stages) * q.c + (double)(pw.n + pd.n) * q.e) / 256.0;
    for (int hw = 0; hw <= most_w; ++hw) {
      if (busy + rw[hw] >= best) break;  // (as in tile_plan; the reduction takes longer with every split)
      for (int hd = 0; hd <= most_d; ++hd) {
        if (busy + rw[hw] + rd[hd] >= best) break;
        const double nw = (double)(pw.n << hw), nd = (double)(pd.n << hd), n256 = (nw + nd) / 256.0;
        const double lw = (pw.stages + (1 << hw) - 1) >> hw, ld = (pd.stages + (1 << hd) - 1) >> hd;
        const double n = std::min((double)q.fit, std::ceil(n256));
        const double tail = (n256 > q.fit ? 0.421 : 0.115) * std::min(lw, ld) * (q.a + q.b);
        const double work = ((nw * lw + nd * ld) * q.c + (nw + nd) * q.e) / 256.0 + tail;
        double t = q.z + std::max(work, std::max(lw, ld) * (q.a + q.b * n) + q.e) + rw[hw] + rd[hd];
        if (t >= best) continue;
        t += q.f * (panels(pw, c, 1 << hw, q.fit) * lw + panels(pd, c, 1 << hd, q.fit) * ld);
        if (t < best) { best = t; out->cfg = c; out->sw = 1 << hw; out->sd = 1 << hd; }
      }
    }
  }
  // Tiles of 256 x 128, one to a compute unit, by dealing them out: 0.88 us a stage and 4 a tile (4096 x 2048 -> 6144 219 -> 195 us; 8192 x
  // 1024 -> 4096 136 -> 124; 4096 x 2048 -> 2048 73 -> 67; 5785 x 2048 -> 2048 103 -> 95).  Against unsplit 128 x 128 tiles, the other
  // choice at such sizes, their time by the table and their time by dealing them out count the same (2.5 % more than the best on
  // average over 700 such linears, by either alone 2.7).
  const Tiling pw = tiling(w.M, w.N, w.K, kWide), pd = tiling(d.M, d.N, d.K, kWide);
  const double tw = pw.stages * 0.88 + 4.0, td = pd.stages * 0.88 + 4.0;
  if (pw.n + pd.n <= 2048 && std::max((pw.n * tw + pd.n * td) / 256.0, std::max(tw, td)) < best * 1.1) {
    const auto dealt = [](const Tiling &a, double ta, const Tiling &b, double tb, long slots) {
      return a.stages >= b.stages ? deal(a.n, ta, b.n, tb, slots) : deal(b.n, tb, a.n, ta, slots);
    };
    const double wide = dealt(pw, tw, pd, td, 256), t = 12.94 + 0.907 * wide;
    double against = best * 0.99 / t;
    if (out->cfg == 0 && out->sw == 1 && out->sd == 1) {
      const Tiling qw = tiling(w.M, w.N, w.K, 0), qd = tiling(d.M, d.N, d.K, 0);
      against = best / t * (2.7 + dealt(qw, qw.stages * 0.95 + 2.2, qd, qd.stages * 0.95 + 2.2, 512)) / (2.7 + wide);
    }
    if (against > 1) { best = std::min(best, t); out->cfg = kWide; out->sw = out->sd = 1; }
  }
  return best;
}

// Predicted time of the 256 x 256 kernels, fitted to 362 products of such layers (standard deviation 9 %): a round of 256 of their
// tiles takes 1.05 us a stage however empty it is and up to 0.42 more when it is full (4096 x 6144 x 2048, 384 tiles: 94 us against
// 107 here).
static bool large_possible(int M, int N, int K, bool transA, bool transB) {
  if (M % 256 || N % 256 || K % 64 || (long)(M / 256) * (N / 256) < 256) return false;
  return K % 128 == 0 || (!transA && transB);  // (gemm_km256_k takes its stages in pairs)
}
static double large_cost(int M, int N, int K) {
  const long tiles = (long)(M / 256) * (N / 256);
  const double rounds = tiles / 256.0, begun = (double)((tiles + 255) / 256);
  return (K / 64) * (1.046 * begun + 0.42 * rounds) + 4.45 * begun + 5.65 * rounds;
}

// Whether they should take a problem that suits both: unless 128 x 128 tiles would be done sooner if they kept every compute unit busy to
// the end, which they are just above 256 tiles of 256 x 256 (5632 x 3072 x 12288, 264 tiles: 534 us, by 128 x 128 477, by 256 x 128 449;
// 8960 x 2048 x 8192, 280 tiles: 346, 343, 309; from 288 tiles on the large ones are ahead).
bool gemm_large_fits(int M, int N, int K, bool transA, bool transB, int dtype) {
  if (dtype != SSDT_BF16 || !large_possible(M, N, K, transA, transB)) return false;
  if (!gemm_tile_fits(M, N, K, transA, transB, dtype)) return true;
  const TileCost &q = kCost[0];
  const Tiling p = tiling(M, N, K, 0);
  return q.z + p.n / 256.0 * (q.c * p.stages + q.e) > large_cost(M, N, K);
}

static bool tiles_take(const Shape &p, bool transA, bool transB) {
  return gemm_tile_fits(p.M, p.N, p.K, transA, transB, SSDT_BF16) && !gemm_large_fits(p.M, p.N, p.K, transA, transB, SSDT_BF16);
}
// No tile takes less: the least of the bounds that tile_plan starts from.
static double least_cost(const Shape &p) {
  double least = 1e30;
  for (int c = 0; c < kCfgs; ++c) {
    const Tiling t = tiling(p.M, p.N, p.K, c);
    least = std::min(least, kCost[c].z + t.n * (kCost[c].c * t.stages + kCost[c].e) / 256.0);
  }
  return least;
}
// Whether the weight gradient w (M x N over K tokens) and the input gradient d of a linear should share a launch, given
// `scratch` bytes; *out is the choice then.
static bool pair_wanted(const Shape &w, const Shape &d, size_t scratch, PairPlan *out) {
  if (!tiles_take(w, true, false) || !tiles_take(d, false, true)) return false;
  const double together = pair_plan(w, d, scratch, out);
  if (together < least_cost(w) + least_cost(d)) return true;
  int c, sp;
  return together < tile_plan(w.M, w.N, w.K, true, scratch, kCfgs, &c, &sp) + tile_plan(d.M, d.N, d.K, false, scratch, kCfgs, &c, &sp);
}

// Scratch that the choices for a linear's two backward products (rows tokens, in -> out) use where there is enough of it, each by
// itself or both in one launch (*plan).
size_t gemm_linear_bwd_scratch_bytes(int rows, int in, int out, int dtype, PairPlan *plan) {
  *plan = PairPlan{rows, in, out};
  if (dtype != SSDT_BF16) return 0;
  const Shape w{in, out, rows}, d{rows, in, out};
  const size_t all = ~(size_t)0;
  const bool tw = tiles_take(w, true, false), td = tiles_take(d, false, true);
  int c = 0, sw = 1, sd = 1;
  double alone = 0;
  if (tw) alone += tile_plan(w.M, w.N, w.K, true, all, kCfgs, &c, &sw);
  if (td) alone += tile_plan(d.M, d.N, d.K, false, all, kCfgs, &c, &sd);
  const auto bytes_w = [&](int s) { return split_bytes(w.M, w.N, std::max(s, pinned_splits(false))); };
  const auto bytes_d = [&](int s) { return split_bytes(d.M, d.N, std::max(s, pinned_splits(true))); };
  size_t bytes = std::max(tw ? bytes_w(sw) : 0, td ? bytes_d(sd) : 0);
  if (tw && td && pair_plan(w, d, all, plan) < alone) {
    plan->pair = true;
    bytes = std::max(bytes, 2 * std::max(bytes_w(plan->sw), bytes_d(plan->sd)) + 512);
  }
  return bytes;
}

// For tests: the tile that a forward product takes, -1 where it goes to the 256 x 256 kernels.
int gemm_tile_choice(int M, int N, int K, bool one_order) {
  if (gemm_large_fits(M, N, K, false, false, SSDT_BF16)) return -1;
  int cfg = 0, splits = 1;
  tile_plan(M, N, K, false, 0, one_order ? kOneOrder : kCfgs, &cfg, &splits);
  return cfg;
}

// Checks what the kernel needs beyond the shape and fills its arguments, the choice of tile aside.  *big: an operand whose extent 31
// bits do not hold in units of 16 bytes (Side::left; w_2 of 524288 tokens, F 32776).
static hipError_t prepare(const Gemm &g, TileP *p, bool *big) {
  if (!gemm_tile_fits(g.M, g.N, g.K, g.transA, g.transB, g.dtype)) return hipErrorNotSupported;
  const bool akm = g.transA, bkm = !g.transB;
  auto al16 = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
  auto al8 = [](const void *q) { return ((uintptr_t)q & 7) == 0; };
  if (!al16(g.A) || !al16(g.B) || g.lda % 8 || g.ldb % 8 || g.lda >= (1L << 21) || g.ldb >= (1L << 21)) return hipErrorNotSupported;
  if (g.lda < (akm ? g.M : g.K) || g.ldb < (bkm ? g.N : g.K)) return hipErrorNotSupported;
  if (g.ldc % 4 || !al8(g.C) || (g.C2 && !al8(g.C2)) || (g.bias && !al8(g.bias)) || (g.aux && !al8(g.aux)) ||
      (g.resid && (!al8(g.resid) || g.ldr % 4)))
    return hipErrorNotSupported;
  const long ea = akm ? (long)(g.K - 1) * g.lda + g.M : (long)(g.M - 1) * g.lda + g.K;
  const long eb = bkm ? (long)(g.K - 1) * g.ldb + g.N : (long)(g.N - 1) * g.ldb + g.K;
  *big = (ea | eb) >> 34;
  if (g.epi == EPI_BIAS_ACT && !g.C2) return hipErrorInvalidValue;
  if (g.epi == EPI_BIAS_RESID && !g.resid) return hipErrorInvalidValue;
  if (g.epi == EPI_ACTBWD && !g.aux) return hipErrorInvalidValue;
  if (g.colsum && (!(akm && bkm) || !al8(g.colsum))) return hipErrorNotSupported;
  *p = TileP{g.M, g.N, g.K, (const uint16_t *)g.A, (const uint16_t *)g.B, g.lda, g.ldb, g.ldc, g.ldr, (uint16_t *)g.C,
             (uint16_t *)g.C2, (const uint16_t *)g.bias, (const uint16_t *)g.resid, (const uint16_t *)g.aux, g.act, g.epi,
             0, 0, 0, 1, stages_of(g.K), nullptr, (uint16_t *)g.colsum, g.colsum_accumulate ? 1 : 0};
  return hipSuccess;
}
static void choose(TileP *p, int cfg, int splits, float *part) {
  p->tiles_m = (p->M + kCfg[cfg].bm - 1) / kCfg[cfg].bm;
  p->tiles_n = (p->N + kCfg[cfg].bn - 1) / kCfg[cfg].bn;
  p->gm = g_force_waves > 0 ? g_force_waves : (p->tiles_m >= p->tiles_n ? 4 : 8);
  const int nk = (p->K + kCfg[cfg].sk - 1) / kCfg[cfg].sk;
  p->stages_per_split = (nk + splits - 1) / splits;
  p->splits = (nk + p->stages_per_split - 1) / p->stages_per_split;  // (every part has a stage)
  p->part = part;
}
static size_t usable_scratch(const Gemm &g) { return g.split && g.scratch && ((uintptr_t)g.scratch & 15) == 0 ? g.scratch_bytes : 0; }

hipError_t gemm_mfma_tile_bf16(const Gemm &g, hipStream_t s) {
  TileP p;
  bool big;
  hipError_t e = prepare(g, &p, &big);
  if (e != hipSuccess) return e;
  int cfg = 0, splits = 1;
  tile_plan(g.M, g.N, g.K, g.transA, usable_scratch(g), g.one_order ? kOneOrder : kCfgs, &cfg, &splits);
  if (g_tile_cfg >= 0) cfg = g_tile_cfg;
  if (g_tile_splits > 0 && split_bytes(g.M, g.N, pinned_splits(g.transB)) <= g.scratch_bytes) splits = pinned_splits(g.transB);
  if (cfg == kWide) splits = 1;
  if (big) cfg = 0;
  choose(&p, cfg, splits, (float *)g.scratch);
  if (big) cfg = kBig;
  if (g.transA) return launch_cfg<true, true>(cfg, p, s);
  if (!g.transB) return launch_cfg<false, true>(cfg, p, s);
  return launch_cfg<false, false>(cfg, p, s);
}

hipError_t gemm_pair_bf16(const Gemm &w, const Gemm &d, const PairPlan *plan, hipStream_t s) {
  TileP pw, pd;
  PairPlan pp;
  const size_t scratch = std::min(usable_scratch(w), usable_scratch(d));
  if (w.transA != true || w.transB || d.transA || !d.transB || w.dtype != SSDT_BF16 || d.dtype != SSDT_BF16 || w.scratch != d.scratch) return hipErrorNotSupported;
  // A plan made for any amount of scratch is the one for this much if it fits: the best of more is the best of fewer that it is among.
  if (plan && plan->rows == w.K && plan->in == w.M && plan->out == w.N && plan->pair &&
      std::max(split_bytes(w.M, w.N, plan->sw), split_bytes(d.M, d.N, plan->sd)) <= half_of(scratch)) pp = *plan;
  else if (!pair_wanted(Shape{w.M, w.N, w.K}, Shape{d.M, d.N, d.K}, scratch, &pp)) return hipErrorNotSupported;
  bool big_w, big_d;
  hipError_t e = prepare(w, &pw, &big_w);
  if (e == hipSuccess) e = prepare(d, &pd, &big_d);
  if (e != hipSuccess) return e;
  if (big_w || big_d) return hipErrorNotSupported;  // (each by itself)
  if (g_tile_cfg >= 0) pp.cfg = g_tile_cfg;
  if (pp.cfg != kWide && !kPairCost[pp.cfg].fit) return hipErrorNotSupported;  // (pinned)
  if (g_tile_splits > 0) {
    const int sw = pinned_splits(false), sd = pinned_splits(true);
    if (std::max(split_bytes(pw.M, pw.N, sw), split_bytes(pd.M, pd.N, sd)) <= half_of(scratch)) { pp.sw = sw; pp.sd = sd; }
  }
  if (pp.cfg == kWide) pp.sw = pp.sd = 1;
  choose(&pw, pp.cfg, pp.sw, (float *)w.scratch);
  choose(&pd, pp.cfg, pp.sd, (float *)((char *)w.scratch + half_of(scratch)));
  switch (pp.cfg) {
    case 0: return launch_pair<128, 128, 2, false>(pw, pd, s);
    case 1: return launch_pair<64, 128, 2, false>(pw, pd, s);
    case 2: return launch_pair<64, 64, 2, false>(pw, pd, s);
    case 3:
      // Eight wavefronts on a tile are no help in the second round of two workgroups to a unit: from 960 workgroups on four took 0.98 of their time
      // on average over 57 linears (512 x 2880 -> 2880 35.8 -> 32.0 us, 512 x 2752 -> 2752 33.4 -> 31.2); below 896, 124 linears, eight are the better
      // by 2 % on average.
      if (blocks_of(pw) + blocks_of(pd) >= 960) return launch_pair<64, 128, 3, false, 4>(pw, pd, s);
      return launch_pair<64, 128, 3, false>(pw, pd, s);
    case 4: return launch_pair<64, 64, 3, false>(pw, pd, s);
    case 7: return launch_pair<32, 64, 3, true>(pw, pd, s);
    case 8: return launch_pair<32, 32, 4, true>(pw, pd, s);
    default: return launch_wide_pair(pw, pd, s);
  }
}

}  // namespace k
}  // namespace ssdt
