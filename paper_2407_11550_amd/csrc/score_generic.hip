// Observation-window scoring (Alg. 2 lines 1-5, group mean of Section 3.5) in 32 bits, on the fp32 matrix instruction
// or, for fp32 inputs with many window rows, with fp32 products made of bf16 ones: fp32 inputs and every shape the
// 16-bit matrix kernels do not take.  It also hosts the two small
// kernels both paths share (the combination of partial softmax statistics, and the max-pool).
//
// The softmax of Alg. 2 l.3 needs each window row's denominator before rows can be added up,
// so the keys are swept twice: once for per-row (max, sum of exp) and once for the normalised
// weights.
#include <math.h>

#include <type_traits>

#include "common.h"

namespace adakv {

namespace {

constexpr int ROW_TILE = 16;   // window rows staged in LDS at a time

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int PER16 = 4;
  static __device__ __forceinline__ void unpack(const uint4 &v, float *o) {
    o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y);
    o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
  }
};
struct bf16_t { unsigned short bits; };
template <> struct Elem<bf16_t> {
  static constexpr int PER16 = 8;
  static __device__ __forceinline__ void unpack(const uint4 &v, float *o) {
    const unsigned a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(a[i] << 16);
      o[2 * i + 1] = __uint_as_float(a[i] & 0xFFFF0000u);
    }
  }
};

struct f16_t { unsigned short bits; };
template <> struct Elem<f16_t> {
  static constexpr int PER16 = 8;
  static __device__ __forceinline__ void unpack(const uint4 &v, float *o) {
    const unsigned a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(a[i] & 0xFFFFu));
      o[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (unsigned short)(a[i] >> 16));
    }
  }
};

template <typename T, int D>
__device__ __forceinline__ void load_row(const T *p, float *o) {
  constexpr int P = Elem<T>::PER16;
  const uint4 *v = reinterpret_cast<const uint4 *>(p);
#pragma unroll
  for (int i = 0; i < D / P; ++i) Elem<T>::unpack(v[i], o + i * P);
}

// Stage rows [r0, r0 + ROW_TILE) of one KV head's g*w window queries as fp32 in LDS.
template <typename T, int D>
__device__ __forceinline__ void stage_q(const T *qhead, int r0, int R, float (*qs)[D]) {
  for (int i = threadIdx.x; i < ROW_TILE * D; i += 256) {
    const int r = i / D, e = i % D;
    float v = 0.0f;
    if (r0 + r < R) {
      float tmp[Elem<T>::PER16];
      const T *src = qhead + (size_t)(r0 + r) * D + (e / Elem<T>::PER16) * Elem<T>::PER16;
      Elem<T>::unpack(*reinterpret_cast<const uint4 *>(src), tmp);
      v = tmp[e % Elem<T>::PER16];
    }
    qs[r][e] = v;
  }
}

template <int D>
__device__ __forceinline__ float logit(const float *qrow, const float *k, float scale) {
  float acc = 0.0f;
#pragma unroll
  for (int e = 0; e < D; ++e) acc = fmaf(qrow[e], k[e], acc);
  return acc * scale;
}

// ---- both sweeps in 32-bit arithmetic on the matrix cores --------------------------------------
//
// v_mfma_f32_32x32x2_f32 multiplies and accumulates in fp32, 64 fused multiply-adds per cycle and
// SIMD: twice the rate of the vector ALUs (packed fp32 is not used here) and no LDS operand per
// multiply-add.  The kernels are bound by it: 2 g w d h n flops per sweep at the 154 TFLOP/s that
// an fp32 matrix product reaches on this part.
//
// A wavefront keeps 32 keys in registers for its whole life (d/2 words per lane, straight from
// memory: every byte of K is read once per sweep) and the window rows stream past them through
// LDS, 32 at a time, converted to fp32 on the way in, one barrier per row block.  So any number
// of window rows per head works, and in sweep 2 the sum over them never leaves a lane's register.
// (Q resident and K streaming, the split of the 16-bit kernels, needs d/2 registers per 32 rows
// and wavefront in fp32, which ends at 256 rows.)  128 keys per workgroup: 8191 keys x 8 heads
// make 512 workgroups, two per compute unit; with 64 keys every workgroup would read all of Q for
// half the work.  (Sweep 1 has a form with eight wavefronts and 256 keys, which leaves half as many
// partial statistics behind; see plan_score.)  32 query heads x 32 rows over 8 KV heads, d = 128, 8191 keys, fp32: the scalar
// kernels before (one thread per key, every operand of Q an LDS broadcast) took 229 + 171 us for
// the two sweeps, these take 25 + 24 us (85 TFLOP/s, launch included).
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr int F32_KEYS = 128;                          // keys per workgroup: four wavefronts of 32 (sweep 1 also: eight)
constexpr int F32_POOL_MAX = 16;                       // largest pool radius that sweep 2 applies itself
constexpr int F32_FUSE_CHUNKS = 32;                    // most partials of a row that sweep 2 combines itself

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// The instruction gives 0 below 2^-126; this one goes down to the last subnormal (keys with weights that
// small are still ordered by them).
constexpr float EXP2_LOW = -126.0f;
__device__ __forceinline__ float exp2_small(float x) {
  const bool small = x < EXP2_LOW;
  const float y = fast_exp2(small ? x + 24.0f : x);
  return small ? y * 0x1p-24f : y;
}

// The 32 window rows r0 .. r0+31 travel memory -> registers (fetch) -> LDS as fp32 (store).  Rows
// past R are fetched from row R-1; their products are left out of every result.
template <typename T, int D, int NT>
struct RowBlock {
  static constexpr int P = Elem<T>::PER16;
  static constexpr int WORDS = 32 * D / P;             // 16-byte words of the block
  static constexpr int LD = (WORDS + NT - 1) / NT;     // per thread
  static constexpr int STRIDE = D + 4;                 // padded LDS row, in floats (16-byte aligned)
  static_assert(WORDS % NT == 0 || WORDS < NT, "the row block must split evenly over the threads");
  uint4 g[LD];
  __device__ __forceinline__ void fetch(const T *qhead, int r0, int R) {
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int wi = min((int)threadIdx.x + i * NT, WORDS - 1);
      const int row = min(r0 + wi / (D / P), R - 1);
      g[i] = *reinterpret_cast<const uint4 *>(qhead + (size_t)row * D + (wi % (D / P)) * P);
    }
  }
  __device__ __forceinline__ void store(float *buf) const {
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int wi = threadIdx.x + i * NT;
      if (WORDS < NT && wi >= WORDS) break;
      float f[P];
      Elem<T>::unpack(g[i], f);
      float *dst = buf + (wi / (D / P)) * STRIDE + (wi % (D / P)) * P;
#pragma unroll
      for (int e = 0; e < P; e += 4) *reinterpret_cast<float4 *>(dst + e) = make_float4(f[e], f[e + 1], f[e + 2], f[e + 3]);
    }
  }
};

// Sweep 1 (PASS 1): partial (reference, sum of exp2(logit - reference)) of every window row over
// the workgroup's 32 NW keys, logits in the base-2 domain.  D = K Q^T: a lane owns one window row and
// 16 keys.  Sweep 2 (PASS 2): weights summed over the rows, divided by g*w, then (pool_r >= 0) the
// max-pool.  D = Q K^T: a lane owns one key and 16 rows.  With the pool applied here a workgroup
// owns the inner 128 - 2 pool_r of its keys; pool_r < 0 leaves the pool to a kernel of its own.
//
// The operands' k index is permuted alike in both: of every two 16-byte words of a row the lower
// half of the wavefront takes the first, the upper half the second.
template <typename T, int D, int PASS, int NW, bool COMBINE>
__global__ __launch_bounds__(64 * NW) void score_f32_kernel(
    SeqTab st, ChunkTab ct, Dims dm, float c_log2, int pool_r, int lse_natural,
    const T *__restrict__ q, const T *__restrict__ K, const float *__restrict__ lse,
    float2 *__restrict__ part, int part_chunk, float *__restrict__ out) {
  typedef RowBlock<T, D, 64 * NW> RB;
  constexpr int KEYS = 32 * NW;
  constexpr int P = RB::P;
  constexpr int KW = D / (2 * P);                      // 16-byte words of a key row per lane
  __shared__ __align__(16) float qs[2][32 * RB::STRIDE];
  __shared__ float sh_a[2][NW][32], sh_b[2][NW][32];   // sweep 1: per-wavefront row statistics
  __shared__ float sh_l2[2][32];                       // sweep 2: the row block's log-sum-exp
  constexpr int SL = 2 * NW;                           // threads that share a row of the statistics combination
  __shared__ float sh_pm[COMBINE ? SL : 1][32], sh_pl[COMBINE ? SL : 1][32];
  __shared__ float sh_raw[KEYS];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const int r = PASS == 2 && pool_r > 0 ? pool_r : 0;
  const int own = KEYS - 2 * r;
  const int k0 = chunk * own - r;                      // first key of the workgroup; keys outside [0, n) are masked
  const int key = k0 + wv * 32 + l32;
  const T *qhead = q + ((size_t)b * RQ + (size_t)c * R) * D;
  const size_t lse0 = (size_t)b * RQ + (size_t)c * R;

  RB rb;
  rb.fetch(qhead, 0, R);
  float kf[KW * P];
  {
    const T *src = K + (st.tok_off[b] + min(max(key, 0), n - 1)) * dm.k_stride_tok + c * dm.k_stride_head + half * P;
#pragma unroll
    for (int s = 0; s < KW; ++s) Elem<T>::unpack(*reinterpret_cast<const uint4 *>(src + s * 2 * P), kf + s * P);
  }
  auto row_l2 = [&](int row) {                         // padding rows: +inf, their weights are exactly zero
    const float v = lse[lse0 + min(row, R - 1)];
    return row < R ? (lse_natural ? v * LOG2E : v) : INFINITY;
  };
  // COMBINE: sweep 2 combines sweep 1's partials of a row block itself (at most
  // F32_FUSE_CHUNKS of them per sequence): SL threads share a row, what they load for the next block
  // travels while this one is multiplied, and 32 threads add the SL slices up.
  static_assert(!COMBINE || PASS == 2, "the weights sweep combines");
  const int prow = tid & 31, slice = tid >> 5;
  constexpr int PB = F32_FUSE_CHUNKS / SL;             // partials per thread
  float2 pml[COMBINE ? PB : 1];
  int nch = 0;
  size_t part0 = 0;
  if (COMBINE) {
    for (int i = 0; i < b; ++i) part0 += (st.n[i] + part_chunk - 1) / part_chunk;
    nch = (n + part_chunk - 1) / part_chunk;
  }
  auto load_partials = [&](int r0) {
#pragma unroll
    for (int u = 0; u < (COMBINE ? PB : 0); ++u)
      pml[u] = part[(part0 + min(slice + u * SL, nch - 1)) * RQ + (size_t)c * R + min(r0 + prow, R - 1)];
  };
  auto fold_partials = [&]() {
    float M = -INFINITY, L = 0.0f;
#pragma unroll
    for (int u = 0; u < (COMBINE ? PB : 0); ++u)
      if (slice + u * SL < nch) M = fmaxf(M, pml[u].x);
    const float ref = (M == -INFINITY) ? 0.0f : M;
#pragma unroll
    for (int u = 0; u < (COMBINE ? PB : 0); ++u)
      if (slice + u * SL < nch) L += pml[u].y * fast_exp2(pml[u].x - ref);
    sh_pm[slice][prow] = M;
    sh_pl[slice][prow] = L;
  };
  rb.store(qs[0]);
  if (COMBINE) {
    load_partials(0);
    fold_partials();
  } else if (PASS == 2 && tid < 32) {
    sh_l2[0][tid] = row_l2(tid);
  }
  __syncthreads();

  float total = 0.0f;
  const int blocks = (R + 31) / 32;
  for (int ib = 0; ib < blocks; ++ib) {
    const int cur = ib & 1;
    const bool more = ib + 1 < blocks;
    float next_l2 = 0.0f;
    if (COMBINE && tid < 32) {
      float M = sh_pm[0][tid];
#pragma unroll
      for (int i = 1; i < SL; ++i) M = fmaxf(M, sh_pm[i][tid]);
      const float ref = (M == -INFINITY) ? 0.0f : M;
      float L = 0.0f;
#pragma unroll
      for (int i = 0; i < SL; ++i) L += sh_pl[i][tid] * fast_exp2(sh_pm[i][tid] - ref);
      sh_l2[cur][tid] = ib * 32 + tid < R ? M + __builtin_amdgcn_logf(L) : INFINITY;
    }
    if (more) {
      rb.fetch(qhead, (ib + 1) * 32, R);
      if (COMBINE) load_partials((ib + 1) * 32);
      else if (PASS == 2 && tid < 32) next_l2 = row_l2((ib + 1) * 32 + tid);
    }
    // two chains of d/2 multiply-adds instead of one of d: the rounding of a logit follows the longest
    floatx16 acc = {0}, acc1 = {0};
    const float *qrow = qs[cur] + l32 * RB::STRIDE + half * P;
#pragma unroll
    for (int s = 0; s < KW; ++s) {
#pragma unroll
      for (int e = 0; e < P; e += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(qrow + s * 2 * P + e);
        const float qv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          floatx16 &a = (i & 1) ? acc1 : acc;
          a = PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s * P + e + i], qv[i], a, 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_32x32x2f32(qv[i], kf[s * P + e + i], a, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] += acc1[i];
    if (PASS == 1) {
      // acc[i]: key k0 + wv*32 + 8*(i/4) + 4*half + i%4, window row ib*32 + l32
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc[i] = (k0 + wv * 32 + 8 * (i / 4) + 4 * half + i % 4 < n) ? acc[i] * c_log2 : -INFINITY;
        m = fmaxf(m, acc[i]);
      }
      m = fmaxf(m, __shfl_xor(m, 32));
      const float ref = (m == -INFINITY) ? 0.0f : m;
      float l = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) l += fast_exp2(acc[i] - ref);
      l += __shfl_xor(l, 32);
      if (half == 0) { sh_a[cur][wv][l32] = m; sh_b[cur][wv][l32] = l; }
    } else {
      if (COMBINE) __syncthreads();                    // the log-sum-exp above; and the slices have been read
      // acc[i]: window row ib*32 + 8*(i/4) + 4*half + i%4, key k0 + wv*32 + l32
      const float *l2 = sh_l2[cur] + 4 * half;
      const float before = total;
      bool careful = ib * 32 + 32 > R;                 // padding rows (row R-1 once more, and an infinite logit
      if (!careful) {                                  // against their infinite log-sum-exp would be a NaN)
        float low = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float x = fmaf(acc[i], c_log2, -l2[8 * (i / 4) + i % 4]);
          low = fminf(low, x);
          total += fast_exp2(x);
        }
        careful = __any(low < EXP2_LOW);               // weights below the normal range
      }
      if (careful) {
        total = before;
#pragma unroll
        for (int j = 0; j < 16; j += 4) {
          if (ib * 32 + 2 * j >= R) break;
#pragma unroll
          for (int i = j; i < j + 4; ++i) {
            const float w = exp2_small(fmaf(acc[i], c_log2, -l2[8 * (i / 4) + i % 4]));
            total += ib * 32 + 8 * (i / 4) + 4 * half + i % 4 < R ? w : 0.0f;
          }
        }
      }
    }
    if (more) {
      rb.store(qs[cur ^ 1]);
      if (COMBINE) fold_partials();
      else if (PASS == 2 && tid < 32) sh_l2[cur ^ 1][tid] = next_l2;
    }
    __syncthreads();
    // (the buffers of this row block are written again two barriers from here)
    if (PASS == 1 && tid < 32 && ib * 32 + tid < R) {
      float M = sh_a[cur][0][tid];
#pragma unroll
      for (int i = 1; i < NW; ++i) M = fmaxf(M, sh_a[cur][i][tid]);
      const float ref = (M == -INFINITY) ? 0.0f : M;
      float L = 0.0f;
#pragma unroll
      for (int i = 0; i < NW; ++i) L += sh_b[cur][i][tid] * fast_exp2(sh_a[cur][i][tid] - ref);
      part[(size_t)blockIdx.x * RQ + (size_t)c * R + ib * 32 + tid] = make_float2(M, L);
    }
  }
  if (PASS == 2) {
    total += __shfl_xor(total, 32);
    const float raw = total * (1.0f / (float)R);
    float *dst = out + st.score_off[b] + (size_t)c * n;
    if (pool_r < 0) {
      if (half == 0 && key < n) dst[key] = raw;
      return;
    }
    // (a window that leaves the sequence takes the key at its end more than once: the same maximum, and
    // scores that are NaN stay so)
    if (half == 0) sh_raw[wv * 32 + l32] = raw;
    __syncthreads();
    const int lo = max(-k0, 0), hi = min(KEYS, n - k0) - 1;
    if (tid < own && k0 + r + tid < n) {
      float m = sh_raw[min(max(tid, lo), hi)];
      for (int t = 1; t <= 2 * r; ++t) m = fmaxf(m, sh_raw[min(max(tid + t, lo), hi)]);
      dst[k0 + r + tid] = m;
    }
  }
}

// ---- the same, with every fp32 product made of bf16 products ---------------------------------------
//
// An fp32 value is the sum of three bf16 values of 8 bits each (rounded to nearest, x = h + m + l without a
// rest), so a product of two is nine products of 16-bit values, each exact in fp32, on instructions sixteen times as
// fast as v_mfma_f32_32x32x2_f32.  Six are taken (hh, hm, mh, hl, lh, mm).  A second part is at most 2^-8 of a value, a
// third 2^-17, so ml and lm, the larger of those left out, are below 2^-25 each and all three below 2^-24 of the whole: no
// more than fp32 rounds a product by.  The five small ones have an accumulator of their own, so that a logit
// is rounded at its own size 8 times where d = 128, and not 64: error against 64 bits 8191 keys x 8 heads, 128 rows
// 6.7e-7 -> 4.7e-7, 16384 7.9e-7 -> 5.4e-7, d = 64, 64 rows, 16000 keys 8.1e-7 -> 6.6e-7.
// What 16-bit parts cannot hold goes through the fp32 instruction, for the keys and rows concerned: values from
// 2^60 on, infinities among them (an infinite part times a part that is zero would be a NaN, and products could
// overflow with different signs).  At the other end a part may lie below bf16's range and be lost, less than 2^-126 of a
// value (2^-134 with subnormal parts), at most 2 * 128 * 2^-126 * 2^60 = 2^-58 of a sum of products: a logit moves by
// less than 2^-27 up to a scale of 2^30, beyond which the caller gets the fp32 instruction (f32_cut()).
//
// Keys, rows and workgroups as above.  A row block's matrix instructions (48 at d = 128) are issued with other work in
// between: the exponentials of the block before, a stage of a value at a time, and the cut of the next block's rows,
// which were fetched a block before that.  Bound by these (two wavefronts of a SIMD take 2.3 us of sweep 1 and 2.75 of
// sweep 2 for a row block each, of which the matrix instructions are 1.3; one alone takes 1.3 to 1.5, with 0.65) and, with
// few row blocks, by K, which has to be there before the first block is done (34 MB of 8191 keys x 8 heads: 6.7 us).  A
// wavefront with values that are not cut takes 2.6 times as long.
// Kernel times in us, fp32 instruction / this, statistics + weights, d = 128: 8191 keys x 8 heads, 128 rows 23 + 25.5 /
// 19 + 20; 16384 45 + 50 / 32 + 31.5; 4000, 512 rows 43.5 + 45.5 / 31 + 32; 1500, 64 rows 8.5 + 9.7 / 8.0 + 9.2.  (Few rows
// keep the fp32 instruction: f32_cut().)
constexpr int PARTS = 3;
constexpr float CUT_MOST = 0x1p60f;                    // values of this size and more are not cut into parts
constexpr float CUT_MOST_SCALE = 0x1p30f;              // with larger scales of the logits nothing is
constexpr int PANEL = 2048;                            // rows whose log-sum-exp sweep 2 keeps at a time
constexpr float LOW_MID = -138.0f, LOW_WIDE = 13.0f;   // exponents of subnormal results (-150 to -126) lie this near to that
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
__device__ __forceinline__ floatx16 mfma_bf16(const uint4 &a, const uint4 &b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two values on their way through the parts, a stage each; most: the larger magnitude (a NaN does not count: its
// first part is one).
struct Pair {
  float a, b, most;
  __device__ __forceinline__ void begin(const uint4 *raw, int k) {
    float x[8];
    Elem<float>::unpack(raw[0], x);
    Elem<float>::unpack(raw[1], x + 4);
    a = x[2 * k];
    b = x[2 * k + 1];
    most = fmaxf(fabsf(a), fabsf(b));
  }
  __device__ __forceinline__ unsigned stage(int p) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const unsigned v = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
    if (p < PARTS - 1) {
      a -= __uint_as_float(v << 16);
      b -= __uint_as_float(v & 0xFFFF0000u);
    }
    return v;
  }
};
// Eight elements of a row as operand words of the matrix instructions, one word per part; the largest magnitude.
__device__ __forceinline__ float cut8(const uint4 *raw, uint4 (&o)[PARTS]) {
  unsigned w[PARTS][4];
  float most = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    Pair x;
    x.begin(raw, k);
    most = fmaxf(most, x.most);
#pragma unroll
    for (int p = 0; p < PARTS; ++p) w[p][k] = x.stage(p);
  }
#pragma unroll
  for (int p = 0; p < PARTS; ++p) o[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
  return most;
}

// The 32 window rows r0 .. r0+31 travel memory -> registers (fetch) -> LDS, cut into operand words of eight values, a
// word per part (store).  Rows past R are fetched from row R-1; their products are left out of every result.
template <int D, int NT>
struct CutRows {
  static constexpr int ROW8 = D / 8;                   // operand words per row and part
  static constexpr int WORDS = 32 * ROW8;
  static constexpr int LD = (WORDS + NT - 1) / NT;     // of them per thread
  static constexpr int STRIDE = ROW8 + 1;              // padded LDS row, in words
  static constexpr int PART = 32 * STRIDE;
  static_assert(WORDS % NT == 0 || WORDS < NT, "the row block must split evenly over the threads");
  uint4 g[LD][2];
  __device__ __forceinline__ void fetch(int i, const float *qhead, int r0, int R) {
    const unsigned wi = min(threadIdx.x + i * NT, (unsigned)WORDS - 1u);
    const unsigned at = min(r0 + wi / ROW8, (unsigned)R - 1u) * (D * 4u) + wi % ROW8 * 32u;
    const uint4 *src = reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(qhead) + at);
    g[i][0] = src[0];
    g[i][1] = src[1];
  }
  // In STEPS: a stage of two elements each, then the word's store.  Rows with values that cannot be cut are marked with
  // the row block's number (marks of other blocks mean nothing).
  static constexpr int PER = 4 * PARTS, STEPS = PER * LD;
  unsigned w[PARTS][4];
  float most;
  Pair x;
  __device__ __forceinline__ void store(int step, uint4 *buf, int *mark, int block) {
    const int i = step / PER, k = step % PER / PARTS, p = step % PARTS, wi = threadIdx.x + i * NT;
    if (p == 0) {
      x.begin(g[i], k);
      most = k == 0 ? x.most : fmaxf(most, x.most);
      asm volatile("" : "+v"(most));                   // (a step's work stays where it is called)
    }
    w[p][k] = x.stage(p);
    asm volatile("" : "+v"(w[p][k]));
    if (step % PER < PER - 1 || (WORDS < NT && wi >= WORDS)) return;
    if (most >= CUT_MOST) mark[wi / ROW8] = block;
#pragma unroll
    for (int o = 0; o < PARTS; ++o)
      buf[o * PART + wi / ROW8 * STRIDE + wi % ROW8] = make_uint4(w[o][0], w[o][1], w[o][2], w[o][3]);
  }
};

// The same 32 x 32 logits by the fp32 instruction, straight from memory: of every two 16-byte words of a row the
// lower half of the wavefront takes the first, the upper half the second, in both operands.
template <int D, bool KEYS_FIRST>
__device__ __forceinline__ floatx16 fp32_products(const float *krow, const float *qrow, int half) {
  floatx16 acc = {0}, acc1 = {0};
#pragma unroll 1
  for (int s = 0; s < D / 8; ++s) {
    float k[4], q[4];
    Elem<float>::unpack(*reinterpret_cast<const uint4 *>(krow + s * 8 + half * 4), k);
    Elem<float>::unpack(*reinterpret_cast<const uint4 *>(qrow + s * 8 + half * 4), q);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      floatx16 &a = (i & 1) ? acc1 : acc;
      a = KEYS_FIRST ? __builtin_amdgcn_mfma_f32_32x32x2f32(k[i], q[i], a, 0, 0, 0)
                     : __builtin_amdgcn_mfma_f32_32x32x2f32(q[i], k[i], a, 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] += acc1[i];
  return acc;
}

// op of a lane's value and that of the lane 32 further, in both.
template <class Op> __device__ __forceinline__ float over_halves(float x, Op op) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// As score_f32_kernel.
template <int D, int PASS, int NW, bool COMBINE>
__global__ __launch_bounds__(64 * NW, 2) void score_cut_kernel(
    SeqTab st, ChunkTab ct, Dims dm, float c_log2, int pool_r, int lse_natural,
    const float *__restrict__ q, const float *__restrict__ K, const float *__restrict__ lse,
    float2 *__restrict__ part, int part_chunk, float *__restrict__ out) {
  typedef CutRows<D, 64 * NW> RB;
  constexpr int KEYS = 32 * NW;
  constexpr int KS = D / 16;                           // matrix instructions per row block and product
  constexpr int PRODUCTS = 6, SLOTS = KS * PRODUCTS;
  __shared__ uint4 qs[2][PARTS * RB::PART];
  __shared__ int sh_mark[2][32];                       // rows whose values could not be cut
  __shared__ float sh_a[2][NW][32], sh_b[2][NW][32];   // sweep 1: per-wavefront row statistics
  __shared__ __align__(16) float sh_l2[PASS == 2 ? PANEL : 4];     // sweep 2: the rows' log-sum-exp, PANEL rows at a time
  __shared__ float sh_raw[KEYS];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const int r = PASS == 2 && pool_r > 0 ? pool_r : 0;
  const int own = KEYS - 2 * r;
  const int k0 = chunk * own - r;                      // first key of the workgroup; keys outside [0, n) are masked
  const int key = k0 + wv * 32 + l32;
  const float *qhead = q + ((size_t)b * RQ + (size_t)c * R) * D;
  const size_t lse0 = (size_t)b * RQ + (size_t)c * R;

  RB rb;
#pragma unroll
  for (int i = 0; i < RB::LD; ++i) rb.fetch(i, qhead, 0, R);
  const float *krow = K + (st.tok_off[b] + min(max(key, 0), n - 1)) * dm.k_stride_tok + c * dm.k_stride_head;
  uint4 raw[KS][2];                                // of every 16 elements the lower half of the wavefront holds the first 8
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int k = 0; k < 2; ++k) raw[s][k] = reinterpret_cast<const uint4 *>(krow + s * 16 + half * 8)[k];
  if (tid < 64) sh_mark[tid >> 5][tid & 31] = -1;
  // Sweep 2, rows r0 .. r0 + PANEL - 1: the log-sum-exp in the base-2 domain; +inf on padding rows, whose weights
  // are exactly zero.  COMBINE: from sweep 1's partials (at most F32_FUSE_CHUNKS of them per sequence), by `share`
  // neighbouring threads a row, so that few rows keep all threads busy.
  static_assert(!COMBINE || PASS == 2, "the weights sweep combines");
  const float2 *pp = part;
  int np = 0;
  if (COMBINE) {
    size_t part0 = 0;
    for (int i = 0; i < b; ++i) part0 += (st.n[i] + part_chunk - 1) / part_chunk;
    np = (n + part_chunk - 1) / part_chunk;
    pp += part0 * RQ + (size_t)c * R;
  }
  auto panel = [&](int r0) {
    const int share = !COMBINE || R > 32 * NW ? 1 : R > 16 * NW ? 2 : R > 8 * NW ? 4 : 8;
    for (int at = tid / share; at < PANEL && r0 + (at & ~31) < R; at += 64 * NW / share) {
      const int row = min(r0 + at, R - 1);
      float v;
      if (COMBINE) {
        constexpr int CB = F32_FUSE_CHUNKS / 2;        // partials asked for at a time
        const int own = tid % share;
        float M = -INFINITY, L = 0.0f;
        auto merge = [&](float m, float l) {
          const float t = fmaxf(M, m), rf = (t == -INFINITY) ? 0.0f : t;
          L = L * fast_exp2(M - rf) + l * fast_exp2(m - rf);
          M = t;
        };
        for (int p0 = own; p0 < np; p0 += CB * share) {
          float2 ml[CB];
#pragma unroll
          for (int u = 0; u < CB; ++u) ml[u] = pp[(unsigned)min(p0 + u * share, np - 1) * (unsigned)RQ + row];
          float m = ml[0].x, l = 0.0f;
#pragma unroll
          for (int u = 1; u < CB; ++u) m = fmaxf(m, ml[u].x);
          const float rf = (m == -INFINITY) ? 0.0f : m;
#pragma unroll
          for (int u = 0; u < CB; ++u)
            if (p0 + u * share < np) l += ml[u].y * fast_exp2(ml[u].x - rf);
          merge(m, l);
        }
        for (int o = 1; o < share; o <<= 1) {
          const float m = __shfl_xor(M, o), l = __shfl_xor(L, o);
          merge(m, l);
        }
        v = M + __builtin_amdgcn_logf(L);
      } else {
        v = lse[lse0 + row] * (lse_natural ? LOG2E : 1.0f);
      }
      if (!COMBINE || tid % share == 0) sh_l2[at] = r0 + at < R ? v : INFINITY;
    }
  };
  __syncthreads();                                     // the marks are cleared
#pragma unroll
  for (int i = 0; i < RB::STEPS; ++i) rb.store(i, qs[0], sh_mark[0], 0);
  if (R > 32) {
#pragma unroll
    for (int i = 0; i < RB::LD; ++i) rb.fetch(i, qhead, 32, R);
  }
  if (PASS == 2) panel(0);
  __syncthreads();

  // The loop over row blocks: a block's matrix instructions are issued with the vector work on the block before in
  // between (SLOTS of them, a value in every SLOTS/16 or several in one), in the first block with the keys' cut,
  // as they arrive.  One barrier a block.
  uint4 kf[KS][PARTS];
  float most = 0.0f;
  unsigned big_keys = 0u;                              // keys whose values could not be cut
  const int blocks = (R + 31) / 32;
  const bool whole = k0 + wv * 32 + 32 <= n;           // (sweep 1: k0 >= 0) no key to mask
  floatx16 prev;                                       // products of the block before
  float total = 0.0f, before = 0.0f, low = 0.0f, kept = 0.0f;      // sweep 2
  float ref = 0.0f, top = 0.0f, usum = 0.0f;           // sweep 1
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 l2[4];
  // sweep 1: prev[i] is key k0 + wv*32 + 8*(i/4) + 4*half + i%4, window row pb*32 + l32; sweep 2: window row
  // pb*32 + 8*(i/4) + 4*half + i%4, key k0 + wv*32 + l32
  auto begin = [&](int pb) {
    if (PASS == 1) {
      if (!whole) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (k0 + wv * 32 + 8 * (i / 4) + 4 * half + i % 4 >= n) prev[i] = -INFINITY;
      }
      float m = prev[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) m = fmaxf(m, prev[i]);
      m = over_halves(m, [](float x, float y) { return fmaxf(x, y); });
      top = m * c_log2;
      ref = (top == -INFINITY) ? 0.0f : top;
      usum = 0.0f;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) l2[i] = *reinterpret_cast<const f32x4 *>(&sh_l2[pb * 32 % PANEL + 8 * i + 4 * half]);
      before = total;
      low = INFINITY;
    }
  };
  // One value in three stages, so that none waits for the one before: exponent, exponential, sum.
  float x[2], e = 0.0f;
  auto exponent = [&](int i) {
    if (PASS == 1) {
      x[i & 1] = fmaf(prev[i], c_log2, -ref);
    } else {
      x[i & 1] = fmaf(prev[i], c_log2, -l2[i / 4][i % 4]);
      low = fminf(low, fabsf(x[i & 1] - LOW_MID));
      asm volatile("" : "+v"(low));
    }
    asm volatile("" : "+v"(x[i & 1]));                 // (stays between the matrix instructions)
  };
  auto exponential = [&](int i) {
    e = fast_exp2(x[i & 1]);
    asm volatile("" : "+v"(e));
  };
  auto sum = [&]() {
    float &s = PASS == 1 ? usum : total;
    s += e;
    asm volatile("" : "+v"(s));
  };
  auto value = [&](int i) {
    exponent(i);
    exponential(i);
    sum();
  };
  auto end = [&](int pb) {
    if (PASS == 1) {
      const float l = over_halves(usum, [](float x, float y) { return x + y; });
      if (half == 0) { sh_a[pb & 1][wv][l32] = top; sh_b[pb & 1][wv][l32] = l; }
    } else if (pb * 32 + 32 > R || __any(low <= LOW_WIDE)) {
      // padding rows (row R-1 once more, and an infinite logit against their infinite log-sum-exp would be a NaN), or
      // weights below the normal range
      total = before;
#pragma unroll
      for (int j = 0; j < 16; j += 4) {
        if (pb * 32 + 2 * j >= R) break;
#pragma unroll
        for (int i = j; i < j + 4; ++i) {
          const float w = exp2_small(fmaf(prev[i], c_log2, -l2[i / 4][i % 4]));
          total += pb * 32 + 8 * (i / 4) + 4 * half + i % 4 < R ? w : 0.0f;
        }
      }
    }
  };
  auto file = [&](int pb) {                            // sweep 1: the wavefronts' statistics of a block together
    if (PASS == 1 && wv == pb % NW && half == 0 && pb * 32 + l32 < R) {
      const int at = pb & 1;
      float M = sh_a[at][0][l32];
#pragma unroll
      for (int i = 1; i < NW; ++i) M = fmaxf(M, sh_a[at][i][l32]);
      const float rf = (M == -INFINITY) ? 0.0f : M;
      float L = 0.0f;
#pragma unroll
      for (int i = 0; i < NW; ++i) L += sh_b[at][i][l32] * fast_exp2(sh_a[at][i][l32] - rf);
      part[(size_t)blockIdx.x * RQ + (size_t)c * R + pb * 32 + l32] = make_float2(M, L);
    }
  };
  auto block = [&](int ib, auto first_tag) {
    constexpr bool FIRST = decltype(first_tag)::value;
    const int cur = ib & 1;
    const uint4 *qrow = qs[cur] + l32 * RB::STRIDE + half;
    uint4 qv[2][PARTS];                             // operand words of this step and the next
#pragma unroll
    for (int p = 0; p < PARTS; ++p) qv[0][p] = qrow[p * RB::PART];
    int mark = 0;
    if (FIRST) most = cut8(raw[0], kf[0]);
    else begin(ib - 1);
    floatx16 acc = {0}, small = {0};
    auto add = [&](floatx16 &a, const uint4 &k, const uint4 &qv) { a = PASS == 1 ? mfma_bf16(k, qv, a) : mfma_bf16(qv, k, a); };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int t = 0; t < PRODUCTS; ++t) {
        const uint4 (&v)[PARTS] = qv[s & 1];
        if (t == PRODUCTS - 1) add(acc, kf[s][0], v[0]);
        else if (t == 0) add(small, kf[s][PARTS - 1], v[0]);
        else if (t == 1) add(small, kf[s][1], v[1]);
        else if (t == 2) add(small, kf[s][0], v[PARTS - 1]);
        else if (t == 3) add(small, kf[s][1], v[0]);
        else add(small, kf[s][0], v[1]);
        if (t == 0 && s + 1 < KS) {
#pragma unroll
          for (int p = 0; p < PARTS; ++p) qv[(s + 1) & 1][p] = qrow[p * RB::PART + 2 * (s + 1)];
        }
        const int slot = s * PRODUCTS + t;
        if constexpr (FIRST) {
          if (t == PRODUCTS / 2 && s + 1 < KS) most = fmaxf(most, cut8(raw[s + 1], kf[s + 1]));
        } else {
#pragma unroll
          for (int i = slot * 16 / SLOTS; i < (slot + 1) * 16 / SLOTS; ++i) {
            if (i > 1) sum();
            if (i > 0) exponential(i - 1);
            exponent(i);
          }
        }
        // the next block's rows, fetched a block ago, and then the fetch of those after it
        constexpr int LAST = SLOTS - 1;
#pragma unroll
        for (int i = 0; i < RB::STEPS; ++i)
          if (slot == min(1 + i * (SLOTS - 4) / RB::STEPS, LAST) && (!FIRST || blocks > 1)) {
            rb.store(i, qs[cur ^ 1], sh_mark[cur ^ 1], ib + 1);
            if (i % RB::PER == RB::PER - 1) rb.fetch(i / RB::PER, qhead, (ib + 2) * 32, R);
          }
        if (slot == SLOTS / 2) mark = sh_mark[cur][l32];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (!FIRST) {
      sum();
      exponential(15);
      sum();
      end(ib - 1);
    }
    if (PASS == 2 && !FIRST && ib * 32 % PANEL == 0) total = kept;
    const unsigned big_rows = (unsigned)__ballot(mark == ib);
    if (FIRST) {
      const unsigned long long big = __ballot(most >= CUT_MOST);
      big_keys = (unsigned)(big >> 32) | (unsigned)big;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) prev[i] = acc[i] + small[i];
    if (__builtin_expect((big_keys | big_rows) != 0u, 0)) {
      const floatx16 exact = fp32_products<D, PASS == 1>(krow, qhead + (size_t)min(ib * 32 + l32, R - 1) * D, half);
      const unsigned col = (PASS == 1 ? big_rows : big_keys) >> l32 & 1u, rows = PASS == 1 ? big_keys : big_rows;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (col | (rows >> (8 * (i / 4) + 4 * half + i % 4) & 1u)) prev[i] = exact[i];
    }
    __syncthreads();
    // (the buffers of this row block are written again two barriers from here)
    if (!FIRST) file(ib - 1);
    if (PASS == 2 && (ib + 1) * 32 % PANEL == 0 && ib + 1 < blocks) {
      // the panel's last block gets its vector work here, what the next block does once more is thrown away
      begin(ib);
#pragma unroll
      for (int i = 0; i < 16; ++i) value(i);
      end(ib);
      kept = total;
      __syncthreads();
      panel((ib + 1) * 32);
      __syncthreads();
    }
  };
  block(0, std::true_type{});
  for (int ib = 1; ib < blocks; ++ib) block(ib, std::false_type{});
  begin(blocks - 1);
#pragma unroll
  for (int i = 0; i < 16; ++i) value(i);
  end(blocks - 1);
  if (PASS == 1) {
    __syncthreads();
    file(blocks - 1);
  }
  if (PASS == 2) {
    total += __shfl_xor(total, 32);
    const float mean = total * (1.0f / (float)R);
    float *dst = out + st.score_off[b] + (size_t)c * n;
    if (pool_r < 0) {
      if (half == 0 && key < n) dst[key] = mean;
      return;
    }
    // (a window that leaves the sequence takes the key at its end more than once: the same maximum, and
    // scores that are NaN stay so)
    if (half == 0) sh_raw[wv * 32 + l32] = mean;
    __syncthreads();
    const int lo = max(-k0, 0), hi = min(KEYS, n - k0) - 1;
    if (tid < own && k0 + r + tid < n) {
      float m = sh_raw[min(max(tid, lo), hi)];
      for (int t = 1; t <= 2 * r; ++t) m = fmaxf(m, sh_raw[min(max(tid + t, lo), hi)]);
      dst[k0 + r + tid] = m;
    }
  }
}

// The other order of Alg. 2 l.4 (as printed there): every window row is max-pooled along the keys
// first, then the g*w rows of the head are averaged.  A block scores 256 consecutive keys and owns
// the middle 256 - 2*radius of them, so that every owned key finds its pool window in LDS; keys
// outside the sequence count as weight 0, which a max over non-negative weights never picks.
template <typename T, int D>
__global__ __launch_bounds__(256) void pooled_generic_kernel(
    SeqTab st, ChunkTab ct, Dims dm, const T *__restrict__ q, const T *__restrict__ K,
    const float *__restrict__ lse, float *__restrict__ scores) {
  __shared__ float qs[ROW_TILE][D];
  __shared__ float sl[ROW_TILE];
  __shared__ float ps[ROW_TILE][256];
  const int tid = threadIdx.x;
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const int r = dm.pool_k / 2, own = 256 - 2 * r;      // the launcher guarantees own >= 1
  const int j = chunk * own - r + tid;                 // the key this thread scores
  const bool valid = j >= 0 && j < n;
  const bool owner = tid >= r && tid < 256 - r && j < n;
  float k[D];
  if (valid) {
    load_row<T, D>(K + (st.tok_off[b] + j) * dm.k_stride_tok + c * dm.k_stride_head, k);
  } else {
#pragma unroll
    for (int e = 0; e < D; ++e) k[e] = 0.0f;
  }
  const T *qhead = q + ((size_t)b * RQ + (size_t)c * R) * D;
  float acc = 0.0f;
  for (int r0 = 0; r0 < R; r0 += ROW_TILE) {
    __syncthreads();                                   // the previous tile's ps and qs are done with
    stage_q<T, D>(qhead, r0, R, qs);
    if (tid < ROW_TILE) sl[tid] = (r0 + tid < R) ? lse[(size_t)b * RQ + (size_t)c * R + r0 + tid] : 0.0f;
    __syncthreads();
    const int rt = min(ROW_TILE, R - r0);
    for (int rr = 0; rr < rt; ++rr)
      ps[rr][tid] = valid ? expf(logit<D>(qs[rr], k, dm.scale) - sl[rr]) : 0.0f;
    __syncthreads();
    if (owner) {
      for (int rr = 0; rr < rt; ++rr) {
        float m = ps[rr][tid - r];
        for (int t = tid - r + 1; t <= tid + r; ++t) m = fmaxf(m, ps[rr][t]);
        acc += m;
      }
    }
  }
  if (owner) scores[st.score_off[b] + (size_t)c * n + j] = acc * (1.0f / (float)R);
}

}  // namespace

// lse[b][row] = log of the sum over the sequence's chunks of l * 2^m.  One wavefront per row:
// the lanes stride over the chunks (independent loads), then the 64 partial (max, sum) pairs are
// merged with shuffles.
// The partials' references are in the base-2 domain (rounded once instead of once more on the
// way to natural logarithms); the result is too, unless natural_out asks for the other.
__global__ __launch_bounds__(256) void lse_combine_kernel(SeqTab st, ChunkTab ct, int RQ,
                                                          const float2 *__restrict__ part,
                                                          float *__restrict__ lse, int natural_out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int b = blockIdx.y;
  if (row >= RQ) return;
  float M = -INFINITY, L = 0.0f;
  for (int k = ct.off[b] + lane; k < ct.off[b + 1]; k += 64) {
    const float2 ml = part[(size_t)k * RQ + row];
    const float m = ml.x, l = ml.y;
    const float nm = fmaxf(M, m);
    if (nm > -INFINITY) L = L * exp2f(M - nm) + l * exp2f(m - nm);
    M = nm;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float m2 = __shfl_xor(M, off), l2 = __shfl_xor(L, off);
    const float nm = fmaxf(M, m2);
    if (nm > -INFINITY) L = L * exp2f(M - nm) + l2 * exp2f(m2 - nm);
    M = nm;
  }
  if (lane == 0) {
    const float v = M + log2f(L);
    lse[(size_t)b * RQ + row] = natural_out ? v * LN2 : v;
  }
}

// scores[j] = max of raw over [j - k/2, j + k/2] clipped to the head's row (stride 1, same length).
__global__ __launch_bounds__(256) void pool_kernel(SeqTab st, ChunkTab ct, int pool_k,
                                                   const float *__restrict__ raw,
                                                   float *__restrict__ scores) {
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const int n = st.n[b];
  const int j = chunk * GEN_CHUNK + threadIdx.x;
  if (j >= n) return;
  const size_t base = st.score_off[b] + (size_t)c * n;
  const int r = pool_k / 2;
  const int lo = max(0, j - r), hi = min(n - 1, j + r);
  float m = raw[base + lo];
  for (int jj = lo + 1; jj <= hi; ++jj) m = fmaxf(m, raw[base + jj]);
  scores[base + j] = m;
}

// fp32 inputs: whether products are made of bf16 parts.  A wavefront's keys have to be cut first, which one row block of
// 128 columns or two of 64 do not bring in again.  us a call, 8 heads, fp32 instruction / parts: 8191 keys, d = 128, 32
// rows 22.9 / 25.3, 40 rows 33.5 / 31.8; d = 64, 64 rows 21.9 / 22.7, 80 rows 28.0 / 24.8; 600 keys 12.9 / 13.7, 17.8 / 17.5,
// 12.9 / 13.0, 15.9 / 14.6.  (From some 16000 keys on parts would win with fewer rows too: d = 128, 32 rows 41.4 / 37.8.)
bool f32_cut(const Dims &dm, int dtype) {
  return dtype == ADAKV_FP32 && dm.g * dm.w * dm.d > 32 * 128 && dm.scale <= CUT_MOST_SCALE;
}

static ScorePlan plan_score_chunk(const SeqTab &st, const Dims &dm, int part_chunk) {
  ScorePlan p;
  // partial statistics: one (max, sum) pair per window row and chunk of keys
  p.part_chunk = part_chunk;
  const size_t chunks = count_chunks(st, p.part_chunk);
  const size_t RQ = (size_t)dm.h_q * dm.w;
  size_t o = 0;
  p.part = o; o += align_up(chunks * RQ * 8, 256);
  p.lse = o; o += align_up((size_t)st.batch * RQ * 4, 256);
  p.raw = o; o += align_up((size_t)st.score_off[st.batch] * 4, 256);
  p.total = o;
  return p;
}

size_t score_workspace(const SeqTab &st, const Dims &dm, int part_chunk) {
  return plan_score_chunk(st, dm, part_chunk).total;
}

// Whether sweep 1 leaves a partial per 256 keys.  With 33 to 64 partials per 128 keys that makes them few enough for
// sweep 2 to combine, which saves the kernel of 4 us and costs sweep 2 1 to 1.7 us.  A workgroup of eight wavefronts
// takes as long as two of four, so the fullest compute unit may get more to do: 1.8 us per unit and row block as in
// f32_pool_fused().  Whole call, us, 128 / 256 keys: 8191 keys x 8 heads, 128 rows 53.4 / 51.4, 5000 keys 49.8 / 46.2,
// d = 64 37.4 / 34.9; 8000 x 8 heads, 8 rows 25.8 / 23.2; 8000 x 4 heads, 32 rows, d = 64 (half a compute unit's
// share more) 17.0 / 14.1.  Refused: 5000 x 4 heads, 128 rows 31.8 / 36.4; five of up to 6000 keys 107.2 / 110.0.  With
// products of parts the same layers are on either side: 8191 x 8 heads, 128 rows 39.5 / 38.5, 5000 35.5 / 33.1, 64 rows
// 28.1 / 26.5 (8191 30.7 / 31.0), d = 64, 128 rows, 5000 24.0 / 22.8; refused: 5000 x 4 heads 25.0 / 27.3, 8000 x 4 28.1 /
// 30.7, d = 64 21.9 / 23.1, five of up to 6000 x 8 75.5 / 83.6.
// The row-pooling order keeps the kernel, and half the partials help it all the same: 8191 x 8 heads, 128 rows 165.9 /
// 165.0, 5000 x 8 heads, 16 rows 35.3 / 33.7, 8000 x 8 heads, 32 rows, d = 64 37.2 / 35.9.
static bool f32_wide_stats(const SeqTab &st, const Dims &dm) {
  int longest = 0;
  for (int b = 0; b < st.batch; ++b) longest = st.n[b] > longest ? st.n[b] : longest;
  if (longest <= F32_FUSE_CHUNKS * F32_KEYS || longest > F32_FUSE_CHUNKS * 2 * F32_KEYS) return false;
  const int narrow = (count_chunks(st, F32_KEYS) * dm.h_kv + 255) / 256;
  const int wide = (count_chunks(st, 2 * F32_KEYS) * dm.h_kv + 255) / 256;
  const int row_blocks = (dm.g * dm.w + 31) / 32;
  return (2 * wide - narrow) * row_blocks * 1.8f * dm.d / 128 <= 1.5f;
}

ScorePlan plan_score(const SeqTab &st, const Dims &dm, int dtype, bool on_mfma) {
  (void)dtype;
  if (on_mfma) {
    const MfmaVariant v = choose_mfma_variant(st, dm);
    ScorePlan p = plan_score_chunk(st, dm, v.part_len);
    p.mfma = v;
    // (the Top-k's shortest form finds room here where partials of the weights sweep's chunks would have made it)
    const size_t lists = topk_spare_bytes(st, dm);
    if (lists > p.total && lists <= score_workspace(st, dm, v.len)) p.total = lists;
    return p;
  }
  // The fp32 kernels' partials are per 128 keys (workgroups of four wavefronts spread best), or per
  // 256 keys where that saves a kernel (f32_wide_stats) or the smaller ones would not fit into the built-in
  // scratch array any more: half the partials, and a sequence that long fills the chip with either.
  const ScorePlan p = plan_score_chunk(st, dm, F32_KEYS);
  const size_t spare = 1024;                           // what the callers add for alignment
  if (!f32_wide_stats(st, dm) && p.total + plan_topk_bytes(st, dm) + spare <= (size_t)ADAKV_STATIC_SCRATCH_BYTES) return p;
  return plan_score_chunk(st, dm, 2 * F32_KEYS);
}

void launch_lse_combine(const SeqTab &st, const ChunkTab &ct, int RQ, const float2 *part,
                        float *lse, hipStream_t s) {
  ADAKV_LAUNCH("score_lse_combine", lse_combine_kernel, dim3((RQ + 3) / 4, st.batch),
               dim3(256), s, st, ct, RQ, part, lse, 0);
}

void launch_pool(const SeqTab &st, const Dims &dm, const float *raw, float *scores,
                 hipStream_t s) {
  const ChunkTab ct = make_chunks(st, GEN_CHUNK);
  ADAKV_LAUNCH("score_pool", pool_kernel, dim3(ct.off[st.batch], dm.h_kv), dim3(256), s, st, ct,
               dm.pool_k, raw, scores);
}

// The pool inside sweep 2 scores 2r keys of every 128 twice; a kernel of its own takes 4 us.  A
// compute unit works through its workgroups at the rate of its matrix cores, so what the overlap
// costs is the workgroups that the fullest compute unit gets more, each 32 rows x 32 keys x d in
// every wavefront (4096 cycles = 1.8 us at d = 128) per row block.  8191 keys x 8 heads, 128 rows:
// 544 workgroups fused (three on some of the 256 compute units) 34.2 us, 512 and a pool kernel
// 24.3 + 4.1 us.
// Where the products are cut into parts two workgroups fit on a compute unit and a third makes a second round, which
// takes longer than the pool kernel however few row blocks there are (fused / apart: 64 rows, d = 128, 8000 keys x 8
// heads 33.4 / 31.0, 16000 x 4 34.0 / 31.9; 128 rows, 8191 x 8 42.8 / 38.6, 16000 x 4 43.5 / 39.9).  Fewer: 128 rows,
// 2011 x 8 23.0 / 25.4, 5000 33.2 / 35.7, 4000 29.4 / 26.4 (apart), 512 rows, 2011 53.2 / 55.5.  A second workgroup
// on a unit that had one costs more than these 1.8 us a row block, which the line does not see where there are few:
// 64 rows, 4000 x 8 23.8 / 21.5 and, d = 64, 128 rows 20.8 / 19.9 are fused.
bool f32_pool_fused(const SeqTab &st, const Dims &dm, int dtype) {
  const int r = dm.pool_k / 2;
  if (r == 0 || r > F32_POOL_MAX) return r == 0;
  const int most = (count_chunks(st, F32_KEYS - 2 * r) * dm.h_kv + 255) / 256;
  const int most_apart = (count_chunks(st, F32_KEYS) * dm.h_kv + 255) / 256;
  if (f32_cut(dm, dtype) && (most + 1) / 2 > (most_apart + 1) / 2) return false;
  const int row_blocks = (dm.g * dm.w + 31) / 32;
  return (most - most_apart) * row_blocks * 1.8f * dm.d / 128 <= 4.0f;
}

bool f32_lse_fused(const SeqTab &st, int part_chunk) {
  for (int b = 0; b < st.batch; ++b)
    if ((st.n[b] + part_chunk - 1) / part_chunk > F32_FUSE_CHUNKS) return false;
  return true;
}

template <typename T, int D>
static void run_generic(const SeqTab &st, const Dims &dm, const void *q, const void *K,
                        const float *row_lse, float *scores, char *ws, const ScorePlan &pl,
                        bool pool_first, hipStream_t s) {
  const float c_log2 = dm.scale * LOG2E;
  const dim3 block(256);
  float2 *part = (float2 *)(ws + pl.part);
  float *lse = (float *)(ws + pl.lse), *raw = (float *)(ws + pl.raw);
  const float *use_lse = row_lse;
  const int dtype = std::is_same<T, float>::value ? ADAKV_FP32 : ADAKV_BF16;
  const bool cut = f32_cut(dm, dtype);
  if (!row_lse) {
    const ChunkTab ct = make_chunks(st, pl.part_chunk);
    const dim3 grid(ct.off[st.batch], dm.h_kv);
#define ADAKV_GO(KERNEL, NW)                                                                      \
  ADAKV_LAUNCH("score_stats_fma", KERNEL, grid, dim3(64 * NW), s, st, ct, dm, c_log2, -1, 0, (const T *)q, \
               (const T *)K, (const float *)nullptr, part, pl.part_chunk, (float *)nullptr)
    const bool narrow = pl.part_chunk == F32_KEYS;
    if constexpr (std::is_same<T, float>::value) {
      if (cut && narrow) ADAKV_GO((score_cut_kernel<D, 1, 4, false>), 4);
      else if (cut) ADAKV_GO((score_cut_kernel<D, 1, 8, false>), 8);
    }
    if (!cut && narrow) ADAKV_GO((score_f32_kernel<T, D, 1, 4, false>), 4);
    else if (!cut) ADAKV_GO((score_f32_kernel<T, D, 1, 8, false>), 8);
#undef ADAKV_GO
    // Up to 32 partials per row (4096 keys) sweep 2 combines them itself, a launch of 4 us less: 2011
    // keys x 8 heads x 128 rows 33.0 -> 29.0 us for both sweeps, 4000 x 512 rows 100.1 -> 97.5; with 64
    // partials its workgroups read more of those than of keys (8000 x 4 heads x 512 rows, d = 64: 65.6 -> 67.6).
    if (pool_first || !f32_lse_fused(st, pl.part_chunk)) {
      const int RQ = dm.h_q * dm.w;
      ADAKV_LAUNCH("score_lse_combine", lse_combine_kernel, dim3((RQ + 3) / 4, st.batch), block, s,
                   st, ct, RQ, (const float2 *)part, lse, pool_first ? 1 : 0);
      use_lse = lse;
    }
  }
  if (pool_first) {
    const ChunkTab co = make_chunks(st, 256 - 2 * (dm.pool_k / 2));
    ADAKV_LAUNCH("score_pooled_fma", (pooled_generic_kernel<T, D>), dim3(co.off[st.batch], dm.h_kv),
                 block, s, st, co, dm, (const T *)q, (const T *)K, use_lse, scores);
    return;
  }
  const int r = dm.pool_k / 2;
  const bool fused = f32_pool_fused(st, dm, dtype);
  const ChunkTab ct = make_chunks(st, fused ? F32_KEYS - 2 * r : F32_KEYS);
  const dim3 grid(ct.off[st.batch], dm.h_kv);
#define ADAKV_GO(KERNEL)                                                                          \
  ADAKV_LAUNCH("score_weights_fma", KERNEL, grid, block, s, st, ct, dm, c_log2, fused ? r : -1, row_lse ? 1 : 0, \
               (const T *)q, (const T *)K, use_lse, part, pl.part_chunk, fused ? scores : raw)
  if constexpr (std::is_same<T, float>::value) {
    if (cut && use_lse) ADAKV_GO((score_cut_kernel<D, 2, 4, false>));
    else if (cut) ADAKV_GO((score_cut_kernel<D, 2, 4, true>));
  }
  if (!cut && use_lse) ADAKV_GO((score_f32_kernel<T, D, 2, 4, false>));
  else if (!cut) ADAKV_GO((score_f32_kernel<T, D, 2, 4, true>));
#undef ADAKV_GO
  if (!fused) launch_pool(st, dm, raw, scores, s);
}

hipError_t launch_score_generic(const SeqTab &st, const Dims &dm, int dtype, const void *q,
                                const void *K, const float *row_lse, float *scores, char *ws,
                                const ScorePlan &pl, bool pool_first, hipStream_t s) {
  if (dtype == ADAKV_FP32) {
    if (dm.d == 64) run_generic<float, 64>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
    else run_generic<float, 128>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
  } else if (dtype == ADAKV_FP16) {
    if (dm.d == 64) run_generic<f16_t, 64>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
    else run_generic<f16_t, 128>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
  } else {
    if (dm.d == 64) run_generic<bf16_t, 64>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
    else run_generic<bf16_t, 128>(st, dm, q, K, row_lse, scores, ws, pl, pool_first, s);
  }
  return hipGetLastError();
}

}  // namespace adakv
