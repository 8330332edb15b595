// Observation-window scoring (Alg. 2 lines 1-5, group mean of Section 3.5) for bf16 and fp16
// inputs on the gfx950 matrix cores: logits = Q_win K^T as v_mfma_f32_32x32x16 tiles with fp32
// accumulation, softmax and reductions in fp32 on the vector ALUs.
//
// The softmax of Alg. 2 l.3 needs every window row's denominator before the rows of a head can
// be added up, so K is swept twice:
//   sweep 1 (PASS 1)  per-row (max, sum of exp) over the keys        -> partial statistics
//   sweep 2 (PASS 2)  exp(logit - lse) summed over the g*w rows      -> pre-pool scores
// A caller-supplied row_lse skips sweep 1.
//
// Work split.  In sweep 2 a workgroup owns chunk_len consecutive keys of one KV head (the fused
// max-pool wants neighbours); in sweep 1 the workgroups of a head take the head's tiles in turn,
// because a (max, sum) pair does not care which keys it saw and the chip then streams one dense
// region of K at a time.  All g query heads of the group share every K tile of 32 keys, and the
// window queries stay in registers as MFMA operands for a workgroup's whole life.  Up to 128 rows
// every wavefront holds all of them and works on tiles of its own (stats_own, weights_own); beyond,
// RS wavefronts of at most 64 rows (128 at d = 64) share the tiles (stats_group, weights_group).  A
// K tile travels straight from HBM into LDS (rows of whole lines, 16 bytes a lane) and from there into
// registers in operand layout.
//
// Operand roles differ between the sweeps because of what the accumulator layout makes cheap
// (D[i][j]: lane = column j, 16 rows i per lane):
//   sweep 1: D = K_tile Q^T, a lane owns ONE window row and 16 keys: running (max, sum) per
//            lane, nothing crosses lanes until the chunk is done;
//   sweep 2: D = Q K_tile^T, a lane owns ONE key and 16 window rows: the sum over rows is
//            lane-local adds plus one cross-half add (partial sums of RS row groups meet
//            in LDS and are added in a fixed order);
//   sweep 2 with the pool in front of the sum over rows: as sweep 1, the pool runs along a
//            lane's registers, and the sum over rows crosses lanes once per tile.
// Sweep 1 hands its (max, sum) pairs to sweep 2 with the maximum in the base-2 domain.
#include <math.h>

#include <type_traits>

#include "common.h"

namespace adakv {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int TILE = 32;           // keys per MFMA tile
constexpr float LOG2E = 1.4426950408889634f;
constexpr int MFMA_POOL_ROWS_MAX_RADIUS = 7;
// From this radius on a row is pooled in steps of up to two keys.  32768 keys x 8 heads, 128 rows, us a call, one key a
// step / up to two: kernel 7 41.4 / 38.7, kernel 13 52.1 / 47.2; a radius of 2 needs two steps of one either way.
constexpr int POOL_WIDE_RADIUS = 3;
constexpr int OWN_MOST = 3840;     // keys of a chunk at 128 rows, d = 128: beside 64 KiB of tiles in half of a compute unit's LDS

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8 as_bf16(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// One 32x32x16 product-accumulate on eight 16-bit elements per lane and operand; the fragments are
// carried as raw 16-byte words (typed bf16x8 above) whatever the element type is.
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
template <bool F16>
__device__ __forceinline__ floatx16 mfma16(bf16x8 a, bf16x8 b, floatx16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The end of a weights sweep: the max-pool (radius r, stride 1, same length, window clipped to the sequence;
// Section 4.1: kernel 7) of the chunk [kc0, kc1) whose scores lie in sh_part from key k0 on, and, in pipeline
// mode, the first radix digits of what is written, counted in sh_hist (cleared; a barrier has passed since).
template <int NT, int CHUNK>
__device__ __forceinline__ void pool_and_file(const float *sh_part, unsigned *sh_hist, float *__restrict__ dst,
                                              int kc0, int kc1, int k0, int n, int chunk_len, int r,
                                              const TopkCarry &tc, int b, int seg) {
  const int tid = threadIdx.x;
  // A thread pools KPT keys at once, one window offset at a time, so that KPT independent LDS
  // reads are in flight instead of one chain per key.  Offsets that leave the sequence are
  // clamped onto its ends (taking an element of the window twice does not change a maximum);
  // a thread's keys past the chunk end repeat the last key and are not written.
  constexpr int KPT = CHUNK / NT;
  static_assert(CHUNK % NT == 0, "every thread pools the same number of keys");
  float pooled[KPT];
  int pk[KPT];
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    pk[i] = min(kc0 + tid + i * NT, kc1 - 1);
    pooled[i] = -INFINITY;
  }
  if (2 * chunk_len > CHUNK) {
    for (int t = -r; t <= r; ++t) {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        pooled[i] = fmaxf(pooled[i], sh_part[min(max(pk[i] + t, 0), n - 1) - k0]);
    }
  } else {
    // a short chunk in a large instantiation: only the keys there are (kept apart, because the test
    // between the reads of a full chunk cost the sweep 2 us of 51 at 131072 keys)
    for (int t = -r; t <= r; ++t) {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if (i * NT < chunk_len) pooled[i] = fmaxf(pooled[i], sh_part[min(max(pk[i] + t, 0), n - 1) - k0]);
    }
  }
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    if (kc0 + tid + i * NT < kc1) {
      dst[pk[i]] = pooled[i];
      if (tc.hist0) atomicAdd(&sh_hist[key_of(pooled[i]) >> 21], 1u);
    }
  }
  if (tc.hist0) {
    __syncthreads();
    unsigned *gh = tc.hist0 + (size_t)seg * RADIX_BINS;
    unsigned *gt = tc.hist_tot0 + (size_t)b * RADIX_BINS;
    for (int i = tid; i < RADIX_BINS; i += NT) {
      const unsigned v = sh_hist[i];
      if (v) {
        atomicAdd(&gh[i], v);
        atomicAdd(&gt[i], v);
      }
    }
  }
}

// ---- up to 128 window rows: every wavefront on its own ------------------------------------------
//
// The wavefronts of a workgroup share nothing but the window queries: each takes tiles of 32 keys in turn,
// keeps all RB = MB * RS row blocks of Q in registers as operands, and has its own tiles on their way, straight
// into its own part of LDS.  No barrier in the loop, no registers for loads in flight, every tile read from
// LDS once.  A row block's products (a chain of D / 16 matrix instructions) are issued with the vector work on
// the row block before it in between.
//
// Bound by reading K (what a kernel with these addresses and no arithmetic reaches: 44 us for 256 MiB, 13.4 us for
// 64 MiB) and close behind by the vector work (27 us of a sweep at 128 rows x 131072 keys x 8 heads, 16 of them
// exponentials at a quarter of the rate).  Against the form before, in which two wavefronts shared a tile that
// came through registers, with a barrier per tile; us a call, d = 128, 8 KV heads, 128 rows:
//   whole step, 2011 keys 39.0 -> 37.6, 32768 keys 70.3 -> 66.5, 131072 keys 151.6 -> 142.0;
//   scores alone, six sequences (217 000 keys) 206 -> 186; with the caller's log-sum-exp, 20000 keys 17.2 -> 13.3,
//   50021 29.3 -> 26.2 (and 58.3 -> 57.1 at 131072 where the form before took 56.5, within 5 us from run to run).
// The window queries come through LDS as well: read from memory as operand words every load touches 32 lines,
// which kept the first tile waiting for 7 us (32768 keys: 22.0 + 25.0 us for the sweeps, 18.2 + 20.3 through LDS).
template <int N> __device__ __forceinline__ void wait_vmem() {
  static_assert(N < 64, "the counter's range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));   // at most N loads on their way (they return in order)
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// An address that is the same in all lanes, in scalar registers even where the compiler would not keep it there.
__device__ __forceinline__ const char *scalar_address(const char *p) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return (const char *)((unsigned long long)hi << 32 | lo);
}
// A barrier for what the workgroup exchanges through LDS; loads on their way stay there.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// 64 x 16 bytes from base + at + the lane's off, straight into 1 KB of LDS.
__device__ __forceinline__ void load_to_lds(const char *base, unsigned off, unsigned at, u32x4 *dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, 0x7fffffff, 0x00027000),
      (__attribute__((address_space(3))) void *)dst, 16, off, at, 0, 0);
}
// The same behind the compiler's back, for loops that wait with wait_vmem alone: where buffers take turns,
// the compiler would wait for every load before it reads any.  (In front of the load stand the wait states
// that follow a write of m0, one, and a scalar register's write by the vector unit, five.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"        // m0 among the clobbers
__device__ __forceinline__ void load_to_lds_untracked(const char *base, unsigned off, unsigned at, u32x4 *dst) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, 0x7fffffff, 0x00027000);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(
                   (unsigned)(size_t)(__attribute__((address_space(3))) void *)dst),
               "v"(off), "s"(rs), "s"(at)
               : "memory", "m0");
}
// 64 x 4 bytes, the same way.
__device__ __forceinline__ void load_words_to_lds_untracked(const char *base, unsigned off, float *dst) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, 0x7fffffff, 0x00027000);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(
                   (unsigned)(size_t)(__attribute__((address_space(3))) void *)dst),
               "v"(off), "s"(rs)
               : "memory", "m0");
}
#pragma clang diagnostic pop
// Lower half of the wavefront + upper half, in every lane.
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// A row's running statistics: reference rm (base 2) and sum rl of exp2(x - rm).  A sum against a kept reference needs
// no search for a maximum in every tile.  It is as accurate as one against the running maximum while the largest
// terms lie near the reference: x - rm is rounded at its own size, which is 3e-7 of a term 16 above it, what the
// log-sum-exp of such a row is rounded to as well, but 1.3e-6 at 60 and 2.6e-6 at 110.  So a lane's terms of a row
// block (16 of them) whose sum goes beyond KEPT_MOST are taken again with the maximum of all so far as the new
// reference, and with them everything that is not a number or not finite.
constexpr float KEPT_MOST = 0x1p16f;
__device__ __forceinline__ void fold_rows(const floatx16 &a, float c_log2, float &rm, float &rl) {
  float tm = a[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) tm = fmaxf(tm, a[r]);
  const float m = fmaxf(rm, tm * c_log2), ref = (m == -INFINITY) ? 0.0f : m;
  float sum = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    sum += fast_exp2(fmaf(a[r], c_log2, -ref));
    asm volatile("" : "+v"(sum));                      // (one at a time: this is rare, and registers are few around it)
  }
  rl = rl * fast_exp2(rm - ref) + sum;
  rm = m;
}
__device__ __forceinline__ void add_kept(const floatx16 &a, float c_log2, float sum, float &rm, float &rl) {
  const float before = rl;                             // (added in any case: a choice would be a second branch in the loop)
  rl += sum;
  if (__builtin_expect(__any(!(sum <= KEPT_MOST)), 0)) {
    rl = before;
    fold_rows(a, c_log2, rm, rl);
  }
}
// Many tiles make a large sum all the same; its logarithm is rounded at the size of its exponent, which therefore
// moves into the reference (the factor is that of the two references as they are stored).
__device__ __forceinline__ void settle(float &m, float &l) {
  if (l > KEPT_MOST) {
    const float to = m + (float)__builtin_amdgcn_frexp_expf(l);
    l *= fast_exp2(m - to);
    m = to;
  }
}

// A wavefront's view of rows of D 16-bit elements in LDS: 32 rows at a time, 16-byte words swizzled so that
// neighbouring lanes' operand reads (row l32, word 2s + half) fall on different banks.
template <int D> struct RowTile {
  static constexpr int KS = D / 16;                    // matrix instructions per row block
  static constexpr int ROW16 = D / 8;                  // 16-byte words per row
  static constexpr int WORDS = TILE * ROW16;
  static constexpr int RPI = 64 / ROW16;               // rows per load instruction
  static constexpr int LD = WORDS / 64;                // load instructions per tile
  static constexpr int NV = D == 128 ? 4 : 2;          // load instructions until the swizzle repeats
  static __device__ __forceinline__ unsigned swz(unsigned row) { return D == 128 ? row & 15u : (row >> 1) & 7u; }
  // byte offset inside its row of the word that lane `ln` of load instruction i loads
  static __device__ __forceinline__ unsigned col(unsigned ln, int i) {
    return ((ln % ROW16) ^ swz((i % NV) * RPI + ln / ROW16)) * 16u;
  }
  // word of LDS that operand word s of this lane's row lies in
  static __device__ __forceinline__ unsigned operand(unsigned l32, unsigned half, int s) {
    return l32 * ROW16 + ((2 * s + half) ^ swz(l32));
  }
  // all rows of a tile are there: off[v] = the lane's row * tok_bytes + col
  template <class Load>
  static __device__ __forceinline__ void whole(const char *sb, unsigned tok_bytes, const unsigned (&off)[NV], Load &&load) {
#pragma unroll
    for (int i = 0; i < LD; ++i) load(sb, off[i % NV], (unsigned)(i * RPI) * tok_bytes, i * 64);
  }
  // rows clamped to [lo, lim], counted from the tile's first
  template <class Load>
  static __device__ __forceinline__ void clamped(const char *sb, unsigned tok_bytes, int lo, int lim, unsigned lane, Load &&load) {
    asm volatile("" : "+v"(lane));                     // (computed here, not kept in registers for the rare tile)
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const unsigned row = (unsigned)max(min((int)(i * RPI + lane / ROW16), lim), lo);
      load(sb, __umul24(row, tok_bytes) + col(lane, i), 0u, i * 64);
    }
  }
};

// The printed order of Alg. 2 l.4 (PR): max-pool along the keys in every window row first, mean over the rows
// afterwards.  A lane then owns one window row and, with the operand rows numbered this way, 16 consecutive keys of
// a tile: D[i][j] has lane j's row and the keys i = 8 (r/4) + 4 half + r%4, and operand row i is key pooled_row(i), so
// that register r is key 16 half + r.  The sliding maximum is then a three-operand maximum per weight and
// unit of radius, between registers; only what lies next to the other half crosses lanes.  (A lane with one key of
// 16 rows, the form before, needed two operations per weight and unit of radius, with neighbouring lanes as
// operands: 20000 keys x 8 heads, 128 rows, d = 128 35.9 us, now 30.8, 512 rows 84.2 and 74.7; kernel 13 over 32768
// keys 62.0 and 51.7.)  Tiles overlap by the radius on either side: their inner
// 32 - 2 radius keys have all their neighbours and produce a score.  Rows outside the sequence repeat its last (first)
// one, which is in every window that reaches them.
__device__ __forceinline__ unsigned pooled_row(unsigned i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// e, pooled over so far `a` keys to either side, goes on to a + S (S <= 2 a + 1, so that no key between is left out):
// three-operand maxima in place.  What lies next to the half's first and last keys comes from the other half; at a
// tile's ends some key of its own stands in, which spoils only what lacks neighbours there anyway.
template <int S> __device__ __forceinline__ void widen(floatx16 &e) {
  unsigned left[S], right[S];
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(e[k]), __float_as_uint(e[16 - S + k]), false, false);
    left[k] = sw[0];                                   // upper half: the lower one's e[16 - S + k]
    right[k] = sw[1];                                  // lower half: the upper one's e[k]
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const unsigned own = __float_as_uint(e[i]);
    e[i] = __uint_as_float(max(max(left[i % S], own), i + S < 16 ? __float_as_uint(e[i + S < 16 ? i + S : 15]) : right[i + S < 16 ? 0 : i + S - 16]));
    left[i % S] = own;
  }
}
// keysum += e, pooled over `radius` keys to either side.  WIDE (radius >= POOL_WIDE_RADIUS): steps of 1, then 2 (of 3 would
// need more registers than there are): two for radius 3, four for 7.  A kernel of its own, because loops for both step
// lengths in one kernel cost the short radii 2 to 4 %.  Weights are not
// negative, so their bit patterns order like they do, and in an unsigned maximum a NaN, whatever its sign, wins (a
// floating-point maximum would drop it): it poisons every mean whose window holds it, which pool_and_file stores as -inf.
template <bool WIDE>
__device__ __forceinline__ void pool_rows(floatx16 &e, int radius, float (&keysum)[16]) {
  if constexpr (WIDE) {
    widen<1>(e);
    if (!(radius & 1)) widen<1>(e);
    for (int t = 2 - (radius & 1); t < radius; t += 2) widen<2>(e);
  } else {
    for (int t = 0; t < radius; ++t) widen<1>(e);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) keysum[i] += e[i];
}
// The 16 keys' sums over the 32 lanes of a half, each step adding lanes and halving the registers: a lane ends up
// with the sum of key summed_key(lane).
__device__ __forceinline__ unsigned summed_key(unsigned lane) {
  return 16 * (lane >> 5) + ((lane >> 4) & 1) + 2 * ((lane >> 3) & 1) + 4 * ((lane >> 2) & 1) + 8 * ((lane >> 1) & 1);
}
template <int CTRL> __device__ __forceinline__ float add_dpp(float x) {
  return x + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_rows(const float (&k)[16], unsigned lane) {
  auto pick = [](bool second, float x, float y) { return second ? y : x; };    // (by value: an lvalue choice would put the arrays into memory)
  float a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {                        // lanes 16 apart; odd rows of 16 lanes go on with key 2i + 1
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(k[2 * i]), __float_as_uint(k[2 * i + 1]), false, false);
    a[i] = add_dpp<0x128>(__uint_as_float(sw[0]) + __uint_as_float(sw[1]));                       // and lanes 8 apart (row_ror:8)
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = add_dpp<0x141>(pick(lane & 8, a[2 * i], a[2 * i + 1]));      // row_half_mirror: lanes j and 7 - j
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = add_dpp<0x4E>(pick(lane & 4, b[2 * i], b[2 * i + 1]));       // quad_perm [2,3,0,1]
  return add_dpp<0xB1>(pick(lane & 2, c[0], c[1]));                                               // quad_perm [1,0,3,2]
}

// Sweep 1.  Tiles of a sequence are dealt out over all wavefronts of the head (the workgroups that the sequence
// has in cp, four wavefronts each), so at any moment the chip reads one dense region of K.  One workgroup per
// compute unit, one wavefront per SIMD with three tiles on their way: of two wavefronts the older one runs ahead
// and leaves the younger one to stream alone (131072 keys: 57.4 us with two of two tiles each, 52 with one).
template <int D, int RB, bool F16>
__device__ __forceinline__ void stats_own(const SeqTab &st, const ChunkTab &cp, const Dims &dm, float c_log2,
                                          const unsigned short *__restrict__ q, const unsigned short *__restrict__ K,
                                          float2 *__restrict__ part, const TopkCarry &tc) {
  typedef RowTile<D> T;
  constexpr int NW = 4, NT = 64 * NW, KS = T::KS, LD = T::LD;
  constexpr int RPAD = 32 * RB;
  constexpr int NBUF = 3;                             // tiles a wavefront has room for
  constexpr int UN = NBUF;
  static_assert(UN * RB % 3 == 0, "a row block's products take turns in three places");
  __shared__ u32x4 kt[NW][NBUF][T::WORDS];
  __shared__ u32x4 qs[RB * T::WORDS];

  const int tid = threadIdx.x, lane = tid & 63;
  // pipeline mode: the Top-k histograms, which the kernel after this one is the first to touch
  if (tc.zero_begin)
    for (unsigned i = blockIdx.x * NT + tid; i < tc.zero_words; i += gridDim.x * NT) tc.zero_begin[i] = 0u;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int h = dm.h_kv;
  const int c = blockIdx.x % h, cg = blockIdx.x / h;
  const int b = find_seq(cp, st.batch, cg);
  const int first = (cg - cp.off[b]) * NW + wv, stride = (cp.off[b + 1] - cp.off[b]) * NW;
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const size_t head_row0 = (size_t)b * RQ + (size_t)c * R;
  const int ntiles = (n + TILE - 1) / TILE;
  const int iters = first < ntiles ? (ntiles - 1 - first) / stride + 1 : 0;
  const char *kbase = reinterpret_cast<const char *>(K) +
                      ((size_t)st.tok_off[b] * dm.k_stride_tok + (size_t)c * dm.k_stride_head) * 2;
  const unsigned tok_bytes = (unsigned)dm.k_stride_tok * 2u;
  unsigned ld_off[T::NV];
#pragma unroll
  for (int v = 0; v < T::NV; ++v) ld_off[v] = __umul24(lane / T::ROW16, tok_bytes) + T::col(lane, v);
  auto issue = [&](int it, int buf) {
    const int key0 = (first + it * stride) * TILE;
    const char *sb = kbase + (long long)key0 * tok_bytes;
    auto load = [&](const char *base, unsigned off, unsigned at, int word) { load_to_lds_untracked(base, off, at, &kt[wv][buf][word]); };
    if (key0 + TILE <= n) T::whole(sb, tok_bytes, ld_off, load);
    else T::clamped(sb, tok_bytes, 0, n - 1 - key0, lane, load);
  };
  // tile `it` has arrived; those asked for behind it, at most NBUF - 1, may be on their way
  auto await = [&](int it) {
    const int behind = min(iters - 1 - it, NBUF - 1);
    if (behind == NBUF - 1) wait_vmem<(NBUF - 1) * LD>();
    else if (behind == NBUF - 2) wait_vmem<(NBUF - 2) * LD>();
    else wait_vmem<0>();
  };

  // the window queries, through LDS: as operand words straight from memory every load would touch 32 lines
  constexpr int QI = RPAD / T::RPI / NW;               // load instructions per wavefront
  static_assert(QI * T::RPI * NW == RPAD, "");
#pragma unroll
  for (int i = 0; i < QI; ++i) {
    const unsigned row = (unsigned)(wv * QI + i) * T::RPI + lane / T::ROW16;     // (rows past R are row R-1, zeroed below)
    load_to_lds_untracked(reinterpret_cast<const char *>(q) + head_row0 * (D * 2),
                          min(row, (unsigned)R - 1u) * (D * 2) + ((lane % T::ROW16) ^ T::swz(row)) * 16u, 0u,
                          &qs[(wv * QI + i) * 64]);
  }
#pragma unroll
  for (int j = 0; j < NBUF; ++j)
    if (j < iters) issue(j, j);
  {
    const int asked = min(iters, NBUF);
    if (asked == NBUF) wait_vmem<NBUF * LD>();
    else if (asked == 2) wait_vmem<2 * LD>();
    else if (asked == 1) wait_vmem<LD>();
    else wait_vmem<0>();
  }
  lds_barrier();
  unsigned rd[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) rd[s] = T::operand(l32, half, s);
  bf16x8 qf[RB][KS];
#pragma unroll
  for (int mb = 0; mb < RB; ++mb) {
    const unsigned keep = mb * 32 + l32 < R ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[mb][s] = as_bf16(qs[mb * T::WORDS + rd[s]] & keep);
  }

  bf16x8 kf[KS];
  floatx16 acc[3];                                     // products of the current row block and of the two before
  float rm[RB], rl[RB];                                // running maximum (or reference) and sum of the row this lane owns
  // The vector work on one row block's products, in KS shares.  Against a kept reference two row blocks of a tile are
  // looked at together (p: the first one's products): a branch per row block took 1 us of 64 at 32768 keys and 3 of 172
  // over six sequences of 217 000 keys.
  float ref = 0.0f, nmx = 0.0f, usum = 0.0f, kept[2] = {0.0f, 0.0f};
  auto share = [&](auto lazy_tag, const floatx16 &p, const floatx16 &a, int mb, int s) {
    if constexpr (decltype(lazy_tag)::value) {
      const int o = mb & 1, of = RB > 1 ? mb & ~1 : mb;
      if (s == 0) kept[o] = 0.0f;
#pragma unroll
      for (int v = s * 16 / KS; v < (s + 1) * 16 / KS; ++v) kept[o] += fast_exp2(fmaf(a[v], c_log2, -rm[mb]));
      if (s == KS - 1 && (RB == 1 || o == 1)) {
        const float both = RB > 1 ? kept[0] + kept[1] : kept[0], first_before = rl[of], before = rl[mb];
        rl[of] += kept[0];                             // (added in any case: a choice would be a second branch)
        if (RB > 1) rl[mb] += kept[1];
        if (__builtin_expect(__any(!(both <= KEPT_MOST)), 0)) {
          rl[of] = first_before;
          if (RB > 1) {
            fold_rows(p, c_log2, rm[of], rl[of]);
            rl[mb] = before;
          }
          fold_rows(a, c_log2, rm[mb], rl[mb]);
        }
      }
    } else {
      if (s == 0) {
        float tm = a[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tm = fmaxf(tm, a[r]);
        nmx = fmaxf(rm[mb], tm * c_log2);
        ref = (nmx == -INFINITY) ? 0.0f : nmx;
        usum = 0.0f;
      } else {
#pragma unroll
        for (int v = (s - 1) * 16 / (KS - 1); v < s * 16 / (KS - 1); ++v) usum += fast_exp2(fmaf(a[v], c_log2, -ref));
      }
      if (s == KS - 1) {
        rl[mb] = rl[mb] * fast_exp2(rm[mb] - ref) + usum;
        rm[mb] = nmx;
      }
    }
  };
  // the sequence's last tile, if it is not full, is the last of its wavefront and comes after the loop
  const int plain = iters > 0 && (first + (iters - 1) * stride) * TILE + TILE > n ? iters - 1 : iters;
  // All full tiles, the first of them in kf; behind it kf holds the tile after them, if there is one.
  auto loop = [&](auto lazy_tag) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = acc[2][r] = -INFINITY;      // (nothing before the first: no weight)
    for (int it0 = 0; it0 < plain; it0 += UN) {
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const int it = it0 + j;
        if (it < plain) {
          wait_lds();                                  // the tile is in registers: its place is free
          if (it + NBUF < iters) issue(it + NBUF, j % NBUF);
#pragma unroll
          for (int mb = 0; mb < RB; ++mb) {
            const int cur = (j * RB + mb) % 3, pmb = mb == 0 ? RB - 1 : mb - 1;
            if (mb == RB - 1) await(it + 1);
            floatx16 a = {0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
              a = mfma16<F16>(kf[s], qf[mb][s], a);
              if (s == 0) __builtin_amdgcn_sched_barrier(0);     // (else the vector work, which waits for the block before, goes first)
              if (mb == RB - 1) kf[s] = as_bf16(kt[wv][(j + 1) % NBUF][rd[s]]);   // (whatever lies there behind the last)
              share(lazy_tag, acc[(cur + 1) % 3], acc[(cur + 2) % 3], pmb, s);
              __builtin_amdgcn_sched_barrier(0);
            }
            acc[cur] = a;
            // the vector work stays in front of this point
            if constexpr (RB > 1) asm volatile("" : "+v"(rl[pmb & ~1]), "+v"(rm[pmb & ~1]), "+v"(rl[pmb | 1]), "+v"(rm[pmb | 1]), "+v"(kept[pmb & 1]));
            else asm volatile("" : "+v"(rl[pmb]), "+v"(rm[pmb]));
          }
        }
      }
    }
    if (plain > 0) {
      auto finish = [&](const floatx16 &p, const floatx16 &last) {
#pragma unroll
        for (int s = 0; s < KS; ++s) share(lazy_tag, p, last, RB - 1, s);
      };
      const int at = (plain * RB + 2) % 3;             // the last row block's place
      if (at == 0) finish(acc[2], acc[0]);
      else if (at == 1) finish(acc[0], acc[1]);
      else finish(acc[1], acc[2]);
    }
  };
#pragma unroll
  for (int mb = 0; mb < RB; ++mb) { rm[mb] = -INFINITY; rl[mb] = 0.0f; }
  auto read_first = [&]() {                            // (in either branch below: both start from its registers)
    await(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = as_bf16(kt[wv][0][rd[s]]);
  };
  // With several tiles to come the first one's maxima are kept as reference (50 instead of 70 vector instructions
  // per row block: 18.2 -> 16.9 us at 32768 keys, 61.5 -> 58.6 at 131072).
  if (plain >= 4) {
    read_first();
#pragma unroll
    for (int mb = 0; mb < RB; ++mb) {
      floatx16 a = {0};
#pragma unroll
      for (int s = 0; s < KS; ++s) a = mfma16<F16>(kf[s], qf[mb][s], a);
      float tm = a[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) tm = fmaxf(tm, a[r]);
      rm[mb] = tm * c_log2;
      asm volatile("" : "+v"(rm[mb]));                 // (one row block's products at a time)
      __builtin_amdgcn_sched_barrier(0);
    }
    loop(std::true_type{});
#pragma unroll
    for (int mb = 0; mb < RB; ++mb) settle(rm[mb], rl[mb]);
  } else {
    if (iters > 0) read_first();
    loop(std::false_type{});
  }
  if (plain < iters) {
    const int base = (first + plain * stride) * TILE;
#pragma unroll
    for (int mb = 0; mb < RB; ++mb) {
      floatx16 a = {0};
#pragma unroll
      for (int s = 0; s < KS; ++s) a = mfma16<F16>(kf[s], qf[mb][s], a);
#pragma unroll
      for (int r = 0; r < 16; ++r)                     // key base + 8 (r/4) + 4 half + r%4
        if (base + 8 * (r / 4) + 4 * half + (r % 4) >= n) a[r] = -INFINITY;
#pragma unroll
      for (int s = 0; s < KS; ++s) share(std::false_type{}, a, a, mb, s);
      asm volatile("" : "+v"(rl[mb]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // merge the two lane halves (same window row, different keys), then the wavefronts
  wait_vmem<0>();
  wait_lds();
  float *own = reinterpret_cast<float *>(&kt[wv][0][0]);
  static_assert(T::WORDS * 16 >= 2 * RPAD * 4, "");
#pragma unroll
  for (int mb = 0; mb < RB; ++mb) {
    const float m2 = __shfl_xor(rm[mb], 32), s2 = __shfl_xor(rl[mb], 32);
    const float M = fmaxf(rm[mb], m2);
    const float rf = (M == -INFINITY) ? 0.0f : M;
    const float L = rl[mb] * fast_exp2(rm[mb] - rf) + s2 * fast_exp2(m2 - rf);
    if (half == 0) { own[mb * 32 + l32] = M; own[RPAD + mb * 32 + l32] = L; }
  }
  __syncthreads();
  if (tid < R) {
    const float *o[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) o[k] = reinterpret_cast<const float *>(&kt[k][0][0]) + tid;
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < NW; ++k) M = fmaxf(M, o[k][0]);
    const float rf = (M == -INFINITY) ? 0.0f : M;
    float L = 0.0f;
#pragma unroll
    for (int k = 0; k < NW; ++k) L += o[k][RPAD] * fast_exp2(o[k][0] - rf);
    part[(size_t)cg * RQ + (size_t)c * R + tid] = make_float2(M, L);            // (base 2, as the weights sweep wants it)
  }
}

// Sweep 2.  A workgroup owns chunk_len consecutive keys (the pool wants neighbours); its wavefronts take the
// chunk's tiles in turn, backwards from a point that differs from workgroup to workgroup: concurrently running
// workgroups then do not ask for addresses that are equal modulo the distance of their chunks.
template <int D, int MB, int RS, int CHUNK, bool F16, bool PR, bool WIDE>
__device__ __forceinline__ void weights_own(const SeqTab &st, const ChunkTab &ct, const ChunkTab &cp, const Dims &dm,
                                            float c_log2, const unsigned short *__restrict__ q,
                                            const unsigned short *__restrict__ K, const float *__restrict__ lse, float lse_mul,
                                            const float2 *__restrict__ part, float *__restrict__ out, int halo,
                                            int chunk_len, const TopkCarry &tc) {
  typedef RowTile<D> T;
  constexpr int NW = 4, NT = 64 * NW, KS = T::KS, LD = T::LD;
  constexpr int RB = MB * RS, RPAD = 32 * RB;
  constexpr int HALO = TILE;                           // keys scored in front of the chunk for the pool
  constexpr int SPAN = (D == 128 && CHUNK == 4096 ? OWN_MOST : CHUNK) + 2 * HALO;
  // (two arrays, so that the compiler sees that reading one does not wait for loads into the other)
  __shared__ u32x4 kt0[NW][T::WORDS], kt1[NW][T::WORDS];
  __shared__ __align__(16) float sh_lse[RPAD < 64 ? 64 : RPAD];
  __shared__ __align__(16) float sh_part[SPAN > 4 * NT ? SPAN : 4 * NT];
  constexpr int SL = 2 * NT / RPAD;                    // threads that share two rows in the statistics combination
  float *sh_cm = sh_part, *sh_cl = sh_part + 2 * NT;   // (the prologue's, before any score is there)
  static_assert(sizeof(kt0) >= RADIX_BINS * sizeof(unsigned), "the digit histogram takes the tiles' place");
  unsigned *sh_hist = reinterpret_cast<unsigned *>(&kt0[0][0]);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int h = dm.h_kv;
  const int c = blockIdx.x % h, cg = ct.off[st.batch] - 1 - (int)blockIdx.x / h;
  const int b = find_seq(ct, st.batch, cg);
  const int chunk = cg - ct.off[b], nch = ct.off[b + 1] - ct.off[b];
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const int kc0 = chunk * chunk_len, kc1 = min(n, kc0 + chunk_len);
  const int pool_r = halo || PR ? dm.pool_k / 2 : 0;
  const int tstep = PR ? TILE - 2 * pool_r : TILE;     // keys a tile advances by
  const int before = PR ? pool_r : 0;                  // keys of a tile in front of its first own
  // with the pool fused: a whole tile in front of the chunk, the pool radius behind it (no tile starts past the
  // last key somebody needs)
  const int k0 = halo && kc0 > 0 ? kc0 - HALO : kc0;
  const int k1 = halo ? min(n, kc1 + pool_r) : kc1;
  const int ntiles = (k1 - k0 + tstep - 1) / tstep;
  const size_t head_row0 = (size_t)b * RQ + (size_t)c * R;

  const int iters = wv < ntiles ? (ntiles - 1 - wv) / NW + 1 : 0;
  const int rot = (int)(((long long)chunk * iters) / nch);
  auto tile_of = [&](int it) {
    const int p = rot - 1 - it;
    return wv + (p < 0 ? p + iters : p) * NW;
  };
  const char *kbase = reinterpret_cast<const char *>(K) +
                      ((size_t)st.tok_off[b] * dm.k_stride_tok + (size_t)c * dm.k_stride_head) * 2;
  const unsigned tok_bytes = (unsigned)dm.k_stride_tok * 2u;
  // rows nobody needs (in front of the pool radius, behind the sequence or the radius) repeat the nearest needed one
  const int need_lo = max(kc0 - pool_r, 0), need_hi = min(kc1 - 1 + pool_r, n - 1);
  unsigned ld_off[T::NV];
#pragma unroll
  for (int v = 0; v < T::NV; ++v) ld_off[v] = __umul24(lane / T::ROW16, tok_bytes) + T::col(lane, v);
  auto issue_clamped = [&](int tile, auto &&load) {
    const int key0 = min(k0 + tile * tstep - before, need_hi);
    T::clamped(kbase + (long long)key0 * tok_bytes, tok_bytes, max(need_lo - key0, 0), need_hi - key0, lane, load);
  };
  auto issue = [&](int tile, int buf) {
    const int key0 = k0 + tile * tstep - before;
    u32x4 *dst = buf ? &kt1[wv][0] : &kt0[wv][0];
    auto load = [&](const char *base, unsigned off, unsigned at, int word) { load_to_lds_untracked(base, off, at, dst + word); };
    if (key0 >= need_lo && key0 + TILE - 1 <= need_hi) T::whole(kbase + (long long)key0 * tok_bytes, tok_bytes, ld_off, load);
    else issue_clamped(tile, load);
  };
  // The first tile and, through LDS (the second tile's place), the window queries.
  constexpr int QI = RPAD / T::RPI / NW;
  static_assert(QI * T::RPI * NW == RPAD && RB * T::WORDS <= NW * T::WORDS, "");
  u32x4 *qs = &kt1[0][0];
  auto first_tile = [&](auto &&load) {
    issue_clamped(iters > 0 ? tile_of(0) : 0, [&](const char *base, unsigned off, unsigned at, int word) { load(base, off, at, &kt0[wv][word]); });
  };
  auto load_queries = [&](auto &&load) {
#pragma unroll
    for (int i = 0; i < QI; ++i) {
      const unsigned row = (unsigned)(wv * QI + i) * T::RPI + lane / T::ROW16;   // (rows past R are row R-1, zeroed below)
      load(reinterpret_cast<const char *>(q) + head_row0 * (D * 2),
           min(row, (unsigned)R - 1u) * (D * 2) + ((lane % T::ROW16) ^ T::swz(row)) * 16u, 0u, qs + (wv * QI + i) * 64);
    }
  };
  unsigned rd[KS], rk[KS];                             // operand words of the queries, of a tile
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    rd[s] = T::operand(l32, half, s);
    rk[s] = PR ? T::operand(pooled_row(l32), half, s) : rd[s];
  }
  // WIDE: word s of a tile is the first one with 2 s exclusive-ored in, worked out for every tile, because registers are
  // few.  (In the short radii's kernel, which has them, it costs 3 %: 32768 keys x 8 heads, 128 rows, kernel 3 37.4 /
  // 38.4 us a call, kernel 5 39.6 / 40.7.)
  unsigned tile_word = T::operand(pooled_row(l32), half, 0);
  auto tile_words = [&]() {
    if constexpr (WIDE) asm volatile("" : "+v"(tile_word));
  };
  auto word = [&](int s) { return WIDE ? tile_word ^ (2u * s) : rk[s]; };
  bf16x8 qf[RB][KS];                                   // kept for the whole chunk
  auto queries = [&]() {
    lds_barrier();
#pragma unroll
    for (int mb = 0; mb < RB; ++mb) {
      const unsigned keep = mb * 32 + l32 < R ? 0xFFFFFFFFu : 0u;
#pragma unroll
      for (int s = 0; s < KS; ++s) qf[mb][s] = as_bf16(qs[mb * T::WORDS + rd[s]] & keep);
    }
  };
  // the rows' log-sum-exp in the base-2 domain; +inf on the padding rows makes their weights zero
  if (lse) {
    // The queries first and the first tile behind them, so that the second one, which takes their place, is asked for
    // while the first is on its way.  (All of it behind the compiler's back: it would wait for the first tile with
    // whatever it waits for first.)  us a call, first tile and queries / queries and first tile, 128 rows, 8 heads:
    // 20000 keys 14.6 / 13.3, 50021 27.0 / 26.2, 131072 58.3 / 57.1; 32 rows, 50021 keys 23.0 / 22.2.
    load_queries(load_to_lds_untracked);
    if (wv < (RPAD + 63) / 64)
      load_words_to_lds_untracked(reinterpret_cast<const char *>(lse + head_row0), (unsigned)min(tid, R - 1) * 4u, sh_lse + wv * 64);
    first_tile(load_to_lds_untracked);
    wait_vmem<LD>();
    queries();
    if (tid < RPAD) sh_lse[tid] = tid < R ? sh_lse[tid] * lse_mul : INFINITY;
  } else {
    // Sweep 1's partials (max, sum) of this head's rows: SL threads take two rows, every SL-th partial each, CB of
    // them at a time; they come from the cache and are asked for before anything else.  (The few partials that
    // are combined here leave their offsets far inside 32 bits.)
    constexpr int CB = 16;
    const int q2 = tid % (RPAD / 2), sl = tid / (RPAD / 2);
    const int row = min(2 * q2, max(R - 2, 0)), np = cp.off[b + 1] - cp.off[b];
    struct __attribute__((packed, aligned(8))) Pair { float m0, l0, m1, l1; };
    const float2 *pp = part + ((size_t)cp.off[b] * RQ + (size_t)c * R);
    Pair pml[CB];
    auto load_parts = [&](int p0) {
#pragma unroll
      for (int u = 0; u < CB; ++u) pml[u] = *reinterpret_cast<const Pair *>(pp + (unsigned)(min(p0 + u * SL, np - 1) * RQ + row));
    };
    float M0 = -INFINITY, L0 = 0.0f, M1 = -INFINITY, L1 = 0.0f;
    // first the largest maximum of a batch, then every sum scaled to it (independent exponentials)
    auto fold = [&](int p0) {
      float n0 = M0, n1 = M1;
#pragma unroll
      for (int u = 0; u < CB; ++u)
        if (p0 + u * SL < np) { n0 = fmaxf(n0, pml[u].m0); n1 = fmaxf(n1, pml[u].m1); }
      const float r0 = (n0 == -INFINITY) ? 0.0f : n0, r1 = (n1 == -INFINITY) ? 0.0f : n1;
      L0 *= fast_exp2(M0 - r0);
      L1 *= fast_exp2(M1 - r1);
#pragma unroll
      for (int u = 0; u < CB; ++u)
        if (p0 + u * SL < np) {
          L0 += pml[u].l0 * fast_exp2(pml[u].m0 - r0);
          L1 += pml[u].l1 * fast_exp2(pml[u].m1 - r1);
        }
      M0 = n0;
      M1 = n1;
    };
    load_parts(sl);
    // (unconditionally, and counted by the compiler, so that its wait for the partials does not stop at these as well)
    __builtin_amdgcn_sched_barrier(0);
    first_tile(load_to_lds);
    load_queries(load_to_lds);
    __builtin_amdgcn_sched_barrier(0);
    fold(sl);
    for (int p0 = sl + CB * SL; p0 < np; p0 += CB * SL) {
      load_parts(p0);
      fold(p0);
    }
    if (2 * q2 == R - 1 && R > 1) { M0 = M1; L0 = L1; }        // (an odd number of rows: the last came as the second of its pair)
    *reinterpret_cast<float2 *>(&sh_cm[sl * RPAD + 2 * q2]) = make_float2(M0, M1);
    *reinterpret_cast<float2 *>(&sh_cl[sl * RPAD + 2 * q2]) = make_float2(L0, L1);
    wait_vmem<0>();
    queries();                                         // (its barrier also shows the above)
    if (tid < RPAD) {
      float Mt = -INFINITY;
#pragma unroll
      for (int i = 0; i < SL; ++i) Mt = fmaxf(Mt, sh_cm[i * RPAD + tid]);
      const float ref = (Mt == -INFINITY) ? 0.0f : Mt;
      float Lt = 0.0f;
#pragma unroll
      for (int i = 0; i < SL; ++i) Lt += sh_cl[i * RPAD + tid] * fast_exp2(sh_cm[i * RPAD + tid] - ref);
      sh_lse[tid] = (tid < R) ? Mt + __builtin_amdgcn_logf(Lt) : INFINITY;
    }
  }
  lds_barrier();                                       // everybody has its queries, and the log-sum-exp is there
  if (iters > 1) issue(tile_of(1), 1);

  bf16x8 kf[KS];
  floatx16 acc[2];                                     // products of the current row block and of the one before
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = -INFINITY;
  float sum[RS];
#pragma unroll
  for (int i = 0; i < RS; ++i) sum[i] = 0.0f;
  const float inv = 1.0f / (float)R;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  // The 16 rows a lane sees of a row block: their log-sum-exp in registers, or, where the queries take 128 of
  // them, four at a time from LDS, two groups ahead of their use.
  constexpr bool L2_REGS = RB <= 2 && !PR;
  float l2[L2_REGS ? RB : 1][16];
  if (L2_REGS) {
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) l2[mb][r] = sh_lse[mb * 32 + 8 * (r / 4) + 4 * half + (r % 4)];
  }
  f32x4 lq[4];
  auto read_lq = [&](int mb, int q4) { return *reinterpret_cast<const f32x4 *>(&sh_lse[mb * 32 + 8 * q4 + 4 * half]); };
  if (!L2_REGS && !PR) {
    lq[0] = read_lq(RB - 1, 0);
    lq[1] = read_lq(RB - 1, 1);
  }
  float l2row[PR ? RB : 1], keysum[PR ? 16 : 1];       // PR: of the row this lane owns; over the tile's rows so far
  if constexpr (PR) {
#pragma unroll
    for (int mb = 0; mb < RB; ++mb) l2row[mb] = sh_lse[mb * 32 + l32];
  }
  // share s of KS of the vector work on a row block's products; a[r]: window row mb*32 + 8*(r/4) + 4*half + r%4
  auto share = [&](floatx16 &a, int mb, int next_mb, int s) {
    constexpr int V = 16 / KS;
#pragma unroll
    for (int v = s * V; v < (s + 1) * V; ++v) {
      float l;
      if constexpr (PR) {
        a[v] = fast_exp2(fmaf(a[v], c_log2, -l2row[mb]));
        continue;
      } else if constexpr (L2_REGS) {
        l = l2[mb][v];
      } else {
        if (v % 4 == 0) lq[(v / 4 + 2) % 4] = v / 4 < 2 ? read_lq(mb, v / 4 + 2) : read_lq(next_mb, v / 4 - 2);
        l = lq[v / 4][v % 4];
      }
      sum[mb / MB] += fast_exp2(fmaf(a[v], c_log2, -l));
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < RS; ++i) sum[i] = 0.0f;
    if constexpr (PR) {
#pragma unroll
      for (int i = 0; i < 16; ++i) keysum[i] = 0.0f;
    }
  };
  clear();
  auto file = [&](int tile) {                          // a finished tile's mean weights (a key per lane; past n: never read)
    if constexpr (PR) {
      const float tot = sum_rows(keysum, lane);
      const int at = summed_key(lane), key = tile * tstep + at - before;
      if (!(lane & 1) && at >= pool_r && at < TILE - pool_r && key < k1 - k0) sh_part[key] = tot * inv;
    } else {
      float tot = sum_halves(sum[0]);
#pragma unroll
      for (int i = 1; i < RS; ++i) tot += sum_halves(sum[i]);
      sh_part[tile * TILE + l32] = tot * inv;
    }
    clear();
  };
  if (iters > 0) {
    if (iters > 1) wait_vmem<LD>(); else wait_vmem<0>();
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = as_bf16(kt0[wv][word(s)]);
  }
  int prev = 0;                                        // tile before the current one
  for (int it0 = 0; it0 < iters; it0 += 2) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int it = it0 + j;
      if (it < iters) {
        const int tile = tile_of(it);
        wait_lds();                                    // the tile is in registers: its place is free
        tile_words();
        if (it + 2 < iters) issue(tile_of(it + 2), j);
#pragma unroll
        for (int mb = 0; mb < RB; ++mb) {
          const int cur = (j * RB + mb) & 1, pmb = mb == 0 ? RB - 1 : mb - 1;
          if (mb == RB - 1) {                          // the next tile, for the reads below
            if (it + 2 < iters) wait_vmem<LD>(); else wait_vmem<0>();
          }
          floatx16 a = {0};
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            a = PR ? mfma16<F16>(kf[s], qf[mb][s], a) : mfma16<F16>(qf[mb][s], kf[s], a);
            if (mb == RB - 1) kf[s] = as_bf16(j == 0 ? kt1[wv][word(s)] : kt0[wv][word(s)]);   // (whatever lies there behind the last)
            share(acc[1 - cur], pmb, mb, s);
            __builtin_amdgcn_sched_barrier(0);
          }
          acc[cur] = a;
          if constexpr (PR) {
            pool_rows<WIDE>(acc[1 - cur], pool_r, keysum);
#pragma unroll
            for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(keysum[i]));
            __builtin_amdgcn_sched_barrier(0);
          } else {
            asm volatile("" : "+v"(sum[pmb / MB]));    // the vector work stays in front of this point
          }
          if (mb == 0) {
            if (it > 0) file(prev);
            else clear();
          }
        }
        prev = tile;
      }
    }
  }
  if (iters > 0) {
    floatx16 last = acc[1];
    if (RB % 2 == 1 && (iters & 1)) last = acc[0];
#pragma unroll
    for (int s = 0; s < KS; ++s) share(last, RB - 1, RB - 1, s);
    if constexpr (PR) pool_rows<WIDE>(last, pool_r, keysum);
    file(prev);
  }
  wait_vmem<0>();                                      // (a wavefront without tiles has asked for one as well)
  __syncthreads();
  if (tc.hist0) {
    for (int i = tid; i < RADIX_BINS; i += NT) sh_hist[i] = 0u;
    __syncthreads();
  }
  pool_and_file<NT, CHUNK>(sh_part, sh_hist, out + st.score_off[b] + (size_t)c * n, kc0, kc1, k0, n, chunk_len,
                           halo ? dm.pool_k / 2 : 0, tc, b, b * h + c);
}

// ---- more than 128 window rows: RS wavefronts share the tiles ---------------------------------------
//
// Every wavefront keeps MB row blocks of Q in registers and works on every tile of the workgroup.  Tiles come in
// sets of ST, straight into LDS, a set ahead of the one that is worked on, and a set is what the wavefronts wait
// for each other for: one barrier per ST tiles, so that the two wavefronts of a SIMD drift apart and one's matrix
// instructions run beside the other's vector work.
//
// The order of things around a barrier, in a set's last tile in front of its last row block's products: the
// wavefront's share of the next set has arrived, its operand reads of this set are done - barrier - all of the next set is there and all of this set is free: the set after next is asked for.
template <int D, int MB, int RS> struct Group {
  typedef RowTile<D> T;
  static constexpr int NT = 64 * RS, RPAD = 32 * MB * RS;
  static constexpr int ST = 4;                         // tiles of a set
  static constexpr int SETW = ST * T::WORDS;
  static constexpr int LDW = ST * T::LD / RS;          // load instructions per wavefront and set
  static_assert(LDW * RS == ST * T::LD, "a set must split evenly over the wavefronts");
  // The queries come through LDS where a row block fits into a wavefront's share of a set and there are two of them:
  // as operand words straight from memory every load touches 32 lines, which cost a workgroup of 256 rows some 2 us.
  // us a call, straight / through LDS, 256 rows, d = 128, 8 heads: with the caller's log-sum-exp 20000 keys 22.2 / 20.9,
  // 50021 41.4 / 39.6 (the form without sets: 21.7, 39.7); both sweeps 2011 keys 16.4 / 15.1, 20000 40.9 / 38.1,
  // 50021 77.4 / 72.4 (42.1, 74.9 at the last two).
  static constexpr bool Q_LDS = MB == 2 && T::WORDS <= SETW / RS;
};
// One row block of the queries of wavefront wv, straight into its share of a set's place (rows past R are row R-1).
template <int D, class Load>
__device__ __forceinline__ void load_query_block(const unsigned short *q, size_t head_row0, int R, int row0, int lane, Load &&load) {
  typedef RowTile<D> T;
#pragma unroll
  for (int i = 0; i < T::LD; ++i)
    load(reinterpret_cast<const char *>(q) + head_row0 * (D * 2),
         (unsigned)min(row0 + i * T::RPI + lane / T::ROW16, R - 1) * (D * 2) + T::col(lane, i), 0u, i * 64);
}

// Elsewhere: the queries of wavefront wv's row blocks as operands, straight from memory (behind the first sets, whose way
// from HBM is longer than the 32 lines that each of these loads touches take).  Rows past R are row R-1, until ...
template <int D, int MB>
__device__ __forceinline__ void group_queries(const unsigned short *q, size_t head_row0, int R, int wv, int l32, int half,
                                              u32x4 (&qw)[MB][RowTile<D>::KS]) {
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const unsigned short *src = q + (head_row0 + min((wv * MB + mb) * 32 + l32, R - 1)) * D + half * 8;
#pragma unroll
    for (int s = 0; s < RowTile<D>::KS; ++s) qw[mb][s] = *reinterpret_cast<const u32x4 *>(src + s * 16);
  }
}
// ... they are zeroed.
template <int MB, int KS>
__device__ __forceinline__ void zero_padding(const u32x4 (&qw)[MB][KS], int R, int wv, int l32, bf16x8 (&qf)[MB][KS]) {
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const unsigned keep = (wv * MB + mb) * 32 + l32 < R ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[mb][s] = as_bf16(qw[mb][s] & keep);
  }
}

// Sweep 1: the sets of a sequence are dealt out over the workgroups of the head.
template <int D, int MB, int RS, bool F16>
__device__ __forceinline__ void stats_group(const SeqTab &st, const ChunkTab &cp, const Dims &dm, float c_log2,
                                            const unsigned short *__restrict__ q, const unsigned short *__restrict__ K,
                                            float2 *__restrict__ part, int part_len, const TopkCarry &tc) {
  typedef Group<D, MB, RS> G;
  typedef RowTile<D> T;
  constexpr int KS = T::KS, ST = G::ST, NT = G::NT;
  __shared__ u32x4 kt[2][G::SETW];
  const int tid = threadIdx.x, lane = tid & 63;
  if (tc.zero_begin)
    for (unsigned i = blockIdx.x * NT + tid; i < tc.zero_words; i += gridDim.x * NT) tc.zero_begin[i] = 0u;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int h = dm.h_kv;
  const int c = blockIdx.x % h, cg = blockIdx.x / h;
  const int b = find_seq(cp, st.batch, cg);
  const int first = cg - cp.off[b], stride = cp.off[b + 1] - cp.off[b];
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const size_t head_row0 = (size_t)b * RQ + (size_t)c * R;
  // Sets of two tiles where those of four would give some workgroups two or three tiles more than their part_len keys
  // are, an eighth of these or more.  The sweep in us, sets of four / two / one, 8 heads, d = 128, by tiles a workgroup:
  //   256 rows   3: 6.5 / 7.4 / 7.2     5: 8.9 / 8.5 / 8.7     6: 9.5 / 8.8 / 9.5     7: 9.5 / 10.0 / 10.4
  //              9: 11.8 / 11.3 / 11.7  10: 11.9 / 11.3 / 12.2  11: 12.0 / 12.5 / 13.1  18: 16.6 / 16.6 / 18.6
  //              21: 19.3 / 19.4 / 21.0  26: 21.1 / 21.4 / 23.9  30: 23.2 / 23.7 / 26.7
  //   512 rows   5: 14.3 / 13.2 / 13.0  7: 15.0 / 15.0 / 14.8  10: 18.4 / 17.2 / 17.8  11: 18.7 / 18.9 / 18.6
  const int ntiles = (n + TILE - 1) / TILE, share_of = part_len / TILE, over = -share_of & (ST - 1);
  const int stt = over >= 2 && over * 8 >= share_of ? 2 : ST;
  const int nsets = (ntiles + stt - 1) / stt;
  const int iters = first < nsets ? (nsets - 1 - first) / stride + 1 : 0;
  const char *kbase = reinterpret_cast<const char *>(K) +
                      ((size_t)st.tok_off[b] * dm.k_stride_tok + (size_t)c * dm.k_stride_head) * 2;
  const unsigned tok_bytes = (unsigned)dm.k_stride_tok * 2u;
  // a wavefront loads every RS-th instruction's rows of a set; rows past the sequence are its last
  auto issue = [&](int it) {
    const int key0 = (first + it * stride) * (stt * TILE), lim = min(n - 1 - key0, stt * TILE - 1);
    const char *sb = scalar_address(kbase + (long long)key0 * tok_bytes);
#pragma unroll
    for (int i = 0; i < G::LDW; ++i) {
      const int at = i * RS + wv;                      // load instruction of the set
      if (i < G::LDW * stt / ST) {
        const unsigned row = (unsigned)min((int)(at * T::RPI + lane / T::ROW16), lim);
        load_to_lds_untracked(sb, __umul24(row, tok_bytes) + T::col(lane, at), 0u, &kt[it & 1][at * 64]);
      }
    }
  };
  unsigned rd[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) rd[s] = T::operand(l32, half, s);
  bf16x8 qf[MB][KS];
  // (the second set is asked for when the first one and the queries are there: loads return in order, and a short
  // sequence would wait for all of it before it starts; 256 rows, 2011 keys: 7.8 us, 7.1 so)
  if constexpr (G::Q_LDS) {
    u32x4 *qs = &kt[1][wv * (G::SETW / RS)], qw[MB][KS];
    auto query_block = [&](int mb) {
      load_query_block<D>(q, head_row0, R, (wv * MB + mb) * 32, lane, [&](const char *base, unsigned off, unsigned at, int word) { load_to_lds_untracked(base, off, at, qs + word); });
    };
    auto read_query_block = [&](int mb) {
#pragma unroll
      for (int s = 0; s < KS; ++s) qw[mb][s] = qs[rd[s]];
    };
    query_block(0);
    if (iters > 0) issue(0);
    if (iters > 0 && stt == ST) wait_vmem<G::LDW>(); else wait_vmem<0>();
    read_query_block(0);
    wait_lds();
    query_block(1);
    wait_vmem<0>();
    read_query_block(1);
    zero_padding<MB, KS>(qw, R, wv, l32, qf);
    lds_barrier();                                     // (the second set takes the queries' place)
  } else {
    if (iters > 0) issue(0);
    u32x4 qw[MB][KS];
    group_queries<D, MB>(q, head_row0, R, wv, l32, half, qw);
    zero_padding<MB, KS>(qw, R, wv, l32, qf);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(qf[mb][KS - 1]));
  }
  wait_vmem<0>();
  if (iters > 1) issue(1);

  bf16x8 kf[KS];
  floatx16 acc[2];
  float rm[MB], rl[MB];
  float ref = 0.0f, nmx = 0.0f, usum = 0.0f;
  auto share = [&](auto lazy_tag, floatx16 &a, int mb, int s) {          // (as in stats_own)
    if constexpr (decltype(lazy_tag)::value) {
      if (s == 0) usum = 0.0f;
#pragma unroll
      for (int v = s * 16 / KS; v < (s + 1) * 16 / KS; ++v) usum += fast_exp2(fmaf(a[v], c_log2, -rm[mb]));
      if (s == KS - 1) add_kept(a, c_log2, usum, rm[mb], rl[mb]);
    } else {
      if (s == 0) {
        float tm = a[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tm = fmaxf(tm, a[r]);
        nmx = fmaxf(rm[mb], tm * c_log2);
        ref = (nmx == -INFINITY) ? 0.0f : nmx;
        usum = 0.0f;
      } else {
#pragma unroll
        for (int v = (s - 1) * 16 / (KS - 1); v < s * 16 / (KS - 1); ++v) usum += fast_exp2(fmaf(a[v], c_log2, -ref));
      }
      if (s == KS - 1) {
        rl[mb] = rl[mb] * fast_exp2(rm[mb] - ref) + usum;
        rm[mb] = nmx;
      }
    }
  };
  // the sequence's last tile, if it is not full, is the last of its workgroup and comes after the loop
  const bool tail = iters > 0 && first + (iters - 1) * stride == nsets - 1 && n % TILE != 0;
  auto tiles_of = [&](int it) { return min(stt, ntiles - (first + it * stride) * stt); };
  const int plain = iters > 0 ? (iters - 1) * stt + tiles_of(iters - 1) - (tail ? 1 : 0) : 0;
  auto loop = [&](auto lazy_tag) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = -INFINITY;      // (nothing before the first: no weight)
    for (int it = 0; it < iters; ++it) {
      const int nt = tiles_of(it), full = nt - (tail && it == iters - 1 ? 1 : 0);
      for (int t = 0; t < full; ++t) {
        const bool leave = t == nt - 1;                // the next tile is the next set's first (behind the last: whatever lies there)
        const u32x4 *src = leave ? &kt[(it + 1) & 1][0] : &kt[it & 1][(t + 1) * T::WORDS];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const int pmb = mb == 0 ? MB - 1 : mb - 1, cur = mb & 1;
          if (mb == MB - 1 && leave && it + 1 < iters) {
            wait_vmem<0>();
            lds_barrier();
            if (it + 2 < iters) issue(it + 2);
          }
          floatx16 a = {0};
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            a = mfma16<F16>(kf[s], qf[mb][s], a);
            if (s == 0) __builtin_amdgcn_sched_barrier(0);       // (as in stats_own)
            if (mb == MB - 1) kf[s] = as_bf16(src[rd[s]]);
            share(lazy_tag, acc[1 - cur], pmb, s);
            __builtin_amdgcn_sched_barrier(0);
          }
          acc[cur] = a;
          asm volatile("" : "+v"(rl[pmb]), "+v"(rm[pmb]));   // the vector work stays in front of this point
        }
      }
    }
    if (plain > 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s) share(lazy_tag, acc[1], MB - 1, s);
    }
  };
  static_assert(MB % 2 == 0, "a row block's products alternate between two places");
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) { rm[mb] = -INFINITY; rl[mb] = 0.0f; }
  lds_barrier();                                       // the first set is there for everybody
  auto read_first = [&]() {
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = as_bf16(kt[0][rd[s]]);
  };
  // (the kept reference as in stats_own)
  if (plain >= 4) {
    read_first();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      floatx16 a = {0};
#pragma unroll
      for (int s = 0; s < KS; ++s) a = mfma16<F16>(kf[s], qf[mb][s], a);
      float tm = a[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) tm = fmaxf(tm, a[r]);
      rm[mb] = tm * c_log2;
      asm volatile("" : "+v"(rm[mb]));
      __builtin_amdgcn_sched_barrier(0);
    }
    loop(std::true_type{});
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) settle(rm[mb], rl[mb]);
  } else {
    if (iters > 0) read_first();
    loop(std::false_type{});
  }
  if (tail) {
    const int base = (ntiles - 1) * TILE;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      floatx16 a = {0};
#pragma unroll
      for (int s = 0; s < KS; ++s) a = mfma16<F16>(kf[s], qf[mb][s], a);
#pragma unroll
      for (int r = 0; r < 16; ++r)                     // key base + 8 (r/4) + 4 half + r%4
        if (base + 8 * (r / 4) + 4 * half + (r % 4) >= n) a[r] = -INFINITY;
#pragma unroll
      for (int s = 0; s < KS; ++s) share(std::false_type{}, a, mb, s);
      asm volatile("" : "+v"(rl[mb]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the two lane halves hold the same window row's statistics over different keys
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const float m2 = __shfl_xor(rm[mb], 32), s2 = __shfl_xor(rl[mb], 32);
    const float M = fmaxf(rm[mb], m2);
    const float rf = (M == -INFINITY) ? 0.0f : M;
    const float L = rl[mb] * fast_exp2(rm[mb] - rf) + s2 * fast_exp2(m2 - rf);
    const int row = (wv * MB + mb) * 32 + l32;
    if (half == 0 && row < R) part[(size_t)cg * RQ + (size_t)c * R + row] = make_float2(M, L);     // (base 2)
  }
}

// Sweep 2: a workgroup owns chunk_len consecutive keys, as in weights_own.
template <int D, int MB, int RS, int CHUNK, bool F16, bool PR, bool WIDE>
__device__ __forceinline__ void weights_group(const SeqTab &st, const ChunkTab &ct, const ChunkTab &cp, const Dims &dm,
                                              float c_log2, const unsigned short *__restrict__ q,
                                              const unsigned short *__restrict__ K, const float *__restrict__ lse, float lse_mul,
                                              const float2 *__restrict__ part, float *__restrict__ out, int halo,
                                              int chunk_len, const TopkCarry &tc) {
  typedef Group<D, MB, RS> G;
  typedef RowTile<D> T;
  constexpr int KS = T::KS, ST = G::ST, NT = G::NT, RPAD = G::RPAD;
  constexpr int HALO = TILE, SPAN = CHUNK + 2 * HALO;
  constexpr int SKEYS = ST * TILE;                     // keys of a set
  // (two arrays, so that the compiler sees that reading one does not wait for loads into the other)
  __shared__ u32x4 kt0[G::SETW], kt1[G::SETW];
  __shared__ float sh_sum[3][RS][SKEYS];               // the row groups' sums over a set's keys, three sets in turn
  __shared__ __align__(16) float sh_lse[RPAD];
  __shared__ __align__(16) float sh_part[SPAN];
  constexpr int SL = 2 * NT / RPAD > 0 ? 2 * NT / RPAD : 1;      // threads that share two rows in the statistics combination
  static_assert(SL * RPAD == 2 * NT && 2 * SL * RPAD <= SPAN, "threads and rows must tile each other");
  float *sh_cm = sh_part, *sh_cl = sh_part + SL * RPAD;          // (the prologue's, before any score is there)
  static_assert(sizeof(kt0) >= RADIX_BINS * sizeof(unsigned), "the digit histogram takes the tiles' place");
  unsigned *sh_hist = reinterpret_cast<unsigned *>(kt0);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int h = dm.h_kv;
  const int c = blockIdx.x % h, cg = ct.off[st.batch] - 1 - (int)blockIdx.x / h;
  const int b = find_seq(ct, st.batch, cg);
  const int chunk = cg - ct.off[b], nch = ct.off[b + 1] - ct.off[b];
  const int n = st.n[b];
  const int R = dm.g * dm.w, RQ = dm.h_q * dm.w;
  const int kc0 = chunk * chunk_len, kc1 = min(n, kc0 + chunk_len);
  const int pool_r = halo || PR ? dm.pool_k / 2 : 0;
  const int tstep = PR ? TILE - 2 * pool_r : TILE;     // keys a tile advances by
  const int before = PR ? pool_r : 0;                  // keys of a tile in front of its first own
  const int k0 = halo && kc0 > 0 ? kc0 - HALO : kc0;
  const int k1 = halo ? min(n, kc1 + pool_r) : kc1;
  const int ntiles = (k1 - k0 + tstep - 1) / tstep, nsets = (ntiles + ST - 1) / ST;
  const size_t head_row0 = (size_t)b * RQ + (size_t)c * R;
  const int rot = (int)(((long long)chunk * nsets) / nch);
  auto set_of = [&](int it) {                          // backwards from a point that differs from workgroup to workgroup
    const int p = rot - 1 - it;
    return p < 0 ? p + nsets : p;
  };
  auto tiles_of = [&](int set) { return min(ST, ntiles - set * ST); };
  const char *kbase = reinterpret_cast<const char *>(K) +
                      ((size_t)st.tok_off[b] * dm.k_stride_tok + (size_t)c * dm.k_stride_head) * 2;
  const unsigned tok_bytes = (unsigned)dm.k_stride_tok * 2u;
  const int need_lo = max(kc0 - pool_r, 0), need_hi = min(kc1 - 1 + pool_r, n - 1);
  auto ask = [&](int it, auto &&load) {
    const int key0 = k0 + set_of(it) * (ST * tstep) - before, lim = need_hi - key0, lo = max(need_lo - key0, 0);     // (no set starts past need_hi)
    const char *sb = scalar_address(kbase + (long long)key0 * tok_bytes);
#pragma unroll
    for (int i = 0; i < G::LDW; ++i) {
      const int at = wv * G::LDW + i;
      const int rel = PR ? at / T::LD * tstep + at % T::LD * T::RPI : at * T::RPI;     // (overlapping tiles have rows of their own)
      const unsigned row = (unsigned)max(min(rel + (int)(lane / T::ROW16), lim), lo);
      load(sb, __umul24(row, tok_bytes) + T::col(lane, at), at * 64);
    }
  };
  auto issue = [&](int it) {
    ask(it, [&](const char *sb, unsigned off, int word) { load_to_lds_untracked(sb, off, 0u, (it & 1 ? kt1 : kt0) + word); });
  };
  unsigned rd[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) rd[s] = T::operand(PR ? pooled_row(l32) : l32, half, s);
  u32x4 qw[MB][KS];
  u32x4 *qs = kt1 + wv * (G::SETW / RS);               // the queries' way: this wavefront's share of the second set's place
  auto query_block = [&](int mb) {
    load_query_block<D>(q, head_row0, R, (wv * MB + mb) * 32, lane, [&](const char *base, unsigned off, unsigned at, int word) { load_to_lds(base, off, at, qs + word); });
  };
  auto read_query_block = [&](int mb) {
#pragma unroll
    for (int s = 0; s < KS; ++s) qw[mb][s] = qs[T::operand(l32, half, s)];
  };
  // The first set and the queries, counted by the compiler, so that its wait for what was asked for before does not
  // stop at them as well (loads return in order).
  auto request = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (G::Q_LDS) query_block(0);
    ask(0, [&](const char *sb, unsigned off, int word) { load_to_lds(sb, off, 0u, kt0 + word); });
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!G::Q_LDS) group_queries<D, MB>(q, head_row0, R, wv, l32, half, qw);
    __builtin_amdgcn_sched_barrier(0);
  };
  // (the first row block is there long before the first set, and the second one's way is hidden by it)
  auto queries = [&]() {
    if constexpr (G::Q_LDS) {
      wait_vmem<G::LDW>();
      read_query_block(0);
      wait_lds();
      query_block(1);
      wait_vmem<0>();
      read_query_block(1);
    }
  };
  float own_lse[(RPAD + NT - 1) / NT];
  if (lse) {
#pragma unroll
    for (int i = 0; i < (RPAD + NT - 1) / NT; ++i) own_lse[i] = lse[head_row0 + min(tid + i * NT, R - 1)] * lse_mul;
    request();
#pragma unroll
    for (int i = 0; i < (RPAD + NT - 1) / NT; ++i)
      if (tid + i * NT < RPAD) sh_lse[tid + i * NT] = tid + i * NT < R ? own_lse[i] : INFINITY;
  } else {
    // sweep 1's partials of this head's rows, two rows and every SL-th partial a thread (as in weights_own)
    constexpr int CB = 16;
    const int q2 = tid % (RPAD / 2), sl = tid / (RPAD / 2);
    const int row = min(2 * q2, max(R - 2, 0)), np = cp.off[b + 1] - cp.off[b];
    struct __attribute__((packed, aligned(8))) Pair { float m0, l0, m1, l1; };
    const float2 *pp = part + ((size_t)cp.off[b] * RQ + (size_t)c * R);
    Pair pml[CB];
    auto load_parts = [&](int p0) {
#pragma unroll
      for (int u = 0; u < CB; ++u) pml[u] = *reinterpret_cast<const Pair *>(pp + (unsigned)(min(p0 + u * SL, np - 1) * RQ + row));
    };
    float M0 = -INFINITY, L0 = 0.0f, M1 = -INFINITY, L1 = 0.0f;
    auto fold = [&](int p0) {
      float n0 = M0, n1 = M1;
#pragma unroll
      for (int u = 0; u < CB; ++u)
        if (p0 + u * SL < np) { n0 = fmaxf(n0, pml[u].m0); n1 = fmaxf(n1, pml[u].m1); }
      const float r0 = (n0 == -INFINITY) ? 0.0f : n0, r1 = (n1 == -INFINITY) ? 0.0f : n1;
      L0 *= fast_exp2(M0 - r0);
      L1 *= fast_exp2(M1 - r1);
#pragma unroll
      for (int u = 0; u < CB; ++u)
        if (p0 + u * SL < np) {
          L0 += pml[u].l0 * fast_exp2(pml[u].m0 - r0);
          L1 += pml[u].l1 * fast_exp2(pml[u].m1 - r1);
        }
      M0 = n0;
      M1 = n1;
    };
    load_parts(sl);
    request();
    fold(sl);
    for (int p0 = sl + CB * SL; p0 < np; p0 += CB * SL) {
      load_parts(p0);
      fold(p0);
    }
    if (2 * q2 == R - 1 && R > 1) { M0 = M1; L0 = L1; }
    *reinterpret_cast<float2 *>(&sh_cm[sl * RPAD + 2 * q2]) = make_float2(M0, M1);
    *reinterpret_cast<float2 *>(&sh_cl[sl * RPAD + 2 * q2]) = make_float2(L0, L1);
  }
  queries();
  lds_barrier();
  if (!lse) {
    for (int r = tid; r < RPAD; r += NT) {
      float Mt = -INFINITY;
#pragma unroll
      for (int i = 0; i < SL; ++i) Mt = fmaxf(Mt, sh_cm[i * RPAD + r]);
      const float ref = (Mt == -INFINITY) ? 0.0f : Mt;
      float Lt = 0.0f;
#pragma unroll
      for (int i = 0; i < SL; ++i) Lt += sh_cl[i * RPAD + r] * fast_exp2(sh_cm[i * RPAD + r] - ref);
      sh_lse[r] = (r < R) ? Mt + __builtin_amdgcn_logf(Lt) : INFINITY;
    }
    lds_barrier();
  }
  float l2[MB][PR ? 1 : 16];                           // log-sum-exp of the 16 rows (PR: the row) a lane sees in each row block
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if constexpr (PR) l2[mb][0] = sh_lse[(wv * MB + mb) * 32 + l32];
      else l2[mb][r] = sh_lse[(wv * MB + mb) * 32 + 8 * (r / 4) + 4 * half + (r % 4)];

  bf16x8 kf[KS];
  floatx16 acc[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = -INFINITY;
  float sum = 0.0f, keysum[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) keysum[i] = 0.0f;
  const float inv = 1.0f / (float)R;
  auto share = [&](floatx16 &a, int mb, int s) {       // a[r]: window row (wv*MB + mb)*32 + 8*(r/4) + 4*half + r%4
    constexpr int V = 16 / KS;
#pragma unroll
    for (int v = s * V; v < (s + 1) * V; ++v)
      if constexpr (PR) a[v] = fast_exp2(fmaf(a[v], c_log2, -l2[mb][0]));
      else sum += fast_exp2(fmaf(a[v], c_log2, -l2[mb][v]));
  };
  // the row groups' sums over the keys of the it-th set, added in a fixed order (all of them are there)
  auto combine = [&](int it) {
    const int set = set_of(it);
    for (int j = tid; j < SKEYS; j += NT) {
      float tot = 0.0f;
#pragma unroll
      for (int i = 0; i < RS; ++i) tot += sh_sum[it % 3][i][j];
      if constexpr (PR) {
        const int at = j % TILE, key = (set * ST + j / TILE) * tstep + at - pool_r;
        if (at >= pool_r && at < TILE - pool_r && key < k1 - k0) sh_part[key] = tot * inv;
      } else {
        if (set * SKEYS + j < ntiles * TILE) sh_part[set * SKEYS + j] = tot * inv;
      }
    }
  };
  bf16x8 qf[MB][KS];
  zero_padding<MB, KS>(qw, R, wv, l32, qf);
  wait_vmem<0>();
  lds_barrier();                                       // (the second set when the first one is there: as in stats_group)
  if (nsets > 1) issue(1);
#pragma unroll
  for (int s = 0; s < KS; ++s) kf[s] = as_bf16(kt0[rd[s]]);
  auto file = [&](int it, int t) {                     // a finished tile's sums over this wavefront's rows
    float *dst = &sh_sum[it % 3][wv][t * TILE];
    if constexpr (PR) {
      const float tot = sum_rows(keysum, lane);
      if (!(lane & 1)) dst[summed_key(lane)] = tot;
#pragma unroll
      for (int i = 0; i < 16; ++i) keysum[i] = 0.0f;
    } else {
      dst[l32] = sum_halves(sum);
      sum = 0.0f;
    }
  };
  int prev_it = 0, prev_t = 0;                         // set (in order of work) and place of the tile before the current one
  for (int it = 0; it < nsets; ++it) {
    const int nt = tiles_of(set_of(it));
    for (int t = 0; t < nt; ++t) {
      const bool leave = t == nt - 1;                  // the next tile is the next set's first (behind the last: whatever lies there)
      const u32x4 *src = leave ? (it & 1 ? kt0 : kt1) : (it & 1 ? kt1 : kt0) + (t + 1) * T::WORDS;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int pmb = mb == 0 ? MB - 1 : mb - 1, cur = mb & 1;
        if (mb == MB - 1 && leave && it + 1 < nsets) {
          wait_vmem<0>();
          lds_barrier();
          if (it + 2 < nsets) issue(it + 2);
          if (it > 0) combine(it - 1);
        }
        floatx16 a = {0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          a = PR ? mfma16<F16>(kf[s], qf[mb][s], a) : mfma16<F16>(qf[mb][s], kf[s], a);
          if (mb == MB - 1) kf[s] = as_bf16(src[rd[s]]);
          share(acc[1 - cur], pmb, s);
          __builtin_amdgcn_sched_barrier(0);
        }
        acc[cur] = a;
        if constexpr (PR) {
          pool_rows<WIDE>(acc[1 - cur], pool_r, keysum);
#pragma unroll
          for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(keysum[i]));
          __builtin_amdgcn_sched_barrier(0);
        } else {
          asm volatile("" : "+v"(sum));                // the vector work stays in front of this point
        }
        if (mb == 0) file(prev_it, prev_t);            // (in front of the first: the place is written again)
      }
      prev_it = it;
      prev_t = t;
    }
  }
#pragma unroll
  for (int s = 0; s < KS; ++s) share(acc[1], MB - 1, s);
  if constexpr (PR) pool_rows<WIDE>(acc[1], pool_r, keysum);
  file(prev_it, prev_t);
  wait_vmem<0>();
  __syncthreads();
  if (nsets > 1) combine(nsets - 2);
  combine(nsets - 1);
  if (tc.hist0)
    for (int i = tid; i < RADIX_BINS; i += NT) sh_hist[i] = 0u;
  __syncthreads();
  pool_and_file<NT, CHUNK>(sh_part, sh_hist, out + st.score_off[b] + (size_t)c * n, kc0, kc1, k0, n, chunk_len,
                           halo ? dm.pool_k / 2 : 0, tc, b, b * h + c);
}

// MB row blocks of 32 window rows times RS are a workgroup's rows, RS * KG its wavefronts.  Up to 128 rows a
// wavefront takes all of them and the wavefronts split the keys; beyond, RS wavefronts share a tile.  CHUNK: what
// a workgroup of sweep 2 has room for (sweep 1 keeps no scores: 0).
template <int D, int MB, int RS, int KG, int CHUNK, int PASS, bool F16, bool PR = false, bool WIDE = false>
__global__ __launch_bounds__(64 * RS * KG, MB * RS <= 4 ? 2 : 1) void score_mfma_kernel(
    SeqTab st, ChunkTab ct, ChunkTab cp, Dims dm, float c_log2, const unsigned short *__restrict__ q,
    const unsigned short *__restrict__ K, const float *__restrict__ lse, float lse_mul,
    float2 *__restrict__ part, float *__restrict__ out, int halo, int chunk_len,
    TopkCarry tc) {
  if constexpr (MB * RS <= 4 && PASS == 1)
    stats_own<D, MB * RS, F16>(st, cp, dm, c_log2, q, K, part, tc);
  else if constexpr (MB * RS <= 4)
    weights_own<D, MB, RS, CHUNK, F16, PR, WIDE>(st, ct, cp, dm, c_log2, q, K, lse, lse_mul, part, out, halo, chunk_len, tc);
  else if constexpr (PASS == 1)
    stats_group<D, MB, RS, F16>(st, cp, dm, c_log2, q, K, part, chunk_len, tc);
  else
    weights_group<D, MB, RS, CHUNK, F16, PR, WIDE>(st, ct, cp, dm, c_log2, q, K, lse, lse_mul, part, out, halo, chunk_len, tc);
}

template <bool F16, int D, int MB, int RS, int KG, int CHUNK>
void run_mfma(const MfmaVariant &v, const SeqTab &st, const Dims &dm, const void *q, const void *K,
              const float *row_lse, float *scores, char *ws, const ScorePlan &pl,
              const TopkCarry &tc, bool pool_rows, hipStream_t s) {
  const ChunkTab ct = make_chunks(st, v.len);
  const ChunkTab cp = make_chunks(st, v.part_len);     // sweep 1's workgroups
  const int nblk = ct.off[st.batch] * dm.h_kv;
  const float c_log2 = dm.scale * LOG2E;
  float2 *part = (float2 *)(ws + pl.part);
  float *lse = (float *)(ws + pl.lse), *raw = (float *)(ws + pl.raw);
  const dim3 block(64 * RS * KG);
  const bool fuse_lse = v.fuse_lse, fuse_pool = v.fuse_pool;
  const float *use_lse = row_lse;              // the caller's in the natural-log domain, the combined one in base 2
  const float lse_mul = row_lse ? LOG2E : 1.0f;
  if (!row_lse) {
    ADAKV_LAUNCH("score_stats_mfma", (score_mfma_kernel<D, MB, RS, KG, 0, 1, F16>), dim3(cp.off[st.batch] * dm.h_kv),
                 block, s, st, cp, cp, dm, c_log2, (const unsigned short *)q,
                 (const unsigned short *)K, (const float *)nullptr, 1.0f, part,
                 (float *)nullptr, 0, v.part_len, tc);
    if (!fuse_lse) {
      launch_lse_combine(st, cp, dm.h_q * dm.w, part, lse, s);
      use_lse = lse;
    }
  } else if (tc.zero_begin) {
    launch_topk_clear(tc, s);                 // no statistics sweep to do the clearing
  }
  if (pool_rows) {
    // the printed order of Alg. 2 l.4: the sweep pools every row itself and writes final scores
    auto *kernel = dm.pool_k / 2 >= POOL_WIDE_RADIUS ? score_mfma_kernel<D, MB, RS, KG, CHUNK, 2, F16, true, true>
                                                     : score_mfma_kernel<D, MB, RS, KG, CHUNK, 2, F16, true>;
    ADAKV_LAUNCH("score_weights_mfma", kernel, dim3(nblk), block, s, st, ct, cp,
                 dm, c_log2, (const unsigned short *)q, (const unsigned short *)K, use_lse, lse_mul, part, scores, 0, v.len, tc);
    return;
  }
  ADAKV_LAUNCH("score_weights_mfma", (score_mfma_kernel<D, MB, RS, KG, CHUNK, 2, F16>), dim3(nblk),
               block, s, st, ct, cp, dm, c_log2, (const unsigned short *)q, (const unsigned short *)K,
               use_lse, lse_mul, part, fuse_pool ? scores : raw, fuse_pool ? 1 : 0, v.len, tc);
  if (!fuse_pool) launch_pool(st, dm, raw, scores, s);
}

template <int D, bool F16>
hipError_t run_mfma_d(const MfmaVariant &v, const SeqTab &st, const Dims &dm, const void *q,
                      const void *K, const float *row_lse, float *scores, char *ws,
                      const ScorePlan &pl, const TopkCarry &tc, bool pool_rows, hipStream_t s) {
#define ADAKV_MFMA_CASE(MB, RS, KG, CHUNK)                                                      \
  if (v.mb == MB && v.rs == RS && v.kg == KG && v.chunk == CHUNK) {                             \
    run_mfma<F16, D, MB, RS, KG, CHUNK>(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s); \
    return hipGetLastError();                                                                   \
  }
  ADAKV_MFMA_CASE(1, 1, 4, 2048)
  ADAKV_MFMA_CASE(2, 1, 4, 2048)
  ADAKV_MFMA_CASE(2, 2, 2, 4096)
  ADAKV_MFMA_CASE(2, 2, 2, 2048)
  ADAKV_MFMA_CASE(2, 2, 2, 1024)
  ADAKV_MFMA_CASE(2, 2, 2, 512)
  ADAKV_MFMA_CASE(2, 4, 1, 2048)
  ADAKV_MFMA_CASE(2, 4, 1, 1024)
  if constexpr (D == 128) { ADAKV_MFMA_CASE(2, 8, 1, 2048) ADAKV_MFMA_CASE(2, 8, 1, 4096) }
  else { ADAKV_MFMA_CASE(4, 4, 1, 1024) }
#undef ADAKV_MFMA_CASE
  return hipErrorInvalidValue;                 // a variant nobody instantiated
}

}  // namespace

// The instantiations are split over four translation units by head dimension and element type,
// so that they compile side by side: ADAKV_MFMA_PART = 1 .. 4 builds one quarter (part 1 also the
// host functions below), 0 or undefined everything.
#ifndef ADAKV_MFMA_PART
#define ADAKV_MFMA_PART 0
#endif
#define ADAKV_MFMA_ARGS                                                                          \
  const MfmaVariant &v, const SeqTab &st, const Dims &dm, const void *q, const void *K,          \
      const float *row_lse, float *scores, char *ws, const ScorePlan &pl, const TopkCarry &tc,   \
      bool pool_rows, hipStream_t s
hipError_t run_mfma_d64_bf16(ADAKV_MFMA_ARGS);
hipError_t run_mfma_d64_fp16(ADAKV_MFMA_ARGS);
hipError_t run_mfma_d128_bf16(ADAKV_MFMA_ARGS);
hipError_t run_mfma_d128_fp16(ADAKV_MFMA_ARGS);
#if ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 1
hipError_t run_mfma_d64_bf16(ADAKV_MFMA_ARGS) { return run_mfma_d<64, false>(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s); }
#endif
#if ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 2
hipError_t run_mfma_d64_fp16(ADAKV_MFMA_ARGS) { return run_mfma_d<64, true>(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s); }
#endif
#if ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 3
hipError_t run_mfma_d128_bf16(ADAKV_MFMA_ARGS) { return run_mfma_d<128, false>(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s); }
#endif
#if ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 4
hipError_t run_mfma_d128_fp16(ADAKV_MFMA_ARGS) { return run_mfma_d<128, true>(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s); }
#endif
#undef ADAKV_MFMA_ARGS

#if ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 1
// 16-bit inputs with at most 512 window rows per KV head (g*w); anything else takes the FMA path.
bool mfma_path_supported(const Dims &dm, int dtype) {
  return (dtype == ADAKV_BF16 || dtype == ADAKV_FP16) && dm.g * dm.w <= 512 && (dm.d == 64 || dm.d == 128) &&
         dm.k_stride_tok * 2 < (1ll << 24);   // 24-bit multiplies address a row inside a tile set
}

// Workgroups that chunks of `len` keys make.
static long long workgroups(const SeqTab &st, const Dims &dm, int len) {
  return (long long)count_chunks(st, len) * dm.h_kv;
}

// The one place that decides which instantiation scores a layer: rows per wavefront and the
// split of a workgroup's wavefronts over window rows (RS) and keys (KG) follow the number of
// window rows per KV head; the chunk length follows the number of workgroups.
MfmaVariant choose_mfma_variant(const SeqTab &st, const Dims &dm) {
  MfmaVariant v;
  const int R = dm.g * dm.w;
  int slots, most;                             // workgroups the chip holds at a time; longest chunk
  // (most: at 128 rows and d = 128 what half of a compute unit's LDS holds beside four wavefronts' tiles)
  if (R <= 64) { v = {R <= 32 ? 1 : 2, 1, 4, 2048, 0, 0, false, false}; slots = 256; most = 2048; }
  else if (R <= 128) { v = {2, 2, 2, 512, 0, 0, false, false}; slots = 512; most = dm.d == 128 ? OWN_MOST : 4096; }
  else if (R <= 256) { v = {2, 4, 1, 1024, 0, 0, false, false}; slots = 512; most = 2048; }
  // 512 rows: eight wavefronts of 64 rows; with d = 64 a row block needs half the registers and
  // a tile half the loads, so four wavefronts of 128 rows.
  else if (dm.d == 128) { v = {2, 8, 1, 2048, 0, 0, false, false}; slots = 256; most = 4096; }
  else { v = {4, 4, 1, 1024, 0, 0, false, false}; slots = 256; most = 1024; }
  // Chunk length.  A workgroup's set-up and epilogue (4 and 7 us) want long chunks, the chip wants
  // to be full, and workgroups beyond what it holds at a time wait for a second round.  So: the
  // shortest chunk that gives every compute unit at most one workgroup, down to 64 keys (128 where
  // four wavefronts take a tile each); if that is longer than `one`, one resident round of
  // `slots`, and as many rounds as the longest chunk makes necessary beyond that.  Both sweeps
  // together, 8 KV heads of dimension 128, against fixed lengths of 512 to 4096 (us):
  //   rows   700 keys       2011           8000           20000          50021          100000
  //     32   20.1 -> 13.7   34.4 -> 13.2   35.3 -> 16.8   36.6 -> 23.2   42.3 -> 42.9   87.4 -> 82.6
  //    128   23.0 -> 14.6   24.9 -> 15.8   26.2 -> 21.4   37.2 -> 32.6   68.6 -> 53.8  109.6 -> 87.6
  //    256   39.3 -> 16.3   51.7 -> 17.8   53.8 -> 25.8   57.1 -> 44.0   84.2 -> 75.6  159.5 -> 130.9
  //    512   55.8 -> 24.2  123.8 -> 25.6  128.4 -> 38.9  132.6 -> 63.1  137.7 -> 119.8 271.9 -> 216.8
  // `one` is 512 keys: two shorter workgroups on a compute unit instead of one pay the set-up
  // twice and fill the chip unevenly (between 256 and 512 of them), while one workgroup of more
  // than 512 keys hides too little latency.  One against two (us, both sweeps):
  //   rows    8000 keys      9600           11000          12500          14400          15800
  //    128   21.4 | 23.2   22.8 | 26.8    24.2 | 27.2    25.5 | 27.6    27.4 | 28.2    28.0 | 28.8
  //    256   25.8 | 30.1   28.8 | 36.0    30.4 | 36.5    33.2 | 36.9    36.0 | 38.2    37.8 | 39.0
  // 4.1 us of two at 256 rows is the kernel that combines their statistics, so where a sequence is short
  // enough that sweep 2 combines either way the two come closer, and at d = 64, where a workgroup's
  // stream is half as long, they win: line at 384 there.  256 rows, 8 heads, 512 | 384:
  //   keys        14000         16000       3200 .. 484    5000 4000 3000    7000 5000    6 x 2000
  //   d = 64    27.5 | 26.7   29.5 | 28.6   27.6 | 26.2     25.9 | 25.4    25.9 | 25.2   26.0 | 25.4
  //   d = 128   31.1 | 31.3   34.0 | 34.0   34.3 | 34.1     30.4 | 32.1    30.3 | 31.8   30.4 | 31.7
  const int unit = TILE * v.kg;
  auto shortest = [&](int from, long long wgs) {       // chunk of at least `from` keys that makes `wgs` workgroups at most
    int lo = from / unit, hi = most / unit;
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (workgroups(st, dm, mid * unit) <= wgs) hi = mid;
      else lo = mid + 1;
    }
    return hi * unit;
  };
  int longest = 0;
  for (int b = 0; b < st.batch; ++b) longest = st.n[b] > longest ? st.n[b] : longest;
  const int one = v.rs == 4 && dm.d == 64 && (longest + 255ll) / 256 * R <= 8192 ? 384 : 512;
  v.len = shortest(unit > 64 ? unit : 64, 256);
  if (v.len > one) {
    const long long rounds = (workgroups(st, dm, most) + slots - 1) / slots;
    v.len = shortest(256, rounds * slots);
  }
  // Sweep 1 of up to 256 rows is not bound to the chunks: one resident round of workgroups over all sequences, as many
  // rounds as there are heads for beyond that, and never more workgroups than sweep 2's chunks.  Up to 128 rows the
  // tiles' place in LDS leaves one workgroup per compute unit at d = 128, two at d = 64.  Beyond 128 rows two would
  // fit, but one halves the partials, so that sweep 2 can combine them itself: 20000 keys x 8 heads, 256 rows
  // 41.3 -> 38.5 us, 50021 74.3 -> 73.3; with chunks of more than 1024 keys a wavefront alone on its SIMD loses more
  // than that kernel takes (131072 keys: 168.7 | 170.2).
  auto stats_len = [&](int len, int least) {           // sweep 1's keys per workgroup beside chunks of len, no fewer than least
    if (!(R <= 128 || (R <= 256 && len <= 1024))) return len;
    const long long room = dm.d == 128 || R > 128 ? 256 : 512, heads = (long long)st.batch * dm.h_kv;
    const long long wgs = (heads + room - 1) / room * room;
    if (workgroups(st, dm, least) <= wgs) return least;
    int lo = least / TILE, hi = longest / TILE + 1 > lo ? longest / TILE + 1 : lo;
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (workgroups(st, dm, mid * TILE) <= wgs) hi = mid;
      else lo = mid + 1;
    }
    return hi * TILE;
  };
  v.part_len = stats_len(v.len, v.len);
  // More workgroups of sweep 1 are more partial statistics: a layer that fits into the built-in scratch array with
  // the longest chunks (at 65 to 128 rows, whose chunks end at OWN_MOST, with partials per 4096 keys) gets no split
  // that would take it past the array's end (1 KiB for the alignment of the parts, asked of the split alone, so that
  // a layer that just fits keeps fitting).
  auto need = [&](int part_len) { return score_workspace(st, dm, part_len) + plan_topk_bytes(st, dm); };
  if (need(v.part_len) + 1024 > (size_t)ADAKV_STATIC_SCRATCH_BYTES) {
    const int fewest = stats_len(most, most == OWN_MOST ? 4096 : most);
    if (need(fewest) <= (size_t)ADAKV_STATIC_SCRATCH_BYTES) { v.len = most; v.part_len = fewest; }
  }
  // The instantiation: the smallest score array in LDS that holds a chunk; with 512 rows a compute
  // unit holds one workgroup either way and long sequences take the larger.
  while (v.chunk < v.len) v.chunk *= 2;
  if (v.rs == 8 && workgroups(st, dm, 4096) >= 256) v.chunk = 4096;
  // Fused forms: sweep 2 combines sweep 1's partial statistics itself unless a head has so many
  // (chunks x rows) that every workgroup re-reading them would cost more than a kernel (one round of
  // the combination's loads: 131072 keys x 512 rows 141.5 us fused, 4.1 + 138.9 apart), and it
  // applies the max-pool itself when the pool radius fits into the one-tile halo.
  int max_chunks = 0;
  for (int b = 0; b < st.batch; ++b) {
    const int k = (st.n[b] + v.part_len - 1) / v.part_len;
    max_chunks = k > max_chunks ? k : max_chunks;
  }
  v.fuse_lse = (long long)max_chunks * R <= (v.rs == 8 ? 16384 : 8192);
  v.fuse_pool = dm.pool_k / 2 <= TILE;
  return v;
}

hipError_t launch_score_mfma(const SeqTab &st, const Dims &dm, int dtype, const void *q,
                             const void *K, const float *row_lse, float *scores, char *ws,
                             const ScorePlan &pl, const TopkCarry &tc, bool pool_rows,
                             hipStream_t s) {
  const MfmaVariant &v = pl.mfma;
  if (dtype == ADAKV_FP16)
    return dm.d == 64 ? run_mfma_d64_fp16(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s)
                      : run_mfma_d128_fp16(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s);
  return dm.d == 64 ? run_mfma_d64_bf16(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s)
                    : run_mfma_d128_bf16(v, st, dm, q, K, row_lse, scores, ws, pl, tc, pool_rows, s);
}

// The printed order of Alg. 2 l.4 (pool every row, then average) runs on the matrix cores as long
// as a tile has at least 18 inner keys of its 32 (pool radius up to 7); wider pools take the FMA path.
bool mfma_pool_rows_supported(const Dims &dm, int dtype) {
  return mfma_path_supported(dm, dtype) && dm.pool_k / 2 <= MFMA_POOL_ROWS_MAX_RADIUS;
}
#endif  // ADAKV_MFMA_PART == 0 || ADAKV_MFMA_PART == 1

}  // namespace adakv
