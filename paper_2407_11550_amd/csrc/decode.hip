// Decode side of the flattened per-head cache (Section 3.5): the cache update of Eq. (1) and
// one decoding step of Eq. (2) per query head over segments of different lengths.
//
// Layout: segment s = b*h_kv + c starts at row cu[s] + s*headroom of K_cache / V_cache and holds
// seg_len[s] rows of ROWB = d*sizeof(T) bytes, so a segment is one contiguous byte range.
//
// Attention: HBM-bound (every cached K and V row is read once, 2*ROWB bytes for 4*g*d flops).
// 16-bit caches run both products on the matrix cores (decode_mfma_kernel); fp32 caches, and 16-bit ones
// with so few query heads per KV head that the matrix instructions stay empty, run on the vector ALUs
// (decode_attn_kernel): there a row is read by LPR = ROWB/16 neighbouring lanes, 16 bytes each: every load
// instruction of a wavefront fetches 64/LPR whole rows = 1 KB of consecutive memory.
// Segment lengths live on the device, so the host launches an upper bound of workgroups
// (capacity / split + segments); each workgroup finds its segment and its part of it from a prefix sum
// of the lengths, writes partial (max, sum, weighted value sum) per query head, and a second kernel
// merges the parts of each segment.  Where no segment of a layer can be long, one workgroup takes each
// segment (decode_mfma_kernel, WHOLE) and writes the result itself: no prefix sum, no merge.
#include <math.h>

#include <type_traits>

#include "common.h"

namespace adakv {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float M_INIT = -1.0e30f;    // finite "no row seen yet" maximum: exp2(-inf - M_INIT) = 0

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false);
  return x + __builtin_bit_cast(float, y);
}

// Sum over the LPR neighbouring lanes that share a row; every one of them gets the sum.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0xB1>(x);                       // quad_perm [1,0,3,2]
  x = dpp_add<0x4E>(x);                       // quad_perm [2,3,0,1]
  if (LPR >= 8) x = dpp_add<0x141>(x);        // row_half_mirror: lane i <-> 7-i
  if (LPR >= 16) x = dpp_add<0x140>(x);       // row_mirror: lane i <-> 15-i
  if (LPR >= 32) x += __shfl_xor(x, 16);
  return x;
}

struct f16_t { unsigned short bits; };        // IEEE half: tag type (bf16: unsigned short)
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int EPL = 4;
  static __device__ __forceinline__ void widen(u32x4 v, float (&f)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned int word = v[i];          // a copy: bit_cast of the vector element itself
      f[i] = __builtin_bit_cast(float, word);  // reads element 0 for every i
    }
  }
};

template <> struct Elem<unsigned short> {     // bf16
  static constexpr int EPL = 8;
  static __device__ __forceinline__ void widen(u32x4 v, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned int word = v[i];
      f[2 * i] = __builtin_bit_cast(float, word << 16);
      f[2 * i + 1] = __builtin_bit_cast(float, word & 0xffff0000u);
    }
  }
};
template <> struct Elem<f16_t> {
  static constexpr int EPL = 8;
  static __device__ __forceinline__ void widen(u32x4 v, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned int word = v[i];
      f[2 * i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(word & 0xffffu));
      f[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (unsigned short)(word >> 16));
    }
  }
};

// Rows of segment s this call works on: the rows held, plus the row the call itself appends
// (`grow` = 1) if the segment has room for it.
__device__ __forceinline__ int rows_held(const int *cu, const int *seg_len, int s, int headroom,
                                         int grow) {
  const int cap = cu[s + 1] - cu[s] + headroom;
  const int held = min(max(seg_len[s], 0), cap);   // a corrupt length can never leave the segment
  return held + (held < cap ? grow : 0);
}

// What a workgroup works on: part `j` of the `parts` that the `rows` rows of segment s are split into.
struct Work {
  int s, j, parts, rows, first_row;
  bool appended;                               // the last row is the one the call appends
};

// Finds it from a prefix sum, over the segments, of the parts that their lengths make (blocks of `split` rows).  The
// same in all lanes.  False: the workgroup has nothing to do (the launch is an upper bound).  The merge kernel finds a
// segment's partial results through seg_tab; the launch has at least one workgroup per segment, and workgroup s
// files the entry of segment s.
//
// Up to 64 segments every wavefront does it for itself, a segment a lane, without LDS or a barrier (by the other way a
// workgroup knew its rows 1.5 us after it had started; the kernel over 8 segments of 512 rows 5.4 -> 4.8 us, over 64 of
// 1500 13.3 -> 12.6).  Beyond, thread t of
// the workgroup takes segments t*per .. t*per+per-1 and the result goes through sh[0..21].
template <int NWV = 4>
__device__ __forceinline__ bool find_work(int nseg, int per, int split, int headroom, int grow, const int *cu,
                                          const int *seg_len, int *sh, int4 *seg_tab, Work &wk) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, blk = (int)blockIdx.x;
  if (nseg <= 64) {
    const int s = min(lane, nseg - 1);
    const int from = cu[s], cap = cu[s + 1] - from + headroom;
    const int held = min(max(seg_len[s], 0), cap);       // (as in rows_held)
    const int now = held + (held < cap ? grow : 0);
    const int nb = lane < nseg ? (now + split - 1) / split : 0;
    const int upto = wave_scan_incl(nb), first = upto - nb;
    if (lane == blk && lane < nseg && wv == 0) seg_tab[s] = make_int4(first, nb, now, now - held);
    const unsigned long long here = __ballot(blk >= first && blk < upto);
    if (here == 0) return false;
    const int L = __ffsll(here) - 1;
    wk.s = L;
    wk.j = blk - __builtin_amdgcn_readlane(first, L);
    wk.parts = __builtin_amdgcn_readlane(nb, L);
    wk.rows = __builtin_amdgcn_readlane(now, L);
    wk.first_row = __builtin_amdgcn_readlane(from, L);
    wk.appended = __builtin_amdgcn_readlane(now - held, L) != 0;
    return true;
  }
  int mine = 0;
  for (int i = 0; i < per; ++i) {
    const int s = tid * per + i;
    if (s < nseg) mine += (rows_held(cu, seg_len, s, headroom, grow) + split - 1) / split;
  }
  const int inc = wave_scan_incl(mine);
  if (lane == 63) sh[wv] = inc;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int i = 0; i < NWV; ++i) {
    const int v = sh[i];
    if (i < wv) before += v;
    total += v;
  }
  int first = before + inc - mine;
  for (int i = 0; i < per; ++i) {
    const int s = tid * per + i;
    if (s >= nseg) break;
    const int now = rows_held(cu, seg_len, s, headroom, grow);
    const int appended = now - rows_held(cu, seg_len, s, headroom, 0);
    const int nb = (now + split - 1) / split;
    if (blk >= first && blk < first + nb) {
      sh[16] = s;
      sh[17] = blk - first;
      sh[18] = now;
      sh[19] = cu[s];
      sh[20] = appended;
      sh[21] = nb;
    }
    if (s == blk) seg_tab[s] = make_int4(first, nb, now, appended);
    first += nb;
  }
  if (blk >= total) return false;
  __syncthreads();
  wk.s = __builtin_amdgcn_readfirstlane(sh[16]);
  wk.j = __builtin_amdgcn_readfirstlane(sh[17]);
  wk.rows = __builtin_amdgcn_readfirstlane(sh[18]);
  wk.first_row = __builtin_amdgcn_readfirstlane(sh[19]);
  wk.appended = __builtin_amdgcn_readfirstlane(sh[20]) != 0;
  wk.parts = __builtin_amdgcn_readfirstlane(sh[21]);
  return true;
}

// ---------------------------------------------------------------------------------------------
// Query heads one wavefront carries: at most four (queries and accumulators take 2*GW*EPL
// registers).  A larger group is split over NGRP sets of four wavefronts that read the
// same rows at the same time (the second read of a row is a cache hit).
template <typename T, int G> struct HeadSplit {
  static constexpr int GW = G > 4 ? 4 : G;
  static constexpr int NGRP = G / GW;
};

template <typename T, int D, int G>
__global__ __launch_bounds__((256 * HeadSplit<T, G>::NGRP)) void decode_attn_kernel(
    int nseg, int h, int per, int split, int headroom, float c_log2, const T *__restrict__ q,
    const char *__restrict__ k_new, const char *__restrict__ v_new, const int *__restrict__ cu,
    const int *__restrict__ seg_len, char *Kc, char *Vc, float *__restrict__ part_acc,
    float *__restrict__ part_ml, int4 *__restrict__ seg_tab) {
  constexpr int EPL = Elem<T>::EPL;
  constexpr int ROWB = D * (int)sizeof(T);
  constexpr int LPR = ROWB / 16;               // lanes per row
  constexpr int RPW = 64 / LPR;                // rows per wavefront load
  constexpr int NW = 4;                        // wavefronts that share the rows of a split
  constexpr int GW = HeadSplit<T, G>::GW, NGRP = HeadSplit<T, G>::NGRP;
  constexpr int NT = 256 * NGRP;
  constexpr int U = 4;                         // row loads in flight per lane, for K and for V

  __shared__ int sh_scan[24];                  // [0..15] the prefix sum's wavefront totals, [16..21] results
  __shared__ float sh_acc[NW][G][D];
  __shared__ float sh_m[NW][G], sh_l[NW][G];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wv_all / NW, wv = wv_all % NW; // head set, and place among the set's wavefronts
  const int col = lane % LPR, slot = lane / LPR;

  // ---- which (segment, split) is this workgroup? -------------------------------------------
  // With k_new/v_new the call appends one row per segment (Eq. 1) and attends over it as well:
  // the row is taken from k_new/v_new by the lanes it falls to, which also store it in the cache.
  const int grow = k_new != nullptr ? 1 : 0;
  Work wk;
  if (!find_work<NW * NGRP>(nseg, per, split, headroom, grow, cu, seg_len, sh_scan, seg_tab, wk)) return;
  const int s = wk.s, len = wk.rows;
  const int b = s / h, c = s % h;
  // (equal parts of the segment, as in decode_mfma_kernel, in multiples of the split's own unit)
  const int part = ((len + wk.parts - 1) / wk.parts + 63) / 64 * 64;
  const int r0 = wk.j * part, r1 = min(len, r0 + part);
  const int new_row = wk.appended ? len - 1 : -1;
  const long long seg_byte = ((long long)wk.first_row + (long long)s * headroom) * ROWB + col * 16;
  char *Kb = Kc + seg_byte;
  char *Vb = Vc + seg_byte;
  const long long new_byte = (long long)s * ROWB + col * 16;

  // ---- the g query rows of this KV head, pre-scaled so that exp() becomes exp2() --------------
  float qf[GW][EPL];
#pragma unroll
  for (int gi = 0; gi < GW; ++gi) {
    const T *qp = q + ((long long)(b * h + c) * G + grp * GW + gi) * D + col * EPL;
    Elem<T>::widen(*reinterpret_cast<const u32x4 *>(qp), qf[gi]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qf[gi][e] *= c_log2;
  }

  float m[GW], l[GW], acc[GW][EPL];
#pragma unroll
  for (int gi = 0; gi < GW; ++gi) {
    m[gi] = M_INIT; l[gi] = 0.0f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[gi][e] = 0.0f;
  }

  const int rows = r1 - r0;
  const int iters = (rows + U * NW * RPW - 1) / (U * NW * RPW);
  for (int it = 0; it < iters; ++it) {
    u32x4 kk[U], vv[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + ((it * U + u) * NW + wv) * RPW + slot;
      ok[u] = r < r1;
      const int rr = min(r, r1 - 1);                           // r1 >= 1: the block exists
      const long long o = (long long)rr * ROWB;
      // lanes past the end re-read the block's last row (and ignore it): if that is the new row,
      // they too must take it from k_new/v_new, its place in the cache is not written yet
      const bool fresh = rr == new_row;
      kk[u] = *reinterpret_cast<const u32x4 *>(fresh ? k_new + new_byte : Kb + o);
      vv[u] = *reinterpret_cast<const u32x4 *>(fresh ? v_new + new_byte : Vb + o);
      if (r == new_row && grp == 0) {
        *reinterpret_cast<u32x4 *>(Kb + o) = kk[u];
        *reinterpret_cast<u32x4 *>(Vb + o) = vv[u];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[EPL], sc[GW];
      Elem<T>::widen(kk[u], kf);
      bool grow = false;
#pragma unroll
      for (int gi = 0; gi < GW; ++gi) {
        float a = 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) a = fmaf(qf[gi][e], kf[e], a);
        a = row_sum<LPR>(a);
        sc[gi] = ok[u] ? a : -INFINITY;
        grow |= sc[gi] > m[gi];
      }
      if (__any(grow)) {                       // a new running maximum somewhere in the wavefront
#pragma unroll
        for (int gi = 0; gi < GW; ++gi) {
          const float mn = fmaxf(m[gi], sc[gi]);
          const float corr = fast_exp2(m[gi] - mn);
          l[gi] *= corr;
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[gi][e] *= corr;
          m[gi] = mn;
        }
      }
      float vf[EPL];
      if (it == iters - 1 && !ok[u]) vv[u] = u32x4{0};         // (a weight of 0 times an infinite value would be a NaN)
      Elem<T>::widen(vv[u], vf);
#pragma unroll
      for (int gi = 0; gi < GW; ++gi) {
        const float p = fast_exp2(sc[gi] - m[gi]);
        l[gi] += p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[gi][e] = fmaf(p, vf[e], acc[gi][e]);
      }
    }
  }

  // ---- merge the RPW row slots of the wavefront, then the NW wavefronts of each head set --------
#pragma unroll
  for (int gi = 0; gi < GW; ++gi) {
    float M = m[gi];
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) M = fmaxf(M, __shfl_xor(M, o));
    const float f = fast_exp2(m[gi] - M);
    float ll = l[gi] * f;
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) ll += __shfl_xor(ll, o);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      float a = acc[gi][e] * f;
#pragma unroll
      for (int o = LPR; o < 64; o <<= 1) a += __shfl_xor(a, o);
      acc[gi][e] = a;
    }
    if (slot == 0) {
      const int head = grp * GW + gi;
#pragma unroll
      for (int e = 0; e < EPL; ++e) sh_acc[wv][head][col * EPL + e] = acc[gi][e];
      if (col == 0) { sh_m[wv][head] = M; sh_l[wv][head] = ll; }
    }
  }
  __syncthreads();
  for (int t = tid; t < G * D; t += NT) {
    const int gi = t / D, e = t % D;
    float M = sh_m[0][gi];
#pragma unroll
    for (int w2 = 1; w2 < NW; ++w2) M = fmaxf(M, sh_m[w2][gi]);
    float a = 0.0f, ll = 0.0f;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) {
      const float f = fast_exp2(sh_m[w2][gi] - M);
      a = fmaf(sh_acc[w2][gi][e], f, a);
      ll = fmaf(sh_l[w2][gi], f, ll);
    }
    part_acc[((long long)blockIdx.x * G + gi) * D + e] = a;
    if (e == 0) {
      part_ml[((long long)blockIdx.x * G + gi) * 2] = M;
      part_ml[((long long)blockIdx.x * G + gi) * 2 + 1] = ll;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// 16-bit caches: both products on the matrix cores (v_mfma_f32_16x16x32), one wavefront per tile of
// 32 rows, nothing staged through LDS and no data crossing lanes between the two products.
//
//   logits   D[row][head] = K Q^T: a lane loads 16-byte words of row l%16 (twice: 32 rows), and
//            ends up with head l%16 and the rows 4 (l/16) + i and 16 + 4 (l/16) + i, i < 4.  The
//            columns past the group repeat its heads.
//   values   D[head][column] += P V: what a lane holds is its part of the P operand if the rows are
//            numbered that way, so V is loaded in that numbering: a lane takes 8 rows x D/16
//            columns and turns its own 8 x (D/16) block with byte permutes.
//
// P stays in 32 bits: it is cut into three bf16 parts whose sum is P to 2^-24 (truncated to 8, 8 and 8
// bits), and the 16 rows of the P operand hold the parts side by side (the repeated heads).  For g = 8
// the third part goes through a product of its own.  Products of 16-bit values and their sums are exact
// in fp32 up to the accumulation, as they were on the vector units.  The parts are bf16 for fp16 caches
// too: fp16 parts run out of exponent 2^-39 below the maximum, so that a weight of 2^-28 kept 11 bits
// and an infinite value row behind a smaller one gave 0 * inf.  An fp16 value is exactly the sum of a
// bf16 value of its upper 8 bits and one of the lower 3, so its product takes two instructions, and P
// travels multiplied by 2^64, which leaves the parts of the smallest weight above the bf16 range's end.
//
// The vector form before this one (16 lanes per row, a dot product and two fused multiply-adds
// per element and head) issued 130 instructions per four rows at g = 4 and 240 at g = 8, which
// made it the bound from g = 8 on: a 134 MB cache at g = 8 took 77.2 us, now 29.8 (a plain
// read of as much: 25); 49 MB at g = 4 19.2, now 12.9 (kernel times, launch included).
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

template <bool F16>
__device__ __forceinline__ floatx4 mfma16(u32x4 a, u32x4 b, floatx4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <bool F16> constexpr float P_SCALE = F16 ? 0x1p64f : 1.0f;    // (|V| < 2^16, 2^31 rows: below the fp32 range's end)
constexpr float LOW_MAX = 1024.0f;             // above the lower 3 bits of any finite fp16 value

// The bf16 value that x is cut to, back in 32 bits, where `on`; 0 elsewhere.
__device__ __forceinline__ float cut(float x, bool on) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) & (on ? 0xffff0000u : 0u));
}
// x0 and x1 cut to bf16, x0 in the lower half of the word.
__device__ __forceinline__ unsigned pack(float x0, float x1) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, x1), __builtin_bit_cast(unsigned, x0), 0x07060302u);
}
// The upper (odd) or lower half of a word of two fp16 values.
__device__ __forceinline__ float half_of(unsigned w, bool odd) {
  return (float)__builtin_bit_cast(_Float16, (unsigned short)(odd ? w >> 16 : w & 0xffffu));
}
// What the cut leaves of an fp16 value in 32 bits.  Of an infinity (whose difference is a NaN) some
// finite number: the upper part alone makes the product infinite.
__device__ __forceinline__ float low_part(float x) { return fminf(x - cut(x, true), LOW_MAX); }

// Where a workgroup's result goes: partial results for the merge kernel, or (WHOLE, one workgroup per
// segment) straight to the caller.
struct DecodeOut {
  float *part_acc, *part_ml;
  int4 *seg_tab;
  float *out, *lse;
  int *new_len, *overflow;                     // null unless the call appends
};

// (seg_len is also written, through res.new_len: after the barrier, by the one workgroup that read it)
template <bool F16, int D, int G, bool WHOLE>
__global__ __launch_bounds__(WHOLE ? 512 : 256) void decode_mfma_kernel(
    int nseg, int h, int per, int split, int headroom, float c_log2, const unsigned short *__restrict__ q,
    const char *__restrict__ k_new, const char *__restrict__ v_new, const int *__restrict__ cu,
    const int *seg_len, char *Kc, char *Vc, DecodeOut res) {
  constexpr int NW = WHOLE ? 8 : 4;            // wavefronts that share the rows of a split
  constexpr int ROWB = D * 2;
  constexpr int KS = D / 32;                   // k-steps of the logits
  constexpr int VC = D / 16;                   // columns of V per lane
  constexpr int TR = 32;                       // rows per tile
  constexpr int PARTS = G == 8 ? 2 : 3;        // parts of P held side by side
  constexpr bool THIRD = G == 8;               // the last part has accumulators of its own
  typedef unsigned int vword __attribute__((ext_vector_type(VC / 2)));

  __shared__ int sh_scan[24];                  // [0..15] the prefix sum's wavefront totals, [16..21] results
  __shared__ __align__(16) float sh_acc[NW][PARTS * G][D];
  __shared__ __align__(16) float sh_third[THIRD ? NW : 1][THIRD ? G : 1][THIRD ? D : 1];
  __shared__ float sh_m[NW][G], sh_l[NW][G];

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- which (segment, split) is this workgroup?  (as in decode_attn_kernel) --------------------
  const int grow = k_new != nullptr ? 1 : 0;
  int s, len, cu_s, new_row, r0, r1;
  if constexpr (WHOLE) {
    s = blockIdx.x;
    cu_s = cu[s];
    len = rows_held(cu, seg_len, s, headroom, grow);
    new_row = len > rows_held(cu, seg_len, s, headroom, 0) ? len - 1 : -1;
    r0 = 0;
    r1 = len;
  } else {
    Work wk;
    if (!find_work<NW>(nseg, per, split, headroom, grow, cu, seg_len, sh_scan, res.seg_tab, wk)) return;
    s = wk.s;
    len = wk.rows;
    cu_s = wk.first_row;
    new_row = wk.appended ? len - 1 : -1;
    // The segment's rows in equal parts, in whole rounds of the workgroup: the call lasts as long as its
    // longest workgroup, and with `split` rows for all but the last one 1024 rows were cut into 896 + 128
    // (40 sequences x 8 heads of as many rows, d = 128, g = 4: 42.9 us, now 34.7; the vector kernel's 832 + 192
    // at g = 1: 37.4, 40.4 with this one, then 33.0).  None is empty.  (Whole tiles instead of rounds: 40 uneven
    // segments of 900 rows 11.8 instead of 11.3 us, 320 of 400 rows 21.7 instead of 22.0.)
    const int rows = min(split, __builtin_amdgcn_readfirstlane(((len + wk.parts - 1) / wk.parts + NW * TR - 1) / (NW * TR) * (NW * TR)));
    r0 = wk.j * rows;
    r1 = min(len, r0 + rows);
  }
  const long long seg_byte = ((long long)cu_s + (long long)s * headroom) * ROWB;
  char *Kb = Kc + seg_byte;
  char *Vb = Vc + seg_byte;
  const char *kn = k_new + (long long)s * ROWB, *vn = v_new + (long long)s * ROWB;

  u32x4 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = *reinterpret_cast<const u32x4 *>(q + ((long long)s * G + l16 % G) * D + (4 * ks + lg) * 8);

  float m = M_INIT, l = 0.0f;                  // of head l16 % G; m the same in all lanes of a head
  floatx4 acc[VC], acc3[THIRD ? VC : 1];
#pragma unroll
  for (int e = 0; e < VC; ++e) acc[e] = floatx4{0};
  if (THIRD) {
#pragma unroll
    for (int e = 0; e < VC; ++e) acc3[e] = floatx4{0};
  }
  const int part = l16 / G;                    // which part of P this lane's operand rows hold

  for (int t0 = r0 + wv * TR; t0 < r1; t0 += NW * TR) {
    u32x4 kk[2][KS];
    vword vv[8];
    const bool edge = t0 + TR > r1 || (new_row >= t0 && new_row < t0 + TR);
    const char *kt = Kb + (long long)t0 * ROWB, *vt = Vb + (long long)t0 * ROWB;
    const unsigned vcol = l16 * (VC * 2);
    if (!edge) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          kk[t][ks] = *reinterpret_cast<const u32x4 *>(kt + (unsigned)((16 * t + l16) * ROWB + (4 * ks + lg) * 16));
#pragma unroll
      for (int j = 0; j < 8; ++j)
        vv[j] = *reinterpret_cast<const vword *>(vt + (unsigned)((16 * (j / 4) + 4 * lg + j % 4) * ROWB + vcol));
    } else {
      // rows past the end repeat the block's last one (and are masked below); the appended row comes from
      // k_new / v_new, its place in the cache is not written yet, and the lanes it falls to store it
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int r = t0 + 16 * t + l16, rr = min(r, r1 - 1);
        const char *src = rr == new_row ? kn : Kb + (long long)rr * ROWB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          kk[t][ks] = *reinterpret_cast<const u32x4 *>(src + (4 * ks + lg) * 16);
          if (r == new_row) *reinterpret_cast<u32x4 *>(Kb + (long long)r * ROWB + (4 * ks + lg) * 16) = kk[t][ks];
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = t0 + 16 * (j / 4) + 4 * lg + j % 4, rr = min(r, r1 - 1);
        const char *src = rr == new_row ? vn : Vb + (long long)rr * ROWB;
        vv[j] = *reinterpret_cast<const vword *>(src + vcol);
        if (r == new_row) *reinterpret_cast<vword *>(Vb + (long long)r * ROWB + vcol) = vv[j];
      }
    }
    float sc[8];                               // row t0 + 16 (j/4) + 4 lg + j%4, not scaled yet
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // a sum of its own per k-step, then a tree: the rounding of a logit is what the result's error
      // against 64 bits consists of (one chain of KS products: 1.3 times as much)
      floatx4 a[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) a[ks] = mfma16<F16>(kk[t][ks], qf[ks], floatx4{0});
#pragma unroll
      for (int o = KS / 2; o > 0; o >>= 1)
#pragma unroll
        for (int ks = 0; ks < o; ++ks) a[ks] += a[ks + o];
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[4 * t + i] = a[0][i];
    }
    if (edge) {
      // the values too: a weight of 0 times an infinite one would be a NaN (here and not between the
      // loads, where every one of them would be waited for: 64 segments of 1500 rows 15.7 -> 17.7 us)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (t0 + 16 * (j / 4) + 4 * lg + j % 4 >= r1) { sc[j] = -INFINITY; vv[j] = vword{0}; }
    }
    float top = sc[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) top = fmaxf(top, sc[j]);
    top *= c_log2;
    if (__any(top > m)) {                      // a new running maximum somewhere in the wavefront
      top = fmaxf(top, __shfl_xor(top, 16));
      top = fmaxf(top, __shfl_xor(top, 32));
      const float mn = fmaxf(m, top);
      const float corr = fast_exp2(m - mn);
      l *= corr;
      m = mn;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ci = __shfl(corr, 4 * lg + i);   // accumulator row 4 lg + i: that lane's head
#pragma unroll
        for (int e = 0; e < VC; ++e) {
          acc[e][i] *= ci;
          if (THIRD) acc3[e][i] *= ci;
        }
      }
    }
    float p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      p[j] = fast_exp2(fmaf(sc[j], c_log2, -m));
      l += p[j];
      p[j] *= P_SCALE<F16>;
    }
    u32x4 pa, pc;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float x0 = p[2 * k], x1 = p[2 * k + 1];
      x0 -= cut(x0, part >= 1);
      x1 -= cut(x1, part >= 1);
      if (!THIRD) {
        x0 -= cut(x0, part >= 2);
        x1 -= cut(x1, part >= 2);
      }
      pa[k] = pack(x0, x1);
      if (THIRD) {
        float y0 = p[2 * k], y1 = p[2 * k + 1];
        y0 -= cut(y0, true); y1 -= cut(y1, true);
        y0 -= cut(y0, true); y1 -= cut(y1, true);
        pc[k] = pack(y0, y1);
      }
    }
#pragma unroll
    for (int e = 0; e < VC; ++e) {
      u32x4 vb, vl;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned w0 = vv[2 * k][e / 2], w1 = vv[2 * k + 1][e / 2];
        if constexpr (F16) {
          const float x0 = half_of(w0, e & 1), x1 = half_of(w1, e & 1);
          vb[k] = pack(x0, x1);
          vl[k] = pack(low_part(x0), low_part(x1));
        } else {
          vb[k] = __builtin_amdgcn_perm(w1, w0, (e & 1) ? 0x07060302u : 0x05040100u);
        }
      }
      acc[e] = mfma16<false>(pa, vb, acc[e]);
      if (THIRD) acc3[e] = mfma16<false>(pc, vb, acc3[e]);
      if constexpr (F16) {
        acc[e] = mfma16<false>(pa, vl, acc[e]);
        if (THIRD) acc3[e] = mfma16<false>(pc, vl, acc3[e]);
      }
    }
  }

  // ---- the wavefronts' results meet in LDS -------------------------------------------------------
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (lane < G) { sh_m[wv][lane] = m; sh_l[wv][lane] = l; }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 4 * lg + i;                // part * G + head
#pragma unroll
    for (int e = 0; e < VC; e += 4) {
      if (row < PARTS * G)
        *reinterpret_cast<float4 *>(&sh_acc[wv][row][l16 * VC + e]) =
            make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
      if (THIRD && row < G)
        *reinterpret_cast<float4 *>(&sh_third[wv][row][l16 * VC + e]) =
            make_float4(acc3[e][i], acc3[e + 1][i], acc3[e + 2][i], acc3[e + 3][i]);
    }
  }
  __syncthreads();
  for (int t = tid; t < G * D; t += 64 * NW) {
    const int gi = t / D, e = t % D;
    float M = sh_m[0][gi];
#pragma unroll
    for (int w2 = 1; w2 < NW; ++w2) M = fmaxf(M, sh_m[w2][gi]);
    float a = 0.0f, ll = 0.0f;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) {
      const float f = fast_exp2(sh_m[w2][gi] - M);
      // an infinite value row makes the first part's sum infinite and 0 * inf = NaN of the others
      const float first = sh_acc[w2][gi][e];
      float rest = sh_acc[w2][G + gi][e];
      rest += THIRD ? sh_third[w2][gi][e] : sh_acc[w2][2 * G + gi][e];
      const float x = first + (__builtin_fabsf(first) < INFINITY ? rest : 0.0f);
      a = fmaf(x * (1.0f / P_SCALE<F16>), f, a);
      ll = fmaf(sh_l[w2][gi], f, ll);
    }
    if constexpr (WHOLE) {
      const long long row = (long long)s * G + gi;
      res.out[row * D + e] = ll > 0.0f ? a / ll : 0.0f;
      if (res.lse && e == 0) res.lse[row] = ll > 0.0f ? (M + log2f(ll)) * LN2 : -INFINITY;
    } else {
      res.part_acc[((long long)blockIdx.x * G + gi) * D + e] = a;
      if (e == 0) {
        res.part_ml[((long long)blockIdx.x * G + gi) * 2] = M;
        res.part_ml[((long long)blockIdx.x * G + gi) * 2 + 1] = ll;
      }
    }
  }
  // (nobody but this workgroup reads the segment's length)
  if (WHOLE && res.new_len && tid == 0) {
    if (new_row >= 0) res.new_len[s] = len;
    else if (res.overflow) *res.overflow = 1;  // the segment was full, its new row was dropped
  }
}

// One workgroup per (segment, query head of its group) merges that segment's splits and
// normalises.  A long segment has hundreds of splits, so they are merged NSLOT side by side
// (each by D/4 lanes holding a float4 of the value sum), four loads deep, then across slots.
template <int D, int G>
__global__ __launch_bounds__(1024) void decode_combine_kernel(
    const int4 *__restrict__ seg_tab, int *__restrict__ seg_len, int *__restrict__ overflow,
    const float *__restrict__ part_acc, const float *__restrict__ part_ml,
    float *__restrict__ out, float *__restrict__ lse) {
  constexpr int LPE = D / 4;
  constexpr int NSLOT = 1024 / LPE;
  constexpr int UC = 4;
  __shared__ float sh_a[NSLOT][D];
  __shared__ float sh_m[NSLOT], sh_l[NSLOT];
  const int tid = threadIdx.x;
  const int s = blockIdx.x, gi = blockIdx.y;
  const int4 ent = seg_tab[s];                 // first partial, partials, rows now, 1 if a row was appended
  const int p0 = ent.x, cnt = ent.y;
  if (seg_len && gi == 0 && tid == 0) {        // the call appended: the new lengths become visible
    if (ent.w) seg_len[s] = ent.z;
    else if (overflow) *overflow = 1;          // the segment was full, its new row was dropped
  }
  const int e4 = tid % LPE, slot = tid / LPE;

  float m = M_INIT, l = 0.0f;
  float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int p = slot; p < cnt; p += NSLOT * UC) {
    float2 ml[UC];
    float4 pa[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int pp = p + u * NSLOT;
      const long long pg = (long long)(p0 + (pp < cnt ? pp : p)) * G + gi;
      ml[u] = *reinterpret_cast<const float2 *>(part_ml + pg * 2);
      pa[u] = *reinterpret_cast<const float4 *>(part_acc + pg * D + e4 * 4);
      if (pp >= cnt) { ml[u] = make_float2(M_INIT, 0.0f); pa[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f); }
    }
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const float mn = fmaxf(m, ml[u].x);
      const float fo = fast_exp2(m - mn), fn = fast_exp2(ml[u].x - mn);
      l = l * fo + ml[u].y * fn;
      a.x = a.x * fo + pa[u].x * fn; a.y = a.y * fo + pa[u].y * fn;
      a.z = a.z * fo + pa[u].z * fn; a.w = a.w * fo + pa[u].w * fn;
      m = mn;
    }
  }
  // (only the slots that had partials: with all of them the end of the kernel took 0.7 us of 32 slots and 1.3 of 64; a step over 8 segments of
  // 512 rows, with the above, 9.1 -> 8.0 us, over 64 of 1500 16.5 -> 16.0)
  // (From half of them on all: the loops below are then of a fixed length, with every load ahead.  One segment's 64
  // slots, d = 64, 8 x 4160 rows: 10.4 us a step with a loop of variable length, 9.65 with this.)
  const int live = cnt > NSLOT / 2 ? NSLOT : cnt;
  if (slot < live) {
    *reinterpret_cast<float4 *>(&sh_a[slot][e4 * 4]) = a;
    if (e4 == 0) { sh_m[slot] = m; sh_l[slot] = l; }
  }
  __syncthreads();
  if (tid < D) {
    float M = M_INIT, acc = 0.0f, ll = 0.0f;
    auto add = [&](int k) {
      const float f = fast_exp2(sh_m[k] - M);
      acc = fmaf(sh_a[k][tid], f, acc);
      ll = fmaf(sh_l[k], f, ll);
    };
    if (live == NSLOT) {
#pragma unroll
      for (int k = 0; k < NSLOT; ++k) M = fmaxf(M, sh_m[k]);
#pragma unroll 8
      for (int k = 0; k < NSLOT; ++k) add(k);
    } else {
#pragma unroll 4
      for (int k = 0; k < live; ++k) M = fmaxf(M, sh_m[k]);
#pragma unroll 4
      for (int k = 0; k < live; ++k) add(k);
    }
    const long long row = (long long)s * G + gi;       // = (b*h + c)*G + gi
    out[row * D + tid] = ll > 0.0f ? acc / ll : 0.0f;
    if (lse && tid == 0) lse[row] = ll > 0.0f ? (M + log2f(ll)) * LN2 : -INFINITY;
  }
}

// Eq. (1) for every segment: LPR lanes move the new K row and the new V row of one segment.
template <int LPR>
__global__ __launch_bounds__(256) void append_kernel(
    int nseg, int headroom, const char *__restrict__ k_new, const char *__restrict__ v_new,
    const int *__restrict__ cu, char *__restrict__ Kc, char *__restrict__ Vc,
    int *__restrict__ seg_len, int *__restrict__ overflow) {
  const int s = (blockIdx.x * 256 + threadIdx.x) / LPR;
  const int col = threadIdx.x % LPR;
  if (s >= nseg) return;
  const int cap = cu[s + 1] - cu[s] + headroom;
  const int len = seg_len[s];                  // read by all LPR lanes before lane 0 stores
  if (len < 0 || len >= cap) {
    if (col == 0 && overflow) *overflow = 1;
    return;
  }
  const uint4 kv = *reinterpret_cast<const uint4 *>(k_new + ((long long)s * LPR + col) * 16);
  const uint4 vv = *reinterpret_cast<const uint4 *>(v_new + ((long long)s * LPR + col) * 16);
  const long long o = (((long long)cu[s] + (long long)s * headroom + len) * LPR + col) * 16;
  *reinterpret_cast<uint4 *>(Kc + o) = kv;
  *reinterpret_cast<uint4 *>(Vc + o) = vv;
  if (col == 0) seg_len[s] = len + 1;
}

template <typename T, int D, int G>
void run_decode(const SeqTab &st, const Dims &dm, int headroom, const DecodePlan &pl,
                const void *q, const void *k_new, const void *v_new, const int *cu, void *Kc,
                void *Vc, int *seg_len, int *overflow, float *out, float *lse, char *ws,
                hipStream_t s) {
  const int nseg = st.batch * dm.h_kv;
  const int per = (nseg + 255) / 256;
  float *part_acc = (float *)(ws + pl.part_acc);
  float *part_ml = (float *)(ws + pl.part_ml);
  int4 *seg_tab = (int4 *)(ws + pl.seg_tab);
  constexpr bool F16 = std::is_same<T, f16_t>::value;
  // The matrix kernel multiplies 16 operand rows whatever the group, so with one head per KV head, and for
  // fp16 (two products per value) with two of 128 columns, the vector kernel is the faster one.  us per
  // step, vector | matrix, d = 128: 64 uneven segments of 4096 rows on average, 64 of 1500, 320 of 1024:
  //   bf16, g = 1   26.8 | 27.2   14.0 | 15.2   31.6 | 33.1      g = 2   30.6 | 29.9   15.0 | 15.0   33.6 | 33.2
  //   fp16, g = 1   26.4 | 29.2   13.7 | 14.9   31.2 | 35.5      g = 2   28.7 | 29.6   15.2 | 15.0   33.5 | 35.9
  // fp16, g = 2, d = 64: 20.1 | 19.5   11.7 | 11.3   22.5 | 22.2.
  // bf16, g = 1, d = 64 (kernels alone): 64 segments of 1500 rows 11.6 | 12.1, 256 of 6000 81.4 | 87.9, but 256
  // of 1500 26.0 | 23.8, the one shape measured that the matrix kernel does faster.
  constexpr bool VECTOR = sizeof(T) == 4 || G == 1 || (F16 && G == 2 && D == 128);
  if constexpr (sizeof(T) == 2) {
    const DecodeOut res = {part_acc, part_ml, seg_tab, out, lse, k_new ? seg_len : nullptr, overflow};
    if (pl.whole) {
      ADAKV_LAUNCH("decode_attn", (decode_mfma_kernel<F16, D, G, true>), dim3(nseg), dim3(512), s, nseg, dm.h_kv,
                   per, pl.split, headroom, dm.scale * LOG2E, (const unsigned short *)q, (const char *)k_new,
                   (const char *)v_new, cu, (const int *)seg_len, (char *)Kc, (char *)Vc, res);
      return;
    }
    if constexpr (!VECTOR)
      ADAKV_LAUNCH("decode_attn", (decode_mfma_kernel<F16, D, G, false>), dim3(pl.nblk), dim3(256), s, nseg,
                   dm.h_kv, per, pl.split, headroom, dm.scale * LOG2E, (const unsigned short *)q, (const char *)k_new,
                   (const char *)v_new, cu, (const int *)seg_len, (char *)Kc, (char *)Vc, res);
  }
  if constexpr (VECTOR)
    ADAKV_LAUNCH("decode_attn", (decode_attn_kernel<T, D, G>), dim3(pl.nblk), dim3(256 * HeadSplit<T, G>::NGRP), s,
                 nseg, dm.h_kv, per, pl.split, headroom, dm.scale * LOG2E, (const T *)q, (const char *)k_new,
                 (const char *)v_new, cu, (const int *)seg_len, (char *)Kc, (char *)Vc, part_acc, part_ml, seg_tab);
  // only a call that appends hands the lengths to the merge kernel for updating
  ADAKV_LAUNCH("decode_combine", (decode_combine_kernel<D, G>), dim3(nseg, G), dim3(1024), s,
               (const int4 *)seg_tab, k_new ? seg_len : nullptr, overflow, (const float *)part_acc,
               (const float *)part_ml, out, lse);
}

struct DecodeArgs {
  const void *q, *k_new, *v_new;
  const int *cu;
  void *Kc, *Vc;
  int *seg_len, *overflow;
  float *out, *lse;
  char *ws;
};

template <typename T, int D>
bool run_decode_g(const SeqTab &st, const Dims &dm, int headroom, const DecodePlan &pl,
                  const DecodeArgs &a, hipStream_t s) {
#define ADAKV_DECODE_G(G)                                                                       \
  run_decode<T, D, G>(st, dm, headroom, pl, a.q, a.k_new, a.v_new, a.cu, a.Kc, a.Vc, a.seg_len,   \
                      a.overflow, a.out, a.lse, a.ws, s)
  switch (dm.g) {
    case 1: ADAKV_DECODE_G(1); return true;
    case 2: ADAKV_DECODE_G(2); return true;
    case 4: ADAKV_DECODE_G(4); return true;
    case 8: ADAKV_DECODE_G(8); return true;
    default: return false;
  }
#undef ADAKV_DECODE_G
}

}  // namespace

bool decode_supported(const Dims &dm) {
  return (dm.g == 1 || dm.g == 2 || dm.g == 4 || dm.g == 8) && (dm.d == 64 || dm.d == 128);
}

DecodePlan plan_decode(const SeqTab &st, const Dims &dm, int dtype, int headroom) {
  DecodePlan pl;
  const long long nseg = (long long)st.batch * dm.h_kv;
  const long long cap = (long long)st.out_off[st.batch] + nseg * headroom;
  // Rows per workgroup: what fills one resident round, so that all workgroups start together and
  // none is left for a thin second round.  Three workgroups fit on a compute unit (768 on the
  // chip), two of the 16-bit kernel for g = 8 at d = 128, whose third part of P takes 32 more
  // registers (134 MB cache: 35.2 us with 500 workgroups, 41.0 with 752, 39.7 with 1500; at g = 4,
  // 49 MB: 17.6, 16.2, 18.2).  The split is a multiple of one round of the workgroup's loads: 128
  // rows in the 16-bit kernels, four wavefronts of 32 (16.2 us against 17.2 with multiples of 64), but of
  // half a round beyond two (segments of 4096 rows on average, uneven, 448 against 512: d = 128, g = 4
  // 28.3 | 30.2, d = 64 18.9 | 20.0; all of them 4096: 27.7 | 27.7, 18.6 | 17.4); 64 rows in the fp32
  // kernel and for caches so small that there are workgroups to spare.
  const bool mfma = dtype != ADAKV_FP32;
  const long long round_wgs = mfma && dm.g == 8 && dm.d == 128 ? 500 : 752;
  const long long room = round_wgs - nseg;                   // the segments' last, partial splits
  long long want = room > 64 ? (cap + room - 1) / room : cap / 512;
  if (want < 64) want = 64;
  const int unit = mfma && want > 64 && want <= 256 ? 128 : 64;
  const int split = (int)((want + unit - 1) / unit * unit);
  // One workgroup of eight wavefronts per segment, and no merge kernel, where no segment can be long: a
  // compute unit walks it alone, and what that takes follows its bytes.  us per step, split / whole, by rows of the
  // longest segment (the others a sixth to a half of it), 8 segments, bf16, d = 128, g = 4: 256 8.2 / 7.0, 384 8.3 / 8.1,
  // 512 8.4 / 9.2, 768 8.6 / 11.2, 1024 9.0 / 13.2; 64 segments 8.6 / 7.2, 8.9 / 9.3, 9.1 / 10.3, 10.1 / 12.5, 11.1 / 14.8;
  // g = 8, 8 segments 9.0 / 7.9, 9.1 / 9.0, 9.3 / 10.0, 9.4 / 12.2, 9.7 / 14.3; d = 64, fp16, g = 4: 512 7.6 / 6.9, 768 7.8 /
  // 8.3, 1024 7.9 / 9.6.  Heads are budgeted unevenly (the longest of a layer holds three to four times the
  // average), so the line is on four times the average, head-room full: 768 rows of 256 bytes; the most that the
  // layer allows, one head with all of its sequence's prefix budget, 1024; and 384 rows of capacity on average.  (768
  // is where both took the same while the split form's workgroups found their rows 1.5 us later.  They meet near 400
  // rows now: a layer at the line, with half to all of its 768 rows in use, takes up to 2.6 us more than in parts.)
  long long likely = 0, longest = 0;
  for (int b = 0; b < st.batch; ++b) {
    const long long most = st.Bp[b] < st.n[b] ? st.Bp[b] : st.n[b];
    const long long four = 4ll * ((st.Bp[b] + dm.h_kv - 1) / dm.h_kv);
    longest = most > longest ? most : longest;
    likely = (four < most ? four : most) > likely ? (four < most ? four : most) : likely;
  }
  const long long fixed = dm.w + headroom;
  pl.whole = mfma && cap <= nseg * 384 && (likely + fixed) * dm.d <= 768 * 128 && (longest + fixed) * dm.d <= 1024 * 128;
  pl.split = split;
  pl.nblk = (int)(cap / split + nseg);          // >= sum over segments of ceil(len / split)
  pl.part_acc = 0;
  pl.part_ml = align_up((size_t)pl.nblk * dm.g * dm.d * sizeof(float), 256);
  pl.seg_tab = pl.part_ml + align_up((size_t)pl.nblk * dm.g * 2 * sizeof(float), 256);
  pl.total = pl.seg_tab + align_up((size_t)nseg * sizeof(int4), 256);
  return pl;
}

hipError_t launch_decode_attn(const SeqTab &st, const Dims &dm, int dtype, int headroom,
                              const void *q, const void *k_new, const void *v_new, const int *cu,
                              void *Kc, void *Vc, int *seg_len, int *overflow, float *out,
                              float *lse, char *ws, hipStream_t s) {
  const DecodePlan pl = plan_decode(st, dm, dtype, headroom);
  const DecodeArgs a = {q, k_new, v_new, cu, Kc, Vc, seg_len, overflow, out, lse, ws};
  bool ok;
  if (dtype == ADAKV_BF16) {
    ok = dm.d == 64 ? run_decode_g<unsigned short, 64>(st, dm, headroom, pl, a, s)
                    : run_decode_g<unsigned short, 128>(st, dm, headroom, pl, a, s);
  } else if (dtype == ADAKV_FP16) {
    ok = dm.d == 64 ? run_decode_g<f16_t, 64>(st, dm, headroom, pl, a, s)
                    : run_decode_g<f16_t, 128>(st, dm, headroom, pl, a, s);
  } else {
    ok = dm.d == 64 ? run_decode_g<float, 64>(st, dm, headroom, pl, a, s)
                    : run_decode_g<float, 128>(st, dm, headroom, pl, a, s);
  }
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_append(const SeqTab &st, const Dims &dm, int dtype, int headroom,
                         const void *k_new, const void *v_new, const int *cu, void *Kc, void *Vc,
                         int *seg_len, int *overflow, hipStream_t s) {
  const int lpr = dm.d * (dtype == ADAKV_FP32 ? 4 : 2) / 16;
  const int nseg = st.batch * dm.h_kv;
  dim3 grid((nseg * lpr + 255) / 256), block(256);
#define ADAKV_LAUNCH_APPEND(LPR)                                                               \
  ADAKV_LAUNCH("append", append_kernel<LPR>, grid, block, s, nseg, headroom,                   \
               (const char *)k_new, (const char *)v_new, cu, (char *)Kc, (char *)Vc, seg_len,  \
               overflow)
  switch (lpr) {
    case 8: ADAKV_LAUNCH_APPEND(8); break;
    case 16: ADAKV_LAUNCH_APPEND(16); break;
    case 32: ADAKV_LAUNCH_APPEND(32); break;
    default: return hipErrorInvalidValue;
  }
#undef ADAKV_LAUNCH_APPEND
  return hipGetLastError();
}

}  // namespace adakv
