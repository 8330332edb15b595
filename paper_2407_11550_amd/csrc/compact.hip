// Gather of the retained K/V rows into the flattened per-head cache (Alg. 2 lines 10-11,
// layout of Section 3.5).  Pure byte movement: a row of d elements is ROWB bytes, moved as
// 16-byte words by LPR = ROWB/16 neighbouring lanes, so a wavefront reads 64/LPR whole rows per
// load instruction and writes them to consecutive output rows (fully coalesced stores).
// With head-room (the decode-side layout) segment s is shifted down by s*headroom rows and its
// length is written to seg_len[s].
#include "common.h"

namespace adakv {

// A row costs a chain of look-ups (segment, position, row), so a block takes RPT rows per LPR lanes
// and has all of them in flight.  The segment of the block's first row is searched once, in scalar
// registers, and the others are counted on from there (a search of six dependent loads per row
// before).  76 800 rows of 256 bytes, K and V, into the cache of 64 segments: 20.2 us, now 17.8 with two
// rows (19.0 with four, 21.5 with eight: fewer blocks hide less; a copy of as many bytes: 15.5).
template <int LPR, int RPT>
__global__ __launch_bounds__(256) void compact_kernel(
    SeqTab st, int h, int nseg, long long k_tok_b, long long k_head_b, long long v_tok_b,
    long long v_head_b, const char *__restrict__ K, const char *__restrict__ V,
    const int *__restrict__ indices, const int *__restrict__ cu, char *__restrict__ K_out,
    char *__restrict__ V_out, int rows_total, int w, int headroom, int *__restrict__ seg_len) {
  constexpr int RPB = 256 / LPR;   // rows side by side
  const int t0 = blockIdx.x * (RPB * RPT);
  const int lane = threadIdx.x % LPR, slot = threadIdx.x / LPR;
  int at[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) at[i] = indices[min(t0 + i * RPB + slot, rows_total - 1)];
  // segment s with cu[s] <= t0 < cu[s+1]; every segment holds at least the w window rows
  int lo = 0, hi = nseg;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= t0) lo = mid; else hi = mid;
  }
  uint4 kv[RPT], vv[RPT];
  int seg[RPT];
  int s = lo;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int t = min(t0 + i * RPB + slot, rows_total - 1);
    while (s + 1 < nseg && cu[s + 1] <= t) ++s;
    seg[i] = s;
    const int b = s / h, c = s % h;
    // clamped into the sequence's own rows, so that a corrupt index can never leave the tensor
    const long long row = st.tok_off[b] + min(max(at[i], 0), st.n[b] + w - 1);
    kv[i] = *reinterpret_cast<const uint4 *>(K + row * k_tok_b + c * k_head_b + lane * 16);
    vv[i] = *reinterpret_cast<const uint4 *>(V + row * v_tok_b + c * v_head_b + lane * 16);
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int t = t0 + i * RPB + slot;
    if (t < rows_total) {
      const long long o = (((long long)t + (long long)seg[i] * headroom) * LPR + lane) * 16;
      if (seg_len && lane == 0 && t == cu[seg[i]]) seg_len[seg[i]] = cu[seg[i] + 1] - cu[seg[i]];
      *reinterpret_cast<uint4 *>(K_out + o) = kv[i];
      *reinterpret_cast<uint4 *>(V_out + o) = vv[i];
    }
  }
}

hipError_t launch_compact(const SeqTab &st, const Dims &dm, int dtype, const void *K,
                          const void *V, const int *indices, const int *cu_seqlens, void *K_out,
                          void *V_out, int headroom, int *seg_len, hipStream_t s) {
  const int esz = dtype == ADAKV_FP32 ? 4 : 2;
  const int rowb = dm.d * esz;
  const int lpr = rowb / 16;
  const int rows = st.out_off[st.batch];
  if (rows == 0) return hipSuccess;
  const int nseg = st.batch * dm.h_kv;
  const int rpb = 256 / lpr;
  const dim3 block(256);
  // two rows per lane group once one each would be more blocks than the chip holds at a time (eight on
  // each of 256 compute units); below that the blocks are what hides the chain (16 384 rows: 5.5 us
  // with one, 6.5 with four)
  const bool many = rows > 2048 * rpb;
  const dim3 grid((rows + (many ? 2 : 1) * rpb - 1) / ((many ? 2 : 1) * rpb));
#define ADAKV_LAUNCH_COMPACT(LPR)                                                              \
  if (many) ADAKV_LAUNCH_COMPACT_N(LPR, 2); else ADAKV_LAUNCH_COMPACT_N(LPR, 1)
#define ADAKV_LAUNCH_COMPACT_N(LPR, RPT)                                                       \
  ADAKV_LAUNCH(seg_len ? "cache_build" : "compact", (compact_kernel<LPR, RPT>), grid, block, s, st,   \
                     dm.h_kv, nseg,                                                            \
                     dm.k_stride_tok * esz, dm.k_stride_head * esz, dm.v_stride_tok * esz,     \
                     dm.v_stride_head * esz, (const char *)K, (const char *)V, indices,        \
                     cu_seqlens, (char *)K_out, (char *)V_out, rows, dm.w, headroom, seg_len)
  switch (lpr) {
    case 8: ADAKV_LAUNCH_COMPACT(8); break;
    case 16: ADAKV_LAUNCH_COMPACT(16); break;
    case 32: ADAKV_LAUNCH_COMPACT(32); break;
    default: return hipErrorInvalidValue;
  }
#undef ADAKV_LAUNCH_COMPACT
#undef ADAKV_LAUNCH_COMPACT_N
  return hipGetLastError();
}

}  // namespace adakv
