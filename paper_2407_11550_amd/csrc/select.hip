// Top-k by radix select, used twice:
//   * layer scope  (Algorithm 1 inside Alg. 2 l.7): the B' largest of a sequence's h*n scores,
//     counted per head, then the safeguard of Alg. 2 l.8 in integer arithmetic;
//   * head scope   (Alg. 2 l.9): the B_c largest of one head's n scores, emitted as ascending
//     positions followed by the window positions.
// Ties are decided by position (lower flat index first) through counts and prefix sums; the
// order in which atomics land never reaches a result, so every output is deterministic.
//
// A score becomes a 32-bit key whose unsigned order is the float order; its digits are the
// key's bits 31..21, 20..10 and 9..0.  Each scope runs two kernels (a kernel boundary is the
// cheapest device-wide synchronisation on this part; a device-scope fence inside a kernel writes
// a whole L2 back), so the whole Top-k is four launches after the first-digit histograms, which
// the scoring kernel leaves behind in pipeline mode (two small kernels make them otherwise), or three
// where the layer's finish and the head's gather share one.  Short rows run a scope, or both, inside
// one block per sequence or segment instead (below):
//
//   gather   every block of 4096 positions finds the first digit d0 of its scope's threshold from
//            the finished first-digit histogram, adds the second digits of its elements under d0
//            to the scope's second-digit histogram, and leaves these elements behind sorted by
//            second digit (a counting sort inside the block: bucket starts + entries), together
//            with the number of its elements above d0;
//   finish / emit
//            finds the second digit d1 from the finished histogram.  The elements that share
//            the threshold's 22-bit prefix are then the bucket d1 of every block: few, and
//            found through the bucket starts without touching the scores again.  The last digit
//            and the number of ties to take come from them inside the block.  The layer scope
//            then counts per head and applies the safeguard; the head scope places every kept
//            position by prefix counts (earlier blocks' counts from the bucket starts; inside the
//            block positions go round by round, wavefront by wavefront, lane by lane, and a ballot
//            gives every lane its place).
//
// When more elements share a 22-bit prefix than a block can hold at once (plateaus: equal or
// almost equal scores), the finishing kernels stream the buckets instead of holding them.
#include "common.h"

namespace adakv {

namespace {

constexpr int ENT_PER_BLOCK = SEL_CHUNK;       // a block's elements under d0: at most all of them
constexpr int HOLD_LAYER = 4096;               // prefix-sharing elements the finishing kernel keeps in LDS
constexpr int HOLD_HEAD = 2048;                // the same for an emit block
constexpr int SERIAL_MAX = 64;                 // longest bucket a single thread copies by itself

struct TopkWs {             // byte offsets inside the Top-k part of the workspace
  size_t hist0;             // u32 [batch*h][RADIX_BINS]  first digits per head
  size_t hist_tot0;         // u32 [batch][RADIX_BINS]    first digits per sequence
  size_t hist1_tot;         // u32 [batch][RADIX_BINS]    layer scope: second digits under the sequence's d0
  size_t hist1;             // u32 [batch*h][RADIX_BINS]  head scope: second digits under the head's d0
  size_t zero_end;          // everything before this starts at zero
  size_t starts;            // u16 [blocks][RADIX_BINS]   bucket starts of a block's sorted entries
  size_t note;              // BlockNote [blocks]
  size_t entries;           // u16 [blocks][SEL_CHUNK]    last digits of a block's elements under d0, by bucket
  size_t bytes;
};

struct BlockNote {          // per gather block
  int entries;              // elements under d0 (= end of the last bucket)
  int above;                // elements above d0
};

TopkWs plan(const SeqTab &st, const Dims &dm) {
  TopkWs p;
  const size_t nseg = (size_t)st.batch * dm.h_kv;
  size_t o = 0;
  p.hist0 = o; o += nseg * RADIX_BINS * 4;
  p.hist_tot0 = o; o += (size_t)st.batch * RADIX_BINS * 4;
  p.hist1_tot = o; o += (size_t)st.batch * RADIX_BINS * 4;
  p.hist1 = o; o += nseg * RADIX_BINS * 4;
  p.zero_end = o;
  const size_t blocks = (size_t)count_chunks(st, SEL_CHUNK) * dm.h_kv;
  p.starts = o; o += align_up(blocks * RADIX_BINS * 2, 256);
  p.note = o; o += align_up(blocks * sizeof(BlockNote), 256);
  p.entries = o; o += align_up(blocks * ENT_PER_BLOCK * 2, 256);
  p.bytes = o;
  return p;
}

// What the kernels of one scope share.
struct TopkBufs {
  const unsigned *hist0;     // first digits: per head
  const unsigned *hist_tot0; // first digits: per sequence
  unsigned *hist1;           // head scope: second digits under the head's d0
  unsigned *hist1_tot;       // layer scope: second digits under the sequence's d0
  unsigned short *starts;
  BlockNote *note;
  unsigned short *entries;   // last digits (10 bits each)
};

// A finished histogram is searched by one wavefront, without a barrier: a lane adds up NB/64 consecutive bins, a scan
// over the lanes finds the lane whose bins hold the rank, a second one over that lane's bins, read once more, finds
// the bin.  (By the threads of a block, eight bins each, with three barriers, as before, a search took 0.6 to 0.8 us of
// which there are up to six one after the other in a kernel; this one 0.25.)  The loads are apart from the search so that
// they travel together with everything else a kernel needs from memory; in LDS every lane starts at another word, so
// that they do not meet on the same banks.
template <int NB> struct WaveBins { uint4 v[NB / 256]; };
template <int NB> __device__ __forceinline__ WaveBins<NB> load_bins(const unsigned *__restrict__ bins) {
  WaveBins<NB> r;
  const uint4 *p = reinterpret_cast<const uint4 *>(bins) + (threadIdx.x & 63) * (NB / 256);
#pragma unroll
  for (int i = 0; i < NB / 256; ++i) r.v[i] = p[i];
  return r;
}
template <int NB> __device__ __forceinline__ WaveBins<NB> lds_bins(const unsigned *bins) {
  WaveBins<NB> r;
  const int lane = threadIdx.x & 63;
  const uint4 *p = reinterpret_cast<const uint4 *>(bins) + lane * (NB / 256);
#pragma unroll
  for (int i = 0; i < NB / 256; ++i) r.v[i] = p[(i + lane) & (NB / 256 - 1)];
  return r;
}

// All lanes of a wavefront: given a finished histogram (`mine`: this lane's part) and the rank krem >= 1 among the
// elements it counts, find the digit whose bin holds that rank, counting from the largest digit down.  Gives the digit
// and the rank inside its bin (>= 1).  A rank beyond the histogram's total gives digit 0 and the rank unchanged
// (callers clamp what they derive from it).
template <int NB>
__device__ __forceinline__ void wave_locate(const WaveBins<NB> &mine, const unsigned *bins, int krem, unsigned &digit,
                                            int &rank_in_bin) {
  constexpr int PER = NB / 64;
  const int lane = threadIdx.x & 63;
  unsigned s = 0;
#pragma unroll
  for (int i = 0; i < NB / 256; ++i) s += (mine.v[i].x + mine.v[i].y) + (mine.v[i].z + mine.v[i].w);
  const unsigned upto = (unsigned)wave_scan_incl((int)s);                      // lanes up to this one
  const unsigned above = (unsigned)__builtin_amdgcn_readlane((int)upto, 63) - upto;
  const unsigned long long in_lane = __ballot(above < (unsigned)krem && (unsigned)krem <= above + s);
  digit = 0u;
  rank_in_bin = krem;
  if (in_lane == 0) return;
  const int L = __ffsll(in_lane) - 1;
  const unsigned r = (unsigned)krem - (unsigned)__builtin_amdgcn_readlane((int)above, L);
  const unsigned x = lane < PER ? bins[L * PER + PER - 1 - lane] : 0u;         // from the largest digit down
  const unsigned cum = (unsigned)wave_scan_incl((int)x);
  const unsigned long long in_bin = __ballot(lane < PER && cum - x < r && r <= cum);
  if (in_bin == 0) return;
  const int j = __ffsll(in_bin) - 1;
  digit = (unsigned)(L * PER + PER - 1 - j);
  rank_in_bin = (int)(r - (unsigned)__builtin_amdgcn_readlane((int)(cum - x), j));
}
// The same for a block, whose first wavefront searches a histogram in LDS that is finished for everybody (a barrier has
// passed); sh: two words that nobody else uses until everybody has passed another barrier.
template <int NB>
__device__ __forceinline__ void block_locate(const unsigned *bins, int krem, unsigned &digit, int &rank_in_bin,
                                             unsigned *sh /*[2]*/) {
  if (threadIdx.x < 64) {
    unsigned d;
    int r;
    wave_locate<NB>(lds_bins<NB>(bins), bins, krem, d, r);
    if (threadIdx.x == 0) { sh[0] = d; sh[1] = (unsigned)r; }
  }
  __syncthreads();
  digit = sh[0];
  rank_in_bin = (int)sh[1];
}

__global__ __launch_bounds__(256) void topk_init_kernel(unsigned *__restrict__ zero_begin,
                                                        size_t zero_words) {
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i = i0; i < zero_words; i += (size_t)gridDim.x * blockDim.x) zero_begin[i] = 0u;
}

// First digits of every score, per head and per sequence (outside pipeline mode, where the
// scoring kernel counts them).  grid.x runs over the SEL_CHUNK-sized chunks of all sequences,
// grid.y over heads.
__global__ __launch_bounds__(256) void topk_digit0_kernel(SeqTab st, ChunkTab ct, int h,
                                                          const float *__restrict__ scores,
                                                          unsigned *__restrict__ hist0,
                                                          unsigned *__restrict__ hist_tot0) {
  __shared__ unsigned lh[RADIX_BINS];
  const int tid = threadIdx.x;
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int n = st.n[b];
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const float *row = scores + st.score_off[b] + (size_t)c * n;
  const int j0 = chunk * SEL_CHUNK, j1 = min(n, j0 + SEL_CHUNK);
  // all of a thread's scores are requested before the first is counted, one trip to memory and not sixteen (indices
  // past the end are clamped): eight sequences of up to 30011 x 8 scores nobody read yet 9.9 -> 5.7 us
  constexpr int EPB = SEL_CHUNK / 256;
  float sc[EPB];
#pragma unroll
  for (int i = 0; i < EPB; ++i) sc[i] = row[min(j0 + tid + 256 * i, j1 - 1)];
  for (int i = tid; i < RADIX_BINS; i += 256) lh[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < EPB; ++i)
    if (j0 + tid + 256 * i < j1) atomicAdd(&lh[key_of(sc[i]) >> 21], 1u);
  __syncthreads();
  unsigned *gh = hist0 + (size_t)(b * h + c) * RADIX_BINS;
  unsigned *gt = hist_tot0 + (size_t)b * RADIX_BINS;
  for (int i = tid; i < RADIX_BINS; i += 256) {
    const unsigned v = lh[i];
    if (v) {
      atomicAdd(&gh[i], v);
      atomicAdd(&gt[i], v);
    }
  }
}

constexpr int GATHER_NT = 1024;
// The gather step of a block: `sc` holds its scores (position j0 + tid + GATHER_NT i, clamped to j1 - 1), d0 the scope's
// first digit, gh the scope's second digits.  The caller has cleared lh and *sh_above; a barrier has passed since.
// (Sixteen wavefronts with four positions a lane: in four with sixteen the counting alone took 1.1 us, now 0.6.  The
// kernel, 64 blocks 4.6 -> 4.1 us, 256 5.2 -> 4.3, 300 7.1 -> 5.8, 500 and more the same.)
__device__ __forceinline__ void gather_block(const float (&sc)[SEL_CHUNK / GATHER_NT], int j0, int j1, unsigned d0, const TopkBufs &tb,
                                             size_t blk, unsigned *gh,
                                             unsigned *lh /*[RADIX_BINS]: second-digit counts, then running bucket fill*/,
                                             int *sh_above, int *sh_wave /*[GATHER_NT / 64]*/) {
  constexpr int NT = GATHER_NT, EPT = SEL_CHUNK / NT, WV = NT / 64;
  static_assert(RADIX_BINS == 2 * NT, "two bins per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  unsigned keys[EPT];
  int above = 0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const bool in = j0 + tid + NT * i < j1;
    const unsigned key = key_of(sc[i]);
    keys[i] = key;
    const unsigned dg = key >> 21;
    if (in && dg == d0) atomicAdd(&lh[(key >> 10) & 2047u], 1u);
    above += __popcll(__ballot(in && dg > d0));
  }
  if (lane == 0 && above) atomicAdd(sh_above, above);
  __syncthreads();
  // bucket starts, largest digit first is not needed: buckets are addressed by digit.  Thread t
  // owns two bins from 2 t: exclusive scan over the block.
  const uint2 cnt = reinterpret_cast<const uint2 *>(lh)[tid];
  const unsigned tsum = cnt.x + cnt.y;
  const unsigned inc = (unsigned)wave_scan_incl((int)tsum);
  if (lane == 63) sh_wave[wv] = (int)inc;
  __syncthreads();
  const unsigned wsum = lane < WV ? (unsigned)sh_wave[lane & (WV - 1)] : 0u;
  const unsigned wupto = (unsigned)wave_scan_incl((int)wsum);
  const unsigned s0 = inc - tsum + (unsigned)__builtin_amdgcn_readlane((int)(wupto - wsum), __builtin_amdgcn_readfirstlane(wv));
  const unsigned s1 = s0 + cnt.x;
  // starts to memory (one store), counts to the scope's histograms, starts into lh
  reinterpret_cast<unsigned *>(tb.starts + blk * RADIX_BINS)[tid] = s0 | (s1 << 16);
  if (tid == NT - 1) { tb.note[blk].entries = (int)(s1 + cnt.y); tb.note[blk].above = *sh_above; }
  reinterpret_cast<uint2 *>(lh)[tid] = make_uint2(s0, s1);
  if (cnt.x) atomicAdd(&gh[tid * 2], cnt.x);
  if (cnt.y) atomicAdd(&gh[tid * 2 + 1], cnt.y);
  __syncthreads();
  // (the order inside a bucket follows the atomics, but only the multiset of a bucket's last
  // digits is ever used)
  unsigned short *ent = tb.entries + blk * ENT_PER_BLOCK;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const bool in = j0 + tid + NT * i < j1;
    if (in && (keys[i] >> 21) == d0) {
      const unsigned slot = atomicAdd(&lh[(keys[i] >> 10) & 2047u], 1u);
      if (slot < (unsigned)ENT_PER_BLOCK) ent[slot] = (unsigned short)(keys[i] & 1023u);
    }
  }
}

// The gather kernel of either scope.  grid as above.  LAYER: the threshold is sought over all
// heads of a sequence (rank B'), else inside the block's own head (rank budgets[segment]).
template <bool LAYER>
__global__ __launch_bounds__(GATHER_NT) void topk_gather_kernel(SeqTab st, ChunkTab ct, int h,
                                                              const float *__restrict__ scores,
                                                              const int *__restrict__ budgets,
                                                              TopkBufs tb) {
  __shared__ __align__(16) unsigned lh[RADIX_BINS];
  __shared__ unsigned sh[2];
  __shared__ int sh_above, sh_wave[GATHER_NT / 64];
  const int tid = threadIdx.x;
  const int b = find_seq(ct, st.batch, blockIdx.x);
  // the first sequence's facts sit at fixed places of the kernel arguments and arrive with the
  // first scalar fetch; only later sequences of a batch cost a dependent one
  int n = st.n[0], cfirst = ct.off[0], soff = st.score_off[0];
  if (b != 0) { n = st.n[b]; cfirst = ct.off[b]; soff = st.score_off[b]; }
  const int chunk = blockIdx.x - cfirst;
  const int c = blockIdx.y;
  const int seg = b * h + c;
  const size_t blk = (size_t)blockIdx.x * h + c;
  // the block's scores are requested first, so they arrive while the prologue below waits for
  // the histogram (indices past the end are clamped, the values ignored)
  const float *row = scores + soff + (size_t)c * n;
  const int j0 = chunk * SEL_CHUNK;
  const int j1 = min(n, j0 + SEL_CHUNK);
  constexpr int NT = GATHER_NT, EPT = SEL_CHUNK / NT;
  float sc[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) sc[i] = row[min(j0 + tid + NT * i, j1 - 1)];
  const unsigned *hist = LAYER ? tb.hist_tot0 + (size_t)b * RADIX_BINS : tb.hist0 + (size_t)seg * RADIX_BINS;
  WaveBins<RADIX_BINS> mine;
  if (tid < 64) mine = load_bins<RADIX_BINS>(hist);
  const int krem = LAYER ? st.Bp[b] : budgets[seg];
  reinterpret_cast<uint2 *>(lh)[tid] = make_uint2(0u, 0u);
  if (tid == 0) sh_above = 0;
  if (krem <= 0) {                                     // nothing to select in this scope
    if (tid == 0) { tb.note[blk].entries = 0; tb.note[blk].above = 0; }
    return;
  }
  if (tid < 64) {
    unsigned d0;
    int r0;
    wave_locate<RADIX_BINS>(mine, hist, krem, d0, r0);
    if (tid == 0) sh[0] = d0;
  }
  __syncthreads();
  unsigned *gh = LAYER ? tb.hist1_tot + (size_t)b * RADIX_BINS : tb.hist1 + (size_t)seg * RADIX_BINS;
  gather_block(sc, j0, j1, sh[0], tb, blk, gh, lh, &sh_above, sh_wave);
}

// Bucket d1 of one gather block: [first, first + count) in its entries.
__device__ __forceinline__ void bucket_of(const TopkBufs &tb, size_t blk, unsigned d1, int &first,
                                          int &count) {
  const unsigned short *s = tb.starts + blk * RADIX_BINS;
  const int total = min(max(tb.note[blk].entries, 0), ENT_PER_BLOCK);
  const int a = min((int)s[d1], total);
  const int e = d1 + 1 < (unsigned)RADIX_BINS ? min((int)s[d1 + 1], total) : total;
  first = a;
  count = max(e - a, 0);
}

// Inclusive scan of one int over the threads of a block of NT threads; returns the block total.
template <int NT>
__device__ __forceinline__ int block_scan_incl(int v, int &incl, int *sh /*[NT/64]*/) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int x = wave_scan_incl(v);
  __syncthreads();
  if (lane == 63) sh[wv] = x;
  __syncthreads();
  int before = 0, total = 0;
  for (int i = 0; i < NT / 64; ++i) {
    if (i < wv) before += sh[i];
    total += sh[i];
  }
  incl = before + x;
  return total;
}

// Last digits of a streamed bucket go to a visitor with two members: same(v, ok, times) when all
// of a lane's `times` entries carry the digit v, in every lane with ok set (a plateau of one
// value), and one(v, ok) for a single entry otherwise.  Both are called by a whole wavefront.
//
// The visitor that files them in a 1024-bin histogram in LDS.  64 atomics on one LDS word run one
// after the other, so while the lanes agree, call after call, the wavefront only keeps a running
// (digit, count) pair and adds it when the digit changes (and in flush() at the end).
struct WaveHist {
  unsigned *lh;
  unsigned run_digit, run_count;                       // the same in all lanes
  __device__ __forceinline__ explicit WaveHist(unsigned *bins) : lh(bins), run_digit(0u), run_count(0u) {}
  __device__ __forceinline__ void flush() {
    if (run_count && (threadIdx.x & 63) == 0) atomicAdd(&lh[run_digit], run_count);
    run_count = 0u;
  }
  __device__ __forceinline__ void same(unsigned digit, bool ok, unsigned times) {
    const unsigned long long act = __ballot(ok);
    if (act == 0) return;
    const int leader = __ffsll((long long)act) - 1;
    const unsigned dl = (unsigned)__builtin_amdgcn_readlane((int)digit, leader);
    if (__ballot(ok && digit != dl) == 0) {
      if (dl != run_digit) flush();
      run_digit = dl;
      run_count += (unsigned)__popcll(act) * times;
    } else if (ok) {
      atomicAdd(&lh[digit], times);
    }
  }
  __device__ __forceinline__ void one(unsigned digit, bool ok) {
    if (ok) atomicAdd(&lh[digit], 1u);
  }
};

// The visitor that counts the entries above and at the last digit d2.
struct CountAbove {
  unsigned d2;
  int gt, eq;
  __device__ __forceinline__ explicit CountAbove(unsigned digit) : d2(digit), gt(0), eq(0) {}
  __device__ __forceinline__ void same(unsigned v, bool ok, unsigned times) {
    gt += (ok && v > d2) ? (int)times : 0;
    eq += (ok && v == d2) ? (int)times : 0;
  }
  __device__ __forceinline__ void one(unsigned v, bool ok) {
    gt += ok && v > d2;
    eq += ok && v == d2;
  }
};

// Every entry of a bucket goes to the visitor f, called by a whole wavefront the same number of
// times in every lane.  Long buckets only occur on plateaus, where a block's elements under d0 all
// share one bucket that starts at entry 0: 16-byte loads (eight entries) when the bucket starts at
// a multiple of eight entries, eight of them in flight per lane (a whole block's 4096 entries in
// one round trip); two-byte loads, eight in flight, otherwise and for the tail.
template <class F>
__device__ __forceinline__ void for_bucket(const unsigned short *ent, int first, int count, F &f) {
  const int lane = threadIdx.x & 63;
  const unsigned short *p = ent + first;
  int done = 0;
  if ((first & 7) == 0) {
    const uint4 *q = reinterpret_cast<const uint4 *>(p);
    const int vecs = count / 8;                        // whole 16-byte words
    for (int v0 = 0; v0 < vecs; v0 += 512) {
      uint4 w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = q[min(v0 + u * 64 + lane, vecs - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = v0 + u * 64 + lane < vecs;
        const unsigned x[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
        const bool all8 = x[0] == x[1] && x[1] == x[2] && x[2] == x[3] && (x[0] >> 16) == (x[0] & 0xFFFFu);
        if (__ballot(ok && !all8) == 0) {
          f.same(x[0] & 1023u, ok, 8u);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            f.one(x[k] & 1023u, ok);
            f.one((x[k] >> 16) & 1023u, ok);
          }
        }
      }
    }
    done = vecs * 8;
  }
  for (int i0 = done; i0 < count; i0 += 512) {
    unsigned v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[min(i0 + u * 64 + lane, count - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) f.one(v[u] & 1023u, i0 + u * 64 + lane < count);
  }
}

// What a block that knows a sequence's whole layer scope holds in LDS: per head the elements above
// the layer's threshold and at it, then the budgets.
constexpr int FIN_NT = 1024;                           // sixteen wavefronts
struct LayerCounts {
  int gt[64], eq[64];
  int base[64];                                        // the budgets, when safeguard() is done
};

// Words of LDS that the searches of one scope share.
struct Searches {
  unsigned prefix[4];                                  // first digit, second digit, rank among those that share both
  unsigned last[2];                                    // last digit, how many at the threshold are taken
  unsigned total, many;                                // elements that share the prefix; 1: a bucket too long for one thread
};
// First and second digit from two finished histograms in memory, by the first wavefront of a block; the barrier that
// shows them to the others is the caller's.
__device__ __forceinline__ void locate_prefix(const WaveBins<RADIX_BINS> &m0, const WaveBins<RADIX_BINS> &m1,
                                              const unsigned *hist0, const unsigned *hist1, int krem, Searches &sr) {
  unsigned d0, d1;
  int r0, r1;
  wave_locate<RADIX_BINS>(m0, hist0, krem, d0, r0);
  wave_locate<RADIX_BINS>(m1, hist1, r0, d1, r1);
  if ((threadIdx.x & 63) == 0) {
    sr.prefix[0] = d0;
    sr.prefix[1] = d1;
    sr.prefix[2] = (unsigned)r1;
  }
}
constexpr int EARLY = 4;                               // entries of a thread's bucket asked for before anybody knows how many there are
struct Bucket {
  int first, count;
  unsigned short early[EARLY];
};
__device__ __forceinline__ void load_early(const TopkBufs &tb, size_t blk, Bucket &bk) {
  const unsigned short *ent = tb.entries + blk * ENT_PER_BLOCK + bk.first;
  const int count = bk.count > SERIAL_MAX ? 0 : bk.count;                  // (a longer one is streamed)
#pragma unroll
  for (int i = 0; i < EARLY; ++i) bk.early[i] = i < count ? ent[i] : (unsigned short)0;
}
// Where a thread puts its `count` elements among those that share the prefix, their order being of no account: a scan
// in its wavefront and an atomic per wavefront, without a barrier.  (With an atomic per thread the compiler goes through
// the active lanes one after the other: allocation alone, 8 heads, scores all equal, 20000 of them 35.5 us, 33.7 with this,
// 131072 91.4 / 89.0.)  All lanes of the wavefront take part.
__device__ __forceinline__ unsigned place(int count, Searches &sr) {
  const int upto = wave_scan_incl(count);
  unsigned first = 0;
  if ((threadIdx.x & 63) == 63 && upto) first = atomicAdd(&sr.total, (unsigned)upto);
  return (unsigned)__builtin_amdgcn_readlane((int)first, 63) + (unsigned)(upto - count);
}

// Layer scope from the gather kernel's results, by a block of sixteen wavefronts: Algorithm 1's
// counts.  Returns the number of threshold-valued elements to take, in flat order.
// scratch: 1024 + HOLD_LAYER words of LDS.
__device__ __forceinline__ int layer_counts(const ChunkTab &ct, int h, int b, int Bp, const TopkBufs &tb,
                                            LayerCounts &lc, Searches &sr, unsigned *scratch) {
  unsigned *lh2 = scratch, *held = scratch + 1024;     // held: (last digit << 6) | head
  int *sh_gt = lc.gt, *sh_eq = lc.eq;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const unsigned *hist0 = tb.hist_tot0 + (size_t)b * RADIX_BINS, *hist1 = tb.hist1_tot + (size_t)b * RADIX_BINS;
  WaveBins<RADIX_BINS> m0, m1;
  if (tid < 64) {
    m0 = load_bins<RADIX_BINS>(hist0);
    m1 = load_bins<RADIX_BINS>(hist1);
    sh_gt[tid] = 0;
    sh_eq[tid] = 0;
  }
  lh2[tid] = 0u;
  static_assert(FIN_NT == 1024, "a bin per thread");
  if (tid == 0) sr.total = sr.many = 0u;
  unsigned d2 = 0;
  int ties = 0;
  const int blk0 = ct.off[b] * h, blk1 = ct.off[b + 1] * h;      // this sequence's gather blocks
  if (Bp > 0) {
    if (tid < 64) locate_prefix(m0, m1, hist0, hist1, Bp, sr);
    __syncthreads();
    const unsigned d1 = sr.prefix[1];
    const int r1 = (int)sr.prefix[2];
    // the elements under (d0, d1): bucket d1 of every block.  Count them first.
    // The block's elements above the prefix go to its head's count right away: those above d0,
    // and under d0 those in the buckets after d1.
    int mine_cnt = 0, longest = 0;
    Bucket mine = {0, 0, {0}};                         // the first of this thread's blocks
    for (int k = blk0 + tid; k < blk1; k += FIN_NT) {
      int first, count;
      bucket_of(tb, (size_t)k, d1, first, count);
      if (k == blk0 + tid) {
        mine.first = first;
        mine.count = count;
        load_early(tb, (size_t)k, mine);
      }
      mine_cnt += count;
      longest = max(longest, count);
      const int total = min(max(tb.note[k].entries, 0), ENT_PER_BLOCK);
      const int over = tb.note[k].above + (total - first - count);
      if (over) atomicAdd(&sh_gt[k % h], over);
    }
    unsigned at = place(mine_cnt, sr);
    if (longest > SERIAL_MAX) sr.many = 1u;
    __syncthreads();
    const int total = (int)sr.total;
    // (a thread copies its blocks' buckets one element after the other: only short ones)
    if (total <= HOLD_LAYER && !sr.many) {
      // few: every thread copies its blocks' buckets into LDS, then digit and counts from there
      for (int k = blk0 + tid; k < blk1; k += FIN_NT) {
        const bool own = k == blk0 + tid;
        int first = mine.first, count = mine.count;
        if (!own) bucket_of(tb, (size_t)k, d1, first, count);
        const unsigned short *ent = tb.entries + (size_t)k * ENT_PER_BLOCK + first;
        const unsigned head = (unsigned)(k % h);
        auto hold = [&](unsigned e) {
          const unsigned v = ((e & 1023u) << 6) | head;
          held[at++] = v;
          atomicAdd(&lh2[v >> 6], 1u);
        };
#pragma unroll
        for (int i = 0; i < EARLY; ++i)
          if (own && i < count) hold(mine.early[i]);
        for (int i = own ? EARLY : 0; i < count; ++i) hold(ent[i]);
      }
      __syncthreads();
      block_locate<1024>(lh2, r1, d2, ties, sr.last);
      for (int i = tid; i < total; i += FIN_NT) {
        const unsigned v = held[i];
        if ((v >> 6) > d2) atomicAdd(&sh_gt[v & 63u], 1);
        if ((v >> 6) == d2) atomicAdd(&sh_eq[v & 63u], 1);
      }
    } else {
      // a plateau: stream the buckets, a wavefront per block, once for the digit and once for
      // the counts
      // (the next block's bucket is looked up while the current one streams)
      WaveHist wh(lh2);
      int nfirst = 0, ncount = 0;
      if (blk0 + wv < blk1) bucket_of(tb, (size_t)(blk0 + wv), d1, nfirst, ncount);
      for (int k = blk0 + wv; k < blk1; k += FIN_NT / 64) {
        const int first = nfirst, count = ncount;
        if (k + FIN_NT / 64 < blk1) bucket_of(tb, (size_t)(k + FIN_NT / 64), d1, nfirst, ncount);
        for_bucket(tb.entries + (size_t)k * ENT_PER_BLOCK, first, count, wh);
      }
      wh.flush();
      __syncthreads();
      block_locate<1024>(lh2, r1, d2, ties, sr.last);
      if (blk0 + wv < blk1) bucket_of(tb, (size_t)(blk0 + wv), d1, nfirst, ncount);
      for (int k = blk0 + wv; k < blk1; k += FIN_NT / 64) {
        const int first = nfirst, count = ncount;
        if (k + FIN_NT / 64 < blk1) bucket_of(tb, (size_t)(k + FIN_NT / 64), d1, nfirst, ncount);
        CountAbove ca(d2);
        for_bucket(tb.entries + (size_t)k * ENT_PER_BLOCK, first, count, ca);
        int gt = ca.gt, eq = ca.eq;
        gt = wave_sum(gt);
        eq = wave_sum(eq);
        if (lane == 0) { atomicAdd(&sh_gt[k % h], gt); atomicAdd(&sh_eq[k % h], eq); }
      }
    }
  }
  __syncthreads();
  return ties;
}

// The safeguard of Alg. 2 l.8 on the counts, by the first wavefront of a block (the others pass
// through; a barrier makes the budgets in lc.base visible to them).  One lane per head (h <= 64), and
// nothing between them but scans and lane reads (through LDS, a read per head and step, it took 0.9 us at
// eight heads, now 0.3).
__device__ __forceinline__ void safeguard(int h, int Bp, int alpha_fix, int ties, LayerCounts &lc) {
  if (threadIdx.x >= 64) return;
  const int c = threadIdx.x;
  const bool live = c < h;
  const int gt = lc.gt[c], eq = lc.eq[c];              // (zero past the last head)
  const long long one = 65536, a = alpha_fix;
  // threshold-valued elements of earlier heads, at most all of a sequence's scores
  const int before = wave_scan_incl(eq) - eq;
  const int avail = max(ties - before, 0);             // ties still to take when head c's turn comes
  const long long f = (long long)gt + min(eq, avail);  // Algorithm 1: B*_c = f_c
  const long long num = (one - a) * h * f + a * (long long)Bp;   // x_c = num / den, den = 65536 h
  // num / 65536 = (1-alpha) h f + alpha B' <= h f + B' < 2^32 (both sums are below 2^31), so
  // the division by den is a shift and one 32-bit division; the remainders recombine exactly
  const unsigned t = (unsigned)(num >> 16);
  const unsigned tq = t / (unsigned)h, tr = t - tq * (unsigned)h;
  int base = live ? (int)tq : 0;
  const int rem = live ? (int)((tr << 16) | (unsigned)(num & 0xFFFF)) : -1;      // below 65536 h <= 2^22
  const int left = Bp - wave_sum(base);                // 0 <= left < h
  int rank = 0;                                        // heads that come first for a spare unit
  for (int i = 0; i < h; ++i) {
    const int other = __builtin_amdgcn_readlane(rem, i);
    rank += other > rem || (other == rem && i < c);
  }
  if (live && rank < left) base += 1;                  // largest remainders, ties to the lower head
  lc.base[c] = base;
}

// Layer scope, second kernel.  One block per sequence.
__global__ __launch_bounds__(FIN_NT) void alloc_finish_kernel(SeqTab st, ChunkTab ct, int h, int w,
                                                              int alpha_fix, TopkBufs tb,
                                                              int *__restrict__ budgets,
                                                              int *__restrict__ cu) {
  __shared__ Searches sr;
  __shared__ __align__(16) unsigned scratch[1024 + HOLD_LAYER];
  __shared__ LayerCounts lc;
  const int b = blockIdx.x, c = threadIdx.x;
  const int Bp = st.Bp[b];
  const int ties = layer_counts(ct, h, b, Bp, tb, lc, sr, scratch);
  safeguard(h, Bp, alpha_fix, ties, lc);
  __syncthreads();
  if (c >= h) return;
  budgets[b * h + c] = lc.base[c];
  int run = st.out_off[b];
  for (int i = 0; i <= c; ++i) run += lc.base[i] + w;
  if (b == 0 && c == 0) cu[0] = 0;
  cu[b * h + c + 1] = run;
}

// Layer scope, second kernel, and head scope, first kernel, in one launch: every block (chunk, head) works the
// layer scope of its sequence out for itself, then gathers for its own head.  `layer` is what the layer's gather
// left behind; the head's lists go to memory of their own (`head`), since other blocks still read the layer's.
// A chain of dependent trips to memory bounds it, so that sixteen wavefronts repeat the layer scope in every
// block in the time in which one block does it.  What it saves is a launch: finish + gather / this kernel, us,
// 32768 keys x 8 heads 5.3 + 4.0 / 7.5, 131072 x 8 6.0 + 4.3 / 8.3, four of up to 30000 x 8 5.2 + 4.7 / 8.3 (whole
// steps: FUSED_BLOCKS).
static_assert(FIN_NT == GATHER_NT, "both halves take the same block");
__global__ __launch_bounds__(FIN_NT) void finish_gather_kernel(SeqTab st, ChunkTab ct, int h, int w, int alpha_fix,
                                                               const float *__restrict__ scores, TopkBufs layer,
                                                               TopkBufs head, int *__restrict__ budgets,
                                                               int *__restrict__ cu) {
  __shared__ Searches sr;
  __shared__ int sh_wave[FIN_NT / 64], sh_above;
  __shared__ unsigned sh_first;
  __shared__ __align__(16) unsigned scratch[1024 + HOLD_LAYER];      // the layer scope's, then the head's second digits
  __shared__ LayerCounts lc;
  static_assert(RADIX_BINS <= 1024 + HOLD_LAYER, "the digits fit into the scratch words");
  const int tid = threadIdx.x;
  const int b = find_seq(ct, st.batch, blockIdx.x);
  const int n = st.n[b], Bp = st.Bp[b];
  const int chunk = blockIdx.x - ct.off[b];
  const int c = blockIdx.y;
  const int seg = b * h + c;
  const float *row = scores + st.score_off[b] + (size_t)c * n;
  const int j0 = chunk * SEL_CHUNK;
  const int j1 = min(n, j0 + SEL_CHUNK);
  constexpr int EPT = SEL_CHUNK / FIN_NT;
  float sc[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) sc[i] = row[min(j0 + tid + FIN_NT * i, j1 - 1)];
  const unsigned *hist = head.hist0 + (size_t)seg * RADIX_BINS;
  WaveBins<RADIX_BINS> mine;
  if (tid < 64) mine = load_bins<RADIX_BINS>(hist);
  const int ties = layer_counts(ct, h, b, Bp, layer, lc, sr, scratch);
  safeguard(h, Bp, alpha_fix, ties, lc);
  // (nobody reads the scratch words any more)
  reinterpret_cast<uint2 *>(scratch)[tid] = make_uint2(0u, 0u);
  if (tid == 0) sh_above = 0;
  if (tid < 64) {                                      // (the wavefront that has the budgets)
    unsigned d0 = 0;
    int r0;
    const int own = __builtin_amdgcn_readfirstlane(lc.base[c]);
    if (own > 0) wave_locate<RADIX_BINS>(mine, hist, own, d0, r0);
    if (tid == 0) sh_first = d0;
  }
  __syncthreads();                                     // the budgets, the first digit and the cleared words
  const int bud = lc.base[c];
  if (chunk == 0 && tid == 0) {
    int run = st.out_off[b] + bud + w;
    for (int i = 0; i < c; ++i) run += lc.base[i] + w;
    budgets[seg] = bud;
    cu[seg + 1] = run;
    if (seg == 0) cu[0] = 0;
  }
  const size_t blk = (size_t)blockIdx.x * h + c;
  if (bud <= 0) {
    if (tid == 0) { head.note[blk].entries = 0; head.note[blk].above = 0; }
    return;
  }
  gather_block(sc, j0, j1, sh_first, head, blk, head.hist1 + (size_t)seg * RADIX_BINS, scratch, &sh_above, sh_wave);
}

// Head scope, second kernel.  Block (chunk, head) writes the kept positions of its 4096.
template <int NT>
__global__ __launch_bounds__(NT) void emit_write_kernel(
    SeqTab st, ChunkTab ct, int h, int w, const float *__restrict__ scores, TopkBufs tb,
    const int *__restrict__ budgets, const int *__restrict__ cu, int *__restrict__ indices,
    int rows_total) {
  constexpr int EPT = SEL_CHUNK / NT, WV = NT / 64;    // positions per thread, NT apart; wavefronts
  __shared__ Searches sr;
  __shared__ int tab[EPT * WV];                   // per round and wavefront: above << 16 | at the threshold
  __shared__ __align__(16) unsigned lh2[1024];
  __shared__ unsigned held[HOLD_HEAD];                 // (last digit << 1) | (lies in an earlier block)
  __shared__ int sh_cnt[2];
  static_assert(EPT * WV == 64, "a lane per table entry");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int b = find_seq(ct, st.batch, blockIdx.x);
  int n = st.n[0], cfirst = ct.off[0], soff = st.score_off[0];   // as in the gather kernel
  if (b != 0) { n = st.n[b]; cfirst = ct.off[b]; soff = st.score_off[b]; }
  const int chunk = blockIdx.x - cfirst;
  const int nchunks = (b != 0 ? ct.off[b + 1] : ct.off[1]) - cfirst;
  const int c = blockIdx.y;
  const int seg = b * h + c;
  const int out0 = cu[seg];
  const int bud = budgets[seg];
  const float *row = scores + soff + (size_t)c * n;

  // Positions are dealt out round by round (chunk start + NT i + tid): the loads are whole lines, and
  // position order is round, wavefront, lane, where a ballot gives every lane its place.  Issued
  // before the searches below; places past the end get key 0, which is never above or at a threshold.
  const int j0 = chunk * SEL_CHUNK + tid;
  unsigned keys[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) keys[i] = __float_as_uint(row[min(j0 + NT * i, n - 1)]);
  const unsigned *hist0 = tb.hist0 + (size_t)seg * RADIX_BINS, *hist1 = tb.hist1 + (size_t)seg * RADIX_BINS;
  WaveBins<RADIX_BINS> m0, m1;
  if (tid < 64) {
    m0 = load_bins<RADIX_BINS>(hist0);
    m1 = load_bins<RADIX_BINS>(hist1);
  }
  for (int i = tid; i < 1024; i += NT) lh2[i] = 0u;
  if (tid < 2) sh_cnt[tid] = 0;
  if (tid == 0) sr.total = sr.many = 0u;

  unsigned thr = 0xFFFFFFFFu;                          // no key is above, no tie is taken
  int ties = 0;
  int pg = 0, pe = 0;                                  // kept / threshold-valued positions of earlier blocks
  if (bud > 0) {
    if (tid < 64) locate_prefix(m0, m1, hist0, hist1, bud, sr);
    __syncthreads();
    const unsigned d0 = sr.prefix[0], d1 = sr.prefix[1];
    const int r1 = (int)sr.prefix[2];
    unsigned d2;
    // Every block of the head (thread k takes block k, k + NT, ...): how many of its elements
    // share the prefix (d0, d1), and, for the blocks in front of this one, how many lie above it:
    // those above d0, and under d0 those in the buckets after d1.
    int mine_cnt = 0, longest = 0;
    Bucket mine = {0, 0, {0}};                         // the first of this thread's blocks
    for (int k = tid; k < nchunks; k += NT) {
      const size_t kb = (size_t)(cfirst + k) * h + c;
      int first, count;
      bucket_of(tb, kb, d1, first, count);
      if (k == tid) {
        mine.first = first;
        mine.count = count;
        load_early(tb, kb, mine);
      }
      mine_cnt += count;
      longest = max(longest, count);
      if (k < chunk) {
        const int total = min(max(tb.note[kb].entries, 0), ENT_PER_BLOCK);
        pg += tb.note[kb].above + (total - first - count);
      }
    }
    unsigned at = place(mine_cnt, sr);
    if (longest > SERIAL_MAX) sr.many = 1u;
    __syncthreads();
    const int total = (int)sr.total;
    if (total <= HOLD_HEAD && !sr.many) {
      for (int k = tid; k < nchunks; k += NT) {
        const size_t kb = (size_t)(cfirst + k) * h + c;
        const bool own = k == tid;
        int first = mine.first, count = mine.count;
        if (!own) bucket_of(tb, kb, d1, first, count);
        const unsigned short *ent = tb.entries + kb * ENT_PER_BLOCK + first;
        const unsigned earlier = k < chunk ? 1u : 0u;
        auto hold = [&](unsigned e) {
          const unsigned v = e & 1023u;
          held[at++] = (v << 1) | earlier;
          atomicAdd(&lh2[v], 1u);
        };
#pragma unroll
        for (int i = 0; i < EARLY; ++i)
          if (own && i < count) hold(mine.early[i]);
        for (int i = own ? EARLY : 0; i < count; ++i) hold(ent[i]);
      }
      __syncthreads();
      block_locate<1024>(lh2, r1, d2, ties, sr.last);
      for (int i = tid; i < total; i += NT) {
        const unsigned v = held[i];
        if (v & 1u) {
          pg += (v >> 1) > d2;
          pe += (v >> 1) == d2;
        }
      }
    } else {
      // a plateau: stream the buckets, a wavefront per block
      WaveHist wh(lh2);
      int nfirst = 0, ncount = 0;
      if (wv < nchunks) bucket_of(tb, (size_t)(cfirst + wv) * h + c, d1, nfirst, ncount);
      for (int k = wv; k < nchunks; k += WV) {
        const size_t kb = (size_t)(cfirst + k) * h + c;
        const int first = nfirst, count = ncount;
        if (k + WV < nchunks) bucket_of(tb, (size_t)(cfirst + k + WV) * h + c, d1, nfirst, ncount);
        for_bucket(tb.entries + kb * ENT_PER_BLOCK, first, count, wh);
      }
      wh.flush();
      __syncthreads();
      block_locate<1024>(lh2, r1, d2, ties, sr.last);
      CountAbove ca(d2);
      if (wv < chunk) bucket_of(tb, (size_t)(cfirst + wv) * h + c, d1, nfirst, ncount);
      for (int k = wv; k < chunk; k += WV) {
        const size_t kb = (size_t)(cfirst + k) * h + c;
        const int first = nfirst, count = ncount;
        if (k + WV < chunk) bucket_of(tb, (size_t)(cfirst + k + WV) * h + c, d1, nfirst, ncount);
        for_bucket(tb.entries + kb * ENT_PER_BLOCK, first, count, ca);
      }
      pg += ca.gt;
      pe += ca.eq;
    }
    thr = (d0 << 21) | (d1 << 10) | d2;
    if (thr == 0u) ties = 0;                           // (no key of a score: inconsistent input)
  } else {
    __syncthreads();                                   // the cleared counters
  }
  if (__ballot((pg | pe) != 0)) {
    pg = wave_sum(pg);
    pe = wave_sum(pe);
    if (lane == 0) { atomicAdd(&sh_cnt[0], pg); atomicAdd(&sh_cnt[1], pe); }
  }

#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const unsigned key = key_of(__uint_as_float(keys[i]));
    keys[i] = j0 + NT * i < n ? key : 0u;
    const int g = __popcll(__ballot(keys[i] > thr)), e = __popcll(__ballot(keys[i] == thr));
    if (lane == 0) tab[i * WV + wv] = (g << 16) | e;    // (a block holds 4096 positions: 13 bits each)
  }
  __syncthreads();
  // every wavefront scans the table for itself
  const int in_table = tab[lane], upto = wave_scan_incl(in_table) - in_table;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const unsigned long long bg = __ballot(keys[i] > thr), be = __ballot(keys[i] == thr);
    if ((bg | be) == 0) continue;
    // over all earlier positions of the head
    const int front = __builtin_amdgcn_readlane(upto, i * WV + __builtin_amdgcn_readfirstlane(wv));
    const int ng = sh_cnt[0] + (front >> 16) +
                   (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bg >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bg, 0u));
    const int ne = sh_cnt[1] + (front & 0xFFFF) +
                   (int)__builtin_amdgcn_mbcnt_hi((unsigned)(be >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)be, 0u));
    const int pos = out0 + ng + min(ne, ties);
    if ((keys[i] > thr || (keys[i] == thr && ne < ties)) && (unsigned)pos < (unsigned)rows_total)
      indices[pos] = j0 + NT * i;
  }
  if (chunk == 0) {
    for (int rr = tid; rr < w; rr += NT)
      if ((unsigned)(out0 + bud + rr) < (unsigned)rows_total) indices[out0 + bud + rr] = n + rr;
  }
}

// ---- short rows: a whole scope inside one block --------------------------------------------------
//
// A kernel boundary costs 4 us here and every dependent trip to memory 2 us, whatever a kernel
// computes, so where a block of 1024 threads can hold all scores of a scope in registers (16 per
// thread) it finds the threshold without leaving LDS: second and last digits are counted in two
// passes over the registers, the first ones are the scoring kernel's (CARRIED) or counted likewise.
// Elements are dealt out round by round (element 1024 i +
// tid), so a wavefront's 64 are neighbours: position order is round, wavefront, lane, and a
// ballot per round gives a lane its place.  Bound by latency: one load of the scores (4 bytes per
// lane, all rounds in flight), three searches of a histogram, one scan.
constexpr int BLK_NT = 1024, BLK_WV = BLK_NT / 64;

// Rounds past the last element are skipped (uniformly); places past it get key 0, which no score has
// and which is never above or at a threshold.
template <int EPT>
__device__ __forceinline__ void load_keys(const float *__restrict__ row, int n, unsigned (&keys)[EPT]) {
  float x[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    x[i] = 0.0f;
    if (i * BLK_NT < n) x[i] = row[min(i * BLK_NT + (int)threadIdx.x, n - 1)];
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) keys[i] = i * BLK_NT + (int)threadIdx.x < n ? key_of(x[i]) : 0u;
}

// Counts a digit per lane where `on`.  64 atomics on one LDS word run one after the other, and equal
// scores (plateaus, repeated keys) stand side by side, so the lanes that agree with the first one
// count once.
__device__ __forceinline__ void count_digit(unsigned *bins, unsigned digit, bool on) {
  const unsigned long long act = __ballot(on);
  if (act == 0) return;
  const int leader = __ffsll((long long)act) - 1;
  const unsigned dl = (unsigned)__builtin_amdgcn_readlane((int)digit, leader);
  const unsigned long long same = __ballot(on && digit == dl);
  if ((int)(threadIdx.x & 63) == leader) atomicAdd(&bins[dl], (unsigned)__popcll(same));
  else if (on && digit != dl) atomicAdd(&bins[digit], 1u);
}

constexpr int BLK_LDS = RADIX_BINS + 1024 + RADIX_BINS;   // second, last and first digits

// The key of rank krem >= 1 among the n keys of the block, and how many equal to it are taken.
// CARRIED: `hist` is the scope's finished first-digit histogram, `first` the first wavefront's part of it.
template <int EPT, bool CARRIED>
__device__ __forceinline__ void block_threshold(const unsigned (&keys)[EPT], int n, int krem, const unsigned *hist,
                                                const WaveBins<RADIX_BINS> &first, unsigned *lds,
                                                Searches &sr, unsigned &thr, int &ties) {
  const int tid = threadIdx.x;
  unsigned d0, d1, d2;
  int r0, r1;
  __syncthreads();                                     // the caller may still use lds
  for (int i = tid; i < BLK_LDS; i += BLK_NT) lds[i] = 0u;
  if (CARRIED) {
    if (tid < 64) {
      wave_locate<RADIX_BINS>(first, hist, krem, d0, r0);
      if (tid == 0) { sr.prefix[0] = d0; sr.prefix[1] = (unsigned)r0; }
    }
    __syncthreads();
    d0 = sr.prefix[0];
    r0 = (int)sr.prefix[1];
  } else {
    __syncthreads();
    unsigned *lh0 = lds + RADIX_BINS + 1024;
#pragma unroll
    for (int i = 0; i < EPT; ++i)
      if (i * BLK_NT < n) count_digit(lh0, keys[i] >> 21, keys[i] != 0u);
    __syncthreads();
    block_locate<RADIX_BINS>(lh0, krem, d0, r0, sr.prefix);
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    if (i * BLK_NT < n) count_digit(lds, (keys[i] >> 10) & 2047u, keys[i] >> 21 == d0);
  __syncthreads();
  block_locate<RADIX_BINS>(lds, r0, d1, r1, sr.prefix + 2);
  const unsigned prefix = (d0 << 11) | d1;
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    if (i * BLK_NT < n) count_digit(lds + RADIX_BINS, keys[i] & 1023u, keys[i] >> 10 == prefix);
  __syncthreads();
  block_locate<1024>(lds + RADIX_BINS, r1, d2, ties, sr.last);
  thr = (prefix << 10) | d2;
  if (thr == 0u) ties = 0;                             // (no key of a score: inconsistent input)
}

// Layer scope of one sequence, h*n <= 1024 EPT: Algorithm 1's counts per head.  Returns the number
// of threshold-valued elements to take, in flat order.
template <int EPT, bool CARRIED>
__device__ __forceinline__ int block_layer_counts(const float *__restrict__ scores, int h, int n, int Bp,
                                                  const TopkBufs &tb, int b, unsigned *lds,
                                                  Searches &sr, LayerCounts &lc) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = h * n;
  if (tid < 64) { lc.gt[tid] = 0; lc.eq[tid] = 0; }
  int ties = 0;
  if (Bp > 0) {
    unsigned keys[EPT], thr;
    const unsigned *hist = tb.hist_tot0 + (size_t)b * RADIX_BINS;
    WaveBins<RADIX_BINS> first;
    if (CARRIED && tid < 64) first = load_bins<RADIX_BINS>(hist);
    load_keys<EPT>(scores, total, keys);
    block_threshold<EPT, CARRIED>(keys, total, Bp, hist, first, lds, sr, thr, ties);
    int c = 0, at = wv * 64;                           // head and position of the wavefront's first element
    while (at >= n && c < h) { at -= n; ++c; }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      if (i * BLK_NT < total) {
        const bool gt = keys[i] > thr, eq = keys[i] == thr && thr != 0u;
        const int g = __popcll(__ballot(gt)), e = __popcll(__ballot(eq));
        if (g + e == 0) {
        } else if (at + 63 < n) {                      // all of them in one head
          if (lane == 0) {
            if (g) atomicAdd(&lc.gt[c], g);
            if (e) atomicAdd(&lc.eq[c], e);
          }
        } else if (gt || eq) {
          int cl = c, r = at + lane;
          while (r >= n) { r -= n; ++cl; }
          atomicAdd(gt ? &lc.gt[cl] : &lc.eq[cl], 1);
        }
        at += BLK_NT;
        while (at >= n && c < h) { at -= n; ++c; }
      }
    }
  }
  __syncthreads();
  return ties;
}

// Head scope of one segment, n <= 1024 EPT: kept positions in ascending order, then the window's.
// lds: BLK_LDS words; tab: two words per round and wavefront.
template <int EPT, bool CARRIED>
__device__ __forceinline__ void block_select(const unsigned (&keys)[EPT], int n, int bud,
                                             const unsigned *hist, const WaveBins<RADIX_BINS> &first, int out0, int w,
                                             int *__restrict__ indices, int rows_total, unsigned *lds,
                                             Searches &sr, int *sh_scan, int (&tab)[2][BLK_WV * 16]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  unsigned thr = 0xFFFFFFFFu;                          // no key is above, no tie is taken
  int ties = 0;
  if (bud > 0) block_threshold<EPT, CARRIED>(keys, n, bud, hist, first, lds, sr, thr, ties);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    int g = 0, e = 0;
    if (i * BLK_NT < n) {
      g = __popcll(__ballot(keys[i] > thr));
      e = __popcll(__ballot(keys[i] == thr));
    }
    if (lane == 0) { tab[0][i * BLK_WV + wv] = g; tab[1][i * BLK_WV + wv] = e; }
  }
  __syncthreads();
  const bool live = tid < EPT * BLK_WV;
  const int vg = live ? tab[0][tid] : 0, ve = live ? tab[1][tid] : 0;
  int ig, ie;
  block_scan_incl<BLK_NT>(vg, ig, sh_scan);
  block_scan_incl<BLK_NT>(ve, ie, sh_scan);
  if (live) { tab[0][tid] = ig - vg; tab[1][tid] = ie - ve; }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if (i * BLK_NT < n) {
      const bool gt = keys[i] > thr, eq = keys[i] == thr;
      const unsigned long long bg = __ballot(gt), be = __ballot(eq);
      if ((bg | be) == 0) continue;
      const int ng = tab[0][i * BLK_WV + wv] +
                     (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bg >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bg, 0u));
      const int ne = tab[1][i * BLK_WV + wv] +
                     (int)__builtin_amdgcn_mbcnt_hi((unsigned)(be >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)be, 0u));
      const int pos = out0 + ng + min(ne, ties);
      if ((gt || (eq && ne < ties)) && (unsigned)pos < (unsigned)rows_total) indices[pos] = i * BLK_NT + tid;
    }
  }
  for (int rr = tid; rr < w; rr += BLK_NT)
    if ((unsigned)(out0 + bud + rr) < (unsigned)rows_total) indices[out0 + bud + rr] = n + rr;
}

// One block per sequence: its budgets and offsets (adakv_allocate for short rows).
template <int EPT>
__global__ __launch_bounds__(BLK_NT) void alloc_block_kernel(SeqTab st, int h, int w, int alpha_fix,
                                                             const float *__restrict__ scores,
                                                             int *__restrict__ budgets,
                                                             int *__restrict__ cu) {
  __shared__ Searches sr;
  __shared__ __align__(16) unsigned lds[BLK_LDS];
  __shared__ LayerCounts lc;
  const int b = blockIdx.x, c = threadIdx.x, Bp = st.Bp[b];
  const int ties = block_layer_counts<EPT, false>(scores + st.score_off[b], h, st.n[b], Bp, TopkBufs(), b, lds, sr, lc);
  safeguard(h, Bp, alpha_fix, ties, lc);
  __syncthreads();
  if (c >= h) return;
  budgets[b * h + c] = lc.base[c];
  int run = st.out_off[b];
  for (int i = 0; i <= c; ++i) run += lc.base[i] + w;
  if (b == 0 && c == 0) cu[0] = 0;
  cu[b * h + c + 1] = run;
}

// One block per segment: its positions (adakv_select for short rows).
template <int EPT, bool CARRIED>
__global__ __launch_bounds__(BLK_NT) void select_block_kernel(SeqTab st, int h, int w,
                                                              const float *__restrict__ scores,
                                                              const unsigned *__restrict__ hist0,
                                                              const int *__restrict__ budgets,
                                                              const int *__restrict__ cu,
                                                              int *__restrict__ indices, int rows_total) {
  __shared__ Searches sr;
  __shared__ int sh_scan[BLK_WV];
  __shared__ __align__(16) unsigned lds[BLK_LDS];
  __shared__ int tab[2][BLK_WV * 16];
  const int seg = blockIdx.x, b = seg / h, c = seg % h, n = st.n[b];
  unsigned keys[EPT];
  const unsigned *hist = hist0 + (size_t)seg * RADIX_BINS;
  WaveBins<RADIX_BINS> first;
  const int out0 = cu[seg], bud = budgets[seg];
  if (CARRIED && threadIdx.x < 64) first = load_bins<RADIX_BINS>(hist);
  load_keys<EPT>(scores + st.score_off[b] + (size_t)c * n, n, keys);
  block_select<EPT, CARRIED>(keys, n, bud, hist, first, out0, w, indices, rows_total, lds, sr, sh_scan, tab);
}

// Layer scope and head scope of one segment in one block (pipeline mode): every block of a sequence
// finds the layer's threshold for itself, from all of the sequence's scores (SHORT, h*n <= 1024 EPT)
// or from the gather kernel's results (n <= 1024 EPT), and goes on with its own head.
template <int EPT, bool SHORT>
__global__ __launch_bounds__(BLK_NT) void topk_block_kernel(SeqTab st, ChunkTab ct, int h, int w,
                                                            int alpha_fix,
                                                            const float *__restrict__ scores, TopkBufs tb,
                                                            int *__restrict__ budgets, int *__restrict__ cu,
                                                            int *__restrict__ indices, int rows_total) {
  static_assert(1024 + HOLD_LAYER >= BLK_LDS, "the head scope's histograms take the layer scope's place");
  __shared__ Searches sr;
  __shared__ int sh_scan[BLK_WV];
  __shared__ __align__(16) unsigned lds[SHORT ? BLK_LDS : 1024 + HOLD_LAYER];
  __shared__ int tab[2][BLK_WV * 16];
  __shared__ LayerCounts lc;
  const int seg = blockIdx.x, b = seg / h, c = seg % h, n = st.n[b], Bp = st.Bp[b];
  const float *all = scores + st.score_off[b];
  unsigned keys[EPT];                                  // requested first, used last
  load_keys<EPT>(all + (size_t)c * n, n, keys);
  const unsigned *hist = tb.hist0 + (size_t)seg * RADIX_BINS;
  WaveBins<RADIX_BINS> first;
  if (threadIdx.x < 64) first = load_bins<RADIX_BINS>(hist);
  const int ties = SHORT ? block_layer_counts<EPT, true>(all, h, n, Bp, tb, b, lds, sr, lc)
                         : layer_counts(ct, h, b, Bp, tb, lc, sr, lds);
  safeguard(h, Bp, alpha_fix, ties, lc);
  __syncthreads();
  int out0 = st.out_off[b];
  for (int i = 0; i < c; ++i) out0 += lc.base[i] + w;
  const int bud = lc.base[c];
  if (threadIdx.x == 0) {
    budgets[seg] = bud;
    cu[seg + 1] = out0 + bud + w;
    if (seg == 0) cu[0] = 0;
  }
  block_select<EPT, true>(keys, n, bud, hist, first, out0, w, indices, rows_total, lds, sr, sh_scan, tab);
}

}  // namespace

size_t plan_topk_bytes(const SeqTab &st, const Dims &dm) { return plan(st, dm).bytes; }

// Pipeline mode needs a scoring kernel that files the first digits itself: the MFMA path with the
// max-pool fused into it.
bool carry_supported(const Dims &dm, int dtype) {
  return mfma_path_supported(dm, dtype) && dm.pool_k / 2 <= 32;
}

TopkCarry plan_carry(const SeqTab &st, const Dims &dm, char *ws_topk) {
  const TopkWs p = plan(st, dm);
  TopkCarry tc;
  tc.zero_begin = (unsigned *)ws_topk;
  tc.zero_words = (unsigned)(p.zero_end / 4);
  tc.hist0 = (unsigned *)(ws_topk + p.hist0);
  tc.hist_tot0 = (unsigned *)(ws_topk + p.hist_tot0);
  return tc;
}

static void launch_clear(const char *name, unsigned *begin, size_t words, hipStream_t s) {
  int zb = (int)((words + 256 * 4 - 1) / (256 * 4));
  if (zb < 1) zb = 1;
  if (zb > 1024) zb = 1024;
  ADAKV_LAUNCH(name, topk_init_kernel, dim3(zb), dim3(256), s, begin, words);
}

void launch_topk_clear(const TopkCarry &tc, hipStream_t s) {
  launch_clear("score_hist_clear", tc.zero_begin, tc.zero_words, s);
}

// The gather lists alone, in other memory: how much, and where.
static size_t list_bytes(size_t blocks) {
  return align_up(blocks * RADIX_BINS * 2, 256) + align_up(blocks * sizeof(BlockNote), 256) + blocks * ENT_PER_BLOCK * 2;
}
static TopkBufs lists_in(TopkBufs tb, char *spare, size_t blocks) {
  tb.starts = (unsigned short *)spare; spare += align_up(blocks * RADIX_BINS * 2, 256);
  tb.note = (BlockNote *)spare; spare += align_up(blocks * sizeof(BlockNote), 256);
  tb.entries = (unsigned short *)spare;
  return tb;
}

static TopkBufs bufs_of(char *ws, const TopkWs &p) {
  TopkBufs tb;
  tb.hist0 = (const unsigned *)(ws + p.hist0);
  tb.hist_tot0 = (const unsigned *)(ws + p.hist_tot0);
  tb.hist1 = (unsigned *)(ws + p.hist1);
  tb.hist1_tot = (unsigned *)(ws + p.hist1_tot);
  tb.starts = (unsigned short *)(ws + p.starts);
  tb.note = (BlockNote *)(ws + p.note);
  tb.entries = (unsigned short *)(ws + p.entries);
  return tb;
}

// Outside pipeline mode a call is self-contained: it clears the histograms and counts the first
// digits itself.
static void first_digits(const char *init_name, const char *pass_name, const SeqTab &st,
                         const ChunkTab &ct, int h, const float *scores, char *ws, const TopkWs &p,
                         hipStream_t s) {
  launch_clear(init_name, (unsigned *)ws, p.zero_end / 4, s);
  dim3 grid(ct.off[st.batch], h), block(256);
  ADAKV_LAUNCH(pass_name, topk_digit0_kernel, grid, block, s, st, ct, h, scores,
               (unsigned *)(ws + p.hist0), (unsigned *)(ws + p.hist_tot0));
}

static int longest_row(const SeqTab &st) {
  int n = 0;
  for (int b = 0; b < st.batch; ++b) n = st.n[b] > n ? st.n[b] : n;
  return n;
}

// Where one block per sequence or segment beats the kernels that spread a scope over the chip: a
// block's passes cost it 0.5 to 0.6 us per 1024 scores, in one compute unit; a launch costs 4 us.
// us a call, spread-out kernels / block (w = 8, h = 8 unless said):
//   allocate alone   4096 scores 14.6 / 9.4, 8192 14.6 / 12.0, 16 384 14.6 / 16.0; eight sequences 15.3 / 8.9, 15.4 / 11.8,
//                    15.5 / 16.0, and 12 288 15.3 / 14.1.  The counts per head make more heads dearer in a block:
//                    h = 32 8192 15.8 / 14.8, 12 288 15.7 / 17.4, h = 64 4096 18.1 / 15.4, 8192 18.0 / 19.3 (eight
//                    sequences 21.3 / 19.7, 12 288 21.3 / 21.7)
//   select alone     4096 per head 15.7 / 8.7, 8192 16.0 / 11.7, 16 384 16.1 / 15.5; eight sequences 18.0 / 15.6 at the last
// A step, d = 128, 128 rows, h = 8, by positions per head: three spread-out kernels / two of them and a block per head /
// one and a block per head / all in a block: 600 36.3 / 32.7 / 31.3 / 30.5, 1000 37.4 / 33.8 / 32.2 / 32.3, 1536 37.3 /
// 34.7 / 32.7 / 34.3, 4096 40.1 / 37.2 / 35.8, 8192 43.8 / 43.6, 10 000 45.2 / 46.0; h = 1, 12 288 39.7 / 40.3 / - / 38.0,
// 16 384 42.2 / 43.3 / - / 43.0.  So the block per head ends at 8192; everything in a block pays up to 12 288 scores where
// rows are too long for the form before it, and up to some 8000 where they are not (beyond, up to the same line, it
// costs 1 to 2 us).  (The line on allocation lies where the two met while a search took 0.7 us instead of 0.25 and the
// gather had 256 threads; with one sequence at the line itself the block is behind by 1.3 to 1.7 us now.)
constexpr long long alloc_block_max(int h) {           // scores of a sequence
  return (h <= 8 ? 16 : h <= 32 ? 12 : 8) * BLK_NT;
}
constexpr long long SELECT_BLOCK_MAX = 16 * BLK_NT;    // of a head; first digits counted here
constexpr long long SELECT_CARRIED_MAX = 8 * BLK_NT;   // of a head; first digits from the scoring kernel
constexpr long long TOPK_BLOCK_MAX = 12 * BLK_NT;      // of a sequence; both scopes in one launch
constexpr long long TOPK_ROW_MAX = 4 * BLK_NT;         // of a head; gather and the rest in one launch
// Longer rows: finish and the head's gather in one launch where every block has a compute unit to itself, each
// repeating the layer scope with a compute unit's whole issue rate, and where the head's lists fit into what the scoring
// sweeps have done with.  A step (d = 128, 128 rows) with four kernels / three, us: 16384 keys x 8 heads 52.1 / 50.8,
// 131072 x 8 139.4 / 137.9, four of up to 30000 x 8 109.0 / 107.5, 20000 x 32 111.9 / 109.4, 32768 x 32 (256 blocks)
// 150.6 / 149.3, but 32768 x 33 160.1 / 162.1, 20000 x 64 189 / 193, two of up to 131072 x 8 193.5 / 195.  On plateaus
// too (scores all equal): 32768 x 8 94.8 / 92.4, 131072 x 8 225 / 220, 20000 x 32 169 / 163.  Below four segments the
// line is not one of speed: a trace of a layer that small is to show each scope's kernels with times of their own (three
// heads of 20000 46.5 / 45.9, two of 60000 52.2 / 51.6, one of 131072 52.4 / 51.6; all scores equal 77.4 / 76.6, 83.0 /
// 81.5).
constexpr int FUSED_BLOCKS = 256, FUSED_SEGMENTS = 4;
size_t topk_spare_bytes(const SeqTab &st, const Dims &dm) {
  if (longest_row(st) <= SELECT_CARRIED_MAX || st.batch * dm.h_kv < FUSED_SEGMENTS) return 0;
  const size_t blocks = (size_t)count_chunks(st, SEL_CHUNK) * dm.h_kv;
  return blocks <= FUSED_BLOCKS ? list_bytes(blocks) : 0;
}
static void launch_gather(bool layer, const SeqTab &st, const ChunkTab &ct, int h, const float *scores, const int *budgets,
                          const TopkBufs &tb, hipStream_t s) {
  const dim3 grid(ct.off[st.batch], h), block(GATHER_NT);
  if (layer) ADAKV_LAUNCH("alloc_gather", (topk_gather_kernel<true>), grid, block, s, st, ct, h, scores, budgets, tb);
  else ADAKV_LAUNCH("select_gather", (topk_gather_kernel<false>), grid, block, s, st, ct, h, scores, budgets, tb);
}
// Emit has as many threads as leave every block resident at once (its registers let a compute unit hold one block of
// 1024, two of 512): the fewer positions a lane has to go through, the better, but a second round costs it all again.
// us, 256 / 512 / 1024 threads: 64 blocks 8.2 / 6.3 / 5.9, 256 8.6 / 6.9 / 6.6, 300 10.2 / 8.5 / 11.6, 400 10.6 / 8.9 / 12.1,
// 560 11.3 / 13.7 / 17.1 (before, with 256: 9.1, 9.4, 10.5, 10.6, 11.6).
static void launch_emit(const SeqTab &st, const ChunkTab &ct, int h, int w, const float *scores, const TopkBufs &tb,
                        const int *budgets, const int *cu, int *indices, int rows, hipStream_t s) {
  const dim3 grid(ct.off[st.batch], h);
#define ADAKV_GO(NT)                                                                              \
  ADAKV_LAUNCH("select_emit", (emit_write_kernel<NT>), grid, dim3(NT), s, st, ct, h, w, scores, tb, budgets, cu, indices, \
               rows)
  const int blocks = ct.off[st.batch] * h;
  if (blocks <= 256) ADAKV_GO(1024);
  else if (blocks <= 512) ADAKV_GO(512);
  else ADAKV_GO(256);
#undef ADAKV_GO
}

hipError_t launch_allocate(const SeqTab &st, const Dims &dm, const float *scores, int *budgets,
                           int *cu_seqlens, char *ws, bool carried, hipStream_t s) {
  const TopkWs p = plan(st, dm);
  const int h = dm.h_kv;
  const TopkBufs tb = bufs_of(ws, p);
  const long long most = (long long)longest_row(st) * h;
  if (!carried && most <= alloc_block_max(h)) {
#define ADAKV_GO(EPT)                                                                            \
  ADAKV_LAUNCH("alloc_block", (alloc_block_kernel<EPT>), dim3(st.batch), dim3(BLK_NT), s, st, h, dm.w, \
               dm.alpha_fix, scores, budgets, cu_seqlens)
    if (most <= 4 * BLK_NT) ADAKV_GO(4);
    else ADAKV_GO(16);
#undef ADAKV_GO
    return hipGetLastError();
  }
  const ChunkTab ct = make_chunks(st, SEL_CHUNK);
  if (!carried) first_digits("alloc_init", "alloc_pass0", st, ct, h, scores, ws, p, s);
  launch_gather(true, st, ct, h, scores, nullptr, tb, s);
  ADAKV_LAUNCH("alloc_finish", alloc_finish_kernel, dim3(st.batch), dim3(FIN_NT), s, st, ct, h, dm.w,
               dm.alpha_fix, tb, budgets, cu_seqlens);
  return hipGetLastError();
}

hipError_t launch_select(const SeqTab &st, const Dims &dm, const float *scores,
                         const int *budgets, const int *cu_seqlens, int *indices, char *ws,
                         bool carried, hipStream_t s) {
  const TopkWs p = plan(st, dm);
  const int h = dm.h_kv, rows = st.out_off[st.batch], n = longest_row(st);
  const TopkBufs tb = bufs_of(ws, p);
  if (n <= (carried ? SELECT_CARRIED_MAX : SELECT_BLOCK_MAX)) {
#define ADAKV_GO(EPT)                                                                            \
  do {                                                                                           \
    if (carried)                                                                                 \
      ADAKV_LAUNCH("select_block", (select_block_kernel<EPT, true>), dim3(st.batch * h), dim3(BLK_NT), s, st, \
                   h, dm.w, scores, tb.hist0, budgets, cu_seqlens, indices, rows);               \
    else                                                                                         \
      ADAKV_LAUNCH("select_block", (select_block_kernel<EPT, false>), dim3(st.batch * h), dim3(BLK_NT), s, st, \
                   h, dm.w, scores, tb.hist0, budgets, cu_seqlens, indices, rows);               \
  } while (0)
    if (n <= 4 * BLK_NT) ADAKV_GO(4);
    else ADAKV_GO(16);
#undef ADAKV_GO
    return hipGetLastError();
  }
  const ChunkTab ct = make_chunks(st, SEL_CHUNK);
  if (!carried) first_digits("select_init", "select_pass0", st, ct, h, scores, ws, p, s);
  launch_gather(false, st, ct, h, scores, budgets, tb, s);
  launch_emit(st, ct, h, dm.w, scores, tb, budgets, cu_seqlens, indices, rows, s);
  return hipGetLastError();
}

hipError_t launch_topk(const SeqTab &st, const Dims &dm, const float *scores, int *budgets,
                       int *cu_seqlens, int *indices, char *ws, bool carried, char *spare, size_t spare_bytes,
                       hipStream_t s) {
  const int h = dm.h_kv, rows = st.out_off[st.batch], nseg = st.batch * h;
  const long long most = (long long)longest_row(st) * h;
  // Every block repeats the layer scope with a compute unit's whole issue rate (sixteen wavefronts), so there
  // are no more of them than compute units; two on one take turns.  The whole step, us, block / the kernels
  // that spread a scope over the chip, d = 64, 8 rows: 4 x 64 heads x 4096 103.9 / 104.6, on plateaus (scores all
  // equal, which every block streams; lengths spread below 4096) 96.7 / 97.6; 5 x 64 145.8 / 133.8, 141 / 116; 8 x 64
  // 177.5 / 164.5, 180 / 151; 8 x 64 heads x 190 62.7 / 45.6; 32 x 8 x 1500 50.0 / 55.0; 40 x 8 71.6 / 67.1; 64 x 8
  // 91.7 / 92.7.
  const bool in_block = most <= TOPK_BLOCK_MAX;
  if (carried && nseg <= 256 && (in_block || longest_row(st) <= TOPK_ROW_MAX)) {
    const TopkBufs tb = bufs_of(ws, plan(st, dm));
    const ChunkTab ct = make_chunks(st, SEL_CHUNK);
    if (!in_block)
      launch_gather(true, st, ct, h, scores, nullptr, tb, s);
#define ADAKV_GO(EPT, SHORT)                                                                     \
  ADAKV_LAUNCH("topk_block", (topk_block_kernel<EPT, SHORT>), dim3(nseg), dim3(BLK_NT), s, st, ct, h, dm.w, \
               dm.alpha_fix, scores, tb, budgets, cu_seqlens, indices, rows)
    if (!in_block) ADAKV_GO(4, false);
    else if (most <= 4 * BLK_NT) ADAKV_GO(4, true);
    else ADAKV_GO(12, true);
#undef ADAKV_GO
    return hipGetLastError();
  }
  const size_t lists = topk_spare_bytes(st, dm);
  if (carried && lists && lists <= spare_bytes) {
    const ChunkTab ct = make_chunks(st, SEL_CHUNK);
    const TopkBufs tb = bufs_of(ws, plan(st, dm)), head = lists_in(tb, spare, (size_t)ct.off[st.batch] * h);
    launch_gather(true, st, ct, h, scores, nullptr, tb, s);
    ADAKV_LAUNCH("topk_finish_gather", finish_gather_kernel, dim3(ct.off[st.batch], h), dim3(FIN_NT), s, st, ct, h, dm.w,
                 dm.alpha_fix, scores, tb, head, budgets, cu_seqlens);
    launch_emit(st, ct, h, dm.w, scores, head, budgets, cu_seqlens, indices, rows, s);
    return hipGetLastError();
  }
  const hipError_t e = launch_allocate(st, dm, scores, budgets, cu_seqlens, ws, carried, s);
  if (e != hipSuccess) return e;
  return launch_select(st, dm, scores, budgets, cu_seqlens, indices, ws, carried, s);
}

}  // namespace adakv
